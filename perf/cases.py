"""Performance cases of the library: the calls a decoding (or training) program makes, at the sizes it makes them.

A case is a dict of plain values.  `kind` names the call:

  step      one whole decode step of one layer: both attention views, then the consensus and the commit
  attn      one attention call of one view over one layer's cache
  verify    the consensus (greedy, or sampling when `temp` > 0) and the commit into every layer's cache
  prefill   the AR view's causal prefill of one layer
  mask      the training block mask's forward: every anchor block of some packed sequences is one batch entry
  cycle     one decode cycle over a layer stack, replayed as a HIP graph

Lengths are ragged where `lo` < `hi`: the batch's lengths are spread evenly from lo to hi and shuffled by the seed,
so that the work of a case does not depend on it.  Calls that append to the cache bump the lengths on the device;
`run` puts the lengths of before the call back first, so that every pass is the same step.
"""
import math

import torch

from paper_2605_12825_amd import runtime as rt

DEV = "cuda:0"
P = 16  # tokens per cache page


def listed():
    heads = dict(hq=32, hkv=8, d=128)          # the 8B model's attention geometry
    return [
        # the smallest call there is: a whole step at toy size, all launches and latency
        dict(name="step_tiny", kind="step", batch=1, hq=4, hkv=2, d=64, K=4, lo=128, hi=128, vocab=512, temp=0.0),
        # an ordinary batch-1 step, T > 0: what an interactive user waits for, per layer, plus the sampled consensus
        dict(name="step_b1_sampled", kind="step", batch=1, K=16, lo=4096, hi=4096, vocab=128256, temp=1.0, **heads),
        # batch 1 through a whole 36-layer stack, greedy: the paper's own setting
        dict(name="cycle_b1", kind="cycle", batch=1, K=16, lo=4096, hi=4096, vocab=128256, layers=36, temp=0.0, **heads),
        # batch 1 at the long end of the paper's context sweep and its block size
        dict(name="attn_40k_k32", kind="attn", batch=1, K=32, lo=40000, hi=40000, view=0, lse=0, splits=0, fused=0, **heads),
        # long contexts, the verification pass, log-sum-exp wanted
        dict(name="attn_long", kind="attn", batch=4, K=16, lo=32768, hi=32768, view=1, lse=1, splits=0, fused=0, **heads),
        # a serving batch with ragged lengths, block inputs read out of a fused projection's output
        dict(name="attn_batch", kind="attn", batch=64, K=16, lo=1025, hi=3071, view=0, lse=0, splits=0, fused=1, **heads),
        # widely ragged lengths, seven query heads per KV head, the balanced partition
        dict(name="attn_ragged", kind="attn", batch=16, hq=28, hkv=4, d=128, K=32, lo=512, hi=8192, view=1, lse=0,
             splits=-1, fused=0),
        # greedy verification of a large batch: logits of a 152k vocabulary, commit into eight layers
        dict(name="verify_b64", kind="verify", batch=64, K=16, lo=200, hi=500, vocab=151936, layers=8, temp=0.0, **heads),
        # sampled verification at the paper's block size
        dict(name="sample_b8", kind="verify", batch=8, K=32, lo=200, hi=500, vocab=151936, layers=1, temp=0.8, **heads),
        # prefill of one long prompt into an empty cache
        dict(name="prefill_8k", kind="prefill", batch=1, lo=0, hi=0, new_lo=8192, new_hi=8192, **heads),
        # chunked prefill of a ragged batch on top of caches of different lengths
        dict(name="prefill_ragged", kind="prefill", batch=6, hq=28, hkv=4, d=128, lo=0, hi=6001, new_lo=333, new_hi=1500),
        # training: packed sequences of 2048 tokens with 256 anchor blocks each
        dict(name="train_mask", kind="mask", seqs=4, length=2048, blocks=256, K=32, **heads),
    ]


HEADS = [(32, 8, 128), (32, 8, 128), (28, 4, 128), (16, 8, 128), (4, 2, 64), (16, 2, 64), (8, 8, 128)]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the ranges above; sizes over their logarithm, trimmed until it costs less than the largest."""
    kind = rng.choice(["step", "attn", "attn", "attn", "verify", "prefill", "prefill", "mask", "cycle"])
    hq, hkv, d = rng.choice(HEADS)
    group = hq // hkv
    K = rng.choice([k for k in (1, 4, 8, 13, 16, 16, 24, 32, 32) if k * group <= 256])
    c = dict(kind=kind, hq=hq, hkv=hkv, d=d)
    if kind == "attn":
        hi = _log(rng, 100, 40000)
        lo = rng.choice([hi, hi, max(1, hi // 16)])
        c.update(batch=_log(rng, 1, 64), K=K, lo=lo, hi=hi, view=rng.randint(0, 1), lse=rng.choice([0, 0, 1]),
                 splits=-1 if lo < hi else 0, fused=rng.randint(0, 1))
        while c["batch"] > 1 and work(c)["bytes"] > 5e8:
            c["batch"] -= 1
    elif kind == "step":
        hi = _log(rng, 100, 16000)
        c.update(batch=_log(rng, 1, 16), K=K, lo=rng.choice([hi, max(1, hi // 4)]), hi=hi, vocab=_log(rng, 500, 160000),
                 temp=rng.choice([0.0, 0.0, 0.7, 1.0]))
        while c["batch"] > 1 and work(c)["bytes"] > 5e8:
            c["batch"] -= 1
    elif kind == "verify":
        c.update(batch=_log(rng, 1, 64), K=K, lo=rng.randint(1, 300), hi=500, vocab=_log(rng, 500, 160000),
                 layers=rng.choice([1, 2, 8, 36]), temp=rng.choice([0.0, 0.7, 1.0]))
        while c["batch"] > 1 and (work(c)["bytes"] > 5e8 or c["batch"] * c["layers"] > 512):
            c["batch"] -= 1
    elif kind == "prefill":
        new = _log(rng, 33, 8192)
        hi = rng.choice([0, _log(rng, 100, 8000)])
        c.update(batch=_log(rng, 1, 8), lo=rng.choice([0, hi]), hi=hi, new_lo=max(1, new // rng.choice([1, 4])), new_hi=new)
        while c["batch"] > 1 and work(c)["flops"] > 5e11:
            c["batch"] -= 1
        while work(c)["flops"] > 5e11:
            c["new_hi"] = c["new_hi"] * 3 // 4
            c["new_lo"] = min(c["new_lo"], c["new_hi"])
    elif kind == "mask":
        c.update(seqs=rng.randint(1, 4), length=_log(rng, 300, 4096), blocks=_log(rng, 32, 256), K=K)
        while c["seqs"] > 1 and work(c)["flops"] > 5e11:
            c["seqs"] -= 1
    else:
        c.update(batch=rng.randint(1, 4), K=K, lo=_log(rng, 200, 4000), hi=4000, vocab=_log(rng, 500, 160000),
                 layers=rng.randint(4, 24), temp=rng.choice([0.0, 0.0, 1.0]))
        while c["layers"] > 4 and work(c)["bytes"] > 8e8:
            c["layers"] -= 1
    return c


# ---------------------------------------------------------------------------------------------------------------
# work, in bytes and operations that the path cannot do without

def _spread(n, lo, hi):
    """n whole numbers from lo to hi, evenly spaced."""
    return [hi] if n == 1 else [lo + (hi - lo) * i // (n - 1) for i in range(n)]


def _attn_work(c, lens, calls=1):
    B, K, hq, hkv, d = len(lens), c["K"], c["hq"], c["hkv"], c["d"]
    tokens = sum(lens)
    kv = 4 * d * hkv * (tokens + B * K)
    return calls * (kv + 4 * B * K * hq * d), calls * 4 * d * hq * K * (tokens + B * K)


def _verify_work(c):
    B, K, V = c["batch"], c["K"], c["vocab"]
    rows = min(K, 3)                       # appended rows per sequence, about
    commit = 2 * B * rows * c.get("layers", 1) * c["hkv"] * c["d"] * 4
    if c["temp"] > 0:
        return 8 * B * K * V + 4 * B * V + commit, 10 * B * K * V
    return 4 * B * K * V + commit, B * K * V


def work(case):
    c = case
    if c["kind"] == "attn":
        by, fl = _attn_work(c, _spread(c["batch"], c["lo"], c["hi"]))
        by += 4 * c["batch"] * c["hq"] * c["K"] if c["lse"] else 0
    elif c["kind"] in ("step", "cycle"):
        by, fl = _attn_work(c, _spread(c["batch"], c["lo"], c["hi"]), 2 * c.get("layers", 1))
        vb, vf = _verify_work(c)
        by, fl = by + vb, fl + vf
    elif c["kind"] == "verify":
        by, fl = _verify_work(c)
    elif c["kind"] == "prefill":
        old, new = _spread(c["batch"], c["lo"], c["hi"]), _spread(c["batch"], c["new_lo"], c["new_hi"])
        keys = sum(o * n + n * (n + 1) // 2 for o, n in zip(old, new))
        by = sum(4 * c["d"] * c["hkv"] * (o + 2 * n) + 4 * c["d"] * c["hq"] * n for o, n in zip(old, new))
        fl = 4 * c["d"] * c["hq"] * keys
    else:
        NB, L, K = c["seqs"] * c["blocks"], c["length"], c["K"]
        by = 4 * c["d"] * c["hkv"] * (c["seqs"] * L + NB * K) + 4 * NB * K * c["hq"] * c["d"]
        fl = 4 * c["d"] * c["hq"] * K * NB * (L // 2 + K)
    return {"bytes": by, "flops": fl}


def tolerance(case):
    """Attention rounds its probabilities and its result to bf16, 2^-9 each: measured against 64 bits over the listed
    and two dozen drawn cases, every output is off by 2.0e-3 to 2.4e-3 (2-norm) and, at its worst value, by 0.005 to
    0.055 of the root mean square (of the value itself where that is larger).  Four times that is allowed.  Tokens,
    lengths and cache rows are comparisons and copies, the same in any correct implementation; only a sampled
    decision can sit within fp32 rounding of a tie."""
    if case["kind"] == "verify":
        return {"rel": 0.0, "differ": 0.01} if case["temp"] > 0 else "exact"
    return {"rel": 1e-2, "max": 0.2, "differ": 0.01 if case.get("temp", 0) > 0 else 0.0}


# ---------------------------------------------------------------------------------------------------------------
# what a program holds before the call

def _gen(seed):
    return torch.Generator(device=DEV).manual_seed(seed * 7919 + 11)


def _normal(g, *shape):
    return torch.randn(shape, generator=g, dtype=torch.bfloat16, device=DEV)


def _lengths(seed, n, lo, hi, salt=0):
    order = torch.randperm(n, generator=torch.Generator().manual_seed(seed * 31 + salt))
    return torch.tensor(_spread(n, lo, hi), dtype=torch.int32)[order].to(DEV)


def _cache(s, g, c, lens, capacity, layers):
    """A paged cache of `layers` layers, its pages in random order, about one in ten of them spare."""
    B = c["batch"]
    slots = (capacity + P - 1) // P
    s["pages"] = B * slots + max(1, B * slots // 10)
    perm = torch.randperm(s["pages"], generator=g, device=DEV).to(torch.int32)
    s["page_table"] = perm[:B * slots].view(B, slots).contiguous()
    shape = (layers, s["pages"], c["hkv"], P, c["d"])
    s["k_pool"], s["v_pool"] = _normal(g, *shape), _normal(g, *shape)
    s["lens0"] = lens
    s["seq_lens"] = lens.clone()


def _block(s, g, c, tag, layers=None, fused=False):
    """One view's queries and block K/V: dense tensors, or column ranges of one fused projection output."""
    B, K, hq, hkv, d = c["batch"], c["K"], c["hq"], c["hkv"], c["d"]
    if fused:
        x = _normal(g, B * K, hq + 2 * hkv, d)
        s["q" + tag], s["k" + tag], s["v" + tag] = x[:, :hq], x[:, hq:hq + hkv], x[:, hq + hkv:]
        return
    pre = () if layers is None else (layers,)
    s["q" + tag] = _normal(g, *pre, B, K, hq, d)
    s["k" + tag], s["v" + tag] = _normal(g, *pre, B, K, hkv, d), _normal(g, *pre, B, K, hkv, d)


def _drafts(s, g, c):
    """Logits and drafts whose accepted prefixes follow a geometric distribution (greedy: a planted row maximum;
    sampled: drafts drawn from a draft distribution close to the target's)."""
    B, K, V = c["batch"], c["K"], c["vocab"]
    if c["temp"] > 0:
        ar = torch.randn((B, K, V), generator=g, device=DEV) * 2
        df = torch.randn((B, K, V), generator=g, device=DEV).mul_(0.5).add_(ar)
        s["draft"] = torch.empty((B, K), dtype=torch.int32, device=DEV)
        for b in range(B):
            e = torch.empty((K, V), device=DEV).exponential_(generator=g)
            s["draft"][b] = (df[b] / c["temp"] - e.log()).argmax(-1).to(torch.int32)
        s["ar"], s["df"] = ar, df
        s["u"] = torch.rand((B, K), generator=g, device=DEV)
        s["gumbel"] = -torch.empty((B, V), device=DEV).exponential_(generator=g).log()
        return
    s["ar"] = torch.randn((B, K, V), generator=g, device=DEV)
    top = torch.randint(0, V, (B, K), generator=g, device=DEV)
    s["ar"].scatter_(2, top[..., None], 8 + torch.rand((B, K, 1), generator=g, device=DEV))
    u = torch.rand((B, 1), generator=g, device=DEV).clamp_min(1e-6)
    n_acc = (u.log() / math.log(0.7)).floor().clamp(0, K).long()
    k = torch.arange(K, device=DEV)[None]
    other = torch.randint(0, V, (B, K), generator=g, device=DEV)
    miss = (top + 1 + other % max(V - 1, 1)) % V
    s["draft"] = torch.where(k < n_acc, top, torch.where(k == n_acc, miss, other)).to(torch.int32)


def _results(s, c):
    B, K = c["batch"], c["K"]
    s["acc"], s["ncm"], s["anchor"] = (torch.zeros(B, dtype=torch.int32, device=DEV) for _ in range(3))
    s["tokens"] = torch.zeros((B, K), dtype=torch.int32, device=DEV)


def _out(c, *pre):
    return torch.zeros(pre + (c["hq"], c["d"]), dtype=torch.bfloat16, device=DEV)


def _step(s, c, bound, **kw):
    return rt.DecodeStep(batch=c["batch"], num_q_heads=c["hq"], num_kv_heads=c["hkv"], head_dim=c["d"], block_k=c["K"],
                         page_size=P, max_pages_per_seq=s["page_table"].shape[1], max_seq_len=bound,
                         num_pages=s["pages"], **kw)


def prepare(case, seed):
    c = dict(case)
    g, s = _gen(seed), {}
    kind = c["kind"]
    if kind == "mask":
        return _prepare_mask(c, g)
    if kind == "prefill":
        c["K"] = 16
        old = _lengths(seed, c["batch"], c["lo"], c["hi"])
        new = _lengths(seed, c["batch"], c["new_lo"], c["new_hi"], 1)
        bound, T = c["hi"] + c["new_hi"], c["new_hi"]
        _cache(s, g, c, old, bound, 1)
        B = c["batch"]
        s.update(case=c, new=new, T=T, q=_normal(g, B, T, c["hq"], c["d"]), kn=_normal(g, B, T, c["hkv"], c["d"]),
                 vn=_normal(g, B, T, c["hkv"], c["d"]), out=_out(c, B, T), step=_step(s, c, bound))
        return s
    lens = _lengths(seed, c["batch"], c["lo"], c["hi"])
    bound = c["hi"] + c["K"]
    if kind == "cycle":
        return _prepare_cycle(c, g, lens, bound)
    layers = c.get("layers", 1)
    _cache(s, g, c, lens, bound, layers)
    s["case"] = c
    if kind == "attn":
        hq, hkv, d, K = c["hq"], c["hkv"], c["d"], c["K"]
        row = (hq + 2 * hkv) * d
        strides = (row, d, row, d, c["batch"] * K * row) if c["fused"] else None
        _block(s, g, c, "", fused=bool(c["fused"]))
        s["out"] = _out(c, c["batch"], K)
        s["lse"] = torch.zeros((c["batch"], hq, K), device=DEV) if c["lse"] else None
        s["step"] = _step(s, c, c["hi"], num_splits=c["splits"], block_strides=strides)
        return s
    _drafts(s, g, c)
    _results(s, c)
    if kind == "verify":
        _block(s, g, c, "_ar", layers=layers)
        s["step"] = _step(s, c, bound, vocab=c["vocab"], num_layers=layers)
        return s
    _block(s, g, c, "_diff")
    _block(s, g, c, "_ar")
    s["out_diff"], s["out_ar"] = _out(c, c["batch"], c["K"]), _out(c, c["batch"], c["K"])
    s["step"] = _step(s, c, bound, vocab=c["vocab"])
    return s


def _prepare_mask(c, g):
    """Anchor blocks of packed sequences; the clean context's K/V stay [token, head, d], which strides describe as
    pages of 16 tokens."""
    n, L, NB, K, hq, hkv, d = c["seqs"], c["length"], c["blocks"], c["K"], c["hq"], c["hkv"], c["d"]
    slots = (L + P - 1) // P
    c["batch"] = n * NB
    s = dict(case=c, pages=n * slots)
    u = torch.rand((n, NB), generator=g, device=DEV)
    anchors = ((torch.arange(NB, device=DEV)[None] + u) * (L / NB)).long().clamp(1, L)   # sorted, one per stratum
    s["seq_lens"] = s["lens0"] = anchors.reshape(-1).to(torch.int32)
    s["page_table"] = torch.arange(n * slots, device=DEV, dtype=torch.int32).view(n, 1, slots).expand(n, NB, slots) \
        .reshape(n * NB, slots).contiguous()
    s["k_pool"], s["v_pool"] = _normal(g, 1, n * slots * P, hkv, d), _normal(g, 1, n * slots * P, hkv, d)
    _block(s, g, c, "")
    s["out"], s["lse"] = _out(c, c["batch"], K), None
    s["step"] = _step(s, c, L, pool_strides=(0, P * hkv * d, d, hkv * d))
    return s


def _prepare_cycle(c, g, lens, bound):
    s = {"case": c}
    _cache(s, g, c, lens, bound, c["layers"])
    st = rt.DecodeStack(num_layers=c["layers"], batch=c["batch"], num_q_heads=c["hq"], num_kv_heads=c["hkv"],
                        head_dim=c["d"], block_k=c["K"], page_size=P, k_pool=s["k_pool"].view(torch.int16),
                        v_pool=s["v_pool"].view(torch.int16), page_table=s["page_table"], seq_lens=s["seq_lens"],
                        max_seq_len=bound, vocab=c["vocab"], temperature=c["temp"])
    for tag in ("_diff", "_ar"):
        _block(s, g, c, tag, layers=c["layers"])
        for x, buf in (("q", "q"), ("k", "k_blk"), ("v", "v_blk")):
            getattr(st, buf + tag).view(torch.bfloat16).copy_(s[x + tag])
            s[x + tag] = getattr(st, buf + tag).view(torch.bfloat16)
    _drafts(s, g, c)
    for x, buf in (("ar", "ar_logits"), ("draft", "draft_tokens"), ("df", "diff_logits"), ("u", "accept_u"),
                   ("gumbel", "gumbel")):
        if x in s:
            getattr(st, buf).copy_(s.pop(x))
    st.capture()
    s["stack"] = st
    return s


# ---------------------------------------------------------------------------------------------------------------
# one pass

def _consensus(s, c):
    step = s["step"]
    args = (s["k_ar"], s["v_ar"], s["k_pool"], s["v_pool"], s["page_table"], s["seq_lens"], s["acc"], s["ncm"],
            s["tokens"], s["anchor"])
    if c["temp"] > 0:
        step.sampling_consensus_commit(c["temp"], s["ar"], s["df"], s["draft"], s["u"], s["gumbel"], *args)
    else:
        step.consensus_commit(s["ar"], s["draft"], *args)


def _state(s):
    bits = torch.int16
    return dict(accepted=s["acc"], committed=s["ncm"], tokens=s["tokens"], anchor=s["anchor"], lens=s["seq_lens"],
                k_pool=s["k_pool"].view(bits), v_pool=s["v_pool"].view(bits))


def run(s):
    c = s["case"]
    kind = c["kind"]
    if kind in ("attn", "mask"):
        s["step"].attn(c.get("view", 0), s["q"], s["k"], s["v"], s["k_pool"], s["v_pool"], s["page_table"],
                       s["seq_lens"], s["out"], s["lse"])
        return dict(out=s["out"]) if s["lse"] is None else dict(out=s["out"], lse=s["lse"])
    s["seq_lens"].copy_(s["lens0"])
    if kind == "prefill":
        s["step"].prefill(s["T"], s["q"], s["kn"], s["vn"], s["new"], s["k_pool"], s["v_pool"], s["page_table"],
                          s["seq_lens"], s["out"])
        return dict(out=s["out"], lens=s["seq_lens"], k_pool=s["k_pool"].view(torch.int16),
                    v_pool=s["v_pool"].view(torch.int16))
    if kind == "cycle":
        st = s["stack"]
        st.replay(torch.cuda.current_stream())
        return dict(out_diff=st.out_diff.view(torch.bfloat16), out_ar=st.out_ar.view(torch.bfloat16),
                    accepted=st.accept_len, committed=st.num_committed, tokens=st.out_tokens, anchor=st.next_anchor,
                    lens=s["seq_lens"], k_pool=s["k_pool"].view(torch.int16), v_pool=s["v_pool"].view(torch.int16))
    if kind == "verify":
        _consensus(s, c)
        return _state(s)
    for view, tag in ((0, "_diff"), (1, "_ar")):
        s["step"].attn(view, s["q" + tag], s["k" + tag], s["v" + tag], s["k_pool"], s["v_pool"], s["page_table"],
                       s["seq_lens"], s["out" + tag])
    _consensus(s, c)
    return dict(_state(s), out_diff=s["out_diff"], out_ar=s["out_ar"])


# ---------------------------------------------------------------------------------------------------------------
# the same in 64 bits

def _gather(pool, pages, n):
    """The first n cached rows behind a row of page ids, [H, n, d] in fp64 ([page, H, slot, d] pools)."""
    x = pool[pages[:(n + P - 1) // P].long()]
    return x.permute(1, 0, 2, 3).reshape(pool.shape[1], -1, pool.shape[3])[:, :n].double()


def _softmax_v(q, k, v, hide):
    """q [R, d], k and v [n, d], hide [R, n] or None."""
    x = (q @ k.t()) / math.sqrt(q.shape[1])
    if hide is not None:
        x = x.masked_fill(hide, -math.inf)
    return torch.softmax(x, -1) @ v, torch.logsumexp(x, -1)


def _exact_block(c, b, view, q, k, v, cached):
    """Attention of one sequence's block: out [K, hq, d], lse [hq, K].  cached(b) -> keys and values [hkv, n, d]."""
    K, hq, hkv, d = c["K"], c["hq"], c["hkv"], c["d"]
    G = hq // hkv
    kc, vc = cached(b)
    n = kc.shape[1]
    i = torch.arange(K, device=DEV)
    hide = torch.zeros((K, n + K), dtype=torch.bool, device=DEV)
    if view == 1:
        hide[:, n:] = i[None] > i[:, None]
    hide = hide.repeat_interleave(G, 0)
    out = torch.empty((K, hq, d), dtype=torch.float64, device=DEV)
    lse = torch.empty((hq, K), dtype=torch.float64, device=DEV)
    q, k, v = (x.reshape(c["batch"], K, -1, d)[b].double() for x in (q, k, v))
    for g in range(hkv):
        rows = q[:, g * G:(g + 1) * G].reshape(K * G, d)
        o, l = _softmax_v(rows, torch.cat((kc[g], k[:, g])), torch.cat((vc[g], v[:, g])), hide)
        out[:, g * G:(g + 1) * G] = o.view(K, G, d)
        lse[g * G:(g + 1) * G] = l.view(K, G).t()
    return out, lse


def exact(case, seed):
    c = case
    if c["kind"] == "verify":
        return None                         # whole numbers and bytes only
    s = prepare(case, seed)
    c = s["case"]
    lens = s["lens0"].tolist()
    if c["kind"] == "prefill":
        return _exact_prefill(s, c, lens)
    if c["kind"] == "mask":
        L = c["length"]
        kp, vp = (s[x][0].view(c["seqs"], -1, c["hkv"], c["d"]) for x in ("k_pool", "v_pool"))

        def cached(b):
            q = b // c["blocks"]
            return tuple(x[q, :lens[b]].permute(1, 0, 2).double() for x in (kp, vp))
        return dict(out=torch.stack([_exact_block(c, b, 0, s["q"], s["k"], s["v"], cached)[0]
                                     for b in range(c["batch"])]))

    def view_of(view, tag, layer=0):
        pick = (lambda x: x[layer]) if c["kind"] == "cycle" else (lambda x: x)

        def cached(b):
            return tuple(_gather(s[x][layer], s["page_table"][b], lens[b]) for x in ("k_pool", "v_pool"))
        got = [_exact_block(c, b, view, pick(s["q" + tag]), pick(s["k" + tag]), pick(s["v" + tag]), cached)
               for b in range(c["batch"])]
        return torch.stack([o for o, _ in got]), torch.stack([l for _, l in got])

    if c["kind"] == "attn":
        out, lse = view_of(c["view"], "")
        return dict(out=out, lse=lse) if c["lse"] else dict(out=out)
    none = dict.fromkeys(("accepted", "committed", "tokens", "anchor", "lens", "k_pool", "v_pool"))
    if c["kind"] == "cycle":
        return dict(none, out_diff=torch.stack([view_of(0, "_diff", l)[0] for l in range(c["layers"])]),
                    out_ar=torch.stack([view_of(1, "_ar", l)[0] for l in range(c["layers"])]))
    return dict(none, out_diff=view_of(0, "_diff")[0], out_ar=view_of(1, "_ar")[0])


def _exact_prefill(s, c, lens):
    G = c["hq"] // c["hkv"]
    out = torch.zeros(s["out"].shape, dtype=torch.float64, device=DEV)
    for b, (L, n) in enumerate(zip(lens, s["new"].tolist())):
        kc, vc = (_gather(s[x][0], s["page_table"][b], L) for x in ("k_pool", "v_pool"))
        for h in range(c["hq"]):
            k = torch.cat((kc[h // G], s["kn"][b, :n, h // G].double()))
            v = torch.cat((vc[h // G], s["vn"][b, :n, h // G].double()))
            for i0 in range(0, n, 2048):
                i1 = min(n, i0 + 2048)
                seen = L + torch.arange(i0, i1, device=DEV)[:, None]
                hide = torch.arange(L + i1, device=DEV)[None] > seen
                out[b, i0:i1, h] = _softmax_v(s["q"][b, i0:i1, h].double(), k[:L + i1], v[:L + i1], hide)[0]
    return dict(out=out, lens=None, k_pool=None, v_pool=None)
