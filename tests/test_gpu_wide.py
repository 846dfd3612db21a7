"""The 64-rows-per-wave attention kernel (the one for launches that fill the chip) against the oracle: decode-mode
batches and prefill at the smallest launches that take it, with lengths on both sides of every tile and ring edge.
Same bars as every other attention parity test."""
from dataclasses import replace

import numpy as np
import pytest

import oracle
from orthrus_inputs import Workload, bf16_bits_to_f32, f32_to_bf16_bits, make_block, make_cache

from test_attn_routes_cpu import decode_is_wide, prefill_waves
from test_gpu_parity import AR, DIFF, GpuCase, _check_attn, _oracle_attn
from test_gpu_prefill import SENTINEL, Case, _check, _new_tokens

pytestmark = pytest.mark.gpu

# empty, inside / at / past a tile, and past the LDS ring (4 or 6 stages of 32 tokens)
EDGES = [0, 1, 31, 32, 33, 63, 64, 96, 127, 128, 129, 160, 161, 191, 192, 193, 224, 255, 257, 300]


def _lens(n, seed):
    rng = np.random.default_rng(seed)
    return rng.permutation(np.concatenate((EDGES, rng.integers(0, 301, size=n)))[:max(n, len(EDGES))])[:n].astype(np.int32)


BOUND = 4096  # the kernel is chosen by the bound on the lengths, not by the lengths


def _roomy(cache, page):
    """The same cache with a page table wide enough for BOUND."""
    pt = cache["page_table"]
    wide = np.full((pt.shape[0], BOUND // page), -1, np.int32)
    wide[:, :pt.shape[1]] = pt
    return dict(cache, page_table=wide)


def _case(w, cache, wide, num_splits=0, num_layers=1):
    rows, units = w.num_q_heads // w.num_kv_heads * w.block_k, w.batch * w.num_kv_heads
    assert decode_is_wide(w.head_dim, rows, BOUND, units) == wide
    return GpuCase(w, _roomy(cache, w.page_size), num_splits=num_splits, num_layers=num_layers, max_seq_len=BOUND)


@pytest.mark.parametrize("view", [DIFF, AR])
@pytest.mark.parametrize("g,K,hkv,batch,d,page", [
    (4, 32, 8, 64, 128, 16),     # 128 rows, two waves, full
    (7, 16, 8, 64, 128, 32),     # 112 rows: the second wave's last block ends in padding
    (8, 32, 4, 80, 128, 16),     # 256 rows, four waves
    (8, 30, 4, 80, 128, 64),     # 240 rows: half a block of padding
    (8, 16, 8, 96, 64, 16),
    (8, 31, 4, 64, 64, 16),
    (7, 32, 4, 96, 64, 64),      # 224 rows: a block of padding
])
def test_decode_batches_that_fill_the_chip(g, K, hkv, batch, d, page, view):
    w = Workload(name="wide", seed=8100 + g * K + d, batch=batch, num_q_heads=g * hkv, num_kv_heads=hkv, head_dim=d,
                 block_k=K, context=300, page_size=page, paging="scattered")
    cache = make_cache(w, seq_lens=_lens(batch, 8200 + K))
    blk = make_block(w, 8300 + K)
    case = _case(w, cache, True)
    got, lse = case.attn(view, blk)
    want, want_lse = _oracle_attn(view, w, blk, cache, want_lse=True)
    _check_attn(got, want)
    np.testing.assert_allclose(lse, want_lse, rtol=0, atol=2e-3)
    assert case.step.device_error() == 0
    again, _ = case.attn(view, blk)
    np.testing.assert_array_equal(again, got)
    case.step.close()


@pytest.mark.parametrize("g,hkv,batch,d,T", [
    (4, 8, 64, 128, 70),         # 64 tokens x 4 heads per workgroup: one full and one short chunk
    (4, 8, 12, 128, 70),         # the same with two waves: 32 tokens
    (1, 8, 70, 128, 40),
    (7, 8, 40, 128, 75),         # 36 tokens x 7 heads: 252 of 256 rows
    (5, 2, 3, 128, 90),          # two waves: 25 tokens x 5 heads
    (8, 2, 3, 64, 90),
])
def test_prefill_that_fills_the_chip(g, hkv, batch, d, T):
    w = Workload(name="widep", seed=8400 + g, batch=batch, num_q_heads=g * hkv, num_kv_heads=hkv, head_dim=d, block_k=8,
                 context=300, page_size=16, paging="shuffled", steps=(T + 7) // 8 + 1)
    cache = make_cache(w, seq_lens=_lens(batch, 8500 + g))
    rng = np.random.default_rng(8600 + g)
    new_lens = rng.integers(0, T + 1, size=batch).astype(np.int32)
    new_lens[:3] = (T, 0, 1)
    q, kn, vn = _new_tokens(w, T, 8700 + g)
    ref_k, ref_v, ref_l = cache["k_pool"].copy(), cache["v_pool"].copy(), cache["seq_lens"].copy()
    want, _ = oracle.prefill_attn(w.sm_scale, q, kn, vn, new_lens, ref_k, ref_v, cache["page_table"], ref_l)
    msl = int(cache["seq_lens"].max()) + T
    assert prefill_waves(d, g, batch * hkv, T, msl) == (2 if batch < 20 and d == 128 else 4)
    case = Case(w, cache, max_seq_len=msl)
    got = case.prefill(q, kn, vn, new_lens)
    _check(got, want, new_lens)
    k, v, l = case.state()
    np.testing.assert_array_equal(l, ref_l)
    np.testing.assert_array_equal(k, ref_k)
    np.testing.assert_array_equal(v, ref_v)
    assert case.step.device_error() == 0
    case.step.close()


@pytest.mark.parametrize("batch,hkv,K", [(2, 2, 8), (64, 8, 32)])
def test_pool_strides_past_32_bit_byte_arithmetic(batch, hkv, K):
    """Pages of 2^23 tokens (only their first rows exist): an in-page offset no longer fits the kernels' 32-bit byte
    arithmetic, which their general address form has to take over, in both attention kernels."""
    d, rows, L = 128, 320, 290
    assert decode_is_wide(d, 4 * K, BOUND, batch * hkv) == (batch == 64)
    w = Workload(name="huge", seed=8800 + batch, batch=batch, num_q_heads=4 * hkv, num_kv_heads=hkv, head_dim=d, block_k=K,
                 context=L, page_size=rows, paging="contiguous", steps=0)
    lens = _lens(batch, 8900)
    rng = np.random.default_rng(8901)
    mk = lambda *s: (rng.standard_normal(s, dtype=np.float32).view(np.uint32) >> 16).astype(np.uint16)
    k_pool, v_pool = mk(batch, hkv, rows, d), mk(batch, hkv, rows, d)
    cache = dict(k_pool=k_pool, v_pool=v_pool, page_table=np.arange(batch, dtype=np.int32)[:, None], seq_lens=np.minimum(lens, L))
    blk = make_block(w, 8902)
    from paper_2605_12825_amd import runtime as rt
    import torch
    step = rt.DecodeStep(batch=batch, num_q_heads=4 * hkv, num_kv_heads=hkv, head_dim=d, block_k=K, page_size=1 << 23,
                         max_pages_per_seq=1, max_seq_len=BOUND, num_pages=batch, pool_strides=(0, hkv * rows * d, rows * d, d))
    D = rt.to_device_bits
    out = torch.zeros((batch, K, 4 * hkv, d), dtype=torch.int16, device="cuda")
    step.attn(AR, D(blk["q"]), D(blk["k_blk"]), D(blk["v_blk"]), D(k_pool), D(v_pool), D(cache["page_table"]),
              D(cache["seq_lens"]), out)
    torch.cuda.synchronize()
    got = bf16_bits_to_f32(rt.bits_to_numpy(out)).astype(np.float64)
    _check_attn(got, _oracle_attn(AR, w, blk, cache))
    assert step.device_error() == 0
    step.close()


def _wider(q):
    return f32_to_bf16_bits(np.float32(2.0) * bf16_bits_to_f32(q))


@pytest.mark.parametrize("g,K,hkv,batch,d", [(4, 32, 8, 64, 128), (8, 32, 4, 80, 128), (7, 32, 4, 96, 64), (8, 16, 8, 96, 64)])
def test_decode_bits_do_not_depend_on_the_batch_size(g, K, hkv, batch, d):
    """A sequence that is not split gets the same bits in a batch that fills the chip (64 rows per wave) and alone (32
    rows): both kernels move a row's softmax reference by the same rule.  Scores of twice the usual size and
    short first tiles, so that references move."""
    w = Workload(name="bits", seed=9000 + g * K + d, batch=batch, num_q_heads=g * hkv, num_kv_heads=hkv, head_dim=d,
                 block_k=K, context=300, page_size=16, paging="scattered")
    cache, blk = make_cache(w, seq_lens=_lens(batch, 9001)), make_block(w, 9002)
    blk["q"] = _wider(blk["q"])
    case = _case(w, cache, True)
    got = case.attn(DIFF, blk, want_lse=False)
    _check_attn(got, _oracle_attn(DIFF, w, blk, cache))
    case.step.close()
    for b in range(0, batch, 2):
        few = _case(replace(w, batch=2), dict(cache, page_table=cache["page_table"][b:b + 2], seq_lens=cache["seq_lens"][b:b + 2]),
                    False, num_splits=1)
        part = few.attn(DIFF, {x: blk[x][b:b + 2] for x in blk}, want_lse=False)
        np.testing.assert_array_equal(part, got[b:b + 2], err_msg="sequences %d, %d" % (b, b + 1))
        few.step.close()


@pytest.mark.parametrize("g,batch,T", [(4, 64, 70), (1, 70, 40)])
def test_prefill_bits_do_not_depend_on_the_batch_size(g, batch, T):
    """The same for prefill, where the chunks of both forms start at whole 32-row blocks."""
    w = Workload(name="bitsp", seed=9100 + g, batch=batch, num_q_heads=g * 8, num_kv_heads=8, head_dim=128, block_k=8,
                 context=300, page_size=16, paging="shuffled", steps=(T + 7) // 8 + 1)
    cache = make_cache(w, seq_lens=_lens(batch, 9101))
    new_lens = np.random.default_rng(9102).integers(1, T + 1, size=batch).astype(np.int32)
    q, kn, vn = _new_tokens(w, T, 9103)
    q = _wider(q)
    msl = int(cache["seq_lens"].max()) + T
    assert prefill_waves(128, g, batch * 8, T, msl) == 4 and prefill_waves(128, g, 16, T, msl) == 0
    case = Case(w, cache, max_seq_len=msl)
    got = case.prefill(q, kn, vn, new_lens)
    case.step.close()
    for b in range(0, batch, 2):
        few = Case(replace(w, batch=2), dict(cache, page_table=cache["page_table"][b:b + 2], seq_lens=cache["seq_lens"][b:b + 2]), msl)
        part = few.prefill(q[b:b + 2], kn[b:b + 2], vn[b:b + 2], new_lens[b:b + 2])
        np.testing.assert_array_equal(part, got[b:b + 2], err_msg="sequences %d, %d" % (b, b + 1))
        few.step.close()


def _check_with_infinities(got, want):
    """Infinities where the 64-bit result has them and nowhere else; everything finite within the usual bars."""
    fin = np.isfinite(want)
    assert not fin.all()
    np.testing.assert_array_equal(got[~fin], want[~fin])
    _check_attn(np.where(fin, got, 0.0), np.where(fin, want, 0.0))


@pytest.mark.parametrize("batch", [2, 96])                        # the 32-row kernel, the 64-row kernel
@pytest.mark.parametrize("g,K,hkv,d", [(4, 32, 8, 128), (8, 32, 4, 128), (8, 16, 8, 64)])
def test_infinite_value_in_the_first_tile_stays_infinite(batch, g, K, hkv, d):
    """An infinite V in a sequence's first 32 tokens, or in its block when the cache is empty, makes its column infinite
    for every row that sees it: zero weights of a pipeline that is still filling must not meet it."""
    lens = np.where(np.arange(batch) % 2, 32 + 37 * (np.arange(batch) % 8), 0).astype(np.int32)
    w = Workload(name="inf", seed=9200 + d + g, batch=batch, num_q_heads=g * hkv, num_kv_heads=hkv, head_dim=d, block_k=K,
                 context=300, page_size=16, paging="shuffled")
    cache, blk = make_cache(w, seq_lens=lens), make_block(w, 9201)
    for b in range(batch):
        bits, head, col = (0x7F80, 0xFF80)[b // 2 % 2], b % hkv, (7 * b) % d
        if lens[b]:
            cache["v_pool"][cache["page_table"][b, b % 2], head, b % 16, col] = bits
        else:
            blk["v_blk"][b, 0, head, col] = bits
    case = _case(w, cache, batch > 2)
    _check_with_infinities(case.attn(DIFF, blk, want_lse=False), _oracle_attn(DIFF, w, blk, cache))
    case.step.close()


@pytest.mark.parametrize("batch", [2, 64])
def test_infinite_value_in_the_first_tile_stays_infinite_in_prefill(batch):
    T, hkv, d = 70, 8, 128
    w = Workload(name="infp", seed=9300, batch=batch, num_q_heads=4 * hkv, num_kv_heads=hkv, head_dim=d, block_k=8, context=300,
                 page_size=16, paging="shuffled", steps=(T + 7) // 8 + 1)
    cache = make_cache(w, seq_lens=(32 + 45 * (np.arange(batch) % 5)).astype(np.int32))
    for b in range(batch):
        cache["v_pool"][cache["page_table"][b, b % 2], b % hkv, b % 16, (7 * b) % d] = 0x7F80
    q, kn, vn = _new_tokens(w, T, 9301)
    new_lens = np.full(batch, T, np.int32)
    ref = [cache[x].copy() for x in ("k_pool", "v_pool", "seq_lens")]
    want, _ = oracle.prefill_attn(w.sm_scale, q, kn, vn, new_lens, ref[0], ref[1], cache["page_table"], ref[2])
    msl = int(cache["seq_lens"].max()) + T
    assert prefill_waves(d, 4, batch * hkv, T, msl) == (4 if batch > 2 else 0)
    case = Case(w, cache, max_seq_len=msl)
    _check_with_infinities(bf16_bits_to_f32(case.prefill(q, kn, vn, new_lens)).astype(np.float64), want)
    case.step.close()


def test_caches_of_their_own_stream_past_the_last_level_cache():
    """The non-temporal form of the tile loads (a model whose layers' caches together outgrow the last-level cache) gives
    the same bits, for every width and head size."""
    for g, K, hkv, batch, d in ((4, 32, 8, 64, 128), (8, 32, 4, 80, 128), (8, 16, 8, 96, 64), (8, 31, 4, 64, 64)):
        w = Workload(name="nt", seed=9400 + K + d, batch=batch, num_q_heads=g * hkv, num_kv_heads=hkv, head_dim=d, block_k=K,
                     context=300, page_size=16, paging="scattered")
        cache, blk = make_cache(w, seq_lens=_lens(batch, 9401)), make_block(w, 9402)
        layers = 2 + int(1.25 * 2**28) // (4 * cache["k_pool"].size)   # K and V: 4 bytes per element of one pool
        plain, streamed = _case(w, cache, True), _case(w, cache, True, num_layers=layers)
        got = plain.attn(AR, blk, want_lse=False)
        _check_attn(got, _oracle_attn(AR, w, blk, cache))
        np.testing.assert_array_equal(streamed.attn(AR, blk, want_lse=False), got)
        plain.step.close()
        streamed.step.close()


@pytest.mark.parametrize("g,K,hkv,batch,d", [(4, 32, 8, 64, 128), (8, 31, 4, 64, 64)])
def test_block_inputs_read_in_place(g, K, hkv, batch, d):
    """q, k_blk and v_blk as column ranges of one fused projection output: the bits of dense inputs."""
    from paper_2605_12825_amd import runtime as rt
    import torch
    w = Workload(name="fusedw", seed=9500 + d, batch=batch, num_q_heads=g * hkv, num_kv_heads=hkv, head_dim=d, block_k=K,
                 context=300, page_size=16, paging="scattered")
    cache, blk = make_cache(w, seq_lens=_lens(batch, 9501)), make_block(w, 9502)
    case = _case(w, cache, True)
    want = case.attn(AR, blk, want_lse=False)
    fused = np.concatenate([blk[x].reshape(batch * K, -1, d) for x in ("q", "k_blk", "v_blk")], axis=1)
    row = fused.shape[1] * d
    step = rt.DecodeStep(batch=batch, num_q_heads=g * hkv, num_kv_heads=hkv, head_dim=d, block_k=K, page_size=16,
                         max_pages_per_seq=BOUND // 16, max_seq_len=BOUND, num_pages=cache["k_pool"].shape[0],
                         block_strides=(row, d, row, d, batch * K * row))
    buf, at = rt.to_device_bits(fused), lambda h: h * d * 2
    out = torch.zeros((batch, K, g * hkv, d), dtype=torch.int16, device="cuda")
    base = buf.data_ptr()
    step.attn(AR, base, base + at(g * hkv), base + at((g + 1) * hkv), case.k_pool, case.v_pool, case.page_table, case.seq_lens, out)
    torch.cuda.synchronize()
    np.testing.assert_array_equal(bf16_bits_to_f32(rt.bits_to_numpy(out)).astype(np.float64), want)
    step.close()
    case.step.close()


@pytest.mark.parametrize("g,K,hkv,batch,d", [(4, 32, 8, 64, 128), (8, 31, 4, 64, 64)])
def test_bad_pages_and_lengths_are_flagged_and_stay_with_their_sequence(g, K, hkv, batch, d):
    """A page id outside the pool in the first, a middle or the last, ragged tile, or a length outside [0, bound]: the error
    word is set, every other sequence keeps its bits."""
    w = Workload(name="bad", seed=9600 + d, batch=batch, num_q_heads=g * hkv, num_kv_heads=hkv, head_dim=d, block_k=K,
                 context=300, page_size=16, paging="scattered")
    lens = np.full(batch, 290, np.int32)
    cache, blk = make_cache(w, seq_lens=lens), make_block(w, 9601)
    case = _case(w, cache, True)
    want = case.attn(DIFF, blk, want_lse=False)
    assert case.step.device_error() == 0
    case.step.close()
    for b, slot, page, length in ((3, 0, -1, 290), (5, 7, cache["k_pool"].shape[0], 290), (9, 18, 1 << 30, 290), (11, 0, None, -1),
                                  (batch - 1, 0, None, BOUND + 1)):
        bad = dict(cache, page_table=cache["page_table"].copy(), seq_lens=lens.copy())
        if page is not None:
            bad["page_table"][b, slot] = page
        bad["seq_lens"][b] = length
        case = _case(w, bad, True)
        got = case.attn(DIFF, blk, want_lse=False)
        assert case.step.device_error() == -4, (b, slot, page, length)
        rest = np.arange(batch) != b
        np.testing.assert_array_equal(got[rest], want[rest])
        case.step.close()


def test_prefill_capacity_error_stays_with_its_sequence():
    """New tokens that fall on an unmapped page leave their sequence alone (cache, length, output); a bad page among the
    cached ones is flagged; the other sequences are as without either."""
    g, hkv, batch, d, T = 4, 8, 64, 128, 70
    w = Workload(name="badp", seed=9700, batch=batch, num_q_heads=g * hkv, num_kv_heads=hkv, head_dim=d, block_k=8, context=300,
                 page_size=16, paging="shuffled", steps=(T + 7) // 8 + 1)
    cache = make_cache(w, seq_lens=np.full(batch, 200, np.int32))
    new_lens = np.full(batch, T, np.int32)
    q, kn, vn = _new_tokens(w, T, 9701)
    msl = 200 + T
    assert prefill_waves(d, g, batch * hkv, T, msl) == 4
    case = Case(w, cache, max_seq_len=msl)
    want = case.prefill(q, kn, vn, new_lens)
    case.step.close()
    bad = dict(cache, page_table=cache["page_table"].copy())
    bad["page_table"][4, 16] = -1                              # position 256 of sequence 4: its 57th new token
    bad["page_table"][6, 3] = cache["k_pool"].shape[0] + 7     # cached positions of sequence 6
    case = Case(w, bad, max_seq_len=msl)
    got = case.prefill(q, kn, vn, new_lens)
    assert case.step.device_error() == -4
    rest = ~np.isin(np.arange(batch), (4, 6))
    np.testing.assert_array_equal(got[rest], want[rest])
    assert (got[4] == SENTINEL).all()
    k, v, lens = case.state()
    np.testing.assert_array_equal(lens, np.where(np.arange(batch) == 4, 200, 200 + T))
    own = cache["page_table"][4][cache["page_table"][4] >= 0]
    np.testing.assert_array_equal(k[own], cache["k_pool"][own])
    np.testing.assert_array_equal(v[own], cache["v_pool"][own])
    case.step.close()


# a wave keeps the addresses of 64 tiles at a time: lengths around one and two such windows, ring turns (4 and 6 tiles) apart
WINDOWS = [2016, 2047, 2048, 2079, 2112, 2143, 2175, 2240, 4050]


@pytest.mark.parametrize("g,K,hkv,batch,d,page", [(4, 32, 8, 64, 128, 16), (8, 32, 4, 80, 128, 64), (8, 31, 4, 64, 64, 32)])
def test_decode_past_a_window_of_addresses(g, K, hkv, batch, d, page):
    w = Workload(name="window", seed=9800 + d, batch=batch, num_q_heads=g * hkv, num_kv_heads=hkv, head_dim=d, block_k=K,
                 context=300, page_size=page, paging="scattered")
    lens = np.full(batch, 5, np.int32)
    lens[:len(WINDOWS)] = WINDOWS
    cache, blk = make_cache(w, seq_lens=lens), make_block(w, 9801)
    case = _case(w, cache, True)
    _check_attn(case.attn(AR, blk, want_lse=False), _oracle_attn(AR, w, blk, cache))
    assert case.step.device_error() == 0
    case.step.close()


@pytest.mark.parametrize("g,d,page", [(7, 128, 16), (5, 128, 64), (8, 64, 32)])
def test_prefill_past_a_window_of_addresses(g, d, page):
    """Against the oracle with two waves (four for d = 64); with four of d = 128, which take a batch that fills the chip,
    the same bits."""
    T, hkv = 51, 1
    w = Workload(name="windowp", seed=9900 + g, batch=len(WINDOWS), num_q_heads=g, num_kv_heads=hkv, head_dim=d, block_k=8,
                 context=300, page_size=page, paging="shuffled", steps=(T + 7) // 8 + 1)
    cache = make_cache(w, seq_lens=np.array(WINDOWS, np.int32))
    new_lens = np.array([T, 1, 25, 26, T, 32, 33, T, 50], np.int32)
    q, kn, vn = _new_tokens(w, T, 9901)
    ref = [cache[x].copy() for x in ("k_pool", "v_pool", "seq_lens")]
    want, _ = oracle.prefill_attn(w.sm_scale, q, kn, vn, new_lens, ref[0], ref[1], cache["page_table"], ref[2])
    msl = max(WINDOWS) + T
    assert prefill_waves(d, g, w.batch, T, msl) == (2 if d == 128 else 4)
    case = Case(w, cache, max_seq_len=msl)
    got = case.prefill(q, kn, vn, new_lens)
    _check(got, want, new_lens)
    np.testing.assert_array_equal(case.state()[0], ref[0])
    case.step.close()
    if g != 5:
        return
    rep = 20                                      # 180 sequences: copies of these nine, which share the cached pages
    assert prefill_waves(d, g, rep * w.batch, T, msl) == 4
    tile = lambda x: np.concatenate([x] * rep)
    pages, slots = cache["page_table"].copy(), cache["page_table"].shape[1]
    own = [np.arange(L // page, (L + T - 1) // page + 1) for L in WINDOWS]   # pages that the new tokens write
    pt, k, v = [pages], [cache["k_pool"]], [cache["v_pool"]]
    at = cache["k_pool"].shape[0]
    for r in range(1, rep):
        p = pages.copy()
        for b, s in enumerate(own):
            k.append(cache["k_pool"][pages[b, s]]), v.append(cache["v_pool"][pages[b, s]])
            p[b, s] = np.arange(at, at + len(s))
            at += len(s)
        pt.append(p)
    big = dict(cache, k_pool=np.concatenate(k), v_pool=np.concatenate(v), page_table=np.concatenate(pt), seq_lens=tile(cache["seq_lens"]))
    case = Case(replace(w, batch=rep * w.batch), big, max_seq_len=msl)
    np.testing.assert_array_equal(case.prefill(tile(q), tile(kn), tile(vn), tile(new_lens)), tile(got))
    case.step.close()
