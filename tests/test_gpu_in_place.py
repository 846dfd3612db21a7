"""Consensus and commit with out_tokens written over draft_tokens, for several layers: every layer's workgroup commits by
the same decision, whatever the order in which the tokens replace the drafts.  Results are the oracle's, bit for bit.
Pages run out inside the block of some sequences, so that a layer that counted one more row would append none, and too
early in others, which are left alone."""
import numpy as np
import pytest
import torch

import oracle
from orthrus_inputs import Workload, make_block, make_cache, make_consensus_case

from test_gpu_sampling import _clear_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("temperature", [0.0, 0.9])
@pytest.mark.parametrize("batch,K,layers", [(1, 4, 1), (1, 4, 36), (9, 16, 1), (9, 16, 3), (24, 32, 36),
                                            (71, 2, 36), (72, 3, 36)])      # either side of the copy as its own launch
def test_tokens_replace_the_drafts_in_place(batch, K, temperature, layers):
    from paper_2605_12825_amd import runtime as rt
    w = Workload(name="inplace", seed=9700 + K, batch=batch, num_q_heads=4, num_kv_heads=2, head_dim=64, block_k=K,
                 context_range=(0, 50), page_size=16, paging="shuffled", vocab=700, accept="uniform", steps=1)
    lens = make_cache(w)["seq_lens"]
    cache = [make_cache(w, seed=9710 + l, seq_lens=lens) for l in range(layers)]
    kp, vp = np.stack([c["k_pool"] for c in cache]), np.stack([c["v_pool"] for c in cache])
    pt = cache[0]["page_table"]
    blk = [make_block(w, 9750 + l) for l in range(layers)]
    kb, vb = np.stack([x["k_blk"] for x in blk]), np.stack([x["v_blk"] for x in blk])
    # every other sequence has pages for exactly the rows that it appends
    c = _clear_case(w, 9790, temperature=temperature)[0] if temperature else make_consensus_case(w, 9790)
    D = rt.to_device_bits

    def oracle_call(k, v, l, table):
        if temperature:
            return oracle.sampling_consensus_commit(c["ar_logits"], c["diff_logits"], c["draft_tokens"], c["accept_u"], c["gumbel"],
                                                    temperature, kb, vb, k, v, table, l)
        return oracle.consensus_commit(c["ar_logits"], c["draft_tokens"], kb, vb, k, v, table, l)

    rk, rv, rl = kp.copy(), vp.copy(), lens.copy()
    want = oracle_call(rk, rv, rl, pt)
    m = want["num_committed"].copy()
    table = pt.copy()
    for b in range(0, batch, 2):
        table[b, (lens[b] + m[b] + 15) // 16:] = -1
    for b in range(7, batch, 8):
        table[b, (lens[b] + m[b] - 1) // 16] = -1
        own = pt[b][pt[b] >= 0]
        rk[:, own], rv[:, own], rl[b], want["num_committed"][b] = kp[:, own], vp[:, own], lens[b], 0
    step = rt.DecodeStep(batch=batch, num_q_heads=4, num_kv_heads=2, head_dim=64, block_k=K, page_size=16,
                         max_pages_per_seq=pt.shape[1], max_seq_len=16 * pt.shape[1], num_pages=kp.shape[1], vocab=700,
                         num_layers=layers)
    for _ in range(3):
        dk, dv, dl, tok = D(kp), D(vp), D(lens), D(c["draft_tokens"])
        acc, ncm, anc = (torch.full((batch,), -7, dtype=torch.int32, device="cuda") for _ in range(3))
        rest = (D(kb), D(vb), dk, dv, D(table), dl, acc, ncm, tok, anc)
        if temperature:
            step.sampling_consensus_commit(temperature, D(c["ar_logits"]), D(c["diff_logits"]), tok, D(c["accept_u"]),
                                           D(c["gumbel"]), *rest)
        else:
            step.consensus_commit(D(c["ar_logits"]), tok, *rest)
        torch.cuda.synchronize()
        assert step.device_error() == (-4 if batch > 7 else 0)
        for name, got in (("accept_len", acc), ("num_committed", ncm), ("out_tokens", tok), ("next_anchor", anc)):
            np.testing.assert_array_equal(got.cpu().numpy(), want[name], err_msg=name)
        np.testing.assert_array_equal(dl.cpu().numpy(), rl)
        np.testing.assert_array_equal(rt.bits_to_numpy(dk), rk)
        np.testing.assert_array_equal(rt.bits_to_numpy(dv), rv)
    step.close()
