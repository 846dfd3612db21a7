"""Calls of at most 16 query rows per KV head (the attention kernel's 16-row form) against the oracle: every count of rows
at which a lane's row, block row and head change, lengths on both sides of the tile and ring edges, every way of cutting."""
from dataclasses import replace

import numpy as np
import pytest

from orthrus_inputs import Workload, make_block, make_cache

from test_gpu_parity import AR, DIFF, GpuCase, _check_attn, _oracle_attn

EDGES = [0, 1, 15, 16, 17, 31, 32, 33, 63, 64, 65, 96, 97, 128, 129, 200, 300]


@pytest.mark.gpu
@pytest.mark.parametrize("splits", [0, 1, 3, 7, -1])
@pytest.mark.parametrize("g,K,d,page", [(1, 1, 128, 16), (1, 16, 128, 16), (4, 4, 128, 32), (5, 3, 128, 16), (2, 8, 64, 16),
                                        (16, 1, 64, 64), (3, 5, 64, 16)])
def test_up_to_16_rows(g, K, d, page, splits):
    hkv, batch = 2, len(EDGES)
    w = Workload(name="thin", seed=9600 + g * K + d, batch=batch, num_q_heads=g * hkv, num_kv_heads=hkv, head_dim=d, block_k=K,
                 context=300, page_size=page, paging="scattered")
    cache = make_cache(w, seq_lens=np.random.default_rng(9700 + K).permutation(EDGES).astype(np.int32))
    blk = make_block(w, 9800 + K)
    case = GpuCase(w, cache, num_splits=splits)
    for view in (DIFF, AR):
        got, lse = case.attn(view, blk)
        want, want_lse = _oracle_attn(view, w, blk, cache, want_lse=True)
        _check_attn(got, want)
        np.testing.assert_allclose(lse, want_lse, rtol=0, atol=2e-3)
    assert case.step.device_error() == 0
    case.step.close()


@pytest.mark.gpu
@pytest.mark.parametrize("d", [64, 128])
def test_unsplit_rows_have_the_same_bits_in_every_launch(d):
    """In a batch whose items start by size, and alone."""
    g, K, hkv, batch = 2, 8, 8, 200
    w = Workload(name="thinb", seed=9900 + d, batch=batch, num_q_heads=g * hkv, num_kv_heads=hkv, head_dim=d, block_k=K, context=100,
                 page_size=16, paging="scattered")
    lens = np.random.default_rng(9901).integers(0, 101, batch).astype(np.int32)
    cache, blk = make_cache(w, seq_lens=lens), make_block(w, 9902)
    whole = GpuCase(w, cache, num_splits=1)
    got, lse = whole.attn(AR, blk)
    whole.step.close()
    for b in (0, 77, batch - 1):
        one = replace(w, batch=1)
        case = GpuCase(one, dict(cache, page_table=cache["page_table"][b:b + 1].copy(), seq_lens=lens[b:b + 1].copy()), num_splits=1)
        o, l = case.attn(AR, {k: v[b:b + 1].copy() for k, v in blk.items()})
        np.testing.assert_array_equal(o[0], got[b])
        np.testing.assert_array_equal(l[0], lse[b])
        case.step.close()
