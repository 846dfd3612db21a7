"""Calls of at most 16 query rows per KV head (the attention kernel's 16-row form) against the oracle: every count of rows
at which a lane's row, block row and head change, lengths on both sides of the tile and ring edges, every way of cutting."""
from dataclasses import replace

import numpy as np
import pytest

from orthrus_inputs import Workload, bf16_bits_to_f32, make_block, make_cache

from test_gpu_parity import AR, DIFF, GpuCase, _check_attn, _oracle_attn
from test_gpu_wide import _check_with_infinities

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


def _some(g, K, d, lens, seed, page=16):
    w = Workload(name="thins", seed=seed, batch=len(lens), num_q_heads=g * 2, num_kv_heads=2, head_dim=d, block_k=K, context=300,
                 page_size=page, paging="scattered")
    return w, make_cache(w, seq_lens=np.asarray(lens, np.int32)), make_block(w, seed + 1)


@pytest.mark.gpu
@pytest.mark.parametrize("splits", [1, 3, -1])
@pytest.mark.parametrize("g,K,d", [(4, 4, 128), (2, 7, 64)])
def test_non_temporal_loads_give_the_same_bits(g, K, d, splits):
    w, cache, blk = _some(g, K, d, EDGES, 10000 + d)
    plain, streamed = (GpuCase(w, cache, num_splits=splits, num_layers=n) for n in (1, 1000))
    for view in (DIFF, AR):
        got, lse = plain.attn(view, blk)
        _check_attn(got, _oracle_attn(view, w, blk, cache))
        again, lse2 = streamed.attn(view, blk)
        np.testing.assert_array_equal(again, got)
        np.testing.assert_array_equal(lse2, lse)
    plain.step.close()
    streamed.step.close()


@pytest.mark.gpu
@pytest.mark.parametrize("splits", [1, 3, -1])
@pytest.mark.parametrize("g,K,d", [(4, 4, 128), (2, 7, 64)])
def test_block_inputs_read_in_place(g, K, d, splits):
    """q, k_blk and v_blk as column ranges of one fused projection output: the bits of dense inputs."""
    from paper_2605_12825_amd import runtime as rt
    import torch
    w, cache, blk = _some(g, K, d, EDGES, 10100 + d)
    batch, hkv = w.batch, w.num_kv_heads
    case = GpuCase(w, cache, num_splits=splits)
    fused = np.concatenate([blk[x].reshape(batch * K, -1, d) for x in ("q", "k_blk", "v_blk")], axis=1)
    row = fused.shape[1] * d
    step = rt.DecodeStep(batch=batch, num_q_heads=g * hkv, num_kv_heads=hkv, head_dim=d, block_k=K, page_size=16,
                         max_pages_per_seq=cache["page_table"].shape[1], max_seq_len=max(EDGES), num_pages=cache["k_pool"].shape[0],
                         num_splits=splits, block_strides=(row, d, row, d, batch * K * row))
    buf = rt.to_device_bits(fused)
    base, at = buf.data_ptr(), lambda h: h * d * 2
    out = torch.zeros((batch, K, g * hkv, d), dtype=torch.int16, device="cuda")
    for view in (DIFF, AR):
        want = case.attn(view, blk, want_lse=False)
        step.attn(view, base, base + at(g * hkv), base + at((g + 1) * hkv), case.k_pool, case.v_pool, case.page_table, case.seq_lens, out)
        torch.cuda.synchronize()
        np.testing.assert_array_equal(bf16_bits_to_f32(rt.bits_to_numpy(out)).astype(np.float64), want)
    step.close()
    case.step.close()


@pytest.mark.gpu
@pytest.mark.parametrize("splits", [1, 3, -1])
def test_strides_past_32_bit_byte_arithmetic(splits):
    """Pages of 2^23 tokens (only their first rows exist) and block rows 2^25 values apart: the general address forms."""
    from paper_2605_12825_amd import runtime as rt
    import torch
    g, K, d, hkv, lens, rows, apart = 4, 3, 128, 2, [290, 65, 0], 320, 1 << 25
    w = Workload(name="huge", seed=10200, batch=3, num_q_heads=g * hkv, num_kv_heads=hkv, head_dim=d, block_k=K, context=300,
                 page_size=rows, paging="contiguous", steps=0)
    rng = np.random.default_rng(10201)
    mk = lambda *s: (rng.standard_normal(s, dtype=np.float32).view(np.uint32) >> 16).astype(np.uint16)
    k_pool, v_pool = mk(3, hkv, rows, d), mk(3, hkv, rows, d)
    cache = dict(k_pool=k_pool, v_pool=v_pool, page_table=np.arange(3, dtype=np.int32)[:, None], seq_lens=np.asarray(lens, np.int32))
    blk = make_block(w, 10202)
    step = rt.DecodeStep(batch=3, num_q_heads=g * hkv, num_kv_heads=hkv, head_dim=d, block_k=K, page_size=1 << 23, max_pages_per_seq=1,
                         max_seq_len=300, num_pages=3, num_splits=splits, pool_strides=(0, hkv * rows * d, rows * d, d),
                         block_strides=(g * hkv * d, d, apart, d, 9 * apart))
    D = rt.to_device_bits
    sparse = torch.zeros(8 * apart + 2 * hkv * d, dtype=torch.int16, device="cuda")   # row r at r * apart: keys, then values
    for r in range(9):
        sparse[r * apart:r * apart + 2 * hkv * d] = D(np.concatenate((blk["k_blk"][r // K, r % K], blk["v_blk"][r // K, r % K]))).reshape(-1)
    out = torch.zeros((3, K, g * hkv, d), dtype=torch.int16, device="cuda")
    for view in (DIFF, AR):
        step.attn(view, D(blk["q"]), sparse, sparse[hkv * d:], D(k_pool), D(v_pool), D(cache["page_table"]), D(cache["seq_lens"]), out)
        torch.cuda.synchronize()
        _check_attn(bf16_bits_to_f32(rt.bits_to_numpy(out)).astype(np.float64), _oracle_attn(view, w, blk, cache))
    assert step.device_error() == 0
    step.close()


@pytest.mark.gpu
@pytest.mark.parametrize("g,K,d", [(4, 4, 128), (2, 8, 64)])
def test_infinite_value_in_the_first_tile_stays_infinite(g, K, d):
    lens = 32 + 37 * (np.arange(8) % 8)
    w, cache, blk = _some(g, K, d, lens, 10300 + d)
    for b in range(8):
        cache["v_pool"][cache["page_table"][b, b % 2], b % 2, b % 16, (7 * b) % d] = (0x7F80, 0xFF80)[b // 2 % 2]
    case = GpuCase(w, cache, num_splits=1)
    _check_with_infinities(case.attn(DIFF, blk, want_lse=False), _oracle_attn(DIFF, w, blk, cache))
    case.step.close()


@pytest.mark.gpu
@pytest.mark.parametrize("splits", [1, 3, -1])
def test_bad_pages_and_lengths_are_flagged_and_stay_with_their_sequence(splits):
    """A page id outside the pool is read as page 0, a length outside the bound as 0 or the bound."""
    w, cache, blk = _some(4, 4, 128, [290] * 6, 10400)
    pages = cache["k_pool"].shape[0]
    for b, slot, page, length in ((0, 0, -1, 290), (2, 7, pages, 290), (5, 18, 1 << 30, 290), (3, 0, None, -1), (5, 0, None, 2 ** 31 - 1)):
        bad = dict(cache, page_table=cache["page_table"].copy(), seq_lens=cache["seq_lens"].copy())
        read = dict(cache, page_table=cache["page_table"].copy())
        if page is not None:
            bad["page_table"][b, slot], read["page_table"][b, slot] = page, 0
        bad["seq_lens"][b] = length
        case = GpuCase(w, bad, num_splits=splits, max_seq_len=290)
        got = case.attn(AR, blk, want_lse=False)
        _check_attn(got, _oracle_attn(AR, w, blk, read, seq_lens=np.clip(bad["seq_lens"], 0, 290)))
        assert case.step.device_error() == -4, (b, slot, page, length)
        case.step.close()
