"""Split attention calls: pieces of every length against the oracle, and what a result's bits depend on (the split count and
the sequence's own data, nothing around them)."""
from dataclasses import replace

import numpy as np
import pytest

from orthrus_inputs import Workload, make_block, make_cache

from test_gpu_parity import AR, DIFF, GpuCase, _check_attn, _oracle_attn

OTHERS = [900, 0, 33, 1, 410, 64]


def _pieces(bound, splits):
    """How many pieces the library makes of `splits` under a host bound: whole tiles of 32 tokens."""
    chunk = -(-(-(-bound // splits)) // 32) * 32
    return -(-bound // chunk)


@pytest.mark.gpu
@pytest.mark.parametrize("g,K,d,hkv,splits,length", [
    (4, 4, 128, 8, 13, 4096), (4, 8, 128, 8, 13, 4096), (4, 16, 128, 8, 13, 4096), (7, 8, 128, 4, 20, 6400), (5, 16, 128, 4, 3, 4096),
    (4, 32, 128, 4, 3, 4096), (7, 32, 128, 2, 4, 4096), (2, 8, 64, 4, 8, 2048), (2, 16, 64, 4, 8, 2048), (4, 16, 64, 4, 8, 2048),
    (4, 32, 64, 4, 4, 2048),
])
def test_a_fixed_split_count_gives_the_same_bits_in_every_launch(g, K, d, hkv, splits, length):
    """Alone, alone under a looser bound that is cut into as many pieces, as one of many layers, and in batches whose
    pieces fit the chip or wait for others."""
    w = Workload(name="bits", seed=10500 + g * K + d, batch=1, num_q_heads=g * hkv, num_kv_heads=hkv, head_dim=d, block_k=K, context=length,
                 page_size=16, paging="scattered")
    batch = max(7, 1 + 1600 // (hkv * splits))
    lens = np.array(([length] + OTHERS * batch)[:batch], np.int32)
    many = replace(w, batch=batch)
    cache, blk = make_cache(many, seq_lens=lens), make_block(many, w.seed + 1)
    loose = max(b for b in range(length, 2 * length, 32) if _pieces(b, splits) == splits)
    table = np.zeros((batch, loose // 16), np.int32)   # as long as the loose bound needs it
    table[:, :cache["page_table"].shape[1]] = cache["page_table"]

    def call(n, bound, layers):
        case = GpuCase(replace(w, batch=n), dict(cache, page_table=table[:n].copy(), seq_lens=lens[:n].copy()),
                       num_splits=splits, num_layers=layers, max_seq_len=bound)
        assert case.step.num_splits == splits
        got = [case.attn(view, {k: v[:n].copy() for k, v in blk.items()}) for view in (DIFF, AR)]
        assert case.step.device_error() == 0
        case.step.close()
        return got

    base = call(1, length, 1)
    for view in (DIFF, AR):
        one = replace(w, batch=1)
        want = _oracle_attn(view, one, {k: v[:1] for k, v in blk.items()}, dict(cache, page_table=cache["page_table"][:1], seq_lens=lens[:1]))
        _check_attn(base[view][0], want)
    for n, bound, layers in ((1, loose, 1), (1, length, 1000), (2, length, 1), (3, loose, 1), (7, length, 1), (batch, length, 1), (batch, length, 1000)):
        for view, (got, lse) in enumerate(call(n, bound, layers)):
            np.testing.assert_array_equal(got[0], base[view][0][0], err_msg=str((n, bound, layers, view)))
            np.testing.assert_array_equal(lse[0], base[view][1][0], err_msg=str((n, bound, layers, view)))


def _short(g, K, d, hi, lens, seed, page=16):
    w = Workload(name="pieces", seed=seed, batch=len(lens), num_q_heads=g * 2, num_kv_heads=2, head_dim=d, block_k=K, context=hi,
                 page_size=page, paging="scattered")
    return w, make_cache(w, seq_lens=np.asarray(lens, np.int32)), make_block(w, seed + 1)


@pytest.mark.gpu
@pytest.mark.parametrize("g,K,d,splits,hi,page", [
    (4, 5, 128, 2, 500, 16), (4, 8, 128, 3, 700, 32), (4, 16, 128, 2, 600, 64), (7, 5, 128, 3, 900, 16), (4, 32, 128, 2, 2560, 16),
    (7, 14, 128, 2, 2560, 16), (8, 3, 64, 2, 450, 16), (8, 8, 64, 3, 700, 16), (8, 13, 64, 2, 900, 16),
])
def test_pieces_of_every_length(g, K, d, splits, hi, page):
    # pieces of one tile, of an odd and an even number, ragged and whole last tiles, empty pieces
    lens = [hi, 0, 1, 31, 32, 33, 64, 95, 96, 97, 160, 193, 256, hi - 1, hi - 32]
    w, cache, blk = _short(g, K, d, hi, lens, 10100 + g * K + d, page)
    case = GpuCase(w, cache, num_splits=splits, num_layers=1000 if g * K > 96 else 1)
    for view in (DIFF, AR):
        got, lse = case.attn(view, blk)
        want, want_lse = _oracle_attn(view, w, blk, cache, want_lse=True)
        _check_attn(got, want)
        np.testing.assert_allclose(lse, want_lse, rtol=0, atol=2e-3)
        again, _ = case.attn(view, blk)
        np.testing.assert_array_equal(again, got)
    assert case.step.device_error() == 0
    case.step.close()


@pytest.mark.gpu
@pytest.mark.parametrize("layers", [1, 1000])
def test_bad_page_and_non_temporal_loads(layers):
    """1000 layers of the pool: the non-temporal form.  A page id past the pool is flagged and read as page 0."""
    w, cache, blk = _short(4, 16, 128, 600, [600, 580, 77], 10300)
    case = GpuCase(w, cache, num_splits=2, num_layers=layers)
    got, _ = case.attn(AR, blk)
    _check_attn(got, _oracle_attn(AR, w, blk, cache))
    assert case.step.device_error() == 0
    case.page_table[1, 3] = cache["k_pool"].shape[-4] + 5
    got, _ = case.attn(AR, blk)
    swapped = dict(cache, page_table=cache["page_table"].copy())
    swapped["page_table"][1, 3] = 0
    _check_attn(got, _oracle_attn(AR, w, blk, swapped))
    assert case.step.device_error() == -4
    case.step.close()
