"""Pieces whose row blocks are shared by two waves (even and odd tiles) against the oracle, where this form is chosen, and the
rule that chooses it."""
import ctypes

import numpy as np
import pytest

import paper_2605_12825_amd as orthrus
from orthrus_inputs import Workload, make_block, make_cache

from test_gpu_parity import AR, DIFF, GpuCase, _check_attn, _oracle_attn

_rule = getattr(ctypes.CDLL(orthrus.library_path()), "_ZN7orthrus16split_pays_pairsEiiliibi")
_rule.restype, _rule.argtypes = ctypes.c_bool, [ctypes.c_int, ctypes.c_int, ctypes.c_int64] + [ctypes.c_int] * 2 + [ctypes.c_bool, ctypes.c_int]


def _case(g, K, d, splits, hi, lens, seed, page=16, kv_nt=False):
    hkv = 2
    assert _rule(d, g * K, len(lens) * hkv * splits, splits, hi, kv_nt, 256)
    w = Workload(name="paired", seed=seed, batch=len(lens), num_q_heads=g * hkv, num_kv_heads=hkv, head_dim=d, block_k=K, context=hi,
                 page_size=page, paging="scattered")
    cache = make_cache(w, seq_lens=np.asarray(lens, np.int32))
    return w, cache, make_block(w, seed + 1)


@pytest.mark.gpu
@pytest.mark.parametrize("g,K,d,splits,hi,page", [
    (4, 5, 128, 2, 500, 16), (4, 8, 128, 3, 700, 32), (4, 16, 128, 2, 600, 64), (7, 5, 128, 3, 900, 16), (4, 32, 128, 2, 2560, 16),
    (7, 14, 128, 2, 2560, 16), (8, 3, 64, 2, 450, 16), (8, 8, 64, 3, 700, 16), (8, 13, 64, 2, 900, 16),
])
def test_two_waves_to_a_row_block(g, K, d, splits, hi, page):
    # pieces of one tile (the second wave has none), of an odd and an even number, ragged and whole last tiles, empty pieces
    lens = [hi, 0, 1, 31, 32, 33, 64, 95, 96, 97, 160, 193, 256, hi - 1, hi - 32]
    w, cache, blk = _case(g, K, d, splits, hi, lens, 10100 + g * K + d, page, g * K > 96)
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
    lens = [600, 580, 77]
    w, cache, blk = _case(4, 16, 128, 2, 600, lens, 10300)
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


@pytest.mark.parametrize("paired,d,rows,items,splits,bound", [
    (False, 128, 16, 104, 13, 4112), (True, 128, 17, 104, 13, 4112), (True, 128, 64, 104, 13, 4112), (True, 128, 64, 144, 18, 6400),
    (False, 128, 64, 152, 19, 6400), (False, 128, 64, 96, 12, 3400), (True, 128, 32, 192, 12, 3000), (False, 128, 32, 193, 12, 3000),
    (False, 128, 96, 240, 30, 40000), (True, 128, 128, 240, 30, 40000), (True, 128, 97, 256, 8, 32768), (False, 128, 128, 257, 8, 32768),
    (False, 128, 128, 112, 14, 4112), (False, 128, 160, 240, 30, 40000), (False, 128, 64, 32, 1, 4112),
    (True, 64, 32, 256, 16, 8000), (True, 64, 64, 112, 14, 3000), (False, 64, 64, 64, 8, 1500), (True, 64, 128, 72, 36, 16000),
    (False, 64, 128, 76, 19, 6000), (False, 64, 96, 72, 36, 16000),
])
def test_where_two_waves_pay(paired, d, rows, items, splits, bound):
    assert _rule(d, rows, items, splits, bound, True, 256) == paired
    assert _rule(d, rows, items, splits, bound, False, 256) == (paired and not (d == 128 and rows > 96))
