"""The order in which the items of a fixed-split decode launch start: batches whose items do not all fit the chip at once,
with lengths that rise, fall, repeat a rise, come in any order or are alike, against the oracle (most of them at few rows, so in
the 16-row form); every kernel and number of row blocks in two of these orders; and the rules on the CPU."""
import ctypes

import numpy as np
import pytest

import paper_2605_12825_amd as orthrus
from orthrus_inputs import Workload, make_block, make_cache

from test_attn_routes_cpu import decode_is_wide
from test_gpu_parity import AR, DIFF, GpuCase, _check_attn, _oracle_attn

_rule = getattr(ctypes.CDLL(orthrus.library_path()), "_ZN7orthrus14decode_by_sizeEilii")
_rule.restype, _rule.argtypes = ctypes.c_bool, [ctypes.c_int, ctypes.c_int64, ctypes.c_int, ctypes.c_int]

_direction = getattr(ctypes.CDLL(orthrus.library_path()), "_ZN7orthrus24decode_direction_on_hostEPKiib")
_direction.restype, _direction.argtypes = ctypes.c_int, [ctypes.POINTER(ctypes.c_int), ctypes.c_int, ctypes.c_bool]
RANKED, ALIKE, RISING, FALLING = range(4)


def _lens(kind, n, hi, seed):
    rng = np.random.default_rng(seed)
    x = rng.integers(0, hi + 1, size=n)
    x[:4] = (0, hi, hi // 2, 0)[:n]
    if kind == "rising":
        x = np.sort(x)
    elif kind == "falling":
        x = np.sort(x)[::-1]
    elif kind == "packed":       # a rise for each packed sequence
        x = np.concatenate([np.sort(p) for p in np.array_split(x, 3)])
    elif kind == "nearly":       # every sample in order, a few lengths not
        x = np.sort(x)
        x[[3, n // 2 + 1, n - 3]] = (hi, 0, 1)
    elif kind == "alike":        # one number of tiles, different lengths
        x = 33 + x % 32
    elif kind == "one":          # a single sequence that differs
        x[:] = 40
        x[n - 2] = 97
    return np.ascontiguousarray(x.astype(np.int32))


@pytest.mark.gpu
@pytest.mark.parametrize("kind,batch,splits,g,hkv,d,K,per_cu", [
    ("any", 200, 1, 2, 8, 64, 4, 6), ("any", 65, 3, 2, 8, 64, 4, 6), ("any", 256, 1, 1, 7, 64, 3, 6), ("any", 64, 4, 2, 8, 64, 4, 6),
    ("rising", 257, 1, 2, 6, 64, 4, 6), ("falling", 300, 1, 2, 6, 64, 4, 6), ("packed", 300, 1, 2, 6, 64, 4, 6),
    ("packed", 129, 2, 2, 8, 64, 4, 6), ("nearly", 200, 1, 2, 8, 64, 4, 6), ("nearly", 260, 1, 2, 6, 64, 4, 6),
    ("alike", 193, 1, 2, 8, 64, 4, 6), ("alike", 385, 1, 2, 4, 64, 4, 6), ("one", 192, 1, 2, 9, 64, 4, 6),
    ("rising", 130, 2, 6, 4, 128, 31, 1), ("any", 2, 1, 1, 1025, 64, 1, 6),
    ("any", 112, 1, 4, 8, 128, 32, 2), ("rising", 112, 1, 4, 8, 128, 32, 2),   # the 64-row kernel
])
def test_items_that_start_by_size(kind, batch, splits, g, hkv, d, K, per_cu):
    assert _rule(batch, batch * hkv * splits, per_cu, 256)
    hi = 130
    assert decode_is_wide(d, g * K, hi, batch * hkv) == (batch == 112)
    w = Workload(name="order", seed=9300 + batch, batch=batch, num_q_heads=g * hkv, num_kv_heads=hkv, head_dim=d, block_k=K,
                 context=hi, page_size=16, paging="scattered")
    lens = _lens(kind, batch, hi, 9400 + batch)
    cache = make_cache(w, seq_lens=lens)
    blk = make_block(w, 9500 + K)
    case = GpuCase(w, cache, num_splits=splits)
    for view in (DIFF, AR):
        got, lse = case.attn(view, blk)
        want, want_lse = _oracle_attn(view, w, blk, cache, want_lse=True)
        _check_attn(got, want)
        np.testing.assert_allclose(lse, want_lse, rtol=0, atol=2e-3)
    assert case.step.device_error() == 0
    case.step.close()


def _check(case, view, w, blk, cache, lens):
    got, lse = case.attn(view, blk)
    want, want_lse = _oracle_attn(view, w, blk, cache, want_lse=True, seq_lens=lens)
    _check_attn(got, want)
    np.testing.assert_allclose(lse, want_lse, rtol=0, atol=2e-3)
    return got, lse


@pytest.mark.gpu
@pytest.mark.parametrize("layers", [1, 1000])   # 1000 layers of the pool: the non-temporal form
@pytest.mark.parametrize("kind", ["any", "rising"])
@pytest.mark.parametrize("g,K,d,splits,batch,per_cu,bound", [
    (2, 4, 64, 1, 200, 6, 130), (1, 16, 128, 2, 50, 3, 130),                                     # up to 16 rows
    (2, 10, 128, 2, 50, 3, 130), (1, 17, 64, 1, 200, 6, 130), (4, 16, 128, 1, 105, 3, 130),      # one to eight row blocks
    (5, 16, 128, 2, 50, 3, 130), (3, 25, 64, 1, 110, 3, 130), (4, 32, 128, 2, 34, 2, 130), (8, 17, 128, 2, 34, 2, 130),
    (6, 31, 128, 2, 18, 1, 130), (7, 32, 128, 2, 18, 1, 130), (7, 29, 64, 1, 34, 1, 130), (8, 32, 128, 2, 18, 1, 130),
    (4, 32, 128, 1, 112, 2, 130), (8, 16, 64, 1, 96, 2, 4096), (8, 32, 128, 1, 40, 1, 4096),      # the 64-row kernel
])
def test_every_kernel_that_starts_its_items_by_size(g, K, d, splits, batch, per_cu, bound, kind, layers):
    """16-row, 32-row and 64-row forms, with lengths in order, in any order, and outside the bound where the samples look."""
    hkv, hi, rows = 8, 130, g * K
    assert _rule(batch, batch * hkv * splits, per_cu, 256)
    assert (splits == 1 and decode_is_wide(d, rows, bound, batch * hkv)) == ((g, K, batch) in ((4, 32, 112), (8, 16, 96), (8, 32, 40)))
    w = Workload(name="by", seed=9600 + rows + d, batch=batch, num_q_heads=g * hkv, num_kv_heads=hkv, head_dim=d, block_k=K,
                 context=hi, page_size=16, paging="scattered")
    lens = _lens(kind, batch, hi, 9700 + batch)
    assert _direction((ctypes.c_int * batch)(*lens), batch, False) == (RISING if kind == "rising" else RANKED)
    cache, blk = make_cache(w, seq_lens=lens), make_block(w, 9800 + K)
    table = np.zeros((batch, max(-(-bound // 16), cache["page_table"].shape[1])), np.int32)
    table[:, :cache["page_table"].shape[1]] = cache["page_table"]
    roomy = dict(cache, page_table=table)
    case = GpuCase(w, roomy, num_splits=splits, num_layers=layers, max_seq_len=bound)
    assert case.step.num_splits == splits
    good = _check(case, AR, w, blk, cache, lens)
    assert case.step.device_error() == 0
    case.step.close()
    # outside the bound on either side, where a sample is taken (or near it): read as 0, and as the bound
    bad = lens.copy()
    bad[[0, batch // 2]] = (-(2 ** 31), -1)
    many = bound == hi
    if many:
        full = int(np.flatnonzero(lens == hi)[-1])
        bad[full] = 2 ** 31 - 1
    case = GpuCase(w, dict(roomy, seq_lens=bad), num_splits=splits, num_layers=layers, max_seq_len=bound)
    got = _check(case, AR, w, blk, cache, np.clip(bad, 0, hi))
    assert case.step.device_error() == -4
    same = bad == lens
    np.testing.assert_array_equal(got[0][same], good[0][same])
    np.testing.assert_array_equal(got[1][same], good[1][same])
    case.step.close()


@pytest.mark.parametrize("by_size,batch,items,per_cu", [(False, 1, 4096, 1), (False, 2, 512, 2), (True, 2, 513, 2), (True, 60000, 257, 1)])
def test_by_size_where_items_wait_for_others(by_size, batch, items, per_cu):
    assert _rule(batch, items, per_cu, 256) == by_size


@pytest.mark.parametrize("lens,wide,others", [
    ([1000] * 128, ALIKE, ALIKE), ([0] * 3, ALIKE, ALIKE), ([7] * 400, ALIKE, ALIKE),
    (list(range(992, 1023)), ALIKE, ALIKE),                  # a token or two apart, one count of whole tiles
    (list(range(1000, 1064, 2)), RISING, ALIKE), (list(range(1063, 1000, -2)), FALLING, ALIKE),
    (list(range(1000, 1240, 2)), RISING, RISING), ([20] * 50 + [40] * 50, RISING, RISING),
    (list(range(1000, 1200)) * 2, RISING, RISING),           # a repeated rise above what is ranked: its two ends
    (list(range(1000, 1128)) * 2, RANKED, ALIKE), ([500, 100, 100] * 67, RANKED, RANKED), ([100] + [500] * 299, RISING, RISING),
    ([-(2 ** 31)] + [5] * 99 + [2 ** 31 - 1], RISING, RISING), ([2 ** 31 - 1, -(2 ** 31)] * 150, FALLING, FALLING),
])
def test_lengths_that_are_nearly_alike_keep_the_plain_order(lens, wide, others):
    got = [_direction((ctypes.c_int * len(lens))(*lens), len(lens), small) for small in (True, False)]
    assert got == [wide, others]
