"""The order in which a prefill launch of a few sequences starts its chunks, checked by brute force on the CPU.

The kernel finds the chunk of rank r from counts of the chunks above a level, four levels at a time.  The library compiles
the same search for the host, over arrays in place of a wave's lanes: its ranks name every chunk of every sequence exactly
once, longest first to within a chunk, and nothing past the last.
"""
import ctypes

import numpy as np
import pytest

import paper_2605_12825_amd as orthrus

_lib = ctypes.CDLL(orthrus.library_path())
_order = getattr(_lib, "_ZN7orthrus20ranked_chunk_on_hostEiiPKiS1_PiS2_")
_order.restype = ctypes.c_bool
_rule = getattr(_lib, "_ZN7orthrus14prefill_rankedEilii")
_rule.restype, _rule.argtypes = ctypes.c_bool, [ctypes.c_int, ctypes.c_int64, ctypes.c_int, ctypes.c_int]


def _ranked_chunk(r, ends, chunks):
    n = len(ends)
    seq, chunk = ctypes.c_int(-1), ctypes.c_int(-1)
    found = _order(r, n, (ctypes.c_int * n)(*ends), (ctypes.c_int * n)(*chunks), ctypes.byref(seq), ctypes.byref(chunk))
    return (seq.value, chunk.value) if found else None


@pytest.mark.parametrize("seed", range(60))
def test_ranks_name_every_chunk_once_longest_first(seed):
    rng = np.random.default_rng(seed)
    B, T = int(rng.integers(2, 17)), int(rng.choice([16, 18, 32, 36, 64, 128, 256]))
    old = rng.integers(0, int(rng.choice([1, 300, 20000, 10 ** 9])), B)
    new = rng.integers(0, int(rng.choice([2, 100, 1500])), B)
    if seed % 7 == 0:
        old[:] = 0
    if seed == 1:
        new[:] = 0
    chunks = [-(-int(n) // T) for n in new]
    ends = [int(o + n) // T if n else 0 for o, n in zip(old, new)]
    total = sum(chunks)
    got = [_ranked_chunk(r, ends, chunks) for r in range(total)]
    assert sorted(got) == [(b, c) for b in range(B) for c in range(chunks[b])]
    last = [int(old[b]) + min((c + 1) * T, int(new[b])) for b, c in got]      # tokens that a chunk sees
    assert all(x >= y - 2 * T for x, y in zip(last, last[1:]))
    assert all(_ranked_chunk(total + x, ends, chunks) is None for x in (0, 1, 70))


@pytest.mark.parametrize("ranked,batch,items,per_cu", [
    (False, 1, 4096, 1), (False, 17, 4096, 1), (False, 16, 256, 1), (True, 16, 257, 1), (False, 2, 512, 2), (True, 2, 513, 2),
])
def test_ranked_where_items_wait_for_others(ranked, batch, items, per_cu):
    assert _rule(batch, items, per_cu, 256) == ranked
