"""The order in which a prefill launch of a few sequences starts its chunks, checked by brute force on the CPU.

The kernel finds the chunk of rank r from counts of the chunks above a level, 64 levels at a time.  This restates the
search with the same rounds and checks that the ranks name every chunk of every sequence exactly once, longest first to
within a chunk, and nothing past the last.
"""
import numpy as np
import pytest


def _ranked_chunk(r, ends, chunks):
    lo, hi, above = -1, max(ends), 0
    while hi - lo > 1:
        step = (hi - lo + 63) >> 6
        level = [min(lo + (lane + 1) * step, hi) for lane in range(64)]
        count = [sum(min(max(e - x, 0), n) for e, n in zip(ends, chunks)) for x in level]
        f = next(i for i, c in enumerate(count) if c <= r)
        above, hi = count[f], min(lo + (f + 1) * step, hi)
        lo += f * step
    active = [b for b, (e, n) in enumerate(zip(ends, chunks)) if 0 <= e - hi < n]
    k = r - above
    return (active[k], chunks[active[k]] - 1 - (ends[active[k]] - hi)) if k < len(active) else None


@pytest.mark.parametrize("seed", range(60))
def test_ranks_name_every_chunk_once_longest_first(seed):
    rng = np.random.default_rng(seed)
    B, T = int(rng.integers(2, 17)), int(rng.choice([16, 18, 32, 36, 64, 128, 256]))
    old = rng.integers(0, int(rng.choice([1, 300, 20000])), B)
    new = rng.integers(0, int(rng.choice([2, 100, 1500])), B)
    if seed % 7 == 0:
        old[:] = 0
    if seed == 1:
        new[:] = 0
    ends = [int(o + n) // T for o, n in zip(old, new)]
    chunks = [-(-int(n) // T) for n in new]
    total = sum(chunks)
    got = [_ranked_chunk(r, ends, chunks) for r in range(total)]
    assert sorted(got) == [(b, c) for b in range(B) for c in range(chunks[b])]
    last = [int(old[b]) + min((c + 1) * T, int(new[b])) for b, c in got]      # tokens that a chunk sees
    assert all(x >= y - 2 * T for x, y in zip(last, last[1:]))
    assert all(_ranked_chunk(total + x, ends, chunks) is None for x in (0, 1, 70))
