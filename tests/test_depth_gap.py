"""The odd n whose first four candidates n - 2, n - 4, n - 8, n - 16 are
multiples of 9, 25, 49 and 121 in some order recur within 169400 odd numbers,
so any longer run of odd n holds one of depth 5 or more, and of depths 2 .. 4:
the column layout's segments (2^18 - 4096 n) rely on it to look for an
interval's least n of these depths in its first segment only."""
import numpy as np


def longest_gap():
    """(gap, odd index after which it starts) over one period 9 25 49 121."""
    q = (9, 25, 49, 121)
    period, pad = 9 * 25 * 49 * 121, 8
    marked = np.zeros(period + pad, dtype=bool)      # position x + pad: odd index x
    for m in q:
        marked[((m - 1) // 2 + pad) % m::m] = True
    deep = np.ones(period, dtype=bool)
    for k in range(1, 5):
        d = 1 << (k - 1)
        deep &= marked[pad - d:pad - d + period]
    at = np.flatnonzero(deep)
    gaps = np.diff(np.append(at, at[0] + period))
    return int(gaps.max()), int(at[gaps.argmax()])


def test_a_whole_segment_holds_an_n_of_depth_five():
    gap, at = longest_gap()
    assert gap == 169400 < (1 << 18) - 4096
    n = 2 * at + 1 + 2 * 9 * 25 * 49 * 121
    assert all(any((n - (1 << k)) % m == 0 for m in (9, 25, 49, 121)) for k in range(1, 5))
