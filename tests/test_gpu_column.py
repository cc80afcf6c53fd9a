"""The column-layout kernel (aggregates-only calls at the default knobs) at the
sizes where it can go wrong: around its segment of 2^18 - 4096 n, near 0,
bounded searches, overflowing hit slots, the ends of the medium range, and
enough segments for the queue's short runs.  Whole-number results: against the
oracle, or, where that would take minutes, against the per-n mode (the row
layout, itself checked against the oracle) on the same interval."""
import pytest
import torch

import oracle
from paper_2411_01964_amd import esq
from tests.test_depth_gap import longest_gap
from tests.test_gpu_parity import DEFAULTS, MAX_HI, assert_same, knobs
from tests.test_zz_no_alloc import KEYS, noalloc_call

pytestmark = pytest.mark.gpu

SEG = (1 << 18) - 4096


@pytest.fixture(scope="module", autouse=True)
def lib_ready():
    esq.init(0, MAX_HI)
    knobs()
    yield
    for k, v in DEFAULTS.items():
        esq.set_param(k, v)


@pytest.mark.parametrize("lo,n", [
    (1, 1), (3, 2), (3, 4095), (8191, 64), (1, SEG - 1), (3, SEG), (5, SEG + 1), (8193, 3 * SEG + 17),
    (2 * SEG + 1, 2 * SEG), (1 << 21, 70001),
])
def test_edges_against_the_oracle(lo, n):
    lo, hi = lo, lo + 2 * n
    g = esq.verify_range(lo, hi, exceptions_cap=16)
    o = oracle.verify_range(lo, hi, per_n=False)
    assert_same(g, o, per_n=False)


@pytest.mark.parametrize("kmax", [5, 6, 13])
def test_bounded_search_lists_its_exceptions(kmax):
    lo, hi = 3, 3 + 2 * (2 * SEG + 999)
    g = esq.verify_range(lo, hi, kmax=kmax, exceptions_cap=4096)
    o = oracle.verify_range(lo, hi, kmax=kmax, per_n=False, exc_cap=1 << 16)
    assert_same(g, o, per_n=False)
    assert g["exceptions"] == o["exceptions"][:4096]


def same_as_per_n(lo, hi):
    g = esq.verify_range(lo, hi)
    p = esq.verify_range(lo, hi, per_n=True)
    k = p.pop("per_n")
    assert g == p
    counts = torch.bincount(k.to(torch.int32), minlength=65).cpu().tolist()
    assert g["hist"] == counts


@pytest.mark.parametrize("kw", [dict(), dict(bucket_cap=1), dict(medium_max=11), dict(medium_max=11000),
                                dict(entry_hits=1), dict(runs_per_wg=3)])
def test_high_interval_equals_the_row_layout(kw):
    knobs(**kw)
    lo = (1 << 50) - (1 << 27) + 12345
    same_as_per_n(lo, lo + 2 * (37 * SEG + 4097))
    knobs()


def test_short_runs_from_the_queue():
    """2^33 odd n: about 33 segments per resident workgroup, the last half
    of them in short runs."""
    lo = (1 << 50) - (1 << 34) - (1 << 20) + 1
    g = esq.verify_range(lo, lo + (1 << 34) + 2 * 31)
    knobs(seg_log2=17)
    r = esq.verify_range(lo, lo + (1 << 34) + 2 * 31)
    knobs()
    assert g == r


def test_batch_of_column_intervals():
    """Intervals of uneven length in one launch equal each alone."""
    ivs = [(3, 4001), ((1 << 40) + 1, (1 << 40) + 1 + 2 * 5 * SEG), ((1 << 44) + 7, (1 << 44) + 7),
           ((1 << 33) + 1, (1 << 33) + 1 + 2 * (SEG + 1)), ((1 << 50) - (1 << 25) + 1, 1 << 50)]
    got = esq.verify_batch([a for a, _ in ivs], [b for _, b in ivs])
    for (a, b), g in zip(ivs, got):
        w = esq.verify_range(a, b)
        assert all(g[k] == w[k] for k in g)


def test_a_scratch_limit_admits_what_the_row_layout_needs():
    """The longest interval below 2^50 whose scratch in the row layout fits the
    static array: the column layout takes it too."""
    hi, limit = 1 << 50, esq.ESQ_NOALLOC_SCRATCH_MAX
    knobs(block=256)
    a, b = 1 << 33, 1 << 37
    while b - a > 1:
        mid = (a + b) // 2
        a, b = (mid, b) if esq.scratch_bytes([hi - 2 * mid + 1], [hi]) <= limit else (a, mid)
    lo = hi - 2 * a + 1
    row = esq.verify_range(lo, hi)
    knobs()
    assert esq.scratch_bytes([lo], [hi]) <= limit
    got = noalloc_call(lo, hi)
    assert all(got[k] == row[k] for k in KEYS)


@pytest.mark.parametrize("base", [0, 1 << 40, (1 << 50) - (1 << 23)])
def test_least_n_of_each_depth_after_the_longest_gap(base):
    """Intervals that start where the n of depth 5 and more are furthest away
    (for 9, 25, 49 and 121 alone): the records come from the first segment."""
    gap, at = longest_gap()
    period = 9 * 25 * 49 * 121
    first = base // 2 + (at - base // 2) % period + 1
    for i in (first, first + gap - SEG):
        same_as_per_n(2 * i + 1, 2 * i + 1 + 2 * 3 * SEG)
