"""k_bucket_own's branches that ordinary calls do not take: integer reductions
(odd indices from 2^52 on), cofactors of n up to 2^56, and lists of primes and
cofactors longer than their room in LDS.  Whole-number results: equal to calls
too short for owned segments, or to other segments."""
import time

import numpy as np
import pytest
import torch

import oracle
from paper_2411_01964_amd import esq
from tests.test_gpu_parity import DEFAULTS, assert_same, knobs

pytestmark = pytest.mark.gpu

SEG = (1 << 18) - 4096


@pytest.fixture(scope="module", autouse=True)
def lib_ready():
    esq.init(0, esq.ESQ_MAX_HI)
    knobs()
    yield
    for k, v in DEFAULTS.items():
        esq.set_param(k, v)


def joined(lo, n, parts, kmax=0):
    """hist and per-n bytes of the interval in equal parts."""
    hist, bytes_ = [0] * 65, []
    for i in range(parts):
        r = esq.verify_range(lo + 2 * (n * i // parts), lo + 2 * (n * (i + 1) // parts), per_n=True)
        hist = [a + b for a, b in zip(hist, r["hist"])]
        bytes_.append(r["per_n"])
    return hist, torch.cat(bytes_)


@pytest.mark.parametrize("at", [1 << 53, 1 << 55, esq.ESQ_MAX_HI])
def test_integer_reductions_equal_short_calls(at):
    """With the primes from 17 on all counted as large, 2^22 odd n have about
    7e4 hits, past the 4e4 of owned segments; a sixteenth of them has too few.
    The upper half lies past odd index 2^52 for at = 2^53, which decides for
    the whole call."""
    knobs(medium_max=11)
    n = 1 << 22
    lo = at - n + 1 if at < esq.ESQ_MAX_HI else at - 2 * n - 1
    hist, per_n = joined(lo, n, 16)
    s = esq.verify_range(lo, lo + 2 * n)                        # column layout
    p = esq.verify_range(lo, lo + 2 * n, per_n=True)            # row layout
    assert s["hist"] == hist and p["hist"] == hist
    assert s["records"] == p["records"] and s["ksum"] == p["ksum"]
    assert torch.equal(p["per_n"], per_n)
    whole = esq.sieve_segment(lo, lo + 2 * n)[2]
    step = n // 16
    words = torch.cat([esq.sieve_segment(lo + 2 * i * step, lo + 2 * (i + 1) * step)[2] for i in range(16)])
    assert torch.equal(whole, words)
    knobs()


@pytest.mark.parametrize("at", [1 << 53, esq.ESQ_MAX_HI])
@pytest.mark.parametrize("kw", [dict(), dict(medium_max=11)])
def test_the_column_layout_past_2pow50(at, kw):
    """Against the row layout on whole segments, and against the oracle on the
    last few hundred n."""
    knobs(**kw)
    n = 5 * SEG + 4097
    lo = at - 2 * n - 1
    s = esq.verify_range(lo, lo + 2 * n)
    p = esq.verify_range(lo, lo + 2 * n, per_n=True)
    k = p.pop("per_n")
    assert s == p
    a = lo + 2 * (n - 300)
    o = oracle.verify_range(a, lo + 2 * n, per_n=True)
    assert np.array_equal(k[-300:].cpu().numpy(), o["per_n"])
    assert_same(esq.verify_range(a, lo + 2 * n, exceptions_cap=16), o, per_n=False)
    knobs()


@pytest.mark.parametrize("weight", [60, 1])
def test_lists_longer_than_their_room(weight):
    """2^36 odd n in segments of 2^20: a workgroup owns 256 of them, 2^28
    numbers, with a hit for each of the 1336 primes from 4093 to 2^14 and for
    1050 to 1400 above (room for 2048); at cof_weight 1 the cofactors take over
    from 2^15.5, 5800 of them with an integer in their range.  Against the
    column layout's segments."""
    n = 1 << 36
    lo = (1 << 50) - 2 * n + 1
    want = esq.verify_range(lo, 1 << 50)
    knobs(seg_log2=20)
    esq.set_param("cof_weight", weight)
    got = esq.verify_range(lo, 1 << 50)
    esq.set_param("cof_weight", 60)
    knobs()
    assert got == want


def batch_time(count, n, top):
    """Seconds per launch of a prepared batch of count intervals of n odd n each
    below 2^top."""
    rng = np.random.default_rng(7)
    lo = [int(rng.integers(1 << (top - 2), (1 << (top - 1)) - n)) * 2 + 1 for _ in range(count)]
    pb = esq.PreparedBatch(lo, [a + 2 * n for a in lo])
    best = 1e9
    for _ in range(5):
        pb.launch(graph=True)
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        for _ in range(10):
            pb.launch(graph=True)
        torch.cuda.synchronize()
        best = min(best, (time.perf_counter() - t0) / 10)
    pb.close()
    return best


def test_wide_cofactor_ranges_cost_no_more_than_narrow_ones():
    """512 intervals of 2^24 odd n: near 2^28 the few cofactors have ranges of a
    thousand numbers in a workgroup's segments, near 2^40 of eight; the segment
    kernel's work is the same.  A lane for each range made the batch a third
    slower."""
    wide, narrow = batch_time(512, 1 << 24, 28), batch_time(512, 1 << 24, 40)
    print("us per batch: %.1f with wide ranges, %.1f with narrow ones" % (wide * 1e6, narrow * 1e6))
    assert wide < 1.15 * narrow


def test_an_interval_from_3_on_costs_no_more_than_a_high_one():
    """2^33 odd n: from 3 on the first workgroup's cofactor 1 has a range of 8192
    numbers, which one lane made three times the whole call."""
    def per_call(lo):
        best = 1e9
        for _ in range(5):
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            for _ in range(10):
                esq.verify_range_async(lo, lo + (1 << 34))
            torch.cuda.synchronize()
            best = min(best, (time.perf_counter() - t0) / 10)
        return best

    low, high = per_call(3), per_call((1 << 40) + 1)
    print("us per call: %.1f from 3, %.1f from 2^40" % (low * 1e6, high * 1e6))
    assert low < 1.15 * high


def test_wide_cofactor_ranges_equal_the_row_layout():
    """8 intervals of 2^28 odd n and 2^31 in one, near 2^33."""
    lo = [(1 << 32) + (i << 29) + 12345 for i in range(8)]
    got = esq.verify_batch(lo, [a + (1 << 29) for a in lo])
    one = esq.verify_range(lo[0], lo[0] + (1 << 32))
    knobs(seg_log2=16)
    want = esq.verify_batch(lo, [a + (1 << 29) for a in lo])
    knobs(seg_log2=17)
    whole = esq.verify_range(lo[0], lo[0] + (1 << 32))
    knobs()
    assert got == want
    assert one == whole


def test_many_short_intervals_at_low_positions():
    """8000 intervals of 2^12 odd n: near 2^30 3000 primes are large, near 2^24
    none (sqrt below 4096), and the rest of the batch's work is the same.  A
    workgroup each to go through so few made the batch 1.4 times as slow."""
    some, none = batch_time(8000, 1 << 12, 30), batch_time(8000, 1 << 12, 24)
    print("us per batch: %.1f with 3000 large primes, %.1f with none" % (some * 1e6, none * 1e6))
    assert some < 1.25 * none


@pytest.mark.parametrize("top", [30, 36, 38])
def test_many_short_intervals_equal_each_alone(top):
    """600 intervals: counters in memory below 3e4 large primes, owned segments
    above (at 3 segments each, past 4e4 hits with medium_max 2047)."""
    knobs(medium_max=2047)
    rng = np.random.default_rng(top)
    n = [int(x) for x in rng.integers(1, 5 << 17, 600)]
    lo = [int(rng.integers(1 << (top - 2), (1 << (top - 1)) - (5 << 17))) * 2 + 1 for _ in n]
    got = esq.verify_batch(lo, [a + 2 * k for a, k in zip(lo, n)])
    for g, a, k in list(zip(got, lo, n))[::7]:
        w = esq.verify_range(a, a + 2 * k)
        assert all(g[x] == w[x] for x in g)
    knobs()


def test_more_intervals_than_a_grid_has_rows():
    """70000 intervals at a low position, whichever form they take."""
    lo = [(1 << 28) + 1 + 200 * i for i in range(70000)]
    got = esq.verify_batch(lo, [a + 200 for a in lo])
    one = esq.verify_range(lo[0], lo[-1] + 200)
    assert [sum(h) for h in zip(*(g["hist"] for g in got))] == one["hist"]
