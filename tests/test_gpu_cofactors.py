"""Large primes found from their cofactors: the ends of a cofactor's range of
primes at the ends of the prime bitmap's words, and the time of wide ranges.
Whole-number results: against the oracle and against the per-n mode (whose
regions lie elsewhere)."""
import time

import numpy as np
import pytest
import torch

import oracle
from paper_2411_01964_amd import esq
from tests.test_gpu_parity import DEFAULTS, MAX_HI, knobs

pytestmark = pytest.mark.gpu

SEG = (1 << 18) - 4096


@pytest.fixture(scope="module", autouse=True)
def lib_ready():
    esq.init(0, MAX_HI)
    knobs()
    yield
    for k, v in DEFAULTS.items():
        esq.set_param(k, v)


def primes_from(a, residues):
    """The least prime from a on in each residue class modulo 64."""
    out = []
    for r in residues:
        p = a + (r - a) % 64
        while any(p % d == 0 for d in range(3, int(p ** 0.5) + 1, 2)):
            p += 64
        out.append(p)
    return out


# above the cut-over 2^20, so by cofactor; the first and last bit of a word and
# the middle
PRIMES = primes_from((1 << 20) + 1, (1, 3, 31, 33, 61, 63))


@pytest.mark.parametrize("j", [1, 3])
@pytest.mark.parametrize("p", PRIMES)
def test_multiples_at_the_ends_of_a_sieve(p, j):
    """j p^2 as the first and as the last number asked for (for p = 1 or 63 mod
    64 and j = 1 also the first of its region)."""
    m = j * p * p
    for lo, hi in ((m, m + 400), (m - 400, m + 1), (m, m + 1)):
        m0, n, w = esq.sieve_segment(lo, hi)
        om0, on, ow = oracle.sieve_bits(lo, hi)
        assert (m0, n) == (om0, on)
        assert np.array_equal(w.cpu().numpy().view(np.uint64), ow)


@pytest.mark.parametrize("p", PRIMES)
def test_a_square_as_the_last_and_first_of_the_regions(p):
    """The last candidate of a whole number of segments is the last number of
    their regions; the first number of the first region lies 4097 odd numbers
    below the first n."""
    for n in (p * p + 2 - 2 * (2 * SEG - 1), p * p + 2 * 4097):
        g = esq.verify_range(n, n + 2 * 2 * SEG)
        r = esq.verify_range(n, n + 2 * 2 * SEG, per_n=True)
        r.pop("per_n")
        assert g == r


def test_an_interval_with_wide_ranges_equals_its_parts():
    """2^29 odd n from 2^40 on: the cofactor 1 has a range of 256 odd numbers."""
    lo, n = (1 << 40) + 12345, 1 << 29
    whole = esq.verify_range(lo, lo + 2 * n)
    parts = [esq.verify_range(lo + 2 * n * i // 64, lo + 2 * n * (i + 1) // 64) for i in range(64)]
    assert whole["hist"] == [sum(g["hist"][k] for g in parts) for k in range(65)]


def test_wide_ranges_cost_no_more_than_none():
    """1.6e9 odd n in one call, by launches that count hits in memory
    (medium_max 11000: about 1.5e4 hits): near 2^40 one cofactor has a range of
    1500 numbers, near 2^36 there is none.  The segment kernel's work is the
    same; ranges read a number at a time doubled the call."""
    knobs(medium_max=11000)

    def per_call(lo):
        best = 1e9
        for _ in range(6):
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            for _ in range(20):
                esq.verify_range_async(lo, lo + 2 * 3 * (1 << 29))
            torch.cuda.synchronize()
            best = min(best, (time.perf_counter() - t0) / 20)
        return best

    near, far = per_call((1 << 36) + 1), per_call((1 << 40) + 1)
    knobs()
    print("us per call: %.1f without cofactors, %.1f with" % (near * 1e6, far * 1e6))
    assert far < 1.35 * near
