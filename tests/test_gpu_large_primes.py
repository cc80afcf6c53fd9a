"""The large primes' hits by workgroups that own their segments (k_bucket_own)
against the launches that count them in memory, and the sieve near the bounds
of the double-precision reductions: whole-number results, equal."""
import numpy as np
import pytest

import oracle
from paper_2411_01964_amd import esq
from tests.test_gpu_parity import DEFAULTS, MAX_HI, knobs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def lib_ready():
    esq.init(0, MAX_HI)
    knobs()
    yield
    for k, v in DEFAULTS.items():
        esq.set_param(k, v)


def parts(lo, hi, n):
    cut = [lo + 2 * ((hi - lo) // 2 * i // n) for i in range(n)] + [hi]
    return list(zip(cut, cut[1:]))


@pytest.mark.parametrize("hi,n", [(1 << 50, 1 << 31), ((1 << 40) + 77, (1 << 31) + 12345), (1 << 34, 1 << 32),
                                  ((1 << 33) + 2, (1 << 32) - 1)])
def test_a_long_interval_equals_its_parts(hi, n):
    """One call with 6e4 or more expected hits (owned segments) against 40
    calls below the bound (counters in memory), which share none of its
    ranges."""
    lo = hi - 2 * n + 1
    whole = esq.verify_range(lo, hi)
    got = [esq.verify_range(a, b) for a, b in parts(lo, hi, 40)]
    assert whole["hist"] == [sum(g["hist"][k] for g in got) for k in range(65)]
    assert whole["n_odd"] == sum(g["n_odd"] for g in got)
    assert whole["status"] == 0


def test_a_batch_of_owned_segments_equals_each_interval():
    rng = np.random.default_rng(11)
    ivs = []
    for i in range(40):
        n = int(2 ** rng.uniform(16, 28.5))
        a = int(rng.integers(1 << 29, 1 << 49)) * 2 + 1
        ivs.append((a, a + 2 * n))
    ivs[3] = (ivs[3][0], ivs[3][0])
    ivs[4] = (3, 3 + (1 << 26))
    for g, (a, b) in zip(esq.verify_batch([a for a, _ in ivs], [b for _, b in ivs]), ivs):
        w = esq.verify_range(a, b)
        assert all(g[k] == w[k] for k in g), (a, b)


@pytest.mark.parametrize("medium_max", [11, 4095])
@pytest.mark.parametrize("at", [1 << 52, 1 << 53, 1 << 54, (1 << 56) - 2000])
def test_sieve_around_the_bound_of_the_double_reductions(at, medium_max):
    esq.init(0, esq.ESQ_MAX_HI)
    knobs(medium_max=medium_max)
    lo, hi = at - 1801, at + 1801
    m0, n, w = esq.sieve_segment(lo, hi)
    om0, on, ow = oracle.sieve_bits(lo, hi)
    assert (m0, n) == (om0, on)
    assert np.array_equal(w.cpu().numpy().view(np.uint64), ow)
    knobs()
