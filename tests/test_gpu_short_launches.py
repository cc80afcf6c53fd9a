"""Launches too short to fill the device at the default segment length take
shorter segments (and fewer threads): the sizes where that length changes,
against the same call with the segment length set by its knob, where the rule
does not apply; and lists of exceptions around the sizes of the finalize
pass's sort.  Whole-number results: equal."""
import pytest
import torch

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


@pytest.mark.parametrize("n", [1, (1 << 14) - 1, (1 << 14) + 1, (1 << 21) + 63, (1 << 22) - 1, 1 << 22,
                               (1 << 23) + 65, (1 << 25) - 1, 1 << 25])
@pytest.mark.parametrize("kmax", [0, 3])
def test_per_n_across_the_segment_lengths(n, kmax):
    lo = (1 << 45) + 12347
    g = esq.verify_range(lo, lo + 2 * n, kmax=kmax, per_n=True, exceptions_cap=100)
    knobs(seg_log2=17)
    w = esq.verify_range(lo, lo + 2 * n, kmax=kmax, per_n=True, exceptions_cap=100)
    knobs()
    assert torch.equal(g.pop("per_n"), w.pop("per_n"))
    assert g == w


@pytest.mark.parametrize("n", [1, (1 << 14) + 1, (1 << 20) - 1, 1 << 20, (1 << 21) + 65, (1 << 26) - 1, 1 << 26])
@pytest.mark.parametrize("lo", [1, (1 << 45) + 12347])
def test_sieve_across_the_segment_lengths(lo, n):
    g = esq.sieve_segment(lo, lo + 2 * n)[2]
    knobs(sieve_seg_log2=19)
    w = esq.sieve_segment(lo, lo + 2 * n)[2]
    knobs()
    assert torch.equal(g, w)


def test_per_n_batch_of_short_intervals():
    ivs = [(3, 3 + 2 * n) for n in (1, 1 << 14, 70001)] + [((1 << 44) + 9, (1 << 44) + 9 + (1 << 23))]
    args = [a for a, _ in ivs], [b for _, b in ivs]
    got = esq.verify_batch(*args, per_n=[True] * len(ivs))
    knobs(seg_log2=17)
    want = esq.verify_batch(*args, per_n=[True] * len(ivs))
    knobs()
    for g, w in zip(got, want):
        assert torch.equal(g.pop("per_n"), w.pop("per_n"))
        assert g == w


@pytest.mark.parametrize("cap", [1, 63, 1000, 1024, 1025, 4095, 4096, 4097, 16383, 16384])
@pytest.mark.parametrize("n,kmax", [(9000, 2), (40000, 2), (1 << 20, 1)])
def test_exception_lists_around_the_sorts_sizes(cap, n, kmax):
    """The listed exceptions are the first zeros of the per-n bytes."""
    lo = 100003
    g = esq.verify_range(lo, lo + 2 * n, kmax=kmax, per_n=True, exceptions_cap=cap)
    zeros = torch.nonzero(g["per_n"] == 0).flatten()[:cap].cpu().tolist()
    assert g["exceptions"] == [lo + 2 * i for i in zeros]
    s = esq.verify_range(lo, lo + 2 * n, kmax=kmax, exceptions_cap=cap)
    assert s["exceptions"] == g["exceptions"] and s["hist"] == g["hist"]
