"""Knobs that decide which tables a call needs and how its work is cut: tables
are resident whatever order the knobs were set in, and a knob set off its
default is taken as it is."""
import pytest
import torch

from paper_2411_01964_amd import esq
from tests.test_gpu_parity import DEFAULTS, MAX_HI, knobs
from tests.test_zz_no_alloc import KEYS, noalloc_call

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def lib_ready():
    esq.init(0, MAX_HI)
    knobs()
    yield
    for k, v in DEFAULTS.items():
        esq.set_param(k, v)


@pytest.mark.parametrize("n,kmax,per_n", [(5003, 0, True), (1 << 21, 0, True), (70001, 3, False),
                                          (1 << 24, 4, False)])
def test_noalloc_after_a_longer_tail_list_was_taken_back(n, kmax, per_n):
    """A tail list above its default keeps launches at the knob's segment
    length; back at the default, short ones take shorter segments, whose tables
    the no-alloc call needs resident.  (A medium_max of its own, so that no
    other test has made them.)"""
    esq.set_param("tail_cap", 1 << 21)
    esq.set_param("medium_max", 3571 + n % 97)
    esq.set_param("tail_cap", 1 << 20)
    lo = (1 << 44) + 12345
    got = noalloc_call(lo, lo + 2 * n, kmax, per_n, 16)
    want = esq.verify_range(lo, lo + 2 * n, kmax=kmax, per_n=per_n, exceptions_cap=16)
    assert all(got[k] == want[k] for k in KEYS)
    if per_n:
        assert torch.equal(got["per_n"], want["per_n"])
    knobs()


@pytest.mark.parametrize("n", [1000, (1 << 21) + 13, (1 << 23) + 1, 1 << 26])
def test_a_sieve_call_of_a_new_length_waits_for_nothing(n):
    """Calls only enqueue: the first sieve of a segment length returns while
    work queued before it still runs (making its tables would wait for it)."""
    knobs(medium_max=3300 + n % 89)
    lo, span = (1 << 49) + 1, 1 << 39
    esq.verify_range(lo, lo + span)            # the stream's scratch block
    out = torch.empty((n + 63) // 64, dtype=torch.int64, device="cuda")
    torch.cuda.synchronize()
    for _ in range(10):                        # 5 ms of work each
        esq.verify_range_async(lo, lo + span)
    queued = torch.cuda.Event()
    queued.record()
    esq.sieve_segment(lo, lo + 2 * n, out=out)
    assert not queued.query()
    torch.cuda.synchronize()
    assert queued.query()
    knobs()


def test_hit_slots_of_every_segment_are_as_many_as_set():
    """1000 whole segments of the column layout (985 of the row layout): 500
    slots more, of 4 bytes, in each."""
    span = 2 * 1000 * ((1 << 18) - 4096)
    figure = {}
    for slots in (500, 1000):
        knobs(bucket_cap=slots)
        figure[slots] = esq.scratch_bytes([(1 << 49) + 1], [(1 << 49) + 1 + span])
    knobs()
    assert abs(figure[1000] - figure[500] - 1000 * 500 * 4) <= 512      # alignment


def test_hit_slots_set_give_way_where_only_the_shared_total_fits():
    """As many segments as the row layout fits into the static array at 4096
    slots: the no-alloc call takes them."""
    knobs(bucket_cap=4096, block=256)
    lo, a, b = (1 << 49) + 1, 1 << 20, 1 << 34
    while b - a > 1:
        mid = (a + b) // 2
        a, b = (mid, b) if esq.scratch_bytes([lo], [lo + 2 * mid]) <= esq.ESQ_NOALLOC_SCRATCH_MAX else (a, mid)
    row = esq.verify_range(lo, lo + 2 * a)
    knobs(bucket_cap=4096)
    got = noalloc_call(lo, lo + 2 * a)
    assert all(got[k] == row[k] for k in KEYS)
    knobs()


def marking_share(**kw):
    """The marking phase's share of the segment kernel's time (phase clock), and
    the aggregates, of 2^30 odd n."""
    knobs(**kw)
    lo = (1 << 49) + 12345
    esq.set_param("phase_clock", 1)
    try:
        esq.phase_take()
        r = esq.verify_range(lo, lo + (1 << 31))
        ph = esq.phase_take()
    finally:
        esq.set_param("phase_clock", 0)
        knobs()
    return ph["mark"] / sum(ph.values()), r


def test_marks_per_task_are_as_many_as_set():
    """With 4096 marks a task the multiples of 17^2, 907 in a region, are one
    lane's, where the default gives a lane about 9: the marking phase is most of
    the kernel."""
    share, r = marking_share()
    for hits in (11, 13, 64):
        assert marking_share(entry_hits=hits)[1] == r
    slow, s = marking_share(entry_hits=4096)
    print("marking: %.2f of the kernel, %.2f with 4096 marks a task" % (share, slow))
    assert s == r
    assert share < 0.5 < slow


@pytest.fixture
def as_set():
    esq.set_param("adapt", 0)
    yield
    esq.set_param("adapt", 1)


def segments_of_a_call(lo, n):
    """Segments of the form that has more, from the figure's growth by 500 slots
    each."""
    f = {}
    for slots in (500, 1000):
        esq.set_param("bucket_cap", slots)
        f[slots] = esq.scratch_bytes([lo], [lo + 2 * n])
    esq.set_param("bucket_cap", 0)
    return (f[1000] - f[500]) / 2000


def test_default_values_are_taken_as_set_where_nothing_adapts(as_set):
    """Segments of 2^18 for a short per-n call (128 of 2^14 otherwise), four runs
    a workgroup for a batch (twelve otherwise), and the same results."""
    lo, n = (1 << 49) + 1, 1 << 21
    assert segments_of_a_call(lo, n) == pytest.approx(9, abs=0.3)
    ivs = [lo + (i << 28) for i in range(4096)], [lo + (i << 28) + (1 << 27) for i in range(4096)]
    esq.set_param("bucket_cap", 64)
    equal = esq.scratch_bytes(*ivs)
    esq.set_param("adapt", 1)
    runs = esq.scratch_bytes(*ivs)
    esq.set_param("bucket_cap", 0)
    assert runs - equal > 16 * 4000
    assert segments_of_a_call(lo, n) > 120

    def results():
        p = esq.verify_range(lo, lo + 2 * n, per_n=True)
        return (p.pop("per_n"), esq.sieve_segment(lo, lo + (1 << 21))[2], p,
                esq.verify_range(lo, lo + (1 << 34)), noalloc_call(lo, lo + 2 * n, 3, False, 16))
    adapted = results()
    esq.set_param("adapt", 0)
    for a, b in zip(adapted, results()):
        assert torch.equal(a, b) if torch.is_tensor(a) else a == b
