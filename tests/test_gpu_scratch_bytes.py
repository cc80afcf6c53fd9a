"""esq_scratch_bytes, by which a server admits: its figure is what a call takes,
and asking for it costs less than making the call."""
import time

import pytest
import torch

from paper_2411_01964_amd import esq, workloads
from tests.test_gpu_parity import DEFAULTS, MAX_HI, knobs
from tests.test_zz_no_alloc import noalloc_call

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def lib_ready():
    esq.init(0, MAX_HI)
    knobs()
    yield
    for k, v in DEFAULTS.items():
        esq.set_param(k, v)


def refused(lo, hi, per_n):
    """Whether the no-alloc call finds its static array too small."""
    try:
        noalloc_call(lo, hi, per_n=per_n)
        return False
    except AssertionError:
        assert b"ESQ_NOALLOC_SCRATCH_MAX" in esq.lib().esq_last_error()
        return True


@pytest.mark.parametrize("kw", [dict(medium_max=11), dict(medium_max=11, seg_log2=17), dict(bucket_cap=4096)])
def test_the_figure_is_what_the_larger_form_of_a_call_takes(kw):
    """Around the longest interval below 2^50 whose figure fits the static array:
    up to it the no-alloc call takes both forms, past it it refuses one."""
    knobs(**kw)
    hi, limit = 1 << 50, esq.ESQ_NOALLOC_SCRATCH_MAX
    a, b = 1 << 18, 1 << 34
    while b - a > 1:
        mid = (a + b) // 2
        a, b = (mid, b) if esq.scratch_bytes([hi - 2 * mid + 1], [hi]) <= limit else (a, mid)
    assert not refused(hi - 2 * a + 1, hi, False) and not refused(hi - 2 * a + 1, hi, True)
    assert refused(hi - 2 * b + 1, hi, False) or refused(hi - 2 * b + 1, hi, True)
    knobs()


@pytest.mark.parametrize("count", [300, 4096])
def test_asking_costs_less_than_the_call(count):
    lo, hi = workloads.batch_intervals(seed=4, count=count, log2_len=(12, 16))

    def best(f):
        t = []
        for _ in range(20):
            t0 = time.perf_counter()
            f()
            t.append(time.perf_counter() - t0)
            torch.cuda.synchronize()
        return min(t)

    ask, call = best(lambda: esq.scratch_bytes(lo, hi)), best(lambda: esq.verify_batch_async(lo, hi))
    print("%d intervals: asking %.1f us, enqueueing %.1f us" % (count, ask * 1e6, call * 1e6))
    assert ask < call
