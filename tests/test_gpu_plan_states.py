"""GPU tests of a batch plan's states: a result before the first run, after a
batch whose upload was reported as failed and after a copy that was, and runs of
a plan that outlives its system."""
import ctypes

import numpy as np
import pytest

import oracle
import workloads

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sess():
    from paper_1709_07781_amd.session import Session
    s = Session()
    yield s
    s.close()


def _check(got, off, v):
    o = oracle.default()
    assert len(got) == len(off) - 1
    for j, g in enumerate(got):
        for a, e in zip(g, o.wah_index(v[off[j]:off[j + 1]])):
            np.testing.assert_array_equal(a, e)


def _batch(seed, sizes, bits):
    off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.uint32)
    return off, workloads.uniform_values(seed, int(off[-1]), 1 << bits)


@pytest.mark.parametrize("cap,nreq,largest", [(100_000, 64, 1024), (100_000, 64, 0), (5, 1, 0), (4_000_000, 700, 0)])
def test_any_batch_plan_starts_with_an_empty_batch(sess, cap, nreq, largest):
    """Each capacity's result before the first run is that of no requests, by the staged copy and (4,000,000
    values, whose run is held to the same afterwards) by the plain one."""
    from paper_1709_07781_amd.session import BatchPlan
    plan = BatchPlan(sess, None, 8, any_batch=(cap, nreq, largest))
    try:
        assert plan.result() == []
        plan.run()  # the empty batch itself
        assert plan.result() == []
        off, v = _batch(7, [3, 0, 2][:nreq] if cap < 100 else [900, 0, 1000, 31], 8)
        plan.run_batch(v, off)
        _check(plan.result(), off, v)
        if cap >= 4_000_000:
            off, v = _batch(8, [1_500_000, 5, 1_400_000], 8)
            plan.run_batch(v, off)
            _check(plan.result(), off, v)
    finally:
        plan.close()


def test_fixed_plan_has_no_result_before_its_run(sess):
    import paper_1709_07781_amd as ka
    from paper_1709_07781_amd.session import BatchPlan
    off, v = _batch(9, [100, 2000], 8)
    plan = BatchPlan(sess, off, 8)
    try:
        with pytest.raises(ka.KaError) as e:
            plan.result()
        assert e.value.code == ka.KA_E_STATE
        plan.run(v)
        _check(plan.result(), off, v)
    finally:
        plan.close()


def _leave_error():
    """A failed call of this thread whose error the next check of a launch reports; False if HIP keeps none."""
    import torch
    import paper_1709_07781_amd as ka
    torch.cuda.synchronize()
    dev = ctypes.c_int()
    ka.lib.hipGetDevice(ctypes.byref(dev))
    assert ka.lib.hipSetDevice(9999) != 0
    return ka.lib.hipGetDevice(ctypes.byref(dev)) == 0 and ka.lib.hipPeekAtLastError() != 0


@pytest.mark.parametrize("second", [[40, 7], [1000, 1000, 1000, 1000, 1000]])
def test_failed_upload_keeps_the_last_batch(sess, second):
    """A batch (smaller, larger) that was reported as failed leaves the last one's result as it was, and the next
    batch is exact."""
    import paper_1709_07781_amd as ka
    from paper_1709_07781_amd.session import BatchPlan
    off1, v1 = _batch(11, [900, 0, 800], 8)
    off2, v2 = _batch(12, second, 8)
    plan = BatchPlan(sess, None, 8, any_batch=(10_000, 16, 1024))
    try:
        plan.run_batch(v1, off1)
        _check(plan.result(), off1, v1)
        if not _leave_error():
            ka.lib.hipGetLastError()
            pytest.skip("no error is kept past a call that succeeds")
        with pytest.raises(ka.KaError):
            plan.run_batch(v2, off2)
        _check(plan.result(), off1, v1)
        with pytest.raises(ka.KaError) as e:  # the table on the device may be the failed batch's
            plan.run()
        assert e.value.code == ka.KA_E_STATE
        plan.run_batch(v2, off2)
        _check(plan.result(), off2, v2)
    finally:
        plan.close()


def test_result_after_a_failed_copy(sess):
    """A copy of the outputs that was reported as failed may have been queued: its pinned memory is not handed out
    before the plan's stream has passed it, and the next result is exact."""
    import torch
    import paper_1709_07781_amd as ka
    from paper_1709_07781_amd.session import BatchPlan
    off, v = _batch(13, [200_000, 3, 100_000], 8)
    plan = BatchPlan(sess, off, 8)
    try:
        plan.run(v)
        plan.result()
        if not _leave_error():
            ka.lib.hipGetLastError()
            pytest.skip("no error is kept past a call that succeeds")
        for _ in range(300):  # keeps the stream busy for longer than the call takes
            plan.run()
        with pytest.raises(ka.KaError):
            plan.result()
        assert torch.cuda.ExternalStream(plan.stream_handle()).query()
        _check(plan.result(), off, v)
    finally:
        plan.close()


def _device_maps_mb():
    """What the device driver has mapped into the process (pinned host memory among it)."""
    total = 0
    with open("/proc/self/maps") as f:
        for line in f:
            if "/dev/dri/" in line:
                lo, hi = line.split()[0].split("-")
                total += int(hi, 16) - int(lo, 16)
    return total / 2 ** 20


def test_plan_outlives_its_system():
    """A plan whose system was destroyed still takes host values and returns host results, and pins no memory
    that stays behind when it is closed: six such plans leave no more mapped than six closed before their systems
    (they left 6 MB a plan)."""
    from paper_1709_07781_amd.session import BatchPlan, Session
    off, v = _batch(14, [200_000, 1, 190_000], 12)
    small_off, small_v = _batch(15, [7, 300], 12)
    grown = []
    for close_first in (False, True):
        for rep in range(8):
            if rep == 2:
                before = _device_maps_mb()
            s = Session()
            fixed = BatchPlan(s, off, 12)
            any_plan = BatchPlan(s, None, 12, any_batch=(400_000, 8, 0))
            any_plan.run_batch(small_v, small_off)
            if close_first:
                s.close()
            _check(any_plan.result(), small_off, small_v)
            any_plan.run_batch(v, off)
            fixed.run(v)
            a, b = fixed.result(), any_plan.result()
            if rep == 0:
                _check(a, off, v)
                _check(b, off, v)
            fixed.close()
            any_plan.close()
            if not close_first:
                s.close()
        grown.append(_device_maps_mb() - before)
    print("mapped:", grown)
    assert grown[1] < grown[0] + 12.0
