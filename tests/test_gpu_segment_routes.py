"""GPU test of the segmented sort's two forms of digit counts (rows summed by each
tile, a scanned table) at the request sizes between them, with digits of 8 bits
and fewer, over uniform and clustered keys."""
import numpy as np
import pytest

import oracle
import workloads

pytestmark = pytest.mark.gpu

TILE = 8192


@pytest.fixture(scope="module")
def sess():
    from paper_1709_07781_amd.session import Session
    s = Session()
    yield s
    s.close()


def _values(n, bits, clustered, seed):
    v = workloads.uniform_values(seed, n // 50 + 2 if clustered else n, 1 << bits)
    return np.repeat(v, 50)[7:n + 7].copy() if clustered else v


def _check(got, off, v):
    for j, g in enumerate(got):
        for a, e in zip(g, oracle.default().wah_index(v[off[j]:off[j + 1]])):
            np.testing.assert_array_equal(a, e, err_msg=f"request {j}")


@pytest.mark.parametrize("clustered", [False, True])
@pytest.mark.parametrize("bits", [8, 12, 14, 15, 16])
@pytest.mark.parametrize("largest", [16 * TILE, 16 * TILE + 1, 128 * TILE, 128 * TILE + 1])
def test_requests_at_the_row_limits(sess, bits, largest, clustered):
    """Batches of more than 384 tiles whose largest request is at a limit, empty requests and shared tiles among
    them."""
    sizes = [largest, 0, 5000, 1]
    while sum(sizes) <= 390 * TILE:
        sizes += [min(largest, 70_001), 3]
    off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.uint32)
    v = _values(int(off[-1]), bits, clustered, bits + largest)
    _check(sess.wah_batch(sess.upload(v), off, bits), off, v)


@pytest.mark.parametrize("shape", [0, 1, 3])
@pytest.mark.parametrize("bits", [8, 12, 16])
def test_clustered_keys_in_every_form(sess, bits, shape):
    """Few tiles (rows): the even and the byte digit split, and the tagged sort."""
    from paper_1709_07781_amd.session import BatchPlan
    sizes = [3000, 100_003, 0, 8192, 1, 40_000]
    off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.uint32)
    plan = BatchPlan(sess, off, bits, shape=shape)
    try:
        for seed in (1, 2):
            v = _values(int(off[-1]), bits, True, seed)
            plan.run(v)
            _check(plan.result(), off, v)
    finally:
        plan.close()


@pytest.mark.parametrize("nreq", [1, 1023, 1024, 1025, 2500])
def test_requests_laid_out_by_one_and_by_many_work_groups(sess, nreq):
    """The batch's layout on both sides of its limit, eager and in a plan of that many requests, of which a batch may
    have fewer."""
    from paper_1709_07781_amd.session import BatchPlan
    rng = np.random.default_rng(nreq)
    sizes = rng.integers(0, 40, nreq)
    sizes[rng.integers(0, nreq, 3)] = [1025, 9000, 20_000]
    off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.uint32)
    v = _values(int(off[-1]), 12, False, nreq)
    _check(sess.wah_batch(sess.upload(v), off, 12), off, v)
    plan = BatchPlan(sess, None, 12, any_batch=(int(off[-1]), nreq, 0))
    try:
        for k in (nreq, max(1, nreq // 2), nreq):
            plan.run_batch(v[: off[k]], off[: k + 1])
            _check(plan.result(), off[: k + 1], v)
    finally:
        plan.close()
