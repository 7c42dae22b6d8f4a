"""GPU parity of the index build's size-dependent paths at the sizes where one hands over to the
next and around their tiles, in every word format, against the oracle (bit-exact)."""
import os

import numpy as np
import pytest

import oracle
import workloads

pytestmark = pytest.mark.gpu

ENC_TILE = 8192


@pytest.fixture(scope="module")
def sess():
    from paper_1709_07781_amd.session import Session
    s = Session()
    yield s
    s.close()


@pytest.fixture(scope="module")
def impatient():
    """A system whose look-backs take the fallback at every stall."""
    from paper_1709_07781_amd.session import Session
    old = os.environ.get("KA_LOOKBACK_SPIN")
    os.environ["KA_LOOKBACK_SPIN"] = "1"
    try:
        s = Session()
        s.wah_index(np.arange(5, dtype=np.uint32))  # the variable is read on first use of the device
    finally:
        if old is None:
            del os.environ["KA_LOOKBACK_SPIN"]
        else:
            os.environ["KA_LOOKBACK_SPIN"] = old
    yield s
    s.close()


def expected(v, fmt):
    o = oracle.default()
    return o.wah_index_format(v, fmt) if fmt else o.wah_index(v)


def check(sess, v, bits, fmt):
    got = sess.wah_index(sess.upload(v), refs=False, value_bits=bits, fmt=fmt)
    for g, e, what in zip(got, expected(v, fmt), ("keys", "offsets", "words")):
        np.testing.assert_array_equal(g, e, err_msg=f"{what} n={v.size} bits={bits} fmt={fmt}")


def columns(n):
    """Columns whose bitmaps have long runs of full groups, runs followed by a group of 30 rows (the missing
    row at each place in turn), single rows after gaps, and everyday ones."""
    r = np.arange(n, dtype=np.int64)
    long_runs = np.where((r // 31) % 600 < 590, 3, 9).astype(np.uint32)
    thirty = np.full(n, 2, np.uint32)
    thirty[(r // 31) % 5 == 4] = 1
    thirty[((r // 31) % 5 == 3) & (r % 31 == (r // 155) % 31)] = 7
    thirty[r % 1031 == 1000] = 11
    return {"long_runs": long_runs, "thirty": thirty, "clusters": (workloads.u32(n, n) % 5 != 0).cumsum(
        dtype=np.int64).astype(np.uint32) // 200 % 50, "zipf": workloads.zipf_values(n + 1, n, 1.1, 1 << 12)}


@pytest.mark.parametrize("fmt", [1, 2])
@pytest.mark.parametrize("n", [ENC_TILE - 1, ENC_TILE + 30, 2 * ENC_TILE + 31, 5 * ENC_TILE - 29])
def test_formats_around_tiles(sess, fmt, n):
    """Runs, 30-row groups and gaps that cross the encoder's tiles, over uint32 and uint16 sorted keys."""
    for v in columns(n).values():
        check(sess, v, 0, fmt)
        check(sess, v, 12, fmt)


@pytest.mark.parametrize("fmt", [1, 2])
def test_formats_with_fallback(impatient, fmt):
    n = 300 * ENC_TILE + 77
    for v in columns(n).values():
        check(impatient, v, 12, fmt)
