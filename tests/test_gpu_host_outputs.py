"""GPU test of host indexes whose outputs could take more than 8 MiB and do or do
not: up to 8 MiB they are staged once their lengths are known, above they are
read one by one."""
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


def _runs(seed, n, bits, run):
    return np.repeat(workloads.uniform_values(seed, n // run + 1, 1 << bits), run)[:n]


# (values, bits, run length, hint, smallest and largest bytes out)
@pytest.mark.parametrize("n,bits,run,hint,lo,hi", [
    (1 << 20, 8, 200, 0, 0, 1 << 20),          # capacities 16 MiB, unhinted
    (1_500_001, 4, 100, 4, 0, 1 << 20),        # 12 MB, nearly all of it words
    (1_048_001, 12, 1, 12, 7 << 20, 8 << 20),  # just below the limit
    (1_250_000, 12, 1, 12, (8 << 20) + 1, 11 << 20),  # above it
])
def test_outputs_below_and_above_the_staged_size(sess, n, bits, run, hint, lo, hi):
    v = _runs(3, n, bits, run)
    exp = oracle.default().wah_index(v)
    assert lo <= sum(e.nbytes for e in exp) <= hi
    for values in (v, sess.upload(v)):
        for _ in range(2):
            for g, e in zip(sess.wah_index(values, value_bits=hint), exp):
                np.testing.assert_array_equal(g, e)


def test_rejected_index_of_large_capacity(sess):
    import paper_1709_07781_amd as ka
    v = _runs(4, 2_000_000, 8, 100)
    v[1_999_999] = 1 << 8
    with pytest.raises(ka.KaError) as e:
        sess.wah_index(v, value_bits=8)
    assert e.value.code == ka.KA_E_ARG
