"""GPU tests of rejected requests in a served batch: values far beyond a small
value_bits, which device-resident requests can hold, leave every request
batched with them exact (the batch's tables are sized by 2^value_bits)."""
import numpy as np
import pytest

import oracle
import workloads

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sess():
    from paper_1709_07781_amd.session import Session
    s = Session(n_streams=2)
    yield s
    s.close()


# one work-group per request; the segmented sort in one and in two passes of even digits
@pytest.mark.parametrize("size", [1000, 3000, 20_000])
@pytest.mark.parametrize("bits", [1, 4, 5, 7, 9, 12])
def test_requests_beyond_small_value_bits_fail_alone(sess, bits, size):
    import paper_1709_07781_amd as ka
    from paper_1709_07781_amd.session import Server
    ora = oracle.default()
    good = [workloads.uniform_values(40 + i, size - 13 * i, 1 << bits) for i in range(4)]
    bad = [workloads.u32(50, size),  # any uint32, nearly all distinct
           np.arange(size, dtype=np.uint32) + np.uint32(1 << bits)]
    held = []
    srv = Server(sess, streams=1, max_batch=64, value_bits=bits)
    try:
        for b in bad:
            t = sess.upload(b)
            held.append((sess.wrap(t), t))
        scan = workloads.u32(60, 8 << 20)
        first = srv.send(workloads.KIND_SCAN, scan)  # keeps the server busy while the others are sent
        sent = [srv.send(workloads.KIND_WAH, x) for x in (good[0], held[0][0], good[1], held[1][0], good[2], good[3])]
        (got,) = sess.receive(first, 1)
        sess.release_ticket(first)
        np.testing.assert_array_equal(got, ora.exclusive_scan(scan))
        for i, t in enumerate(sent):
            if i in (1, 3):
                with pytest.raises(ka.KaError) as e:
                    sess.receive(t, 3)
                assert e.value.code == ka.KA_E_ARG
            else:
                exp = ora.wah_index(good[{0: 0, 2: 1, 4: 2, 5: 3}[i]])
                for g, x in zip(sess.receive(t, 3), exp):
                    np.testing.assert_array_equal(g, x, err_msg=f"request {i}")
            sess.release_ticket(t)
        assert srv.stats()["mean_batch"] > 1.5  # merged: in two batches but for a slow host
    finally:
        srv.close()
        for r, _ in held:
            sess.release_ref(r)
