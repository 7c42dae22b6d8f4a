"""GPU test of compactions around the size where the tile and the loads change."""
import numpy as np
import pytest

import workloads

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [(1 << 25) + 1, 3 << 24, (3 << 24) + 1, (3 << 24) + 16_389])
def test_compaction_at_the_large_limit(n):
    import paper_1709_07781_amd as ka
    from paper_1709_07781_amd.session import Session
    s = Session()
    try:
        x = np.tile(workloads.u32(5, 1 << 20), n // (1 << 20) + 1)[:n]
        x[x % 3 == 0] = 0
        r = s.wrap(s_x := s.upload(x))
        act = s.spawn("compact_nonzero_u32", [ka.arg(ka.KA_IN), ka.arg(ka.KA_OUT, out_mode=ka.KA_VAL)])
        (got,) = s.request(act, ka.ref(r), n_out=1)
        np.testing.assert_array_equal(got, x[x != 0])
        s.release_actor(act)
        s.release_ref(r)
        del s_x
    finally:
        s.close()
