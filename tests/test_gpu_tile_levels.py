"""GPU test of AND / OR over more tiles than a tile walks over: nearly empty and
nearly full results, whose fills and runs begin and end in other tiles, blocks
of 64 tiles and blocks of 4096, against the oracle."""
import ctypes

import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

TILE, FULL = 2048, 0x7FFFFFFF
MANY = 4096 * TILE  # groups in the most tiles without levels


@pytest.fixture(scope="module")
def sess():
    from paper_1709_07781_amd.session import Session
    s = Session()
    yield s
    s.close()


def _words(base, at, values, ng, fmt):
    """The bitmap of ng groups `base` (0 or full) but for values at the ascending groups `at`, in a format."""
    length = 0x1FFFFFF if fmt == 2 else 0x3FFFFFFF
    if base == 0:
        at, values = at[values != 0], values[values != 0]
        zero = np.zeros(at.size, np.uint32)
        return oracle.default().wah_encode_groups(zero, at.astype(np.uint32), values, fmt)[2] if at.size else zero
    out, g = [], 0
    for p, v in list(zip(at.tolist(), values.tolist())) + [(ng, None)]:  # full runs and literals, unfused: still decodable
        while p > g:
            n = min(p - g, length)
            out.append(0xC0000000 | n)
            g += n
        if v is not None:
            out.append(v if v else 0x80000001)
            g += 1
    return np.array(out, np.uint32)


def _positions(ng, seed):
    rng = np.random.default_rng(seed)
    edges = [0, TILE - 1, TILE, 64 * TILE - 1, 64 * TILE, 65 * TILE, MANY - 1, MANY, MANY + 64 * TILE, ng - 1]
    at = [e for e in edges if rng.random() < 0.6] + rng.integers(0, ng, 3).tolist()
    return np.unique(np.array(at, np.int64)[np.array(at) < ng])


@pytest.mark.parametrize("seed,ng", [(1, MANY), (2, MANY + 1), (3, MANY + 64 * TILE + 5), (4, 2 * MANY + 130 * TILE)])
@pytest.mark.parametrize("fin,fout", [(1, 0), (1, 1), (2, 2), (1, 2)])
def test_nearly_empty_and_nearly_full_results(sess, ng, fin, fout, seed):
    import paper_1709_07781_amd as ka
    rng = np.random.default_rng(seed)
    ora = oracle.default()

    def values(k, zeros):
        v = rng.integers(1, FULL + 1, k).astype(np.uint32)
        v[rng.random(k) < 0.3] = FULL & ~(1 << 4)  # one row missing, one row present, empty
        v[rng.random(k) < 0.3] = 1 << 9
        if zeros:
            v[rng.random(k) < 0.3] = 0
        return v

    def bitmap(base):
        at = _positions(ng, int(rng.integers(1 << 30)))
        return _words(base, at, values(at.size, base != 0), ng, fin)

    empty1, empty2, full1, full2, none = bitmap(0), bitmap(0), bitmap(FULL), bitmap(FULL), np.zeros(0, np.uint32)
    cases = [(empty1, empty2, 1), (empty1, full1, 0), (none, full2, 0), (empty2, none, 1)]
    if fout:  # nearly full results are literals in the paper's form: as many words as groups
        cases += [(full1, full2, 0), (full1, empty1, 1), (full2, none, 1)]
    for a, b, op in cases:
        act = sess.spawn("wah_combine", [ka.arg(ka.KA_IN, in_mode=ka.KA_VAL), ka.arg(ka.KA_IN, in_mode=ka.KA_VAL),
                                         ka.arg(ka.KA_PRIV, count=4, init=(ctypes.c_uint32 * 4)(op, fin, fout, ng)),
                                         ka.arg(ka.KA_OUT, out_mode=ka.KA_VAL)])
        (got,) = sess.request(act, *(ka.val(x.ctypes.data if x.size else None, x.size) for x in (a, b)), n_out=1)
        sess.release_actor(act)
        np.testing.assert_array_equal(got, ora.wah_combine(a, b, fin, ng, op, fout))
