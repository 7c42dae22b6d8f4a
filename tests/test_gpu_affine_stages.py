"""GPU parity of composed affine actors, whose consecutive stages run as one launch: lengths around the 16 stages of
one pass, nested compositions, a repeated actor, sub-ranges, device-resident counts and mapping functions between
stages, against the stages applied one after another in numpy."""
import ctypes

import numpy as np
import pytest

import workloads

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sess():
    from paper_1709_07781_amd.session import Session
    s = Session()
    yield s
    s.close()


def staged(x, params):
    x = x.copy()
    for a, b in params:
        x = x * np.uint32(a) + np.uint32(b)
    return x


def params_of(k):
    a, b = workloads.affine_params(900 + k, k)
    return [(int(p), int(q)) for p, q in zip(a, b)]


def chain_of(sess, actors, balanced=False):
    """The composition of actors, first to last; balanced: halves composed first (an inner composition is a stage)."""
    if len(actors) == 1:
        return actors[0], []
    if balanced:
        h = len(actors) // 2
        (x, cx), (y, cy) = chain_of(sess, actors[:h], True), chain_of(sess, actors[h:], True)
        c = sess.compose(y, x)
        return c, cx + cy + [c]
    c, made = actors[0], []
    for a in actors[1:]:
        c = sess.compose(a, c)
        made.append(c)
    return c, made


@pytest.mark.parametrize("k", [1, 2, 16, 17, 33])
@pytest.mark.parametrize("n", [1, 4097])
@pytest.mark.parametrize("balanced", [False, True])
def test_stage_counts(sess, k, n, balanced):
    import paper_1709_07781_amd as ka
    x, p = workloads.u32(n + k, n), params_of(k)
    acts = [sess.affine_actor(a, b) for a, b in p]
    c, made = chain_of(sess, acts, balanced)
    t = sess.upload(x)
    r = sess.wrap(t)
    for want in (staged(x, p), staged(staged(x, p), p)):  # in place: the second request goes on from the first
        (o,) = sess.request(c, ka.ref(r), n_out=1)
        np.testing.assert_array_equal(sess.read(o), want)
        sess.release_ref(o)
    sess.release_ref(r)
    for a in made + acts:
        sess.release_actor(a)


def test_repeated_actor_and_other_ranges(sess):
    """An actor that occurs twice, and neighbours over another index space, which are not one run."""
    import paper_1709_07781_amd as ka
    n, off, m = 10_000, 1003, 5001
    x = workloads.u32(7, n)
    (a, b), (c, d) = params_of(2)
    ca, cb = (ctypes.c_uint32 * 1)(c), (ctypes.c_uint32 * 1)(d)
    whole = sess.affine_actor(a, b)
    part = [sess.spawn("affine_u32", [ka.arg(ka.KA_IN_OUT), ka.arg(ka.KA_PRIV, count=1, init=ca),
                                      ka.arg(ka.KA_PRIV, count=1, init=cb)],
                       rng=ka.nd_range(m, off)) for _ in range(2)]
    c_, made = chain_of(sess, [whole, whole, part[0], part[1], whole])
    t = sess.upload(x)
    r = sess.wrap(t)
    (o,) = sess.request(c_, ka.ref(r), n_out=1)
    want = staged(x, [(a, b)] * 2)
    want[off:off + m] = staged(want[off:off + m], [(c, d)] * 2)
    want = staged(want, [(a, b)])
    np.testing.assert_array_equal(sess.read(o), want)
    for q in (o, r):
        sess.release_ref(q)
    for q in made + part + [whole]:
        sess.release_actor(q)


def test_count_on_the_device(sess):
    import paper_1709_07781_amd as ka
    x = workloads.u32(8, 9000) % 3
    p = params_of(3)
    acts = [sess.affine_actor(a, b) for a, b in p]
    comp = sess.spawn("compact_nonzero_u32", [ka.arg(ka.KA_IN, in_mode=ka.KA_VAL), ka.arg(ka.KA_OUT)])
    c, made = chain_of(sess, [comp] + acts)
    (o,) = sess.request(c, ka.val(x.ctypes.data, x.size), n_out=1)
    np.testing.assert_array_equal(sess.read(o), staged(x[x != 0], p))
    sess.release_ref(o)
    for q in made + acts + [comp]:
        sess.release_actor(q)


def test_mapping_between_stages(sess):
    """A mapping function on a stage runs at its place: such a stage is none of a run."""
    import paper_1709_07781_amd as ka
    n = 500
    x, p = workloads.u32(9, n), params_of(4)
    acts = [sess.affine_actor(a, b) for a, b in p]
    calls = []

    @ka.ka_map_fn
    def post(vals, n_in, outs, n_out, cap, ud):
        calls.append(n_in)
        for i in range(n_in):
            outs[i] = vals[i]
        n_out[0] = n_in
        return 0

    ka.check(ka.lib.ka_actor_set_mapping(acts[1], ka.ka_map_fn(), post, None), "ka_actor_set_mapping")
    c, made = chain_of(sess, acts)
    t = sess.upload(x)
    r = sess.wrap(t)
    (o,) = sess.request(c, ka.ref(r), n_out=1)
    np.testing.assert_array_equal(sess.read(o), staged(x, p))
    assert calls == [1]
    for q in (o, r):
        sess.release_ref(q)
    for q in made + acts:
        sess.release_actor(q)
