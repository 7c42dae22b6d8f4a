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


SMALL_MAX = 8192


@pytest.mark.parametrize("fmt", [0, 1, 2])
@pytest.mark.parametrize("n", [1, 63, 1024, 1025, 2049, 4096, 4097, SMALL_MAX - 1, SMALL_MAX, SMALL_MAX + 1])
def test_small_inputs(sess, fmt, n):
    """One work-group's sort and encode: each count of values per work-item, digits that start at any bit, equal
    values, all values distinct."""
    u = workloads.u32(n + fmt, n)
    cases = [(u % 1024, 10), (u, 0), (u & np.uint32(0x00FFF000), 24), (np.full(n, 1 << 31, np.uint32), 32),
             (np.arange(n, dtype=np.uint32)[::-1].copy(), 14), (columns(n)["thirty"], 8)]
    for v, bits in cases:
        check(sess, v.astype(np.uint32), bits, fmt)


@pytest.mark.parametrize("bits", [1, 9, 16, 31])
def test_small_input_beyond_its_hint(sess, bits):
    from paper_1709_07781_amd import KaError
    v = np.zeros(5000, np.uint32)
    v[4999] = 1 << bits
    with pytest.raises(KaError):
        sess.wah_index(v, value_bits=bits)
    v[4999] -= 1
    check(sess, v, bits, 0)


# capacities where the sort's tile grows (1024, 2048, 4096, 8192 keys) and where its digit counts are scanned instead
# of summed by every tile (by digit width), with the encoder's tiles of 2048, 4096 and 8192 pairs
SORT_EDGES = [1 << 18, 1 << 19, 1 << 20, 352 << 13, 1 << 22]


@pytest.mark.parametrize("n", [SMALL_MAX + 1, 70_001] + [e + d for e in SORT_EDGES for d in (0, 1)])
def test_sort_tile_shapes(sess, n):
    """Every digit width (2, 4, 6, 8 bits, one and two passes), skipped passes of unhinted values, skewed values."""
    u = workloads.u32(n, n)
    z = workloads.zipf_values(n, n, 1.1, 1 << 16)
    for bits in (1, 4, 7, 12, 16):
        check(sess, (u & np.uint32((1 << bits) - 1)), bits, 0)
    check(sess, z, 16, 0)
    if n <= (1 << 21) + 1:
        check(sess, (u & np.uint32(0xFF00FF)), 0, 0)
        check(sess, z, 20, 2)


@pytest.mark.parametrize("n", [513 * 8192 + 1, 2050 * 8192 - 5])
def test_scanned_digit_rows(sess, n):
    """Tiles whose row is the scanned one or up to three after it, both widths of the scan, and skipped passes."""
    u = workloads.u32(n, n)
    check(sess, u & np.uint32(0xFFF), 12, 0)
    check(sess, u & np.uint32(0x3FF00FF), 0, 0)
    check(sess, np.where(u % 64 == 0, u & np.uint32(0xFFFF), np.uint32(7)), 16, 0)


@pytest.mark.parametrize("cap,n", [(4_300_000, 4_200_001), (4_300_000, 9), (300_000, 299_000), (300_000, 5), (300_000, 0), (6000, 17), (6000, 0)])
@pytest.mark.parametrize("bits", [0, 12])
def test_counts_on_the_device(sess, cap, n, bits):
    """The same paths behind a compaction: the grid covers its capacity, the count is read on the device."""
    import ctypes
    import paper_1709_07781_amd as ka
    x = np.zeros(cap, np.uint32)
    x[np.sort(workloads.u32(cap + n, cap).argsort(kind="stable")[:n])] = workloads.u32(3, n) % 4095 + 1
    priv = (ctypes.c_uint32 * 1)(bits)
    comp = sess.spawn("compact_nonzero_u32", [ka.arg(ka.KA_IN, in_mode=ka.KA_VAL), ka.arg(ka.KA_OUT)])
    idx = sess.spawn("wah_index", [ka.arg(ka.KA_IN), ka.arg(ka.KA_PRIV, count=1, init=priv)] +
                     [ka.arg(ka.KA_OUT, out_mode=ka.KA_VAL)] * 3)
    both = sess.compose(idx, comp)
    got = sess.request(both, ka.val(x.ctypes.data, x.size), n_out=3)
    for a in (both, comp, idx):
        sess.release_actor(a)
    for g, e in zip(got, oracle.default().wah_index(x[x != 0])):
        np.testing.assert_array_equal(g, e)


@pytest.mark.parametrize("n", [3000, 40_000])
def test_lengths_of_requests_in_flight(sess, n):
    """Lengths that arrive on the host: requests queued before any is received, some dropped unread (their words
    are reused by later requests while the kernels may still have to write them), lengths read in any order."""
    import ctypes
    import paper_1709_07781_amd as ka
    priv = (ctypes.c_uint32 * 1)(10)
    idx = sess.spawn("wah_index", [ka.arg(ka.KA_IN), ka.arg(ka.KA_PRIV, count=1, init=priv)] + [ka.arg(ka.KA_OUT)] * 3)
    cols = [workloads.uniform_values(50 + i, n - 7 * i, 3 + 90 * i) for i in range(9)]
    dev = [sess.upload(c) for c in cols]
    refs = [sess.wrap(d) for d in dev]
    for round_ in range(3):
        tickets = [sess.send(idx, ka.ref(r)) for r in refs]
        for i in (0, 3, 4):
            sess.release_ticket(tickets[i])
        more = [sess.send(idx, ka.ref(refs[i])) for i in (8, 7, 6)]
        todo = [(i, tickets[i]) for i in (8, 1, 7, 2, 6, 5)] + list(zip((8, 7, 6), more))
        for i, t in todo:
            got = sess.receive(t, 3)
            sess.release_ticket(t)
            for g, e in zip(got, oracle.default().wah_index(cols[i])):
                np.testing.assert_array_equal(sess.read(g), e)
                sess.release_ref(g)
    for r in refs:
        sess.release_ref(r)
    sess.release_actor(idx)


GROUP_TILE = 2048  # groups per tile of the decoder and of the AND / OR


def bitmap(groups, fmt):
    """The words of a bitmap given as 31-bit groups, by the oracle's own encoder."""
    bits = ((groups[:, None] >> np.arange(31, dtype=np.uint32)) & 1).astype(np.uint32).ravel()
    bits = np.append(bits, np.uint32(0))  # value 0 exists too: it sorts first
    keys, off, words = expected(bits, fmt)
    d = int(np.searchsorted(keys, 1))
    return words[off[d]:off[d + 1]].copy() if d < keys.size and keys[d] == 1 else np.zeros(0, np.uint32)


def group_patterns(ng):
    """Bitmaps with fills and runs of full groups longer than tiles, ending and starting at their edges, groups of 30
    rows after runs and of one row after gaps."""
    full, i = np.uint32(0x7FFFFFFF), np.arange(ng)
    sparse = np.zeros(ng, np.uint32)
    sparse[[0, ng // 2, ng - 1]] = [1, 1 << 30, 6]
    runs = np.where((i // (GROUP_TILE + 1)) % 2 == 0, full, 0).astype(np.uint32)
    runs[GROUP_TILE - 1::GROUP_TILE] = full ^ np.uint32(1 << 7)
    ones = np.full(ng, full)
    mixed = workloads.u32(ng, ng) & full
    mixed[(i % 7) < 4] = 0
    mixed[(i % 53) > 40] = full
    mixed[(i % 53) == 52] = full ^ np.uint32(1)
    return [sparse, runs, ones, mixed]


@pytest.mark.parametrize("fmt", [0, 1, 2])
@pytest.mark.parametrize("ng", [1, 7, GROUP_TILE - 1, GROUP_TILE + 1, 5 * GROUP_TILE, 70 * GROUP_TILE + 9])
def test_bitmap_queries_around_tiles(sess, fmt, ng):
    """Decode, AND and OR of bitmaps around the tile of groups; 70 tiles: more than one window of summaries."""
    import ctypes
    import paper_1709_07781_amd as ka
    pats = group_patterns(ng)
    words = [bitmap(p, fmt) for p in pats]
    val = lambda w: ka.val(w.ctypes.data if w.size else None, w.size)  # noqa: E731
    dec = sess.spawn("wah_decode", [ka.arg(ka.KA_IN, in_mode=ka.KA_VAL),
                                    ka.arg(ka.KA_PRIV, count=2, init=(ctypes.c_uint32 * 2)(fmt, ng)),
                                    ka.arg(ka.KA_OUT, out_mode=ka.KA_VAL)])
    for p, w in zip(pats, words):
        (g,) = sess.request(dec, val(w), n_out=1)
        np.testing.assert_array_equal(g, p)
    sess.release_actor(dec)
    for op in (0, 1):
        for fout in (0, 1, 2):
            act = sess.spawn("wah_combine", [ka.arg(ka.KA_IN, in_mode=ka.KA_VAL), ka.arg(ka.KA_IN, in_mode=ka.KA_VAL),
                                             ka.arg(ka.KA_PRIV, count=4, init=(ctypes.c_uint32 * 4)(op, fmt, fout, ng)),
                                             ka.arg(ka.KA_OUT, out_mode=ka.KA_VAL)])
            for i, j in ((0, 1), (1, 2), (3, 1), (3, 0), (2, 2), (3, 3)):
                (o,) = sess.request(act, val(words[i]), val(words[j]), n_out=1)
                want = bitmap(pats[i] | pats[j] if op else pats[i] & pats[j], fout)
                np.testing.assert_array_equal(o, want, err_msg=f"op={op} out={fout} {i},{j}")
            sess.release_actor(act)


@pytest.mark.parametrize("fmt", [0, 2])
def test_bitmaps_of_unlike_sizes(sess, impatient, fmt):
    """Both bitmaps' words are scanned in one launch: one tile and several, in both orders, with the fallback too."""
    import ctypes
    import paper_1709_07781_amd as ka
    ng = 40 * GROUP_TILE + 3
    pats = group_patterns(ng)
    words = [bitmap(p, fmt) for p in pats]
    assert words[0].size < 10 and words[3].size > 3 * ENC_TILE
    for s in (sess, impatient):
        act = s.spawn("wah_combine", [ka.arg(ka.KA_IN, in_mode=ka.KA_VAL), ka.arg(ka.KA_IN, in_mode=ka.KA_VAL),
                                      ka.arg(ka.KA_PRIV, count=4, init=(ctypes.c_uint32 * 4)(1, fmt, fmt, ng)),
                                      ka.arg(ka.KA_OUT, out_mode=ka.KA_VAL)])
        for i, j in ((0, 3), (3, 0), (3, 3)):
            (o,) = s.request(act, ka.val(words[i].ctypes.data, words[i].size),
                             ka.val(words[j].ctypes.data, words[j].size), n_out=1)
            np.testing.assert_array_equal(o, bitmap(pats[i] | pats[j], fmt))
        s.release_actor(act)


def test_combine_scans_many_tiles(sess):
    """More tiles than one work-group sums up: their words are scanned in a launch of their own."""
    import ctypes
    import paper_1709_07781_amd as ka
    ng = 2048 * GROUP_TILE + 77
    a, b = (workloads.u32(k, ng) & np.uint32(0x7FFFFFFF) for k in (1, 2))
    a[np.arange(ng) % 3 == 0] = 0
    act = sess.spawn("wah_combine", [ka.arg(ka.KA_IN, in_mode=ka.KA_VAL), ka.arg(ka.KA_IN, in_mode=ka.KA_VAL),
                                     ka.arg(ka.KA_PRIV, count=4, init=(ctypes.c_uint32 * 4)(0, 0, 0, ng)),
                                     ka.arg(ka.KA_OUT, out_mode=ka.KA_VAL)])

    def paper(x):  # literals with a fill before each that follows empty groups
        at = np.flatnonzero(x)
        gap = np.diff(np.concatenate([[-1], at])) - 1
        w = np.zeros(at.size + int((gap > 0).sum()), np.uint32)
        end = np.cumsum(1 + (gap > 0))
        w[end - 1] = x[at]
        w[end[gap > 0] - 2] = np.uint32(0x80000000) | gap[gap > 0].astype(np.uint32)
        return w

    wa, wb = paper(a), paper(b)
    (o,) = sess.request(act, ka.val(wa.ctypes.data, wa.size), ka.val(wb.ctypes.data, wb.size), n_out=1)
    sess.release_actor(act)
    np.testing.assert_array_equal(o, paper(a & b))


@pytest.mark.parametrize("sizes", [[3000] * 400, [1 << 20, 0, 5, (1 << 20) - 1, 1] + [9000] * 20,
                                   [(1 << 20) + 1] * 4, [0, 0, 8192, 8193, 0, 77] * 3, [2] * 17_000 + [1500]])
@pytest.mark.parametrize("bits", [3, 12, 16])
def test_batch_tile_layouts(sess, sizes, bits):
    """Rows and table, requests that share tiles, empty ones, more requests than one work-group lays out; a batch in
    which some value exceeds its hint is refused."""
    from paper_1709_07781_amd import KaError
    if bits == 16 and len(sizes) > 1 << 16:
        pytest.skip("request ids and values exceed 32 bits")
    off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.uint32)
    v = workloads.u32(len(sizes), int(off[-1])) & np.uint32((1 << bits) - 1)
    got = sess.wah_batch(sess.upload(v), off, bits)
    some = range(len(sizes)) if len(sizes) < 500 else list(range(0, len(sizes), 997)) + [len(sizes) - 1]
    for j in some:
        for g, e in zip(got[j], oracle.default().wah_index(v[off[j]:off[j + 1]])):
            np.testing.assert_array_equal(g, e, err_msg=f"request {j}")
    v[int(off[-1]) // 2] = 1 << bits
    with pytest.raises(KaError):
        sess.wah_batch(sess.upload(v), off, bits)


@pytest.mark.parametrize("variant", [0, 1])
@pytest.mark.parametrize("size", [1, 255, 256, 257, 1023, 1024])
def test_small_requests_of_a_batch(sess, size, variant):
    """The small-request forms' sort: one and four values per work-item, values of 1 to 22 bits, equal and distinct."""
    from paper_1709_07781_amd.session import BatchPlan
    for bits in (1, 8, 12, 22):
        sizes = [size, 0, size, 1, size]
        off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.uint32)
        v = workloads.u32(size + bits, int(off[-1])) & np.uint32((1 << bits) - 1)
        v[off[2]:off[3]] = (1 << bits) - 1
        plan = BatchPlan(sess, off, bits, shape=variant)
        plan.run(v)
        for j, got in enumerate(plan.result()):
            for g, e in zip(got, oracle.default().wah_index(v[off[j]:off[j + 1]])):
                np.testing.assert_array_equal(g, e)
        plan.close()


@pytest.mark.parametrize("n,bits", [(1, 10), (31_337, 10), (1_030_000, 10), (1_060_000, 10), (300_000, 0)])
def test_host_outputs_of_every_size(sess, n, bits):
    """Results copied by a kernel behind the request, and those too large for it, of an index and of a batch."""
    v = workloads.u32(n, n) & np.uint32((1 << bits) - 1 if bits else 0xFFFFFFFF)
    for g, e in zip(sess.wah_index(v, value_bits=bits), oracle.default().wah_index(v)):
        np.testing.assert_array_equal(g, e)
    if not bits:
        return
    off = np.array([0, n // 3, n // 3, n], np.uint32)
    for j, got in enumerate(sess.wah_batch(v, off, bits)):
        for g, e in zip(got, oracle.default().wah_index(v[off[j]:off[j + 1]])):
            np.testing.assert_array_equal(g, e)


@pytest.mark.parametrize("n", [40, 70_000, 900_000])
def test_plan_results_of_every_size(sess, n):
    """One plan for any batch, host and device values, batches that grow and shrink."""
    from paper_1709_07781_amd.session import BatchPlan
    plan = BatchPlan(sess, None, 9, any_batch=(n, 8, 0))
    for k, m in enumerate((n, n // 2, 0, n)):
        off = np.array([0, m // 4, m // 4, m], np.uint32)
        v = workloads.u32(n + k, m) & np.uint32(511)
        plan.run_batch(sess.upload(v) if k % 2 else v, off)
        for j, got in enumerate(plan.result()):
            for g, e in zip(got, oracle.default().wah_index(v[off[j]:off[j + 1]])):
                np.testing.assert_array_equal(g, e)
    plan.close()


@pytest.mark.parametrize("n", [1 << 22, (1 << 22) + 1, 1 << 25, (1 << 25) + 16384 * 3 + 5])
def test_scan_and_compaction_tile_sizes(sess, impatient, n):
    """Where the scan's and the compaction's tiles double, with and without the look-back's fallback."""
    import paper_1709_07781_amd as ka
    x = workloads.u32(n, n)
    x[workloads.u32(n + 1, n) % 3 == 0] = 0
    for s in (sess, impatient):
        t = s.upload(x)
        r = s.wrap(t)
        for kernel, want in (("exclusive_scan_u32", np.concatenate([[0], np.cumsum(x[:-1], dtype=np.uint32)])),
                             ("compact_nonzero_u32", x[x != 0])):
            act = s.spawn(kernel, [ka.arg(ka.KA_IN), ka.arg(ka.KA_OUT)])
            (o,) = s.request(act, ka.ref(r), n_out=1)
            np.testing.assert_array_equal(s.read(o), want.astype(np.uint32))
            s.release_ref(o)
            s.release_actor(act)
        s.release_ref(r)
