"""What the framework's time is measured on: calls a user's program makes, through the public
entry points, over the sizes, value widths, word formats and forms (one request, composed actors,
batch, graph-replayed plan, served burst, queries, primitives) that this repository's benchmark,
workloads and tests use.

Inputs are drawn on the GPU; results stay on the device as references where the entry point
offers that, and come back as numpy arrays where the call is host to host.  The length of an index
depends on which rows hold equal values, and results of different seeds are laid side by side, so a
case fixes that pattern and the seed assigns the values to it (a dictionary-encoded column under
another assignment of its codes): every seed has other keys in another order, and other bitmaps
under each, at the same total lengths.
"""
from __future__ import annotations

import ctypes
import math
import random

import numpy as np
import torch

import paper_1709_07781_amd as ka
from paper_1709_07781_amd.session import BatchPlan, Server, Session

_kept: dict = {}


def _session() -> Session:
    """The program's one actor system (a user's program keeps it for its lifetime)."""
    if "session" not in _kept:
        _kept["session"] = Session()
    return _kept["session"]


def _server() -> Server:
    """The program's one server: two batches in flight, value requests below 2^12, 8-stage chains."""
    if "server" not in _kept:
        r = random.Random(2)
        a = np.array([r.getrandbits(32) | 1 for _ in range(8)], dtype=np.uint32)
        b = np.array([r.getrandbits(32) for _ in range(8)], dtype=np.uint32)
        _kept["server_session"] = Session(n_streams=4, use_torch_stream=False)
        _kept["server"] = Server(_kept["server_session"], streams=2, max_batch=1024, value_bits=12, chain_a=a,
                                 chain_b=b, max_batch_bytes=16 << 20)
    return _kept["server"]


# ---- the cases ---------------------------------------------------------------------------------
def listed() -> list[dict]:
    return [
        # the smallest served request sizes, one at a time: launches and host work are all there is
        {"name": "index_tiny", "kind": "index", "n": 777, "bits": 10, "hint": 10, "dist": "uniform", "fmt": 0, "host": False},
        # the plain configuration: 2^16 values below 1024 from host memory to a host index
        {"name": "index_plain", "kind": "index", "n": 1 << 16, "bits": 10, "hint": 10, "dist": "uniform", "fmt": 0, "host": True},
        # an ordinary column of 12-bit values, odd length, resident in HBM
        {"name": "index_mid", "kind": "index", "n": 1_500_007, "bits": 12, "hint": 12, "dist": "uniform", "fmt": 0, "host": False},
        # the benchmark's large request: 2^26 Zipf(1.1) values over 2^16
        {"name": "index_large", "kind": "index", "n": 1 << 26, "bits": 16, "hint": 16, "dist": "zipf", "fmt": 0, "host": False},
        # the two stage actors composed, any uint32 values (four digit passes, nearly all values distinct)
        {"name": "compose_u32", "kind": "compose", "n": 4_194_309, "bits": 32, "dist": "uniform"},
        # a clustered column (runs of equal values) in canonical WAH, whose 1-fills such columns are stored for
        {"name": "index_canonical", "kind": "index", "n": 6_000_011, "bits": 16, "hint": 16, "dist": "runs", "fmt": 1, "host": False},
        # the batched form: requests of log-uniform sizes 2^10..2^20, 12-bit values, one pass
        {"name": "batch_mixed", "kind": "batch", "nreq": 192, "lo": 10, "hi": 20, "bits": 12, "sizes": 4},
        # a serving tick of small requests through a recorded plan, host results
        {"name": "plan_small", "kind": "plan", "nreq": 256, "lo": 4, "hi": 10, "bits": 12, "sizes": 7},
        # the two data-parallel primitives on a large array of device values
        {"name": "scan_compact", "kind": "primitives", "n": 30_000_001, "zeros": 50},
        # eight composed affine stages, in place: the actor-overhead experiment's ordinary size
        {"name": "chain", "kind": "chain", "n": 1 << 20, "stages": 8},
        # a query on an index: slots of 4096 values, two values' bitmaps ORed, the result decoded
        {"name": "query_plwah", "kind": "query", "n": 20_000_003, "bits": 6, "dist": "uniform", "fmt": 2, "op": 1, "queries": 4096},
        # a burst of 24 served requests (index, scan and chain) from host memory to host results
        {"name": "served_burst", "kind": "served", "nreq": 24, "lo": 8, "hi": 18, "sizes": 5},
    ]


def _log_int(rng: random.Random, lo: float, hi: float) -> int:
    return int(2.0 ** rng.uniform(lo, hi)) | rng.getrandbits(1)


def draw(rng: random.Random) -> dict:
    kind = rng.choice(["index", "index", "index", "index", "compose", "batch", "plan", "primitives", "chain", "query",
                       "served"])
    if kind == "index":
        # formats beyond the paper's and unhinted values cost more per value: smaller columns
        fmt = rng.choice([0, 0, 0, 1, 2])
        bits = rng.choice([6, 8, 10, 12, 14, 16, 16, 20, 32])
        hint = bits if rng.random() < 0.75 else 0
        host = rng.random() < 0.25
        n = _log_int(rng, 8, 20 if host else 25.5 if fmt == 0 and 0 < hint <= 16 else 23.5)
        dist = rng.choice(["uniform", "zipf", "runs"]) if bits <= 16 else "uniform"
        return {"kind": kind, "n": n, "bits": bits, "hint": hint, "dist": dist, "fmt": fmt, "host": host}
    if kind == "compose":
        bits = rng.choice([8, 12, 16, 24, 32])
        return {"kind": kind, "n": _log_int(rng, 10, 23.5), "bits": bits, "dist": "uniform"}
    if kind == "batch":
        hi = rng.choice([10, 14, 18, 20])
        return {"kind": kind, "nreq": _log_int(rng, 2, 7.5 if hi > 14 else 12), "lo": 4 if hi == 10 else 10, "hi": hi,
                "bits": rng.choice([8, 12, 16]), "sizes": rng.getrandbits(16)}
    if kind == "plan":
        return {"kind": kind, "nreq": _log_int(rng, 4, 11), "lo": 4, "hi": rng.choice([8, 10]),
                "bits": rng.choice([8, 12]), "sizes": rng.getrandbits(16)}
    if kind == "primitives":
        return {"kind": kind, "n": _log_int(rng, 10, 26), "zeros": rng.choice([10, 50, 90])}
    if kind == "chain":
        return {"kind": kind, "n": _log_int(rng, 10, 24), "stages": rng.choice([2, 8])}
    if kind == "query":
        return {"kind": kind, "n": _log_int(rng, 14, 25), "bits": rng.choice([3, 6, 10]),
                "dist": rng.choice(["uniform", "runs"]), "fmt": rng.choice([0, 1, 2]), "op": rng.choice([0, 1]),
                "queries": _log_int(rng, 6, 16)}
    return {"kind": kind, "nreq": rng.choice([6, 12, 24]), "lo": 8, "hi": rng.choice([12, 16, 18]),
            "sizes": rng.getrandbits(16)}


# ---- inputs ------------------------------------------------------------------------------------
RUN = 100  # mean length of a run of equal values in a clustered column


def _gen(seed: int) -> torch.Generator:
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return g


def _zipf_cdf(nvals: int) -> np.ndarray:
    w = np.arange(1, nvals + 1, dtype=np.float64) ** -1.1
    c = np.cumsum(w)
    return c / c[-1]


def _values(n: int, bits: int, dist: str, seed: int, pattern: int = 0) -> torch.Tensor:
    """n values below 2^bits as the int32 tensor that holds their bits: the equality pattern of the sizes
    and `pattern`, under the seed's assignment of values.  Uniform and clustered columns: every code XORed
    with one mask.  Zipf: rank - 1, as the benchmark's large request has it (the smallest values are the
    most frequent), with the tail's values rotated."""
    g = _gen(1_000_003 * pattern + n)
    top = 1 << bits
    if dist == "zipf":
        cdf = torch.from_numpy(_zipf_cdf(top)).cuda()
        u = torch.rand(n, generator=g, device="cuda", dtype=torch.float64)
        v = torch.searchsorted(cdf, u, right=True).clamp_(max=top - 1).to(torch.int32)
        hot = 1 << (bits // 2)
        shift = random.Random(seed).randrange(top - hot)
        return torch.where(v < hot, v, hot + (v - hot + shift) % (top - hot)).to(torch.int32)
    if dist == "runs":
        run = torch.cumsum(torch.rand(n, generator=g, device="cuda") < 1.0 / RUN, 0)
        v = torch.randint(0, top, (n,), generator=g, device="cuda", dtype=torch.int64)[run.clamp_(max=n - 1)]
    else:
        v = torch.randint(0, top, (n,), generator=g, device="cuda", dtype=torch.int64)
    v ^= random.Random(seed).randrange(top)
    return torch.where(v >= 1 << 31, v - (1 << 32), v).to(torch.int32)


def _host_u32(t: torch.Tensor) -> np.ndarray:
    return t.cpu().numpy().view(np.uint32)


def _sizes(case: dict) -> list[int]:
    r = random.Random(case["sizes"])
    return [int(2.0 ** r.uniform(case["lo"], case["hi"])) for _ in range(case["nreq"])]


def _offsets(case: dict) -> np.ndarray:
    return np.concatenate([[0], np.cumsum(_sizes(case))]).astype(np.uint32)


class _State:
    """What a program has in hand before the call; gives its handles back at the end."""

    def __init__(self, case: dict):
        self.case = case
        self.refs: list = []
        self.actors: list = []
        self.plan = None

    def __del__(self):
        try:
            s = _session()
            for r in self.refs:
                s.release_ref(r)
            for a in self.actors:
                s.release_actor(a)
            if self.plan is not None:
                self.plan.close()
        except Exception:
            pass


def prepare(case: dict, seed: int):
    s, st, kind = _session(), _State(case), case["kind"]
    if kind == "index":
        v = _values(case["n"], case["bits"], case["dist"], seed)
        st.values = _host_u32(v) if case["host"] else v
    elif kind == "compose":
        st.values = _values(case["n"], case["bits"], case["dist"], seed)
        st.refs.append(s.wrap(st.values))
        sort = s.spawn("radix_sort_rows_u32", [ka.arg(ka.KA_IN), ka.arg(ka.KA_OUT), ka.arg(ka.KA_OUT)])
        enc = s.spawn("wah_encode_sorted", [ka.arg(ka.KA_IN), ka.arg(ka.KA_IN), ka.arg(ka.KA_OUT), ka.arg(ka.KA_OUT),
                                            ka.arg(ka.KA_OUT)])
        st.actor = s.compose(enc, sort)
        st.actors += [st.actor, sort, enc]
    elif kind == "batch":
        st.off = _offsets(case)
        st.values = _values(int(st.off[-1]), case["bits"], "uniform", seed)
    elif kind == "plan":
        st.off = _offsets(case)
        st.values = _host_u32(_values(int(st.off[-1]), case["bits"], "uniform", seed))
        st.plan = BatchPlan(s, None, case["bits"],
                            any_batch=(int(st.off[-1]), case["nreq"], 1 << case["hi"]))
    elif kind == "primitives":
        v = torch.randint(1, 1 << 31, (case["n"],), generator=_gen(seed), device="cuda", dtype=torch.int64)
        v = v.to(torch.int32).masked_fill_(torch.rand(case["n"], generator=_gen(case["n"]), device="cuda") <
                                           case["zeros"] / 100.0, 0)
        st.values = v
        st.refs.append(s.wrap(v))
        st.scan = s.spawn("exclusive_scan_u32", [ka.arg(ka.KA_IN), ka.arg(ka.KA_OUT)])
        st.compact = s.spawn("compact_nonzero_u32", [ka.arg(ka.KA_IN), ka.arg(ka.KA_OUT)])
        st.actors += [st.scan, st.compact]
    elif kind == "chain":
        st.values = _values(case["n"], 32, "uniform", seed)
        st.refs.append(s.wrap(st.values))
        r = random.Random(seed)
        acts = [s.affine_actor(r.getrandbits(32) | 1, r.getrandbits(32)) for _ in range(case["stages"])]
        st.actor = acts[0]
        st.actors += acts
        for a in acts[1:]:
            st.actor = s.compose(a, st.actor)
            st.actors.append(st.actor)
    elif kind == "query":
        n, fmt = case["n"], case["fmt"]
        ng = (n + 30) // 31
        column = _values(n, case["bits"], case["dist"], seed)
        idx = s.wah_index(column, refs=True, value_bits=case["bits"], fmt=fmt)
        keys, off, words = (t.clone() for t in _tensors([idx.keys_ref, idx.offsets_ref, idx.words_ref]))
        st.values = [keys]
        for row in (0, n // 2):  # the bitmaps of the values that these rows hold
            d = int(torch.searchsorted(keys, column[row:row + 1]))
            st.values.append(words[int(off[d]):int(off[d + 1])].clone())
        st.values.append(torch.randint(0, 1 << (case["bits"] + 1), (case["queries"],), generator=_gen(seed + 1),
                                       device="cuda", dtype=torch.int64).to(torch.int32))
        st.refs += [s.wrap(t) for t in st.values]
        priv4 = (ctypes.c_uint32 * 4)(case["op"], fmt, fmt, ng)
        priv2 = (ctypes.c_uint32 * 2)(fmt, ng)
        st.lookup = s.spawn("wah_lookup", [ka.arg(ka.KA_IN), ka.arg(ka.KA_IN), ka.arg(ka.KA_OUT)])
        st.combine = s.spawn("wah_combine", [ka.arg(ka.KA_IN), ka.arg(ka.KA_IN), ka.arg(ka.KA_PRIV, count=4, init=priv4),
                                             ka.arg(ka.KA_OUT)])
        st.decode = s.spawn("wah_decode", [ka.arg(ka.KA_IN), ka.arg(ka.KA_PRIV, count=2, init=priv2), ka.arg(ka.KA_OUT)])
        st.actors += [st.lookup, st.combine, st.decode]
    else:  # served: 10 of 24 requests are indexes, 7 scans, 7 chains
        _server()
        kinds = [0, 1, 2, 0, 1, 2, 0, 0, 1, 2, 0, 1]
        st.requests = []
        for j, m in enumerate(_sizes(case)):
            k = kinds[j % len(kinds)]
            st.requests.append((k, _host_u32(_values(m, 12 if k == 0 else 32, "uniform", seed, j))))
    return st


# ---- one pass ----------------------------------------------------------------------------------
class _Device:
    """A device reference's data, for torch: the reference is released with the last tensor on it."""

    def __init__(self, ref):
        self.ref = ref
        self.__cuda_array_interface__ = {"shape": (_session().length(ref),), "typestr": "<i4", "version": 2,
                                         "data": (_session().device_ptr(ref), False)}

    def __del__(self):
        try:
            _session().release_ref(self.ref)
        except Exception:
            pass


def _tensors(refs) -> list[torch.Tensor]:
    return [torch.as_tensor(_Device(r if isinstance(r, ctypes.c_void_p) else ctypes.c_void_p(r)), device="cuda")
            for r in refs]


def run(st):
    s, case = _session(), st.case
    kind = case["kind"]
    if kind == "index":
        if case["host"]:
            return s.wah_index(st.values, value_bits=case["hint"], fmt=case["fmt"])
        r = s.wah_index(st.values, refs=True, value_bits=case["hint"], fmt=case["fmt"])
        return _tensors([r.keys_ref, r.offsets_ref, r.words_ref])
    if kind == "compose":
        return _tensors(s.request(st.actor, ka.ref(st.refs[0]), n_out=3))
    if kind == "batch":
        r = s.wah_batch(st.values, st.off, case["bits"], refs=True)
        return _tensors([r.keys_ref, r.offsets_ref, r.words_ref, r.key_start_ref, r.word_start_ref])
    if kind == "plan":
        st.plan.run_batch(st.values, st.off)
        got = st.plan.result()
        return [np.concatenate([g[i] for g in got]) for i in range(3)]
    if kind == "primitives":
        x = ka.ref(st.refs[0])
        return _tensors(s.request(st.scan, x, n_out=1) + s.request(st.compact, x, n_out=1))
    if kind == "chain":
        (r,) = s.request(st.actor, ka.ref(st.refs[0]), n_out=1)
        s.release_ref(r)
        return st.values
    if kind == "query":
        keys, a, b, q = st.refs
        (slots,) = s.request(st.lookup, ka.ref(q), ka.ref(keys), n_out=1)
        (words,) = s.request(st.combine, ka.ref(a), ka.ref(b), n_out=1)
        (groups,) = s.request(st.decode, ka.ref(words), n_out=1)
        return _tensors([slots, words, groups])
    srv = _server()
    reqs = [srv.submit(k, d) for k, d in st.requests]
    out = []
    for (k, _), r in zip(st.requests, reqs):
        if srv.wait(r) != 0:
            raise RuntimeError("a served request failed")
        out.append([srv.result(r, i) for i in range(3 if k == 0 else 1)])
        srv.release(r)
    return out


# ---- what a pass cannot do without -------------------------------------------------------------
def _index_words(n: int, bits: int, dist: str, fmt: int) -> tuple[float, float]:
    """Expected (distinct values, words) of an index: over the values v of probability p, a 31-row group
    holds a literal with q = 1 - (1 - p)^31, and a fill stands before it unless the group before is
    non-empty too.  Runs: about four words a run (two partly filled groups, a gap, a 1-fill)."""
    groups = n / 31.0
    if dist == "runs":
        runs = n / RUN
        per = 4.0 if fmt else 1.0 + (RUN / 31.0 + 1.0)
        return min(runs, 2.0 ** bits), per * runs
    if dist == "zipf":
        p = np.diff(_zipf_cdf(1 << bits), prepend=0.0)
        m = 1.0
    else:
        k = min(2.0 ** bits, 65536.0)  # classes of equal probability stand for all of them
        p, m = np.full(int(k), 2.0 ** -bits), 2.0 ** bits / k
    q = -np.expm1(31.0 * np.log1p(-np.minimum(p, 1 - 1e-12)))
    lit = groups * q
    d = float(m * np.sum(-np.expm1(n * np.log1p(-np.minimum(p, 1 - 1e-12)))))
    absorbed = lit * (1 - q) if fmt == 2 else 0.0  # most groups after a fill hold one row: in PLWAH one word
    return d, float(m * np.sum(lit + lit * (1 - q) - absorbed))


def _index_bytes(n: int, bits: int, dist: str, fmt: int) -> float:
    d, w = _index_words(n, bits, dist, fmt)
    return 4.0 * n + 4.0 * (w + 2 * d + 1)


def work(case: dict) -> dict:
    kind = case["kind"]
    if kind in ("index", "compose"):
        b = _index_bytes(case["n"], case["bits"], case["dist"], case.get("fmt", 0))
    elif kind in ("batch", "plan"):
        b = sum(_index_bytes(m, case["bits"], "uniform", 0) for m in _sizes(case))
    elif kind == "primitives":
        b = 4.0 * case["n"] * (1 + 1 + 1 + (1 - case["zeros"] / 100.0))
    elif kind == "chain":
        b = 8.0 * case["n"]  # the stages are separate actors of one request: one read, one write
    elif kind == "query":
        ng = case["n"] / 31.0
        _, w = _index_words(case["n"], case["bits"], case["dist"], case["fmt"])
        b = 4.0 * (ng + 8 * case["queries"] / 4.0 + 5.0 * w / 2 ** case["bits"])
    else:
        kinds = [0, 1, 2, 0, 1, 2, 0, 0, 1, 2, 0, 1]
        b = sum(_index_bytes(m, 12, "uniform", 0) if kinds[j % 12] == 0 else 8.0 * m
                for j, m in enumerate(_sizes(case)))
    return {"bytes": b, "flops": 0}


# ---- the same results from plain numpy ---------------------------------------------------------
def _plain_index(v: np.ndarray):
    """(keys, offsets, words) in the paper's word form, by sorting and reducing with numpy."""
    v = v.astype(np.int64)
    rows = np.argsort(v, kind="stable")
    k, c, bit = v[rows], rows // 31, rows % 31
    seg = np.ones(k.size, bool)
    seg[1:] = k[1:] != k[:-1]
    head = seg.copy()
    head[1:] |= c[1:] != c[:-1]
    at = np.flatnonzero(head)
    lit = np.bitwise_or.reduceat(np.int64(1) << bit, at)
    gk, gc, gs = k[at], c[at], seg[at]
    gap = gc.copy()
    gap[1:] = np.where(gs[1:], gc[1:], gc[1:] - gc[:-1] - 1)
    emits = 1 + (gap > 0)
    end = np.cumsum(emits)
    words = np.empty(int(end[-1]), np.int64)
    words[end - 1] = lit
    fill = gap > 0
    words[end[fill] - 2] = 0x80000000 | gap[fill]
    off = np.append((end - emits)[gs], end[-1])
    return [x.astype(np.uint32) for x in (gk[gs], off, words)]


def exact(case: dict, seed: int):
    """Every output is whole numbers.  The indexes in the paper's form and the primitives are made again with
    numpy; the other formats, the queries, the served bursts and the in-place chain (whose result depends on
    how often it ran) have no such value here."""
    kind = case["kind"]
    if kind == "primitives" and case["n"] <= 1 << 25:
        st = prepare(case, seed)
        x = _host_u32(st.values)
        scan = np.cumsum(x, dtype=np.uint64).astype(np.uint32)
        return [np.concatenate([[0], scan[:-1]]).astype(np.uint32).view(np.int32), x[x != 0].view(np.int32)]
    if kind in ("index", "compose") and case.get("fmt", 0) == 0 and case["n"] <= 1 << 23:
        v = prepare(case, seed).values
        host = isinstance(v, np.ndarray)
        got = _plain_index(v if host else _host_u32(v))
        return tuple(got) if host else [x.view(np.int32) for x in got]
    return None
