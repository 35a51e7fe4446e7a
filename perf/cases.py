"""Timing cases of the framework's paths through its public entry points.

Each case is one call (or the short call sequence) that a program using the
library makes on an index it keeps: device selects from a single window to a
million, the stream-ordered select with the library's own workspace, the
server's two-stage select, joins, index rebuilds, a batch over independent
trees, and the host-array select.  Data follow the repository's synthetic
configurations (uniform, clustered and mixed rectangles in the unit square,
square windows of log-uniform area), drawn on the GPU from the seed.

Every result is a set of integer ids decided by exact fp32 comparisons, so
there is no rounding to compare against 64 bits.
"""

from __future__ import annotations

import math

import numpy as np
import torch

import paper_2309_16913_amd as rt

# Largest expected number of ids of a drawn select (the two listed large ones
# return 1.4e9 and 2.1e9).
MAX_IDS = 1.4e9


def listed():
    return [
        # latency of one user request against a resident index
        dict(name="select_one_window", op="select", n=1_000_000, nq=1, data="uniform", side=1e-4, sel_lo=1e-4,
             sel_hi=1e-3, fanout=32, layout="soa", split=0),
        # the plain configuration: 100k rectangles, 1000 windows of area 1e-4
        dict(name="select_1k_on_100k", op="select", n=100_000, nq=1000, data="uniform", side=1e-3, sel_lo=1e-4,
             sel_hi=1e-4, fanout=16, layout="soa", split=0),
        # an application's batch through the library-held workspace, ragged sizes
        dict(name="async_50k_on_1m", op="async", n=1_234_567, nq=50_001, data="mixed", side=1e-4, sel_lo=1e-6,
             sel_hi=1e-3, fanout=32, layout="d2", split=0),
        # the benchmark's default step: 10M rectangles, 1M windows
        dict(name="select_1m_on_10m", op="select", n=10_000_000, nq=1_000_000, data="mixed", side=1e-4, sel_lo=1e-6,
             sel_hi=1e-3, fanout=64, layout="soa", split=0),
        # the served window mix as one select: results of up to a million ids
        dict(name="select_50k_on_50m", op="select", n=50_000_000, nq=50_000, data="dense", side=5e-5, sel_lo=1e-7,
             sel_hi=1e-2, fanout=32, layout="soa", split=16),
        # one batch of the server at a moderate request rate
        dict(name="served_100_on_50m", op="served", n=50_000_000, nq=100, data="dense", side=5e-5, sel_lo=1e-7,
             sel_hi=1e-2, fanout=32, layout="soa", split=16),
        # join of two relations indexed with the builder's defaults, host result
        dict(name="join_200k", op="join_host", n=200_000, m=200_000, side=5e-4, fanout=32, layout="soa",
             sorted_lx=False),
        # the benchmark's join: low-x-sorted nodes, pairs left on the device
        dict(name="join_2m", op="join", n=2_000_000, m=2_000_000, side=5e-4, fanout=32, layout="soa",
             sorted_lx=True),
        # moving data: rebuild the index, answer a batch of windows on it
        dict(name="rebuild_100k", op="rebuild", n=100_000, nq=1000, data="uniform", side=1e-3, sel_lo=1e-4,
             sel_hi=1e-4, fanout=16, layout="soa", sorted_lx=False),
        dict(name="rebuild_10m", op="rebuild", n=10_000_000, nq=10_000, data="mixed", side=1e-4, sel_lo=1e-6,
             sel_hi=1e-3, fanout=32, layout="soa", sorted_lx=True),
        # independent trees answered by one graph, results fetched per tree
        dict(name="batch_16_trees", op="batch", trees=16, n=100_000, nq=3000, side=1e-4, sel_lo=1e-6, sel_hi=1e-3,
             fanout=32, layout="soa"),
        # host arrays in, host arrays out
        dict(name="host_10k_on_1m", op="host", n=1_000_000, nq=10_000, data="mixed", side=1e-4, sel_lo=1e-6,
             sel_hi=1e-4, fanout=32, layout="soa"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    op = rng.choice(["select", "select", "async", "served", "join", "join_host", "rebuild", "batch", "host"])
    case = dict(op=op, fanout=rng.choice([16, 20, 32, 32, 50, 64, 64]), layout=rng.choice(["soa", "soa", "aos", "d2"]))
    if op in ("join", "join_host"):
        case.update(n=_log_int(rng, 20_000, 2_000_000), m=_log_int(rng, 20_000, 2_000_000), side=5e-4,
                    sorted_lx=rng.random() < 0.5)
        return case
    if op == "batch":
        case.update(trees=rng.randint(2, 24), n=_log_int(rng, 3000, 300_000), nq=_log_int(rng, 100, 5000), side=1e-4,
                    sel_lo=1e-6, sel_hi=rng.choice([1e-4, 1e-3]))
        return case
    hi_n, hi_q = dict(select=(10_000_000, 1_000_000), served=(50_000_000, 2000), rebuild=(10_000_000, 10_000),
                      host=(3_000_000, 20_000)).get(op, (10_000_000, 200_000))
    data = rng.choice(["uniform", "mixed", "dense"])
    case.update(n=_log_int(rng, 10_000, hi_n), nq=_log_int(rng, 1, hi_q), data=data, side=rng.choice([5e-5, 1e-4]))
    if op == "rebuild":
        case.update(sorted_lx=rng.random() < 0.5)
    if op in ("select", "async", "served"):
        case.update(split=rng.choice([0, 16]))
    case.update(sel_lo=1e-6, sel_hi=rng.choice([1e-4, 1e-3, 1e-2]))
    limit = {"host": 1e6, "rebuild": 3e7, "served": 1e8}.get(op, MAX_IDS)
    if _ids(case) > limit:
        case["nq"] = max(1, int(case["nq"] * limit / _ids(case)))
    return case


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------

def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(int(seed))


def _u(g, *shape):
    return torch.rand(*shape, generator=g, device="cuda", dtype=torch.float64)


def _pack(lo, wh):
    """(low corner, sides) in float64 -> float32 rectangles, subnormals flushed."""
    r = torch.cat([lo, lo + wh]).t().to(torch.float32).contiguous()
    r[r.abs() < 2.0 ** -126] = 0.0
    return r


def _clustered(g, n, k, sigma, side):
    c = _u(g, 2, k)
    which = torch.randint(0, k, (n,), generator=g, device="cuda")
    lo = c[:, which] + torch.randn(2, n, generator=g, device="cuda", dtype=torch.float64) * sigma
    return _pack(lo, _u(g, 2, n) * side)


def _rects(g, n, data, side):
    """uniform; mixed: half uniform, half in 64 clusters, permuted; dense: 256
    tight clusters (the serving tree)."""
    if data == "uniform":
        return _pack(_u(g, 2, n), _u(g, 2, n) * side)
    if data == "dense":
        return _clustered(g, n, 256, 0.005, side)
    if data == "clusters":
        return _clustered(g, n, 32, 0.02, side)
    h = n // 2
    a = torch.cat([_pack(_u(g, 2, h), _u(g, 2, h) * side), _clustered(g, n - h, 64, 0.01, side)])
    return a[torch.randperm(n, generator=g, device="cuda")].contiguous()


def _windows(g, nq, sel_lo, sel_hi):
    c = _u(g, 2, nq)
    side = torch.exp((math.log(sel_lo) + _u(g, nq) * (math.log(sel_hi) - math.log(sel_lo))) * 0.5)
    return _pack(c - side / 2, side.expand(2, nq))


def _build(case, rects):
    t = rt.build_str_device(rects.data_ptr(), rects.shape[0], case["fanout"], case["layout"], _stream(),
                            sort_lx=case.get("sorted_lx", False))
    if case.get("split"):
        t.set_split(case["split"])
    return t


def _stream():
    return torch.cuda.current_stream().cuda_stream


def _cap(case, n=None, nq=None):
    """Ids an output buffer is made for: the expected number, a sixth more,
    and four standard deviations of the windows' sizes (on clustered data a
    window can hold whole clusters)."""
    n = case["n"] if n is None else n
    nq = case["nq"] if nq is None else nq
    per = 0.5 * case["sel_hi"]
    if case.get("data", "mixed") != "uniform":
        per = case["sel_hi"] + 0.005 * math.sqrt(case["sel_hi"] / 1e-2)
    return int(1.16 * _ids(case, n, nq) + 4 * math.sqrt(nq) * n * per) + 64


def prepare(case, seed):
    g = _gen(seed)
    op = case["op"]
    st = dict(case=case)
    if op in ("join", "join_host"):
        a = _rects(g, case["n"], "uniform", case["side"])
        b = _rects(g, case["m"], "clusters", case["side"])
        st.update(a=_build(case, a), b=_build(case, b))
        cap = st["cap"] = int(1.3 * _pairs(case)) + 5000
        st["pairs"] = (torch.zeros(2 * cap, dtype=torch.int32, device="cuda") if op == "join" else
                       np.zeros((cap, 2), np.uint32))
        return st
    if op == "batch":
        trees, queries, st["ids"] = [], [], []
        for k in range(case["trees"]):   # sizes spread over a factor of ten each
            f = 10.0 ** (k / max(1, case["trees"] - 1) - 0.5)
            n, nq = max(1, int(case["n"] * f)), max(1, int(case["nq"] / f))
            trees.append(_build(case, _rects(g, n, "uniform" if k % 2 else "mixed", case["side"])))
            queries.append(_windows(g, nq, case["sel_lo"], case["sel_hi"]).cpu().numpy())
            st["ids"].append(np.zeros(_cap(case, n, nq), np.uint32))
        st["batch"] = rt.Batch(trees, queries)
        return st
    r = _rects(g, case["n"], case["data"], case["side"])
    q = _windows(g, case["nq"], case["sel_lo"], case["sel_hi"])
    tree = _build(case, r)
    if op == "host":
        st.update(tree=tree, q=q.cpu().numpy(), ids=np.zeros(_cap(case), np.uint32))
        return st
    nq, cap = case["nq"], _cap(case)
    st.update(q=q, tree=tree, cap=cap, off=torch.empty(nq + 1, dtype=torch.int64, device="cuda"),
              ids=torch.zeros(cap, dtype=torch.int32, device="cuda"),
              status=torch.zeros(2, dtype=torch.int64, device="cuda"))
    if op != "async":   # room for the count pass's records
        st["wb"] = rt.select_replay_workspace_bytes(nq, cap)
        st["work"] = torch.empty(st["wb"], dtype=torch.uint8, device="cuda")
    if op == "rebuild":
        st["rects"] = r
    return st


# ---------------------------------------------------------------------------
# one pass
# ---------------------------------------------------------------------------

def _select(st):
    rt.range_select_device(st["tree"], st["q"].data_ptr(), st["q"].shape[0], st["off"].data_ptr(),
                           st["ids"].data_ptr(), st["cap"], st["work"].data_ptr(), st["wb"],
                           st["status"].data_ptr(), _stream())
    return st["off"], st["ids"], st["status"]


def _take(buf, got):
    """A host result taken over into the program's own array."""
    buf[: got.shape[0]] = got
    return buf


def run(st):
    case = st["case"]
    op = case["op"]
    if op == "select":
        return _select(st)
    if op == "async":
        fits = rt.range_select_async(st["tree"], st["q"].data_ptr(), st["q"].shape[0], st["off"].data_ptr(),
                                     st["ids"].data_ptr(), st["cap"], st["status"].data_ptr(), _stream())
        return st["off"], st["ids"], st["status"][:1], fits
    if op == "served":
        # the server reads a batch's size between the stages and places it
        nq = st["q"].shape[0]
        rt.range_select_device_count(st["tree"], st["q"].data_ptr(), nq, st["off"].data_ptr(), st["work"].data_ptr(),
                                     st["wb"], _stream())
        total = int(st["off"][nq].item())
        rt.range_select_device_fill(st["tree"], st["q"].data_ptr(), nq, st["off"].data_ptr(), st["ids"].data_ptr(),
                                    total, st["work"].data_ptr(), st["wb"], st["status"].data_ptr(), _stream())
        return st["off"], st["ids"], st["status"]
    if op == "join":
        n = rt.spatial_join_device(st["a"], st["b"], st["pairs"].data_ptr(), st["cap"], stream=_stream())
        return st["pairs"], n
    if op == "join_host":
        return _take(st["pairs"], rt.spatial_join(st["a"], st["b"]))
    if op == "rebuild":
        old = st["tree"]
        st["tree"] = _build(case, st["rects"])
        old.free()
        return _select(st)
    if op == "batch":
        b = st["batch"]
        b.run(_stream())
        got = [b.result(i) for i in range(case["trees"])]
        return [(off, _take(buf, ids)) for buf, (off, ids) in zip(st["ids"], got)]
    off, ids = rt.range_select(st["tree"], st["q"])
    return off, _take(st["ids"], ids)


# ---------------------------------------------------------------------------
# compulsory work
# ---------------------------------------------------------------------------

def _ids(case, n=None, nq=None):
    """Expected result size: n objects, square windows of log-uniform area."""
    n = case["n"] if n is None else n
    nq = case["nq"] if nq is None else nq
    lo, hi, s = case["sel_lo"], case["sel_hi"], case["side"]
    area = lo if lo == hi else (hi - lo) / math.log(hi / lo)
    edge = math.sqrt(lo) if lo == hi else (math.sqrt(hi) - math.sqrt(lo)) * 2 / math.log(hi / lo)
    return n * nq * (area + edge * s + s * s / 4)


def _select_bytes(case, n, nq):
    """Windows and offsets, every id written, every id read once (at most the
    whole index's ids)."""
    ids = _ids(case, n, nq)
    return 16 * nq + 8 * (nq + 1) + 4 * ids + min(4 * n, 4 * ids)


def _pairs(case):
    """Expected join pairs: sides U[0, s] on both sides, mean edge s."""
    return case["n"] * case["m"] * case["side"] ** 2


def work(case):
    op = case["op"]
    if op in ("join", "join_host"):
        return dict(bytes=20 * (case["n"] + case["m"]) + 8 * _pairs(case), flops=0)
    if op == "batch":
        b = 0.0
        for k in range(case["trees"]):
            f = 10.0 ** (k / max(1, case["trees"] - 1) - 0.5)
            b += _select_bytes(case, max(1, int(case["n"] * f)), max(1, int(case["nq"] / f)))
        return dict(bytes=b, flops=0)
    b = _select_bytes(case, case["n"], case["nq"])
    if op == "rebuild":   # rectangles in, entries (16 B MBR, 4 B ptr) out
        b += (16 + 20 * (1 + 1 / case["fanout"])) * case["n"]
    return dict(bytes=b, flops=0)


def exact(case, seed):
    """Ids are whole numbers; there is no floating output."""
    return None
