"""Performance cases: the work a user of this library has it do.

A case is one call of a public entry point on a synthetic graph.  The graph
families are the repository's own: R-MAT with (a, b, c, d) = (.57, .19, .19,
.05), G(n, m) random graphs, Chung-Lu power-law graphs (exponent 2.1) with planted
cliques, and uneven batches of small graphs.  Graphs are drawn on the GPU
from the seed; a single graph has exactly n vertex ids and m edges, so sizes do
not depend on the seed.  Sizes run from the 20 thousand edges of the
G(2000, 0.01) parity graph to an R-MAT graph of scale 23 (the R-MAT 24 of the
benchmark takes more than two seconds a call).

What is timed is the call: the graph lies in device memory (in host memory for
the bottom-up path, which is made for that), the output array and the workspace
are the caller's and are kept between calls, and the learned scheduler's model
is loaded once.
"""
import random

import numpy as np
import torch

import paper_1205_6693_amd as T
from paper_1205_6693_amd import sched

RMAT = (0.57, 0.19, 0.19, 0.05)
DEVICE = "cuda:0"


# ---- cases -------------------------------------------------------------------------------------

def listed():
    return [
        # the smallest single call: an edge list of the G(2000, 0.01) size, default options;
        # a few dozen launches over 20 thousand edges, so latency counts
        dict(name="decompose_er2000", op="decompose", graph="er", n=2000, m=20000, fmt="edges", sched="heuristic"),
        # an ordinary small graph of odd size (vertex ids not a power of two), edge list in no order
        dict(name="decompose_rmat17_odd", op="decompose", graph="rmat", n=100003, m=1234567, fmt="edges",
             sched="heuristic"),
        # the mid-size benchmark graph: R-MAT scale 20, CSR, learned scheduler
        dict(name="decompose_rmat20", op="decompose", graph="rmat", n=1 << 20, m=15699017, fmt="csr",
             sched="learned"),
        # power-law graph with planted cliques (the other benchmark family, at a quarter of its size)
        dict(name="decompose_chunglu1m", op="decompose", graph="chunglu", n=1 << 20, m=15500003, fmt="csr",
             sched="learned", max_deg=100000, cliques=16, clique_lo=50, clique_hi=500),
        # the largest call: R-MAT scale 23 with edge factor 20, CSR, learned scheduler
        dict(name="decompose_rmat23", op="decompose", graph="rmat", n=1 << 23, m=161000003, fmt="csr",
             sched="learned"),
        # triangle support alone, on a large CSR graph
        dict(name="support_rmat22", op="support", graph="rmat", n=1 << 22, m=64000001, fmt="csr"),
        # triangle support alone, on a small edge list
        dict(name="support_er16k", op="support", graph="er", n=16001, m=400009, fmt="edges"),
        # many small graphs at once, replayed plan: n ~ U{64..8192}, mean degree ~ U[4, 64], even G(n, m), odd
        # R-MAT, as the 4096-graph benchmark, a quarter of its graphs
        dict(name="batch_plan_1024", op="batch_plan", graphs=1024, n_lo=64, n_hi=8192, d_lo=4.0, d_hi=64.0),
        # one-shot batch of little graphs
        dict(name="batch_256_small", op="batch", graphs=256, n_lo=16, n_hi=600, d_lo=2.0, d_hi=20.0),
        # the ten densest classes of a mid-size graph, top-down (upper bound, selection, subgraph runs)
        dict(name="topdown_rmat19", op="topdown", graph="rmat", n=500009, m=7000003, fmt="csr", sched="learned", t=10),
        # core numbers of the mid-size benchmark graph
        dict(name="cores_rmat20", op="cores", graph="rmat", n=1 << 20, m=15699017, fmt="csr"),
        # a graph in host memory decomposed bottom-up, half of its edges on the device at a time: hundreds of
        # small subgraphs one after another, where the latency of a small device run counts
        dict(name="bottomup_rmat11", op="bottomup", graph="rmat", n=1 << 11, m=13001, cap=6500),
    ]


def _log_int(rng, lo, hi):
    return int(round(float(np.exp(rng.uniform(np.log(lo), np.log(hi))))))


def draw(rng):
    op = rng.choice(["decompose", "decompose", "decompose", "support", "batch_plan", "batch", "topdown", "cores",
                     "bottomup"])
    if op == "batch_plan":
        n_lo = rng.randint(16, 64)
        return dict(op=op, graphs=_log_int(rng, 32, 1024), n_lo=n_lo, n_hi=_log_int(rng, 512, 8192), d_lo=4.0,
                    d_hi=float(rng.randint(16, 64)))
    if op == "batch":
        return dict(op=op, graphs=_log_int(rng, 16, 1024), n_lo=16, n_hi=_log_int(rng, 64, 1000), d_lo=2.0,
                    d_hi=float(rng.randint(8, 24)))
    if op == "bottomup":
        n = _log_int(rng, 1000, 2500)
        m = int(n * rng.uniform(4.0, 6.5))
        return dict(op=op, graph="rmat", n=n, m=m, cap=int(m * rng.uniform(0.5, 1.0)))
    m = _log_int(rng, 20000, {"decompose": 100e6, "support": 64e6, "topdown": 8e6, "cores": 16e6}[op])
    graph = rng.choice(["rmat", "rmat", "chunglu", "er"])
    # no more edges than the vertices leave room for: mean degrees 12 to 60
    n = max(512, int(2 * m / rng.uniform(12.0, 60.0)))
    case = dict(op=op, graph=graph, n=n, m=m, fmt=rng.choice(["edges", "csr"]))
    if graph == "chunglu":
        k = max(1, min(16, m // 400000))
        hi = 500 if m > 4000000 else 60
        case.update(max_deg=max(64, n // 20), cliques=k, clique_lo=hi // 4, clique_hi=hi)
    if op in ("decompose", "topdown"):
        case["sched"] = rng.choice(["heuristic", "learned"])
    if op == "topdown":
        case["t"] = rng.randint(1, 20)
    return case


# ---- inputs ------------------------------------------------------------------------------------

def _rmat_pairs(gen, n, count):
    """count R-MAT samples over 2^ceil(log2 n) ids, those with an id >= n left out."""
    a, b, c, _ = RMAT
    u = torch.zeros(count, dtype=torch.int32, device=DEVICE)
    v = torch.zeros(count, dtype=torch.int32, device=DEVICE)
    for _ in range(max(1, (n - 1).bit_length())):
        r = torch.rand(count, generator=gen, device=DEVICE)
        u.mul_(2).add_((r >= a + b).to(torch.int32))
        v.mul_(2).add_((((r >= a) & (r < a + b)) | (r >= a + b + c)).to(torch.int32))
    keep = (u < n) & (v < n) if n & (n - 1) else None
    return (u, v) if keep is None else (u[keep], v[keep])


def _er_pairs(gen, n, count):
    return tuple(torch.randint(0, n, (count,), generator=gen, device=DEVICE, dtype=torch.int32) for _ in range(2))


def _chunglu_cdf(n, m, max_deg):
    w = torch.arange(1, n + 1, device=DEVICE, dtype=torch.float64).pow_(-1.0 / 1.1)
    for _ in range(20):
        w = (w * (2.0 * m / w.sum())).clamp_(max=float(max_deg))
    return torch.cumsum(w / w.sum(), 0)


def _keys(u, v, n):
    lo, hi = torch.minimum(u, v).to(torch.int64), torch.maximum(u, v)
    return (lo * n + hi)[lo != hi]


def _graph(case, seed):
    """Endpoints (int32, on the GPU) of m distinct edges, u < v, sorted."""
    n, m = case["n"], case["m"]
    gen = torch.Generator(device=DEVICE).manual_seed(seed)
    planted = torch.zeros(0, dtype=torch.int64, device=DEVICE)
    cdf = None
    if case["graph"] == "chunglu":
        sizes = random.Random(seed)
        ids, at, parts = torch.randperm(n, generator=gen, device=DEVICE), 0, []
        for _ in range(case["cliques"]):
            k = sizes.randint(case["clique_lo"], case["clique_hi"])
            i, j = torch.triu_indices(k, k, 1, device=DEVICE)
            parts.append(_keys(ids[at + i], ids[at + j], n))
            at += k
        planted = torch.cat(parts)
        cdf = _chunglu_cdf(n, m, case["max_deg"])
    name = torch.randperm(n, generator=gen, device=DEVICE).to(torch.int32)  # ids say nothing about degrees
    have = torch.zeros(0, dtype=torch.int64, device=DEVICE)
    want = m - planted.numel()
    count = int(1.1 * m) + 64
    while have.numel() < want:
        if cdf is not None:
            u, v = (torch.searchsorted(cdf, torch.rand(count, generator=gen, device=DEVICE, dtype=torch.float64))
                    .clamp_(max=n - 1) for _ in range(2))
        else:
            u, v = (_rmat_pairs if case["graph"] == "rmat" else _er_pairs)(gen, n, count)
        key = _keys(name[u.long()], name[v.long()], n)
        del u, v
        have = torch.unique(torch.cat([have, key]))
        if planted.numel():
            have = have[~torch.isin(have, planted)]
        del key
        count = max(count // 4, 2 * (want - have.numel()))
    drop = torch.randperm(have.numel(), generator=gen, device=DEVICE)[want:]
    keep = torch.ones(have.numel(), dtype=torch.bool, device=DEVICE)
    keep[drop] = False
    key = have[keep]
    if planted.numel():
        key = torch.cat([key, planted]).sort().values
    return (key // n).to(torch.int32), (key % n).to(torch.int32)


def _shuffled(u, v, seed):
    gen = torch.Generator(device=DEVICE).manual_seed(seed + (1 << 20))
    order = torch.randperm(u.numel(), generator=gen, device=DEVICE)
    flip = torch.rand(u.numel(), generator=gen, device=DEVICE) < 0.5
    u, v = u[order], v[order]
    return torch.where(flip, v, u), torch.where(flip, u, v)


def _csr(n, u, v):
    key = torch.cat([u.to(torch.int64) * n + v, v.to(torch.int64) * n + u]).sort().values
    col = (key % n).to(torch.int32)
    key //= n
    row_ptr = torch.zeros(n + 1, dtype=torch.int64, device=DEVICE)
    row_ptr[1:] = torch.cumsum(torch.bincount(key, minlength=n), 0)
    return row_ptr, col


def _input(case, seed):
    """The graph as the call takes it: endpoints of an edge list in no order, or CSR."""
    u, v = _graph(case, seed)
    return _csr(case["n"], u, v) if case.get("fmt") == "csr" else _shuffled(u, v, seed)


def _batch_sizes(case):
    """(n, m) of every graph: fixed by the case, the edges by the seed.  Mean
    degrees of tiny graphs stay below a quarter of the complete graph's."""
    rng = random.Random(case["graphs"] * 1000003 + case["n_hi"])
    out = []
    for _ in range(case["graphs"]):
        n = rng.randint(case["n_lo"], case["n_hi"])
        d = rng.uniform(case["d_lo"], case["d_hi"])
        out.append((n, int(n * min(d, (n - 1) / 4.0) / 2)))
    return out


def _batch_keys(gen, g, n, bits):
    """One pair for each entry of g (a graph's index): uniform in even graphs, R-MAT in odd ones."""
    ng, bg = n[g], bits[g]
    a, b, c, _ = RMAT
    u, v = torch.zeros_like(g), torch.zeros_like(g)
    for level in range(int(bits.max())):
        r = torch.rand(g.numel(), generator=gen, device=DEVICE)
        on = level < bg
        u = torch.where(on, 2 * u + (r >= a + b), u)
        v = torch.where(on, 2 * v + (((r >= a) & (r < a + b)) | (r >= a + b + c)), v)
    er = g % 2 == 0
    ru, rv = (torch.rand(g.numel(), generator=gen, device=DEVICE, dtype=torch.float64) for _ in range(2))
    u = torch.where(er, (ru * ng).long(), u)
    v = torch.where(er, (rv * ng).long(), v)
    ok = (u != v) & (u < ng) & (v < ng)
    return ((g << 26) + (torch.minimum(u, v) << 13) + torch.maximum(u, v))[ok]


def _batch_input(case, seed):
    """Packed batch: host offsets, device endpoints with graph-local ids."""
    sizes = _batch_sizes(case)
    gen = torch.Generator(device=DEVICE).manual_seed(seed)
    n, m = (torch.tensor(x, device=DEVICE) for x in zip(*sizes))
    bits = torch.tensor([(s[0] - 1).bit_length() for s in sizes], device=DEVICE)
    index = torch.arange(len(sizes), device=DEVICE)
    key = torch.zeros(0, dtype=torch.int64, device=DEVICE)
    need = m + m // 4
    while int(need.max()) > 0:
        key = torch.unique(torch.cat([key, _batch_keys(gen, torch.repeat_interleave(index, need), n, bits)]))
        short = m - torch.bincount(key >> 26, minlength=len(sizes))
        need = torch.where(short > 0, 4 * short + 16, torch.zeros_like(short))
    # m of each graph's pairs, in no order
    g = key >> 26
    order = torch.argsort(g * 2.0 + torch.rand(g.numel(), generator=gen, device=DEVICE, dtype=torch.float64))
    key, g = key[order], g[order]
    first = torch.cumsum(torch.bincount(g, minlength=len(sizes)), 0) - torch.bincount(g, minlength=len(sizes))
    key = key[torch.arange(g.numel(), device=DEVICE) - first[g] < m[g]]
    u, v = (key >> 13) & 8191, key & 8191
    flip = torch.rand(key.numel(), generator=gen, device=DEVICE) < 0.5
    src, dst = torch.where(flip, v, u).to(torch.int32), torch.where(flip, u, v).to(torch.int32)
    vo, eo = (np.concatenate([[0], np.cumsum(x)]).astype(np.int64) for x in zip(*sizes))
    return vo, eo, src, dst


# ---- the calls ---------------------------------------------------------------------------------

def prepare(case, seed):
    op = case["op"]
    st = {"op": op, "t": case.get("t")}
    if op in ("batch", "batch_plan"):
        vo, eo, src, dst = _batch_input(case, seed)
        if op == "batch_plan":
            st["plan"] = T.BatchPlan(vo, eo, src, dst)
        else:
            ws = torch.empty(T.truss_batch_workspace_size(vo, eo), dtype=torch.uint8, device=DEVICE)
            st.update(vo=vo, eo=eo, src=src, dst=dst, ws=ws, out=torch.empty_like(src))
        return st
    if op == "bottomup":
        src, dst = _input(case, seed)
        st.update(n=case["n"], cap=case["cap"], src=src.cpu().numpy(), dst=dst.cpu().numpy())
        return st
    x, y = _input(case, seed)
    torch.cuda.empty_cache()
    g = (T.Graph.from_csr if case["fmt"] == "csr" else T.Graph.from_edges)(case["n"], x, y)
    st["graph"] = g
    if op in ("decompose", "topdown"):
        learned = case["sched"] == "learned"
        st["opts"] = T.make_options(scheduler=T.SCHED_LEARNED if learned else T.SCHED_HEURISTIC,
                                    model=sched.load_model(device=DEVICE) if learned else None)
    if op in ("decompose", "support"):
        st["ws"] = T.workspace(g)
    st["out"] = torch.empty(case["n"] if op == "cores" else case["m"], dtype=torch.int32, device=DEVICE)
    return st


def run(state):
    op = state["op"]
    if op == "decompose":
        out, st = T.truss_decompose(state["graph"], state["opts"], out=state["out"], ws=state["ws"])
        return [out, st["kmax"], st["triangles"]]
    if op == "support":
        out, triangles = T.truss_support(state["graph"], out=state["out"], ws=state["ws"])
        return [out, triangles]
    if op == "topdown":
        out, kmin, kmax, _ = T.truss_topdown(state["graph"], state["t"], state["opts"], out=state["out"])
        return [out, kmin, kmax]
    if op == "cores":
        out, cmax = T.truss_core_numbers(state["graph"], out=state["out"])
        return [out, cmax]
    if op == "batch_plan":
        out, st = state["plan"].run()
        return [out, st["kmax"], st["triangles"]]
    if op == "batch":
        out, st = T.truss_batch(state["vo"], state["eo"], state["src"], state["dst"], out=state["out"],
                                ws=state["ws"])
        return [out, st["kmax"], st["triangles"]]
    phi, low, _ = T.truss_bottomup(state["n"], state["src"], state["dst"], state["cap"])
    return [phi, low]


def work(case):
    """The graph read once and the result written once; the integer work of
    triangle listing and peeling depends on the graph and is left out."""
    if case["op"] in ("batch", "batch_plan"):
        n, m = map(sum, zip(*_batch_sizes(case)))
        return {"bytes": 12 * m + 16 * case["graphs"], "flops": 0}
    n, m = case["n"], case["m"]
    graph = 8 * (n + 1) + 8 * m if case.get("fmt") == "csr" else 8 * m
    out = 4 * n if case["op"] == "cores" else 8 * m if case["op"] == "bottomup" else 4 * m
    return {"bytes": graph + out, "flops": 0}


# ---- the same results in plain torch -----------------------------------------------------------

def _dense_truss(n, u, v):
    """Supports and truss numbers of the edges (u, v) by the definitions, on a dense adjacency matrix."""
    u, v = u.long(), v.long()
    adj = torch.zeros((n, n), dtype=torch.float64, device=DEVICE)
    adj[u, v] = 1.0
    adj[v, u] = 1.0
    sup = (adj @ adj)[u, v]
    first = sup.to(torch.int32)
    phi = torch.zeros(u.numel(), dtype=torch.int32, device=DEVICE)
    live = torch.ones(u.numel(), dtype=torch.bool, device=DEVICE)
    k = 2
    while bool(live.any()):
        gone = live & (sup <= k - 2)
        if not bool(gone.any()):
            k = max(k + 1, int(sup[live].min()) + 2)
            continue
        phi[gone] = k
        live &= ~gone
        adj[u[gone], v[gone]] = 0.0
        adj[v[gone], u[gone]] = 0.0
        sup = (adj @ adj)[u, v]
    return first, phi


def _cores(n, u, v):
    u, v = torch.cat([u, v]).long(), torch.cat([v, u]).long()
    deg = torch.bincount(u, minlength=n)
    core = torch.zeros(n, dtype=torch.int32, device=DEVICE)
    live = torch.ones(n, dtype=torch.bool, device=DEVICE)
    c = 0
    while bool(live.any()):
        gone = live & (deg <= c)
        if not bool(gone.any()):
            c = int(deg[live].min())
            continue
        core[gone] = c
        live &= ~gone
        deg = deg - torch.bincount(v[gone[u]], minlength=n)
    return core, int(core.max())


def exact(case, seed):
    op = case["op"]
    if op in ("batch", "batch_plan"):
        if case["graphs"] > 300 or case["n_hi"] > 1024:
            return None
        vo, eo, src, dst = _batch_input(case, seed)
        out, kmax, tri = torch.empty_like(src), 0, 0
        for i in range(case["graphs"]):
            lo, hi = int(eo[i]), int(eo[i + 1])
            if lo < hi:
                sup, out[lo:hi] = _dense_truss(int(vo[i + 1] - vo[i]), src[lo:hi], dst[lo:hi])
                kmax, tri = max(kmax, int(out[lo:hi].max())), tri + int(sup.sum()) // 3
        return [out, kmax, tri]
    if op == "cores":
        if case["m"] > 20000000:
            return None
        u, v = _graph(case, seed)
        return list(_cores(case["n"], u, v))
    if case["n"] > 4096:
        return None
    u, v = _graph(case, seed) if case.get("fmt") == "csr" else _input(case, seed)
    sup, phi = _dense_truss(case["n"], u, v)
    if op == "support":
        return [sup, int(sup.sum()) // 3]
    kmax = int(phi.max())
    if op == "decompose":
        return [phi, kmax, int(sup.sum()) // 3]
    if op == "topdown":
        kmin = max(2, kmax - case["t"] + 1)
        return [torch.where(phi >= kmin, phi, torch.zeros_like(phi)), kmin, kmax]
    return [phi.cpu().numpy(), None]
