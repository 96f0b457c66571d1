"""Performance cases of the segmented-traversal library: what its users run,
from a one-tile graph to the R-MAT 25 headline graph, through the public entry
points of paper_1608_01362_amd.

A case is a dict of plain values. `prepare` makes what a user's program holds
before the call (the graph on the GPU, its segments, the vectors), `run` is one
call of the path, `exact` the same outputs in 64 bits by plain torch, `work` the
bytes and operations the path cannot do without. Graphs are R-MAT
(.57/.19/.19/.05), vertex ids permuted, self-loops and duplicates removed; a
vertex count that is not a power of two scales the R-MAT ids onto [0, V).
"""
from __future__ import annotations

import ctypes
import math

import numpy as np
import torch

from paper_1608_01362_amd import cagra, warmstart

DAMPING = 0.85
QUADRANTS = (0.57, 0.19, 0.19, 0.05)
CHUNK = 1 << 26  # edges sampled at a time


# ------------------------------------------------------------------ the cases

def listed():
    return [
        # a graph of one service request: 20 iterations of three short launches each
        {"name": "pagerank-4k", "kind": "pagerank", "V": 4096, "ef": 16, "N": 1024, "B": 1024, "tile": 4096,
         "dtype": "f32", "iters": 20},
        # the headline graph: R-MAT 25, edge factor 32, FP32 contributions
        {"name": "pagerank-rmat25", "kind": "pagerank", "V": 1 << 25, "ef": 32, "N": 32768, "B": 8192,
         "tile": 262144, "dtype": "f32", "iters": 4},
        # PageRank to an L1 residual of 1e-6, BF16 gathers finishing in FP32, a vertex count of no special form
        {"name": "solve-bf16-3m", "kind": "solve", "V": 3000017, "ef": 16, "N": 32768, "B": 8192, "tile": 65536,
         "dtype": "bf16", "switch": 1e-3, "restart": -1},
        # connected components of an undirected graph: minimum labels to the fixed point
        {"name": "labelprop-rmat22", "kind": "labelprop", "V": 1 << 22, "ef": 16, "N": 32768, "B": 8192,
         "tile": 262144},
        # the out-edge traversal of the same kind of graph
        {"name": "push-rmat22", "kind": "push", "V": 1 << 22, "ef": 16, "N": 20480, "B": 8192, "tile": 65536,
         "iters": 4},
        # 64 personalized PageRank vectors at once (recommendations for a batch of users)
        {"name": "ppr64-rmat21", "kind": "ppr", "V": 1 << 21, "ef": 16, "N": 1 << 20, "B": 512, "tile": 16384,
         "cols": 64, "iters": 4},
        # many small graphs of uneven sizes, all iterations replayed as one HIP graph
        {"name": "multigraph-48", "kind": "multi", "graphs": 48, "lo": 10, "hi": 17, "iters": 20},
        # preprocessing of a new graph: frequency-based clustering, then the segments
        {"name": "preprocess-rmat24", "kind": "prep", "V": 1 << 24, "ef": 24, "N": 32768, "B": 8192,
         "tile": 262144, "cluster": True},
        # matrix factorization on a rating graph (64 factors), one gradient step
        {"name": "cf-128k-8k", "kind": "cf", "users": 1 << 17, "items": 1 << 13, "ef": 120, "N": 65536, "B": 512,
         "tile": 65536},
        # betweenness centrality from sampled starts: levels with sparse and dense frontiers
        {"name": "bc-rmat21", "kind": "bc", "V": 1 << 21, "ef": 16, "N": 32768, "B": 8192, "tile": 65536,
         "starts": 2},
        # one training step of the warm-start network: minibatch, gradient, Adam
        {"name": "train-64k", "kind": "train", "rows": 1 << 20, "batch": 65536},
        # the learned start vector of a new graph: degree features, network, softmax
        {"name": "start-rmat22", "kind": "start", "V": 1 << 22, "ef": 24, "N": 32768, "B": 8192, "tile": 262144},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["pagerank", "pagerank", "solve", "labelprop", "push", "ppr", "multi", "prep", "cf", "bc",
                       "train", "start"])
    V = _log_int(rng, 600, 5_000_000)
    if rng.random() < 0.3:
        V = 1 << max(9, V.bit_length() - 1)
    seg = {"V": V, "ef": rng.randint(4, 32), "N": rng.choice([4096, 10000, 16384, 32768]),
           "B": rng.choice([2048, 4096, 8192]), "tile": rng.choice([4096, 16384, 65536, 262144])}
    if kind == "pagerank":
        return {"kind": kind, **seg, "dtype": rng.choice(["f32", "bf16"]), "iters": rng.randint(1, 20)}
    if kind == "solve":
        dtype = rng.choice(["f32", "bf16"])
        return {"kind": kind, **seg, "dtype": dtype, "switch": 1e-3 if dtype == "bf16" else 0.0,
                "restart": rng.choice([-1, -1, rng.randrange(V)])}
    if kind in ("labelprop", "start"):
        return {"kind": kind, **seg}
    if kind == "push":
        seg["N"] = rng.choice([4096, 10000, 16384, 20480])
        return {"kind": kind, **seg, "iters": rng.randint(1, 8)}
    if kind == "ppr":
        seg["V"] = _log_int(rng, 600, 1_500_000)
        seg.update(N=rng.choice([1 << 18, 1 << 20, 1 << 21]), B=rng.choice([128, 256, 512]),
                   tile=rng.choice([4096, 16384, 65536]))
        return {"kind": kind, **seg, "cols": rng.choice([64, 64, 17, rng.randint(1, 64)]), "iters": rng.randint(1, 4)}
    if kind == "multi":
        lo = rng.randint(9, 12)
        return {"kind": kind, "graphs": _log_int(rng, 3, 48), "lo": lo, "hi": rng.randint(lo, 16),
                "iters": rng.randint(2, 20)}
    if kind == "prep":
        return {"kind": kind, **seg, "cluster": rng.random() < 0.6}
    if kind == "cf":
        return {"kind": kind, "users": _log_int(rng, 300, 130_000), "items": _log_int(rng, 100, 20_000),
                "ef": rng.randint(8, 100), "N": rng.choice([8192, 65536, 262144]), "B": rng.choice([128, 512]),
                "tile": rng.choice([4096, 16384, 65536])}
    if kind == "bc":
        seg["V"] = _log_int(rng, 600, 2_000_000)
        return {"kind": kind, **seg, "starts": rng.randint(1, 2)}
    return {"kind": "train", "rows": _log_int(rng, 2000, 1 << 20), "batch": _log_int(rng, 256, 131072)}


# ------------------------------------------------------------------ inputs

def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return g


def _rmat_ids(bits_u, bits_v, m, g):
    """m R-MAT edges: (row, column) ids of bits_u and bits_v bits. Five levels
    are drawn at a time from the joint distribution of their quadrants."""
    a, b, c, d = QUADRANTS
    u = torch.zeros(m, dtype=torch.int64, device="cuda")
    v = torch.zeros(m, dtype=torch.int64, device="cuda")
    left = max(bits_u, bits_v)
    while left > 0:
        n = min(5, left)
        quads = np.array([a, b, c, d])
        prob, rows, cols = np.ones(1), np.zeros(1, np.int64), np.zeros(1, np.int64)
        for _ in range(n):
            prob = np.outer(prob, quads).ravel()
            rows = (rows[:, None] * 2 + np.array([0, 0, 1, 1])).ravel()
            cols = (cols[:, None] * 2 + np.array([0, 1, 0, 1])).ravel()
        cdf = torch.from_numpy(np.cumsum(prob)[:-1].astype(np.float32)).cuda()
        rows, cols = torch.from_numpy(rows).cuda(), torch.from_numpy(cols).cuda()
        i = torch.bucketize(torch.rand(m, generator=g, device="cuda"), cdf, out_int32=True, right=True)
        u = u.mul_(1 << n).add_(rows[i])
        v = v.mul_(1 << n).add_(cols[i])
        left -= n
    left = max(bits_u, bits_v)
    return u >> (left - bits_u), v >> (left - bits_v)


def _edge_keys(V, ef, seed):
    """Sorted unique keys destination * V + source of an R-MAT graph."""
    g = _gen(seed)
    bits = max(1, (V - 1).bit_length())
    perm = torch.randperm(V, generator=g, device="cuda")
    m = ef * V
    keys = torch.empty(m, dtype=torch.int64, device="cuda")
    for lo in range(0, m, CHUNK):
        n = min(CHUNK, m - lo)
        u, v = _rmat_ids(bits, bits, n, g)
        if V != 1 << bits:
            u, v = (u * V) >> bits, (v * V) >> bits
        u, v = perm[u], perm[v]
        v = v.mul_(V).add_(u)
        keys[lo:lo + n] = torch.where(u * (V + 1) == v, torch.full_like(v, -1), v)
    return _unique(keys)


def _unique(keys):
    keys = torch.sort(keys).values
    keep = keys >= 0
    keep[1:] &= keys[1:] != keys[:-1]
    return keys[keep]


def _csc(V, keys):
    """In-edge CSC arrays (offsets, sources, out-degrees) of sorted keys."""
    E = keys.numel()
    off = torch.searchsorted(keys, torch.arange(V + 1, device="cuda") * V).to(torch.int32)
    src = torch.empty(max(E, 1), dtype=torch.int32, device="cuda")
    deg = torch.zeros(V, dtype=torch.int32, device="cuda")
    for lo in range(0, E, CHUNK):
        s = keys[lo:lo + CHUNK] % V
        src[lo:lo + s.numel()] = s.to(torch.int32)
        deg += torch.bincount(s, minlength=V).to(torch.int32)
    return off, src[:E] if E else src, deg


def _graph(V, off, src, deg):
    dg = cagra.DeviceGraph(V, int(off[-1].item()), off, src, deg)
    dg.c = cagra.CGraph(V, dg.E, off.data_ptr(), src.data_ptr(), deg.data_ptr())
    return dg


def _rmat(V, ef, seed, symmetric=False, reverse=False):
    """(graph, reversed graph or None) as CSC array triples."""
    keys = _edge_keys(V, ef, seed)
    back = None
    if symmetric or reverse:
        back = _unique((keys % V) * V + keys // V)
    if symmetric:
        keys, back = _unique(torch.cat([keys, back])), None
    return _csc(V, keys), _csc(V, back) if reverse else None


def _ratings(case, seed):
    """Rating graph: every (user, item) pair an edge in both directions, with its
    rating in 1..5. CSC arrays and the ratings in CSC order."""
    U, I = case["users"], case["items"]
    g = _gen(seed)
    bu, bi = max(1, (U - 1).bit_length()), max(1, (I - 1).bit_length())
    u, i = _rmat_ids(bu, bi, case["ef"] * U, g)
    pu, pi = torch.randperm(U, generator=g, device="cuda"), torch.randperm(I, generator=g, device="cuda")
    pairs = torch.unique(pu[(u * U) >> bu] * I + pi[(i * I) >> bi])
    u, i = pairs // I, pairs % I + U
    r = torch.randint(1, 6, (pairs.numel(),), generator=g, device="cuda").float()
    V = U + I
    keys, order = torch.sort(torch.cat([u * V + i, i * V + u]))
    off, src, deg = _csc(V, keys)
    x0 = torch.rand(V, cagra.CF_FACTORS, generator=g, device="cuda") * 0.1
    return V, off, src, deg, torch.cat([r, r])[order], x0


def _multi_sizes(case):
    n = case["graphs"]
    rng = np.random.default_rng(n)
    return [(1 << int(s), int(e)) for s, e in zip(rng.integers(case["lo"], case["hi"] + 1, n),
                                                  rng.integers(8, 33, n))]


def _network(seed):
    """Network parameters rounded to BF16, Adam state of a run under way, standardization."""
    rng = np.random.default_rng(seed)
    p = np.zeros(warmstart.NPARAM, np.float32)
    p[:192] = rng.normal(0, 1 / np.sqrt(3), 192)
    p[192:256] = rng.normal(0, 0.1, 64)
    p[256:4352] = rng.normal(0, 1 / 8, 4096)
    p[4352:4416] = rng.normal(0, 0.1, 64)
    p[4416:4480] = rng.normal(0, 1 / 8, 64)
    m = rng.normal(0, 1e-2, p.size).astype(np.float32)
    v = (m * m + rng.uniform(1e-5, 1e-4, p.size)).astype(np.float32)
    norm = np.array([2.0, 1.5, 3.0, 0.7, 0.6, 0.4], np.float32)
    return (torch.from_numpy(x).cuda() for x in (p, m, v, norm))


def _rows(case, seed):
    """Training rows: log-degree features and log-rank targets."""
    g = _gen(seed)
    n = case["rows"]
    deg = torch.floor(torch.rand(n, 3, generator=g, device="cuda").clamp_min(1e-6) ** -0.8) - 1
    F = torch.log1p(deg)
    F[:, 2] = 3 + torch.randn(n, generator=g, device="cuda")
    T = 0.9 * F[:, 0] - 1 + 0.3 * torch.randn(n, generator=g, device="cuda")
    return F.contiguous(), T.contiguous()


def _prep_edges(case):
    """Edges of a preprocessing case: below what remains of ef * V samples once
    duplicates are removed (R-MAT repeats more of them the smaller the graph)."""
    share = 0.4 if case["V"] < 20_000 else 0.75 if case["V"] < 1_000_000 else 0.9
    return int(share * case["ef"] * case["V"])


def _segment_room(case, E):
    """Caller-owned arrays for the segments of any graph of E edges (at most one
    row per edge), as a program holds that segments one graph after another."""
    V, N, B = case["V"], case["N"], case["B"]
    k, nb, tiles = -(-V // N), -(-V // B), -(-V // N) + E // case["tile"]
    word = torch.int16 if N <= cagra.EDGE16_MAX_N else torch.int32
    size = {"seg_row_begin": k + 1, "row_ptr": E + 1, "row_dst": E, "edge_src": -(-E // 8) * 8,
            "block_ptr": (nb + 1) * k, "tile_edge": tiles + 1, "tile_seg": tiles,
            "tile_span_row": tiles * cagra.TILE_WAVES, "row_dst_lo": E, "block_items": nb + 1}
    types = {"edge_src": word, "row_dst_lo": torch.int16}
    return {n: torch.zeros(c, dtype=types.get(n, torch.int32), device="cuda") for n, c in size.items()}


def _build_into(dg, case, room):
    """The query call and the build call of cagra_build_segments into `room`."""
    L, c = cagra.lib(), cagra.CSegments()
    c.N, c.B, c.tile_edges = case["N"], case["B"], case["tile"]
    for fill in (False, True):
        n = c.build_workspace_bytes if fill else L.cagra_query_workspace_bytes(dg.V, dg.E, c.N)
        ws = torch.empty(n, dtype=torch.uint8, device="cuda")
        if fill:
            for name, t in room.items():
                setattr(c, name, t.data_ptr())
        status = L.cagra_build_segments(ctypes.byref(dg.c), ctypes.byref(c), ctypes.c_void_p(ws.data_ptr()), n,
                                        ctypes.c_void_p(torch.cuda.current_stream().cuda_stream))
        if status != cagra.OK:
            raise cagra.CagraError(status, "cagra_build_segments", L.cagra_last_error().decode())
    return c


def _starts(case, seed, deg):
    ok = torch.nonzero(deg > 0).flatten()
    pick = torch.randint(0, ok.numel(), (case["starts"],), generator=_gen(seed + 1), device="cuda")
    return [int(s) for s in ok[pick].cpu()]


def _seeds(case, seed):
    return np.random.default_rng(seed + 1).choice(case["V"], case["cols"], replace=False).astype(np.int32)


def prepare(case, seed):
    kind = case["kind"]
    s = {"kind": kind, "case": case}
    if kind == "train":
        s["F"], s["T"] = _rows(case, seed)
        p, m, v, norm = _network(seed)
        s["start"] = torch.cat([p, m, v])
        s["start_weights"] = p.to(torch.bfloat16).view(torch.int16)
        n = warmstart.NPARAM
        buf = s["buf"] = s["start"].clone()
        s["net"] = warmstart.Network(buf[:n], s["start_weights"].clone(), buf[n:2 * n], buf[2 * n:], norm)
        s["batch"] = (torch.empty(case["batch"], 3, device="cuda"), torch.empty(case["batch"], device="cuda"))
        s["seed"] = seed
        return s
    if kind == "multi":
        graphs = [_graph(V, *_rmat(V, ef, seed + 100 + i)[0]) for i, (V, ef) in enumerate(_multi_sizes(case))]
        segs = [cagra.build_segments(d, 16384, 4096, 65536) for d in graphs]
        s["multi"] = cagra.MultiPageRank(graphs, segs)
        s["multi"].capture(case["iters"], DAMPING)
        return s
    if kind == "cf":
        V, off, src, deg, r, x0 = _ratings(case, seed)
        s["dg"] = _graph(V, off, src, deg)
        s["seg"] = cagra.build_segments(s["dg"], case["N"], case["B"], case["tile"])
        s["state"] = cagra.CFState(s["dg"], s["seg"], cagra.segment_edge_values(s["dg"], s["seg"], r), x0)
        return s
    if kind == "prep":
        keys = _edge_keys(case["V"], case["ef"], seed)
        E = _prep_edges(case)  # evenly thinned to a count that the seed does not change
        keys = keys[torch.arange(E, device="cuda") * keys.numel() // E]
        s["dg"] = _graph(case["V"], *_csc(case["V"], keys))
        s["room"] = _segment_room(case, E)
        return s
    fwd, back = _rmat(case["V"], case["ef"], seed, kind == "labelprop", kind in ("push", "bc"))
    dg = s["dg"] = _graph(case["V"], *fwd)
    N, B, tile = case["N"], case["B"], case["tile"]
    if kind != "push":
        seg = s["seg"] = cagra.build_segments(dg, N, B, tile)
    if back is not None:
        s["dgt"] = _graph(case["V"], *back)
        s["seg_t"] = cagra.build_segments(s["dgt"], N, B, tile)
    if kind == "pagerank":
        s["state"] = cagra.PageRankState(dg, seg, cagra.BF16 if case["dtype"] == "bf16" else cagra.F32)
    elif kind == "solve":
        s["contrib"] = cagra.BF16 if case["dtype"] == "bf16" else cagra.F32
        s["buffers"] = cagra.SolveBuffers(dg, seg, s["contrib"], case["switch"])
    elif kind == "push":
        s["state"] = cagra.PushPageRankState(dg, s["seg_t"])
    elif kind == "ppr":
        s["state"] = cagra.PPRState(dg, seg, _seeds(case, seed))
    elif kind == "bc":
        s["state"] = cagra.BCState(seg, s["seg_t"])
        s["sources"] = _starts(case, seed, fwd[2])
    elif kind == "start":
        p, m, v, norm = _network(seed)
        s["net"] = warmstart.Network(p, p.to(torch.bfloat16).view(torch.int16), m, v, norm)
    return s


# ------------------------------------------------------------------ one pass

def run(s):
    kind, case = s["kind"], s["case"]
    if kind in ("pagerank", "push"):
        st = s["state"]
        st.start()
        for _ in range(case["iters"]):
            st.step(DAMPING)
        return {"rank": st.rank_now, "scalars": st.scalars_now}
    if kind == "solve":
        r = cagra.pagerank_solve(s["dg"], s["seg"], tol=1e-6, damping=DAMPING, contrib_type=s["contrib"],
                                 switch_tol=case["switch"], state=s["buffers"], restart=case["restart"])
        return {"rank": r.rank, "iterations": r.iters}
    if kind == "labelprop":
        labels, iters = cagra.labelprop(s["seg"])
        return {"labels": labels, "iterations": iters}
    if kind == "ppr":
        st = s["state"]
        st.start()
        for _ in range(case["iters"]):
            st.step(DAMPING)
        return {"ranks": st.ranks(), "scalars": st.scalars_now}
    if kind == "multi":
        m = s["multi"]
        m.replay()
        return {"ranks": m.rank[m.cur], "scalars": m.scalars[m.cur]}
    if kind == "prep":
        dg, out = s["dg"], {}
        if case["cluster"]:
            dg, out["perm"], out["hot"] = cagra.cluster(dg)
            out["offsets"], out["sources"], out["degrees"] = dg.in_offsets, dg.in_sources, dg.out_degree
        c = _build_into(dg, case, s["room"])
        out["segments"], out["sizes"] = s["room"], [c.k, c.nb, c.Q, c.ntiles]
        return out
    if kind == "cf":
        st = s["state"]
        st.cur = 0
        st.step(3e-5, 0.05)
        return {"x": st.x_now, "squares": st.sq}
    if kind == "bc":
        st = s["state"]
        st.bc.zero_()
        for v in s["sources"]:
            st.add_source(v)
        return {"bc": st.bc, "depth": st.depth, "sigma": st.sigma}
    if kind == "train":
        net = s["net"]
        s["buf"].copy_(s["start"])
        net.weights.copy_(s["start_weights"])
        net.step = 10
        F, T = warmstart.sample_rows(s["F"], s["T"], s["seed"], 7, case["batch"], s["batch"])
        grad, loss = net.grad(F, T)
        net.adam(grad, lr=3e-3)
        return {"grad": grad, "loss": loss, "master": net.master, "m": net.m, "v": net.v}
    rank0, usable = warmstart.learned_start(s["net"], s["dg"], s["seg"])
    return {"rank0": rank0, "usable": usable}


# ------------------------------------------------------------------ 64 bits

def _pull(off, src, x):
    """sum over the in-edges u -> v of x[u] (float64), for every v: differences
    of prefix sums over short runs of edges, so that no prefix grows large."""
    return _row_sums(off, lambda lo, hi: x[src[lo:hi].long()], x.shape[1:])


def _row_sums(off, terms, shape=()):
    """Row sums of per-edge terms(lo, hi) ([hi - lo, *shape], float64)."""
    V, E = off.numel() - 1, int(off[-1].item())
    out = torch.zeros((V,) + tuple(shape), dtype=torch.float64, device="cuda")
    rows = off.long()
    step = (CHUNK >> 4) // (32 if shape else 1)
    cuts = list(range(0, E, step)) + [E]
    edges = torch.tensor(cuts, device="cuda")
    firsts = (torch.searchsorted(rows, edges[:-1], right=True) - 1).tolist()  # row of each run's first edge
    lasts = (torch.searchsorted(rows, edges[1:] - 1, right=True) - 1).tolist()
    for lo, hi, first, last in zip(cuts[:-1], cuts[1:], firsts, lasts):
        t = terms(lo, hi)
        t = torch.cumsum(t.T.contiguous(), 1).T if shape else torch.cumsum(t, 0)
        t = torch.cat([torch.zeros_like(t[:1]), t])
        ends = t[rows[first:last + 2].clamp(lo, hi) - lo]
        out[first:last + 1] += ends[1:] - ends[:-1]
    return out


def _power(V, off, src, deg, iters, bf16=False, restart=-1, tol=0.0):
    """(rank, scalars, iterations) of the float64 power iteration."""
    r = torch.full((V,), 1.0 / V, dtype=torch.float64, device="cuda")
    if restart >= 0:
        r.zero_()
        r[restart] = 1.0
    d, hangs = deg.double(), deg == 0
    scalars = None
    for it in range(1, iters + 1):
        x = torch.where(hangs, torch.zeros_like(r), r / d)
        if bf16:
            x = x.float().bfloat16().double()
        new = DAMPING * _pull(off, src, x)
        back = DAMPING * r[hangs].sum()
        if restart >= 0:
            new[restart] += (1 - DAMPING) + back
        else:
            new += (1 - DAMPING) / V + back / V
        res = (new - r).abs().sum()
        r = new
        scalars = torch.stack([r[hangs].sum(), res, r.sum(), torch.zeros_like(res)])
        if tol > 0 and float(res) < tol:
            break
    return r, scalars, it


def _mlp(p, norm, F):
    """Network output in float64; p: the 4481 parameters."""
    x = (F.double() - norm[:3].double()) * norm[3:].double()
    g = torch.nn.functional.gelu
    h = g(x @ p[:192].view(64, 3).T + p[192:256])
    h = g(h @ p[256:4352].view(64, 64).T + p[4352:4416])
    return h @ p[4416:4480] + p[4480]


def _sampled(case, seed):
    """Rows of minibatch 7 (SplitMix64 by counter, multiply-shift range reduction)."""
    M = (1 << 64) - 1
    i = np.arange(case["batch"], dtype=np.uint64) + np.uint64(7 * case["batch"] + 1)
    with np.errstate(over="ignore"):
        z = np.uint64(seed & M) + i * np.uint64(0x9e3779b97f4a7c15)
        z = (z ^ (z >> np.uint64(30))) * np.uint64(0xbf58476d1ce4e5b9)
        z = (z ^ (z >> np.uint64(27))) * np.uint64(0x94d049bb133111eb)
        z ^= z >> np.uint64(31)
        n, low = np.uint64(case["rows"]), np.uint64(0xffffffff)
        rows = ((z >> np.uint64(32)) * n + (((z & low) * n) >> np.uint64(32))) >> np.uint64(32)
    return torch.from_numpy(rows.astype(np.int64)).cuda()


def _brandes(V, fwd, back, starts):
    """Betweenness of the starts, and path counts of the last, in float64. fwd
    and back: (offsets, sources) of the graph and of its reverse."""
    bc = torch.zeros(V, dtype=torch.float64, device="cuda")
    for s in starts:
        depth = torch.full((V,), -1, dtype=torch.int32, device="cuda")
        sigma = torch.zeros(V, dtype=torch.float64, device="cuda")
        zero = torch.zeros_like(sigma)
        depth[s], sigma[s], d = 0, 1.0, 0
        while True:
            got = _pull(*fwd, torch.where(depth == d, sigma, zero))
            new = (got > 0.5) & (depth < 0)  # path counts are whole numbers
            if not bool(new.any()):
                break
            d += 1
            depth[new] = d
            sigma = torch.where(new, got.round(), sigma)
        delta = torch.zeros_like(sigma)
        for lev in range(d - 1, -1, -1):
            share = torch.where(depth == lev + 1, (1 + delta) / sigma.clamp_min(1), zero)
            delta = torch.where(depth == lev, sigma * _pull(*back, share), delta)
        delta[s] = 0
        bc += delta
    return bc, sigma


def exact(case, seed):
    kind = case["kind"]
    if kind in ("labelprop", "prep"):
        return None  # whole numbers
    if kind == "multi":
        got = [_power(V, *_rmat(V, ef, seed + 100 + i)[0], case["iters"])
               for i, (V, ef) in enumerate(_multi_sizes(case))]
        return {"ranks": torch.cat([g[0] for g in got]), "scalars": torch.cat([g[1] for g in got])}
    if kind == "cf":
        V, off, src, deg, r, x0 = _ratings(case, seed)
        x, sq = x0.double(), []
        dst = torch.repeat_interleave(torch.arange(V, device="cuda"), (off[1:] - off[:-1]).long())

        def terms(lo, hi):
            xu = x[src[lo:hi].long()]
            err = r[lo:hi].double() - (xu * x[dst[lo:hi]]).sum(1)
            sq.append((err * err).sum())
            return err[:, None] * xu

        g = _row_sums(off, terms, x.shape[1:])
        return {"x": x + 3e-5 * (g - 0.05 * x), "squares": torch.stack(sq).sum().reshape(1)}
    if kind == "train":
        F, T = _rows(case, seed)
        p0, m, v, norm = _network(seed)
        rows = _sampled(case, seed)
        p = p0.to(torch.bfloat16).double().requires_grad_(True)
        loss = ((_mlp(p, norm, F[rows]) - T[rows].double()) ** 2).mean()
        loss.backward()
        grad, b1, b2 = p.grad, 0.9, 0.999
        m, v = b1 * m.double() + (1 - b1) * grad, b2 * v.double() + (1 - b2) * grad * grad
        step = 3e-3 * (m / (1 - b1 ** 11)) / ((v / (1 - b2 ** 11)).sqrt() + 1e-8)
        return {"grad": grad, "loss": loss.detach().reshape(1), "master": p0.double() - step, "m": m, "v": v}
    (off, src, deg), back = _rmat(case["V"], case["ef"], seed, reverse=kind == "bc")
    V = case["V"]
    if kind in ("pagerank", "push"):
        r, scalars, _ = _power(V, off, src, deg, case["iters"], case.get("dtype") == "bf16")
        return {"rank": r, "scalars": scalars}
    if kind == "solve":
        bf16 = case["dtype"] == "bf16"  # its answer is the fixed point up to the stopping rule
        r, _, _ = _power(V, off, src, deg, 100, restart=case["restart"], tol=1e-12 if bf16 else 1e-6)
        return {"rank": r, "iterations": None}
    if kind == "ppr":
        r = torch.zeros(V, case["cols"], dtype=torch.float64, device="cuda")
        seeds = torch.from_numpy(_seeds(case, seed).astype(np.int64)).cuda()
        cols = torch.arange(case["cols"], device="cuda")
        r[seeds, cols] = 1.0
        hangs = deg == 0
        for _ in range(case["iters"]):
            x = torch.where(hangs[:, None], torch.zeros_like(r), r / deg.double()[:, None])
            new = DAMPING * _pull(off, src, x)
            new[seeds, cols] += (1 - DAMPING) + DAMPING * r[hangs].sum(0)
            res, r = (new - r).abs().sum(0), new
        return {"ranks": r, "scalars": torch.stack([r[hangs].sum(0), res, r.sum(0), torch.zeros_like(res)], 1)}
    if kind == "bc":
        bc, sigma = _brandes(V, (off, src), back[:2], _starts(case, seed, deg))
        return {"bc": bc, "depth": None, "sigma": sigma}
    p, _, _, norm = _network(seed)
    indeg = (off[1:] - off[:-1]).double()
    od = torch.log1p(deg.double())
    mean = torch.where(indeg > 0, _pull(off, src, od) / indeg.clamp_min(1), torch.zeros_like(indeg))
    y = _mlp(p.to(torch.bfloat16).double(), norm, torch.stack([torch.log1p(indeg), od, mean], 1))
    return {"rank0": torch.softmax(y, 0), "usable": None}


# ------------------------------------------------------------------ floors

def work(case):
    """Inputs read once and outputs written once (edges at their word width)."""
    kind = case["kind"]
    if kind == "train":
        n = case["batch"]
        return {"bytes": 32.0 * n + 30.0 * warmstart.NPARAM, "flops": 6.0 * 4352 * n}
    if kind == "multi":
        V = case["graphs"] * ((2 << case["hi"]) - (1 << case["lo"])) / (case["hi"] - case["lo"] + 1)
        return {"bytes": case["iters"] * (2.0 * 20 * V + 20.0 * V), "flops": case["iters"] * 20.0 * V}
    if kind == "cf":
        V, E = case["users"] + case["items"], 2.0 * case["ef"] * case["users"]
        return {"bytes": 8 * E + 512.0 * V, "flops": 4 * 64 * E}
    V, E = case["V"], float(case["ef"] * case["V"])
    word = 2 if case["N"] <= cagra.EDGE16_MAX_N else 4
    if kind in ("pagerank", "push"):
        c = 2 if case.get("dtype") == "bf16" else 4
        return {"bytes": case["iters"] * (word * E + (12 + 2 * c) * V), "flops": case["iters"] * E}
    if kind == "solve":
        return {"bytes": 12 * (word * E + 18.0 * V), "flops": 12 * E}
    if kind == "labelprop":
        return {"bytes": 6 * (2 * word * E + 8.0 * V), "flops": 12 * E}
    if kind == "ppr":
        return {"bytes": case["iters"] * (word * E + 4 * 256.0 * V), "flops": case["iters"] * 64 * E}
    if kind == "prep":
        E = float(_prep_edges(case))
        once = 8 * E + 16.0 * V if case["cluster"] else 0.0
        return {"bytes": once + (4 + word) * E + 8.0 * V, "flops": E}
    if kind == "bc":
        return {"bytes": case["starts"] * (2 * word * E + 32.0 * V), "flops": case["starts"] * 2 * E}
    return {"bytes": word * E + 16.0 * V, "flops": E + 8700.0 * V}
