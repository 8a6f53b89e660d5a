"""The work that programs have this library do, as cases that can be timed.

Four kinds of calls, each through the public entry points of
``paper_2511_05895_amd.mf``:

* ``solve``: a static solve of a resident graph (``MaxFlow.solve``), with the
  minimum cut read back where a program would use it;
* ``update``: dynamic updates of a resident, solved graph from host arrays
  (``MaxFlow.update``) or device arrays (``MaxFlow.update_device``);
* ``oneshot``: a graph given once as host arrays: build, solve, cut, release;
* ``batch`` and ``serve``: many independent instances in one call, and several
  resident graphs behind the server with one request each per pass.

Graphs are those of the library's benchmark: uniform random graphs of 8 edges
per vertex, 4-connected segmentation grids with source and sink links, and
R-MAT power-law graphs of about 16 edges per vertex.  Everything is integers:
capacities int32, values int64, cut sides uint8.

An update state holds a few batches over disjoint edges and, for each, the
batch that restores the capacities it changed; successive passes apply them in
turn, so every pass changes the graph, passes go on for ever, and the
capacities after pass k depend on k alone.  ``raise_share`` is the share of a
batch's edges that are raised (0.5: mixed; 1: every other pass raises only and
the next lowers only; 0: the reverse).

Per-edge flows (``MaxFlow.edge_flow``) are left out: a maximum flow is not
unique, so two correct runs return different arrays."""
from __future__ import annotations

from types import SimpleNamespace

import numpy as np
import torch

from paper_2511_05895_amd import mf

# R-MAT quadrant probabilities (0.57, 0.19, 0.19, 0.05) in units of 2^-16
_T1, _T2, _T3 = 37356, 49807, 62259


def listed():
    return [
        # The smallest call in use: 100 changed edges on a graph of a thousand
        # vertices; nothing but launches and latency.
        {"name": "update_random_1k", "op": "update", "graph": "random", "n": 1000, "edges": 8000, "k": 100,
         "batches": 4, "raise_share": 0.5, "device_arrays": False, "cut": False},
        # The smallest static solve, with its cut.
        {"name": "solve_random_1k", "op": "solve", "graph": "random", "n": 1000, "edges": 8000, "cut": True},
        # A mid-size uniform graph of odd size under batches that lower
        # capacities (and batches that put them back), cut wanted every time.
        {"name": "update_random_20k", "op": "update", "graph": "random", "n": 20011, "edges": 160093, "k": 801,
         "batches": 4, "raise_share": 0.0, "device_arrays": False, "cut": True},
        # Interactive segmentation: 1 % of a 512 x 512 grid's edges change and
        # the labels are read back.
        {"name": "update_grid_512", "op": "update", "graph": "grid", "side": 512, "k": 15708, "batches": 2,
         "raise_share": 0.5, "device_arrays": False, "cut": True},
        # The same image segmented from scratch.
        {"name": "solve_grid_512", "op": "solve", "graph": "grid", "side": 512, "cut": True},
        # A power-law graph of 16.8 M edges: 1 % mixed batches already in
        # device memory, value wanted.
        {"name": "update_rmat_20", "op": "update", "graph": "rmat", "scale": 20, "edges": 1 << 24, "k": 167772,
         "batches": 2, "raise_share": 0.5, "device_arrays": True, "cut": False},
        # The same graph from scratch, with the cut.
        {"name": "solve_rmat_20", "op": "solve", "graph": "rmat", "scale": 20, "edges": 1 << 24, "cut": True},
        # The largest resident graph: requests of 10 to 100,000 edges
        # (log-uniform; k = 0 stands for that) against 67 M edges.
        {"name": "requests_rmat_22", "op": "update", "graph": "rmat", "scale": 22, "edges": 1 << 26, "k": 0,
         "batches": 8, "raise_share": 0.5, "device_arrays": False, "cut": False},
        # The largest static solve.
        {"name": "solve_rmat_22", "op": "solve", "graph": "rmat", "scale": 22, "edges": 1 << 26, "cut": False},
        # A graph that is seen once: build from host arrays, solve, cut.
        {"name": "oneshot_rmat_18", "op": "oneshot", "graph": "rmat", "scale": 18, "edges": 4000037},
        # Uneven independent instances in one call: grids of side 32..256 and
        # random graphs of 1k..50k vertices, alternating.
        {"name": "batch_64", "op": "batch", "count": 64},
        # Four tenants behind the server, grids of different sides, one
        # mixed request each.
        {"name": "serve_4_grids", "op": "serve", "tenants": 4, "side_lo": 120, "side_hi": 250, "share": 0.01,
         "batches": 2},
    ]


def _log_int(rng, lo, hi):
    return int(round(lo * (hi / lo) ** rng.random()))


def _draw_graph(rng, op):
    kind = rng.choice(["random", "grid", "rmat"])
    if kind == "random":
        n = _log_int(rng, 500, 50000) | 1
        return {"graph": kind, "n": n, "edges": 8 * n + rng.randrange(97)}
    if kind == "grid":
        return {"graph": kind, "side": _log_int(rng, 32, 500)}
    scale = rng.randint(12, 19 if op == "oneshot" else 22)
    return {"graph": kind, "scale": scale, "edges": rng.randint(12 << scale, 16 << scale)}


def _edge_count(case):
    if case["graph"] == "grid":
        s = case["side"]
        return 4 * s * (s - 1) + 2 * s * s
    return case["edges"]


def draw(rng):
    op = rng.choice(["update", "update", "update", "solve", "solve", "oneshot", "batch", "serve"])
    if op == "batch":
        return {"op": op, "count": rng.randint(9, 63)}
    if op == "serve":
        lo = _log_int(rng, 40, 150)
        return {"op": op, "tenants": rng.randint(2, 6), "side_lo": lo, "side_hi": lo + rng.randint(1, 100),
                "share": round(10 ** rng.uniform(-4, -1.5), 6), "batches": 2}
    c = {"op": op, **_draw_graph(rng, op)}
    if op == "oneshot":
        return c
    c["cut"] = rng.random() < 0.5
    if op == "update":
        m = _edge_count(c)
        c["batches"] = rng.choice([2, 4])
        c["k"] = min(m // c["batches"], max(1, int(m * 10 ** rng.uniform(-5, -1.3))))
        c["raise_share"] = rng.choice([0.0, 0.5, 0.5, 1.0])
        c["device_arrays"] = rng.random() < 0.3
    return c


# ---------------------------------------------------------------- inputs

def _gen(*key):
    """A generator on the GPU whose stream depends on the key alone."""
    seed = int(np.random.SeedSequence([int(x) for x in key]).generate_state(1, np.uint64)[0] >> np.uint64(1))
    return torch.Generator(device="cuda").manual_seed(seed)


def _rand(lo, hi, shape, gen, dtype=torch.int64):
    """Uniform integers of [lo, hi]."""
    return torch.randint(lo, hi + 1, shape, generator=gen, device="cuda", dtype=dtype)


def _csr(n, src, dst, cap, s, t):
    """Host CSR arrays, rows sorted by head."""
    order = torch.sort(src * n + dst, stable=True).indices
    src, dst, cap = src[order], dst[order], cap[order]
    row_ptr = torch.zeros(n + 1, dtype=torch.int64, device="cuda")
    row_ptr[1:] = torch.cumsum(torch.bincount(src, minlength=n), 0)
    return SimpleNamespace(n=int(n), row_ptr=row_ptr.cpu().numpy(), col=dst.to(torch.int32).cpu().numpy(),
                           cap=cap.to(torch.int32).cpu().numpy(), s=int(s), t=int(t))


def _random_graph(n, m, cap_hi, gen):
    """Uniform endpoints, no self-loops, capacities U[1, cap_hi]."""
    src = _rand(0, n - 1, (m,), gen)
    dst = (src + 1 + _rand(0, n - 2, (m,), gen)) % n
    return _csr(n, src, dst, _rand(1, cap_hi, (m,), gen), 0, n - 1)


def _grid_ends(side):
    idx = torch.arange(side * side, device="cuda").reshape(side, side)
    a = torch.cat([idx[:, :-1].reshape(-1), idx[:-1, :].reshape(-1)])
    b = torch.cat([idx[:, 1:].reshape(-1), idx[1:, :].reshape(-1)])
    return idx.reshape(-1), a, b


def _blur(img, sigma=2.0, radius=6):
    w = torch.exp(-torch.arange(-radius, radius + 1, device="cuda", dtype=torch.float64) ** 2 / (2 * sigma * sigma))
    w = (w / w.sum()).tolist()
    for dim in (0, 1):
        size = img.shape[dim]
        at = torch.arange(-radius, size + radius, device="cuda")
        at = torch.where(at < 0, -at - 1, at)
        at = torch.where(at >= size, 2 * size - 1 - at, at)
        wide = img.index_select(dim, at)
        img = sum(w[k] * wide.narrow(dim, k, size) for k in range(2 * radius + 1))
    return img


def _seg_grid(side, gen):
    """Segmentation grid: neighbour links 1 + round(100 exp(-dI^2 / 0.02)) of a
    blurred noise image, source and sink links U[0, 200] at every pixel."""
    px, a, b = _grid_ends(side)
    img = _blur(torch.randn(side, side, generator=gen, device="cuda", dtype=torch.float64)).reshape(-1)
    img = (img - img.min()) / (img.max() - img.min())
    w = 1 + torch.floor(100 * torch.exp(-((img[a] - img[b]) ** 2) / 0.02) + 0.5).to(torch.int64)
    s, t = side * side, side * side + 1
    src = torch.cat([a, b, torch.full_like(px, s), px])
    dst = torch.cat([b, a, px, torch.full_like(px, t)])
    return _csr(side * side + 2, src, dst, torch.cat([w, w, _rand(0, 200, (2 * px.numel(),), gen)]), s, t)


def _plain_grid(side, gen):
    """Grid with every capacity U[1, 1000] (the batched solver's instances)."""
    px, a, b = _grid_ends(side)
    s, t = side * side, side * side + 1
    src = torch.cat([a, b, torch.full_like(px, s), px])
    dst = torch.cat([b, a, px, torch.full_like(px, t)])
    return _csr(side * side + 2, src, dst, _rand(1, 1000, (src.numel(),), gen), s, t)


def _rmat(scale, m, gen):
    """R-MAT(0.57, 0.19, 0.19) with permuted vertex ids, no self-loops,
    capacities U[1, 1000]; s and t are the two vertices of highest degree."""
    n = 1 << scale
    src = torch.zeros(m, dtype=torch.int32, device="cuda")
    dst = torch.zeros(m, dtype=torch.int32, device="cuda")
    for bit in range(scale):
        r = _rand(0, 65535, (m,), gen, torch.int32)
        src |= (r >= _T2).to(torch.int32) << bit
        dst |= (((r >= _T1) & (r < _T2)) | (r >= _T3)).to(torch.int32) << bit
    perm = torch.randperm(n, generator=gen, device="cuda")
    src, dst = perm[src.long()], perm[dst.long()]
    dst = torch.where(src == dst, (src + 1 + _rand(0, n - 2, (m,), gen)) % n, dst)
    deg = torch.bincount(src, minlength=n) + torch.bincount(dst, minlength=n)
    s, t = torch.topk(deg * n + (n - 1 - torch.arange(n, device="cuda")), 2).indices.tolist()
    return _csr(n, src, dst, _rand(1, 1000, (m,), gen), s, t)


def _graph(case, seed):
    gen = _gen(seed, 1)
    if case["graph"] == "random":
        return _random_graph(case["n"], case["edges"], 100, gen)
    if case["graph"] == "grid":
        return _seg_grid(case["side"], gen)
    return _rmat(case["scale"], case["edges"], gen)


def _batches(cap, sizes, raise_share, inc_hi, seed):
    """One batch per size over disjoint edges, as (ids, capacities); after
    each of them all, the batches that restore what they changed."""
    rng = np.random.default_rng([int(seed), 2])
    total = sum(sizes)
    m = cap.shape[0]
    if 4 * total < m:  # distinct ids without a permutation of all m
        ids = np.unique(rng.integers(0, m, 2 * total + 64))
        while ids.size < total:
            ids = np.unique(np.concatenate([ids, rng.integers(0, m, total)]))
        ids = rng.permutation(ids)[:total]
    else:
        ids = rng.permutation(m)[:total]
    out, back, at = [], [], 0
    for k in sizes:
        e = ids[at:at + k].astype(np.int64)
        at += k
        old = cap[e].astype(np.int64)
        up = int(np.ceil(k * raise_share))
        new = rng.integers(0, old + 1)
        new[:up] = old[:up] + rng.integers(1, inc_hi + 1, up)
        out.append((e, new.astype(np.int32)))
        back.append((e, old.astype(np.int32)))
    return out + back


def _update_inputs(case, seed):
    g = _graph(case, seed)
    if case["k"] > 0:
        sizes = [case["k"]] * case["batches"]
    else:  # log-uniform, one size from each part of the range
        rng = np.random.default_rng([int(seed), 3])
        b = case["batches"]
        u = rng.permutation((np.arange(b) + rng.random(b)) / b)
        sizes = [min(g.cap.shape[0] // b, int(round(10 * 10000 ** x))) for x in u]
    return g, _batches(g.cap, sizes, case["raise_share"], 100 if case["graph"] != "rmat" else 1000, seed)


def _batch_graphs(case, seed):
    # the sizes go with the case (one from each part of the range), edges and
    # capacities with the seed
    rng = np.random.default_rng([case["count"], 4])
    out = []
    for i in range(case["count"]):
        u = ((i // 2) + rng.random()) / ((case["count"] + 1) // 2)
        if i % 2 == 0:
            out.append(_plain_grid(int(round(32 * 8 ** u)), _gen(seed, 5, i)))
        else:
            n = int(round(1000 * 50 ** u))
            out.append(_random_graph(n, 8 * n, 1000, _gen(seed, 5, i)))
    return out


def _serve_sides(case):
    rng = np.random.default_rng([case["side_lo"], case["tenants"], 6])
    return rng.integers(case["side_lo"], case["side_hi"] + 1, case["tenants"]).tolist()


def prepare(case, seed):
    op = case["op"]
    if op == "oneshot":
        return {"case": case, "graph": _graph(case, seed)}
    if op == "batch":
        graphs = _batch_graphs(case, seed)
        largest = max(range(len(graphs)), key=lambda i: graphs[i].col.shape[0])
        return {"case": case, "batch": mf.Batch(graphs), "largest": largest}
    if op == "serve":
        server = mf.Server(workers=case["tenants"])
        tenants = []
        for i, side in enumerate(_serve_sides(case)):
            g = _seg_grid(side, _gen(seed, 7, i))
            gid, _ = server.add_graph(g)
            k = max(1, int(g.col.shape[0] * case["share"]))
            tenants.append((gid, _batches(g.cap, [k] * case["batches"], 0.5, 100, seed + 1000003 * i)))
        return {"case": case, "server": server, "tenants": tenants, "pass": 0}
    if op == "solve":
        return {"case": case, "flow": mf.MaxFlow(_graph(case, seed))}
    g, batches = _update_inputs(case, seed)
    flow = mf.MaxFlow(g)
    flow.solve()
    if case["device_arrays"]:
        batches = [(torch.from_numpy(e).cuda(), torch.from_numpy(c).cuda()) for e, c in batches]
    return {"case": case, "flow": flow, "batches": batches, "pass": 0}


def run(state):
    case = state["case"]
    op = case["op"]
    if op == "oneshot":
        with mf.MaxFlow(state["graph"]) as flow:
            value = flow.solve()
            side, cut = flow.min_cut()
        return {"value": value, "side": side, "cut": cut}
    if op == "batch":
        values = state["batch"].solve()
        side, cut = state["batch"].min_cut(state["largest"])
        return {"values": values, "side": side, "cut": cut}
    if op == "serve":
        server, at = state["server"], state["pass"]
        state["pass"] += 1
        ids = [server.submit(gid, *batches[at % len(batches)]) for gid, batches in state["tenants"]]
        results = [server.wait(i) for i in ids]
        for i in ids:
            server.release(i)
        return {"values": [r["value"] for r in results], "status": [r["status"] for r in results]}
    flow = state["flow"]
    if op == "solve":
        out = {"value": flow.solve()}
    else:
        ids, caps = state["batches"][state["pass"] % len(state["batches"])]
        state["pass"] += 1
        out = {"value": flow.update_device(ids, caps) if case["device_arrays"] else flow.update(ids, caps)}
    if case["cut"]:
        out["side"], out["cut"] = flow.min_cut()
    return out


# ---------------------------------------------------------------- floors

def _solve_bytes(n, m):
    """Read a graph of n vertices and m edges once (row bounds, head and
    capacity of every edge), write its residuals and heights once."""
    return 4 * (n + 1) + 8 * m + 4 * m + 4 * n


def _sizes(case):
    if case["graph"] == "grid":
        return case["side"] ** 2 + 2, _edge_count(case)
    return (case["n"] if case["graph"] == "random" else 1 << case["scale"]), case["edges"]


def work(case):
    op = case["op"]
    if op == "batch":
        total, parts = 0, (case["count"] + 1) // 2
        for i in range(case["count"]):
            u = ((i // 2) + 0.5) / parts
            side, n = int(round(32 * 8 ** u)), int(round(1000 * 50 ** u))
            total += _solve_bytes(side * side + 2, 6 * side * side - 4 * side) if i % 2 == 0 else _solve_bytes(n, 8 * n)
        return {"bytes": total + 8 * case["count"], "flops": 0}
    per_update = 12 + 16  # id and capacity in; both residuals of the edge's pair, read and written
    if op == "serve":
        side = (case["side_lo"] + case["side_hi"]) / 2
        return {"bytes": case["tenants"] * (max(1, int(6 * side * side * case["share"])) * per_update + 8), "flops": 0}
    n, m = _sizes(case)
    if op == "oneshot":
        return {"bytes": _solve_bytes(n, m) + n + 16, "flops": 0}
    cut = n + 8 if case["cut"] else 0
    if op == "solve":
        return {"bytes": _solve_bytes(n, m) + cut + 8, "flops": 0}
    k = case["k"] if case["k"] > 0 else (100000 - 10) / np.log(10000)  # mean of the log-uniform sizes
    return {"bytes": float(k * per_update + cut + 8), "flops": 0}


# ---------------------------------------------------------------- exact values

def _max_flow(g, cap):
    """Dinic's algorithm in plain Python: value, source side (the vertices
    that cannot reach t in the residual graph), cut capacity."""
    n, s, t = g.n, g.s, g.t
    tails = np.repeat(np.arange(n), np.diff(g.row_ptr)).tolist()
    heads, out = [], [[] for _ in range(n)]
    res = []
    for u, v, c in zip(tails, g.col.tolist(), cap.tolist()):
        out[u].append(len(heads))
        heads.append(v)
        res.append(c)
        out[v].append(len(heads))
        heads.append(u)
        res.append(0)
    value = 0
    while True:
        dist = [-1] * n  # distance to t
        dist[t] = 0
        queue = [t]
        for v in queue:
            for a in out[v]:
                if res[a ^ 1] > 0 and dist[heads[a]] < 0:
                    dist[heads[a]] = dist[v] + 1
                    queue.append(heads[a])
        if dist[s] < 0:
            break
        at = [0] * n
        path, v = [], s
        while True:
            if v == t:
                d = min(res[a] for a in path)
                value += d
                for a in path:
                    res[a] -= d
                    res[a ^ 1] += d
                path, v = [], s
                continue
            while at[v] < len(out[v]):
                a = out[v][at[v]]
                if res[a] > 0 and dist[heads[a]] == dist[v] - 1:
                    break
                at[v] += 1
            else:
                if v == s:
                    break
                a = path.pop()
                v = heads[a ^ 1]
                at[v] += 1
                continue
            path.append(a)
            v = heads[a]
    side = (np.array(dist) < 0).astype(np.uint8)
    crossing = (side[np.array(tails)] == 1) & (side[g.col] == 0)
    return value, side, int(cap[crossing].astype(np.int64).sum())


def exact(case, seed):
    """What the first pass returns, for the graphs that plain Python solves
    within seconds."""
    if case["op"] not in ("solve", "update") or case["graph"] != "random" or case["edges"] > 20000:
        return None
    if case["op"] == "solve":
        g = _graph(case, seed)
        cap = g.cap
    else:
        g, batches = _update_inputs(case, seed)
        cap = g.cap.copy()
        cap[batches[0][0]] = batches[0][1]
    value, side, cut = _max_flow(g, cap)
    return {"value": value, "side": side, "cut": cut} if case["cut"] else {"value": value}
