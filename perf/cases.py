"""Workloads of the CL-DIAM framework, each one pass through its public entry
points (paper_1506_03265_amd): what a program that estimates diameters has it
do, from a 4,096-node mesh to an R-MAT graph of 520 million arcs.

Paths
  pipeline  resident graph -> decomposition, quotient graph, estimate (all
            three variants of the decomposition)
  quotient  a clustering in hand -> quotient graph and estimate, with the
            thousands of clusters of a larger tau
  batch     many graphs decomposed in one device job
  server    a queue of requests through the continuous-batching server
  sssp      the Delta-stepping competitor, from one source
  ingest    a CSR in device memory -> validated, weight-sorted packed arcs

Graphs are the families of graphgen (meshes, road-like meshes, R-MAT, random
geometric graphs, with its weight laws, largest components), drawn here on the
GPU with torch so that a new one of any size takes well under two seconds.
The topology belongs to the case (sizes stay the same from seed to seed); the
weights and the random centers come from the seed, as when a network's travel
times change.

Every output is a whole number (ids, distances, counts) and is determined by
the inputs; quantities that depend on the schedule (sweeps, times) are left out.
"""
import math

import torch

import paper_1506_03265_amd as cd

DEV = "cuda"
MOST_K = 3072   # quotients of more nodes (rare at these tau) are returned without the all-pairs estimate


# ---------------------------------------------------------------- graphs --

def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    return g


def _components(n, u, v):
    """Component labels of an edge list: hooking on smaller labels and pointer jumping."""
    f = torch.arange(n, device=DEV)
    while u.numel():
        fu, fv = f[u], f[v]
        live = fu != fv
        u, v, fu, fv = u[live], v[live], fu[live], fv[live]
        f.scatter_reduce_(0, torch.maximum(fu, fv), torch.minimum(fu, fv), "amin")
        while True:
            ff = f[f]
            if torch.equal(ff, f):
                break
            f = ff
    return f


def _largest(part, parts, u, v, w):
    """Keeps the largest component of every part (part: the part of each node,
    ascending); node ids stay ascending.  Returns nodes per part and the edges."""
    n = part.numel()
    f = _components(n, u, v)
    size = torch.bincount(f, minlength=n)
    best = torch.zeros(parts, dtype=torch.int64, device=DEV)
    best.scatter_reduce_(0, part, size * n + (n - 1 - torch.arange(n, device=DEV)), "amax")
    keep = f == (n - 1 - best % n)[part]
    new = torch.cumsum(keep, 0) - 1
    e = keep[u]
    return torch.bincount(part[keep], minlength=parts).tolist(), new[u[e]], new[v[e]], w[e]


def _csr(n, u, v, w):
    """Symmetric CSR, rows sorted by column, of an edge list."""
    key = torch.cat([u * n + v, v * n + u])
    key, at = torch.sort(key)
    m = w.numel()
    w = w[torch.where(at < m, at, at - m)]
    col = (key % n).to(torch.int32)
    rp = torch.zeros(n + 1, dtype=torch.int64, device=DEV)
    rp[1:] = torch.cumsum(torch.bincount(key // n, minlength=n), 0)
    return n, rp, col, w


def _topology():
    return _gen(1)


def _weights(m, top, g):
    return torch.randint(1, top + 1, (m,), generator=g, device=DEV, dtype=torch.int32)


def _mesh(rows, cols, road, g):
    """rows x cols mesh, weights in [1, 10^4]; road: 5% of the edges dropped,
    a diagonal in 1% of the cells, largest component."""
    at = torch.arange(rows * cols, device=DEV).view(rows, cols)
    u = torch.cat([at[:, :-1].reshape(-1), at[:-1].reshape(-1)])
    v = torch.cat([at[:, 1:].reshape(-1), at[1:].reshape(-1)])
    if road:
        t = _topology()
        keep = torch.rand(u.numel(), generator=t, device=DEV) >= 0.05
        x = torch.rand((rows - 1) * (cols - 1), generator=t, device=DEV)
        nw = at[:-1, :-1].reshape(-1)
        down, up = nw[x < 0.005], nw[(x >= 0.005) & (x < 0.01)]
        u = torch.cat([u[keep], down, up + 1])
        v = torch.cat([v[keep], down + cols + 1, up + cols])
    w = _weights(u.numel(), 10000, g)
    n = rows * cols
    if road:
        (n,), u, v, w = _largest(torch.zeros(n, dtype=torch.int64, device=DEV), 1, u, v, w)
    return _csr(n, u, v, w)


def _rmat(scale, g):
    """R-MAT(scale, 16) with (a, b, c) = (.57, .19, .19), simple, largest
    component, random node numbers, weights in [1, 2^20]."""
    n, m = 1 << scale, 16 << scale
    u = torch.zeros(m, dtype=torch.int32, device=DEV)
    v = torch.zeros(m, dtype=torch.int32, device=DEV)
    t = _topology()
    for _ in range(scale):
        x = torch.rand(m, generator=t, device=DEV)
        u = 2 * u + (x >= 0.76)
        v = 2 * v + (((x >= 0.57) & (x < 0.76)) | (x >= 0.95))
    perm = torch.randperm(n, generator=t, device=DEV)
    u, v = perm[u], perm[v]
    key = torch.minimum(u, v) * n + torch.maximum(u, v)
    key = torch.unique(key[u != v])
    u, v = key // n, key % n
    w = _weights(u.numel(), 1 << 20, g)
    (n,), u, v, w = _largest(torch.zeros(n, dtype=torch.int64, device=DEV), 1, u, v, w)
    return _csr(n, u, v, w)


def _rgg(sizes, g):
    """Random geometric graphs of the given sizes, average degree 8, largest
    components, weight round(10^4 length x) + 1 with x in [1, 1.25] (a travel
    time: the length times the day's factor)."""
    n = sum(sizes)
    part = torch.repeat_interleave(torch.arange(len(sizes), device=DEV), torch.tensor(sizes, device=DEV))
    rad = [math.sqrt(8 / (math.pi * s)) for s in sizes]
    side = [max(1, int(1 / r)) for r in rad]
    base = [0]
    for s in side:
        base.append(base[-1] + s * s)
    rad, side, first = (torch.tensor(x, device=DEV)[part] for x in (rad, side, base[:-1]))
    xy = torch.rand((n, 2), generator=_topology(), device=DEV)
    cx, cy = ((xy[:, i] * side).long().clamp_(max=10**9) for i in (0, 1))
    cx, cy = torch.minimum(cx, side - 1), torch.minimum(cy, side - 1)
    order = torch.argsort(first + cx * side + cy)   # node numbers follow the cells
    xy, cx, cy = xy[order], cx[order], cy[order]
    count = torch.bincount(first + cx * side + cy, minlength=base[-1])
    start = torch.cumsum(count, 0) - count
    me = torch.arange(n, device=DEV)
    us, vs, ds = [], [], []
    most = int(count.max())
    for dx, dy in ((0, 0), (0, 1), (1, -1), (1, 0), (1, 1)):
        inside = (cx + dx < side) & (cy + dy >= 0) & (cy + dy < side)
        cell = torch.where(inside, first + (cx + dx) * side + cy + dy, 0)
        for k in range(most):
            i = me[inside & (count[cell] > k)]
            j = start[cell[i]] + k
            d = torch.linalg.vector_norm(xy[i] - xy[j], dim=1)
            ok = (d <= rad[i]) & ((j > i) | (dx != 0 or dy != 0))
            us.append(i[ok])
            vs.append(j[ok])
            ds.append(d[ok])
    u, v = torch.cat(us), torch.cat(vs)
    x = 1 + 0.25 * torch.rand(u.numel(), generator=g, device=DEV)
    w = (torch.cat(ds).double() * 1e4 * x).round().to(torch.int32) + 1
    ns, u, v, w = _largest(part, len(sizes), u, v, w)
    key = torch.argsort(u, stable=True)
    u, v, w = u[key], v[key], w[key]
    out, lo = [], 0
    ends = torch.searchsorted(u, torch.tensor([sum(ns[:i + 1]) for i in range(len(ns))], device=DEV)).tolist()
    for i, k in enumerate(ns):
        off = sum(ns[:i])
        out.append(_csr(k, u[lo:ends[i]] - off, v[lo:ends[i]] - off, w[lo:ends[i]]))
        lo = ends[i]
    return out


def _graph(case, g):
    if case["graph"] == "rmat":
        return _rmat(case["scale"], g)
    if case["graph"] == "rgg":
        return _rgg([case["nodes"]], g)[0]
    return _mesh(case["rows"], case["cols"], case["graph"] == "road", g)


def _sizes(case):
    """Sizes of a batch: evenly spread over the logarithm of the range."""
    k, lo, hi = case["count"], math.log(case["least"]), math.log(case["most"])
    return [round(math.exp(lo + (hi - lo) * ((i * 0.6180339887) % 1.0))) for i in range(k)]


def _served(case, g):
    """Graphs of a request queue: meshes and R-MAT graphs in turn."""
    out = []
    for i in range(case["count"]):
        t = (i * 0.6180339887) % 1.0
        if i % 2:
            out.append(_rmat(case["scale_lo"] + round(t * (case["scale_hi"] - case["scale_lo"])), g))
        else:
            side = case["side_lo"] + round(t * (case["side_hi"] - case["side_lo"]))
            out.append(_mesh(side, side, False, g))
    return out


# ----------------------------------------------------------------- cases --

def listed():
    return [
        # the smallest call: the 64 x 64 mesh of the smoke test, bound by latency and launches
        dict(name="mesh64", path="pipeline", graph="grid", rows=64, cols=64, tau=1, variant=0),
        # an ordinary served request on a mesh (the serving mix has sides 256 to 2048), odd sides
        dict(name="mesh1153", path="pipeline", graph="grid", rows=1153, cols=1021, tau=1, variant=0),
        # an ordinary served request on a social-like graph (scales 12 to 22)
        dict(name="rmat18", path="pipeline", graph="rmat", scale=18, tau=1, variant=0),
        # the benchmark's default workload
        dict(name="road4096", path="pipeline", graph="road", rows=4096, cols=4096, tau=4, variant=0),
        # the benchmark's social-like workload: the largest listed pass
        dict(name="rmat24", path="pipeline", graph="rmat", scale=24, tau=4, variant=0),
        # the paper's step-synchronous PartialGrowth, with its round and work counters
        dict(name="steps_road2048", path="pipeline", graph="road", rows=2048, cols=2048, tau=1, variant=1),
        # CLUSTER2 (Algorithm 2), the variant that the paper's estimate is stated for
        dict(name="cluster2_road2048", path="pipeline", graph="road", rows=2048, cols=2048, tau=4, variant=2),
        # a finer clustering: a larger quotient graph, so the estimate's all-pairs step counts
        dict(name="quotient_tau12", path="quotient", graph="road", rows=2048, cols=2048, tau=12),
        # a batch of random geometric graphs of 10^3 to 10^6 nodes in one job
        dict(name="batch_rgg64", path="batch", count=64, least=1000, most=1000000, tau=1),
        # a queue of two dozen mixed requests through the server
        dict(name="serve24", path="server", count=24, side_lo=256, side_hi=1024, scale_lo=12, scale_hi=18, tau=1),
        # the competitor on the benchmark's mesh, its default bucket width
        dict(name="sssp_road4096", path="sssp", graph="road", rows=4096, cols=4096, width=0),
        # a new graph's first step, rows of every length up to hubs
        dict(name="ingest_rmat21", path="ingest", graph="rmat", scale=21),
    ]


def _log_size(rng, lo, hi):
    return round(math.exp(rng.uniform(math.log(lo), math.log(hi))))


def _draw_graph(rng, mesh_hi, scale_hi, rgg_hi):
    kind = rng.choice(["grid", "road", "rmat", "rgg"])
    if kind == "rmat":
        return dict(graph=kind, scale=rng.randint(10, scale_hi))
    if kind == "rgg":
        return dict(graph=kind, nodes=_log_size(rng, 1000, rgg_hi))
    return dict(graph=kind, rows=_log_size(rng, 40, mesh_hi), cols=_log_size(rng, 40, mesh_hi))


def draw(rng):
    path = rng.choice(["pipeline"] * 5 + ["variant"] * 2 + ["quotient", "batch", "server", "sssp", "sssp", "ingest", "ingest"])
    if path == "pipeline":
        return dict(_draw_graph(rng, 4096, 23, 4000000), path="pipeline", tau=rng.choice([1, 2, 4]), variant=0)
    if path == "variant":
        return dict(_draw_graph(rng, 2048, 19, 1000000), path="pipeline", tau=1, variant=rng.choice([1, 2]))
    if path == "quotient":
        return dict(_draw_graph(rng, 2048, 20, 1000000), path="quotient", tau=rng.randint(4, 14))
    if path == "batch":
        return dict(path="batch", count=rng.randint(2, 96), least=1000, most=_log_size(rng, 3000, 1000000), tau=rng.choice([1, 2]))
    if path == "server":
        return dict(path="server", count=rng.randint(2, 28), side_lo=rng.randint(40, 256), side_hi=rng.randint(257, 1400),
                    scale_lo=rng.randint(10, 14), scale_hi=rng.randint(15, 18), tau=rng.choice([1, 2]))
    if path == "sssp":
        return dict(_draw_graph(rng, 4096, 20, 1000000), path="sssp", width=rng.choice([0, 0, 20000, 200000]))
    return dict(_draw_graph(rng, 4096, 22, 4000000), path="ingest")


# ------------------------------------------------------------------- run --

def _load(csr):
    return cd.cldiam_load_csr_device(csr[0], csr[2].numel(), csr[1], csr[2], csr[3])


def prepare(case, seed):
    """Resident graphs and the reusable jobs (outputs and workspaces) of a program."""
    g = _gen(seed)
    path = case["path"]
    if path == "ingest":
        return dict(path=path, csr=_graph(case, g))
    if path == "batch":
        graphs = [_load(c) for c in _rgg(_sizes(case), g)]
        job = cd.DecomposeJob(graphs, [(case["tau"], (i << 32) | (seed + 1), 0) for i in range(len(graphs))])
        return dict(path=path, job=job)
    if path == "server":
        graphs = [_load(c) for c in _served(case, g)]
        sizes = sorted((x.n for x in graphs), reverse=True)
        return dict(path=path, graphs=graphs, tau=case["tau"], seed=seed, server=cd.Server(sum(sizes[:8]), 64))
    dg = _load(_graph(case, g))
    if path == "sssp":
        return dict(path=path, graph=dg, width=case["width"], source=(seed * 2654435761 + 12345) % dg.n)
    quotient = cd.QuotientJob(dg)
    for t in (quotient.center, quotient.row_ptr, quotient.col, quotient.w):
        t.zero_()   # a quotient fills the first k and qm entries of the job's buffers: the rest reads as zero
    state = dict(path=path, quotient=quotient, estimate=cd.EstimateJob(1, 1, DEV),
                 job=cd.DecomposeJob([dg], [(case["tau"], seed + 1, 0, case.get("variant", 0), 0)]))
    if path == "quotient":
        job = state.pop("job")
        st = job.run()[0]
        state["clustering"] = (job.cluster[0], job.D[0], st.radius)
    return state


def _finish(state, cluster, D, radius):
    """Quotient graph and estimate of a clustering."""
    job = state["quotient"]
    q = job.run(cluster, D)
    phi, approx = state["estimate"].run(q, radius) if q.k <= MOST_K else (0, 0)
    return dict(k=q.k, qm=q.qm, center=job.center, row_ptr=job.row_ptr, col=job.col, w=job.w, phi=phi, approx=approx)


def _counts(st):
    return dict(clusters=st.num_clusters, singletons=st.singletons, stages=st.stages, levels=st.levels,
                delta_end=st.delta_end, radius=st.radius, radius1=st.radius1, rounds=st.rounds, messages=st.messages,
                updates=st.updates)


def run(state):
    path = state["path"]
    if path == "pipeline":
        job = state["job"]
        st = job.run()[0]
        out = _finish(state, job.cluster[0], job.D[0], st.radius)
        return dict(out, cluster=job.cluster[0], D=job.D[0], **_counts(st))
    if path == "quotient":
        return _finish(state, *state["clustering"])
    if path == "batch":
        job = state["job"]
        st = job.run()
        return dict(cluster=torch.cat(job.cluster), D=torch.cat(job.D),
                    radius=torch.tensor([s.radius for s in st]), clusters=torch.tensor([s.num_clusters for s in st]))
    if path == "server":
        srv, found = state["server"], {}
        for i, g in enumerate(state["graphs"]):
            srv.submit(g, state["tau"], state["seed"] + i, i)
        while len(found) < len(state["graphs"]):
            srv.step(8)
            for tag, st, _, cluster, D in srv.poll():
                found[tag] = (cluster, D, st.radius)
        return [list(found[i][:2]) for i in range(len(found))] + [torch.tensor([found[i][2] for i in range(len(found))])]
    if path == "sssp":
        dist, far = cd.cldiam_sssp_delta_stepping(state["graph"], state["source"], state["width"])
        return dict(dist=dist, far=far)
    n, rp, col, w = state["csr"]
    g = cd.cldiam_load_csr_device(n, col.numel(), rp, col, w)
    return dict(arcs=g.arcs, weight_sum=g.weight_sum)


# ------------------------------------------------------------------ work --

def _nm(case):
    """Nodes and arcs of a case's graph, in expectation."""
    if case["graph"] == "rmat":
        s = case["scale"]
        return (1 << s) * (0.53 if s > 20 else 0.6), (32 << s) * (0.97 if s > 20 else 0.9)
    if case["graph"] == "rgg":
        return case["nodes"], 8 * case["nodes"]
    n = case["rows"] * case["cols"]
    return n, (4 if case["graph"] == "grid" else 3.82) * n


def work(case):
    """The graph read once and the results written once; one addition and one
    comparison per arc (no path has a dense contraction)."""
    path = case["path"]
    if path == "batch":
        n = sum(_sizes(case))
        return dict(bytes=8 * n + 64 * n + 12 * n, flops=16 * n)
    if path == "server":
        n = m = 0
        for i in range(case["count"]):
            t = (i * 0.6180339887) % 1.0
            c = (dict(graph="rmat", scale=case["scale_lo"] + round(t * (case["scale_hi"] - case["scale_lo"]))) if i % 2 else
                 dict(graph="grid", rows=case["side_lo"] + round(t * (case["side_hi"] - case["side_lo"])), cols=1))
            if not i % 2:
                c["cols"] = c["rows"]
            a, b = _nm(c)
            n, m = n + a, m + b
        return dict(bytes=20 * n + 8 * m, flops=2 * m)
    n, m = _nm(case)
    if path == "ingest":
        return dict(bytes=8 * n + 16 * m, flops=2 * m)
    if path == "sssp":
        return dict(bytes=12 * n + 8 * m, flops=2 * m)
    graph = 8 * n + 8 * m
    if path == "quotient":
        return dict(bytes=graph + 12 * n, flops=2 * m)
    return dict(bytes=2 * graph + 24 * n, flops=4 * m)


def exact(case, seed):
    """Ingest: every row's packed arcs in order.  The other paths return whole
    numbers that have to be equal, and have no quick form in plain torch."""
    if case["path"] != "ingest":
        return None
    n, rp, col, w = _graph(case, _gen(seed))
    row = torch.repeat_interleave(torch.arange(n, device=DEV), rp[1:] - rp[:-1])
    arcs = (w.long() << 32) | col.long()
    arcs, at = torch.sort(arcs)
    arcs = arcs[torch.argsort(row[at], stable=True)]
    return dict(arcs=arcs, weight_sum=int(w.long().sum()))
