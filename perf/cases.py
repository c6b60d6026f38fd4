"""The label-propagation work that programs have this library do, as cases to
be timed: whole solves of one graph in both modes, the first solve of a graph
just received, many graphs in one batch or through the server, and the
scoring of a labelling.

Graphs are those of the repository's benchmark and tests (R-MAT, planted
partitions, the rewired grid), drawn on the GPU from the seed: the same families, parameters and weights as
``paper_2411_19901_amd.inputs``, without its host generators' run time.
Parameters that a case does not carry are the binding's defaults (tol 0.05,
at most 20 iterations, pick-less every 8, validation on, no workspace).
The in-place mode's labels depend on scheduling, so its cases are large
weighted R-MAT graphs, where they hardly do.
"""
import math

import torch

from paper_2411_19901_amd import inputs, lpa, serve

DEVICE = "cuda"


# ------------------------------------------------------------------- cases
def listed():
    return [
        # the smallest request of a serving mix: launches and latency are all of it
        dict(name="sbm 1e3 det", kind="solve", graph="sbm", n=1009, blocks=8, weights=False,
             mode="det", k=8),
        # the planted partition of the tests and the smoke run (10,000 vertices in 50 blocks)
        dict(name="sbm 1e4 wU det", kind="solve", graph="sbm", n=10_000, blocks=50, weights=True,
             mode="det", k=8),
        # a graph that a program has just received: set-up, solve, labels and score
        dict(name="sbm 1e5 wU first solve", kind="first", graph="sbm", n=99_991, blocks=120,
             weights=True, mode="det", k=8),
        # the same for a power-law graph at the top of the served range
        dict(name="rmat20 wU first solve", kind="first", graph="rmat", scale=20, edge_factor=16,
             weights=True, mode="det", k=8),
        # the benchmark's power-law graph with unit weights, reproducible labels
        dict(name="rmat22 det", kind="solve", graph="rmat", scale=22, edge_factor=16,
             weights=False, mode="det", k=8),
        # weighted, with fewer slots and the ranked layout
        dict(name="rmat21 wU det k4 ranked", kind="solve", graph="rmat", scale=21, edge_factor=16,
             weights=True, mode="det", k=4, ranked=True),
        # the in-place mode of the paper's GPU runs, default layout
        dict(name="rmat23 wU async", kind="solve", graph="rmat", scale=23, edge_factor=16,
             weights=True, mode="async", k=8),
        # the benchmark's flagship graph, in the layout that is fastest on it
        dict(name="rmat24 wU async ranked", kind="solve", graph="rmat", scale=24, edge_factor=16,
             weights=True, mode="async", k=8, ranked=True),
        # the road-network stand-in: many short rows and many iterations
        dict(name="grid 4096 det", kind="solve", graph="grid", rows=4096, cols=4096,
             weights=False, mode="det", k=8),
        # many graphs with one set of launches per iteration
        dict(name="batch of 512 sbm det", kind="batch", graphs=512, n_lo=1000, n_hi=200_000,
             weights=False, mode="det", k=8),
        # requests in host memory through the server: planted partitions and power-law graphs
        dict(name="served mix", kind="serve", requests=24, weights=True, mode="det", k=8),
        # scoring a caller's labelling of a large power-law graph
        dict(name="rmat23 wU modularity", kind="score", graph="rmat", scale=23, edge_factor=16,
             weights=True, mode="async", k=8),
    ]


def draw(rng):
    """One more case of the listed ranges: every kind and graph family, sizes
    from the smallest served graph to the benchmark's, odd ones included."""
    def log(lo, hi):
        return int(math.exp(rng.uniform(math.log(lo), math.log(hi))))

    kind = rng.choice(["solve"] * 5 + ["first"] * 2 + ["batch", "serve", "score"])
    case = dict(kind=kind, weights=rng.random() < 0.5, mode="det",
                k=rng.choice([4, 8, 8, 8, 16]))
    if kind == "batch":
        lo = log(1000, 4000)
        case.update(graphs=log(8, 512), n_lo=lo, n_hi=lo * log(8, 50))
    elif kind == "serve":
        case.update(requests=log(4, 24))
    else:
        family = rng.choice(["sbm", "rmat", "rmat", "grid"])
        case.update(graph=family, offsets64=rng.random() < 0.15)
        if family == "sbm":
            n = log(1000, 1_000_000)
            case.update(n=n, blocks=max(1, min(log(8, 4000), n // 16)))
        elif family == "grid":
            case.update(rows=log(40, 4096), cols=log(40, 4096))
        elif kind == "solve" and case["weights"] and rng.random() < 0.4:
            # in place: power-law graphs whose labels hardly depend on scheduling
            case.update(mode="async", scale=rng.choice([22, 23]), edge_factor=rng.randint(9, 20))
        else:
            case.update(scale=rng.randint(14, 22 if kind == "score" else 21),
                        edge_factor=rng.randint(6, 20))
        if kind == "solve" and rng.random() < 0.25:
            case.update(ranked=True)
    return case


# ------------------------------------------------------------------ graphs
def _gen(seed):
    g = torch.Generator(device=DEVICE)
    g.manual_seed(seed)
    return g


def _csr(n, u, v):
    """Symmetric CSR (sorted rows, no self-loops, no duplicates) of edge lists."""
    keep = u != v
    u, v = u[keep], v[keep]
    keys = torch.unique(torch.cat([u * n + v, v * n + u]))
    del u, v, keep
    rp = torch.searchsorted(keys, torch.arange(n + 1, device=DEVICE) * n)
    return rp.to(torch.int32), keys.remainder_(n).to(torch.int32)


def _rmat(scale, edge_factor, gen):
    """R-MAT edges of quadrant probabilities (0.57, 0.19, 0.19, 0.05)."""
    n, m = 1 << scale, edge_factor << scale
    us, vs = [], []
    for e in range(0, m, 1 << 26):
        c = min(1 << 26, m - e)
        u = torch.zeros(c, dtype=torch.int64, device=DEVICE)
        v = torch.zeros(c, dtype=torch.int64, device=DEVICE)
        for _ in range(scale):
            r = torch.rand(c, device=DEVICE, generator=gen)
            right = (r >= 0.76)
            u.mul_(2).add_(right)
            v.mul_(2).add_(((r >= 0.57) & ~right) | (r >= 0.95))
        us.append(u)
        vs.append(v)
    return _csr(n, torch.cat(us), torch.cat(vs))


def _sbm(sizes, blocks, gen):
    """Planted partitions of mean degree 12 inside and 2 between near-equal
    blocks, one after another in one id space."""
    size = torch.tensor(sizes, device=DEVICE)
    nb = torch.tensor(blocks, device=DEVICE)
    first = torch.cumsum(size, 0) - size
    N = int(sum(sizes))

    def pick(count):
        u = torch.randint(N, (count,), device=DEVICE, generator=gen)
        g = torch.searchsorted(first, u, right=True) - 1
        return u, g, torch.rand(count, device=DEVICE, generator=gen, dtype=torch.float64)

    u, g, r = pick(6 * N)
    b = (u - first[g]) * nb[g] // size[g]  # block of u: ids [ceil(b n / B), ceil((b + 1) n / B))
    lo = -((-b * size[g]) // nb[g])
    hi = -((-(b + 1) * size[g]) // nb[g])
    v = first[g] + lo + (r * (hi - lo)).to(torch.int64)
    u2, g2, r2 = pick(N)
    v2 = first[g2] + (r2 * size[g2]).to(torch.int64)
    return _csr(N, torch.cat([u, u2]), torch.cat([v, v2]))


def _grid(rows, cols, gen):
    """Lattice with 5% of the edges deleted and 1% of the rest rewired."""
    n = rows * cols
    i = torch.arange(n, device=DEVICE).view(rows, cols)
    u = torch.cat([i[:, :-1].reshape(-1), i[:-1].reshape(-1)])
    v = torch.cat([i[:, 1:].reshape(-1), i[1:].reshape(-1)])
    r = torch.rand(u.numel(), device=DEVICE, generator=gen, dtype=torch.float64)
    u, v, r = u[r >= 0.05], v[r >= 0.05], r[r >= 0.05]
    far = torch.randint(n, (u.numel(),), device=DEVICE, generator=gen)
    return _csr(n, u, torch.where(r < 0.05 + 0.95 * 0.01, far, v))


def _weights(rp, col, seed):
    """fp32 weights in (0, 1], multiples of 2^-24, the same both ways."""
    n, nnz = rp.numel() - 1, col.numel()
    w = torch.empty(nnz, dtype=torch.float32, device=DEVICE)
    for b in range(0, nnz, 1 << 26):
        e = min(nnz, b + (1 << 26))
        at = torch.arange(b, e, dtype=rp.dtype, device=DEVICE)
        u = torch.searchsorted(rp, at, right=True).sub_(1)
        v = col[b:e].to(torch.int64)
        x = torch.minimum(u, v) * 0x9E3779B1 + torch.maximum(u, v) * 0x85EBCA77 + seed * 0x27D4EB2F
        x = (x ^ (x >> 29)) * 0x1B873593
        x = (x ^ (x >> 32)) * 0x2545F491
        x = ((x ^ (x >> 27)) & 0xFFFFFF) + 1
        w[b:e] = x.to(torch.float32) * 2.0 ** -24
    return w


def _graph(case, seed):
    gen = _gen(seed)
    if case["graph"] == "rmat":
        rp, col = _rmat(case["scale"], case["edge_factor"], gen)
    elif case["graph"] == "sbm":
        rp, col = _sbm([case["n"]], [case["blocks"]], gen)
    else:
        rp, col = _grid(case["rows"], case["cols"], gen)
    return rp, col, _weights(rp, col, seed) if case["weights"] else None


def _options(case):
    return dict(k=case["k"], mode=case["mode"], ranked=case.get("ranked", False))


# -------------------------------------------------------- many graphs at once
def _mix(requests):
    """Sizes of the served mix: 70% planted partitions of 1e3 to 1e5 vertices,
    30% R-MAT graphs of scale 14 to 17 (None in the place of their blocks)."""
    out = []
    for i, s in enumerate(inputs.batch_specs(requests, 3, 1e3, 1e5)):
        r = inputs.uniform(4, i, 0)
        out.append((14 + int(r / 0.3 * 4), None) if r < 0.3 else (s.n, s.blocks))
    return out


def _many(case, seed):
    """(row_ptr, col, w) of every graph of a batch or a served mix."""
    if case["kind"] == "batch":
        sizes = [(s.n, s.blocks) for s in inputs.batch_specs(case["graphs"], 512, case["n_lo"],
                                                             case["n_hi"])]
    else:
        sizes = _mix(case["requests"])
    gen = _gen(seed)
    planted = [s for s in sizes if s[1] is not None]
    rp, col = _sbm([n for n, _ in planted], [b for _, b in planted], gen)
    ids = torch.tensor([0] + [n for n, _ in planted]).cumsum(0)
    ends = rp[ids.to(DEVICE)].tolist()
    graphs, at = [], 0
    for n, blocks in sizes:
        if blocks is None:
            r, c = _rmat(n, 16, gen)
        else:
            lo = int(ids[at])
            r = rp[lo:lo + n + 1] - ends[at]
            c = col[ends[at]:ends[at + 1]] - lo
            at += 1
        graphs.append((r, c, _weights(r, c, seed) if case["weights"] else None))
    return graphs


# ------------------------------------------------------------------- the path
def prepare(case, seed):
    kind = case["kind"]
    if kind == "batch":
        graphs = _many(case, seed)
        return dict(kind=kind, solvers=[lpa.LPA(*g, **_options(case)) for g in graphs],
                    batch=lpa.Batch(len(graphs), k=case["k"], mode=case["mode"]))
    if kind == "serve":
        host = [tuple(None if t is None else t.cpu().numpy() for t in g)
                for g in _many(case, seed)]
        return dict(kind=kind, requests=host,
                    backend=serve.Backend(k=case["k"], mode=case["mode"], capacity=32))
    rp, col, w = _graph(case, seed)
    if case.get("offsets64"):
        rp = rp.to(torch.int64)
    state = dict(kind=kind, mode=case["mode"], graph=(rp, col, w), options=_options(case))
    if kind != "first":
        state["solver"] = lpa.LPA(rp, col, w, **state["options"])
    if kind == "score":
        state["labels"] = _labels(rp.numel() - 1, seed)
    return state


def _labels(n, seed):
    """A labelling as a solve of a power-law graph leaves it: one community
    with half of the vertices, small ones, and vertices on their own."""
    r = torch.rand(n, device=DEVICE, generator=_gen(seed + 1))
    v = torch.arange(n, device=DEVICE)
    return torch.where(r < 0.5, 0, torch.where(r < 0.8, v // 16 * 16, v)).to(torch.int32)


def run(state):
    kind = state["kind"]
    if kind == "batch":
        state["batch"].reset(state["solvers"])
        state["batch"].run(state["solvers"])
        return torch.cat([s.labels() for s in state["solvers"]])
    if kind == "serve":
        server = serve.Server(state["backend"], max_resident=32)
        requests = [server.submit(*g) for g in state["requests"]]
        server.run_until_idle()
        return [r.labels for r in requests]
    if kind == "score":
        return state["solver"].modularity(state["labels"])
    if kind == "first":
        solver = lpa.LPA(*state["graph"], **state["options"])
        out = dict(iterations=solver.run(), labels=solver.labels(), q=solver.modularity())
        solver.close()
        return out
    solver = state["solver"]
    solver.reset()
    iterations = solver.run()
    if state["mode"] == "async":  # in place: the iteration count may vary with scheduling
        return solver.labels()
    return dict(iterations=iterations, labels=solver.labels())


def exact(case, seed):
    """Modularity of the given labelling in 64 bits; labels are whole numbers."""
    if case["kind"] != "score":
        return None
    rp, col, w = _graph(case, seed)
    n, nnz = rp.numel() - 1, col.numel()
    lab = _labels(n, seed).to(torch.int64)
    strength = torch.zeros(n + 1, dtype=torch.float64, device=DEVICE)  # weight of each row
    inside = 0.0
    for b in range(0, nnz, 1 << 26):
        e = min(nnz, b + (1 << 26))
        u = torch.searchsorted(rp, torch.arange(b, e, dtype=rp.dtype, device=DEVICE),
                               right=True).sub_(1)
        x = (torch.ones(e - b, dtype=torch.float64, device=DEVICE) if w is None
             else w[b:e].to(torch.float64))
        inside += float(x[lab[u] == lab[col[b:e].to(torch.int64)]].sum())
        strength[1:] += _ends(x, rp[1:].to(torch.int64).clamp(b, e) - b)
    by_label = torch.argsort(lab)
    last = torch.searchsorted(lab[by_label], torch.arange(n, device=DEVICE), right=True)
    total = _ends(strength.diff()[by_label], last).diff(prepend=strength.new_zeros(1))
    two_m = float(strength[-1])
    return inside / two_m - float(total.square().sum()) / (two_m * two_m)


def _ends(x, at):
    """Sums of the first at[i] values of x."""
    return torch.cat([x.new_zeros(1), torch.cumsum(x, 0)])[at]


# ------------------------------------------------------------------------ work
def _rmat_entries(scale, edge_factor):
    """Expected CSR entries: distinct unordered pairs among the sampled ones,
    over the classes of vertex pairs of one probability."""
    m, total = edge_factor << scale, 0.0
    for i in range(scale + 1):          # levels in the first quadrant
        for j in range(1, scale - i + 1):   # levels in the two mixed quadrants
            d = scale - i - j
            pairs = math.comb(scale, i) * math.comb(scale - i, j) * 2.0 ** j
            p = 2 * 0.57 ** i * 0.19 ** j * 0.05 ** d
            total += pairs * -math.expm1(m * math.log1p(-p))
    return total


def _size(case):
    """(vertices, expected CSR entries) of all of a case's graphs."""
    if case["kind"] == "batch":
        n = sum(s.n for s in inputs.batch_specs(case["graphs"], 512, case["n_lo"], case["n_hi"]))
        return n, 14.0 * n
    if case["kind"] == "serve":
        mix = _mix(case["requests"])
        return (sum(n if b else 1 << n for n, b in mix),
                sum(14.0 * n if b else _rmat_entries(n, 16) for n, b in mix))
    if case["graph"] == "rmat":
        return 1 << case["scale"], _rmat_entries(case["scale"], case["edge_factor"])
    if case["graph"] == "sbm":
        return case["n"], 14.0 * case["n"]
    r, c = case["rows"], case["cols"]
    return r * c, 2 * 0.95 * (2 * r * c - r - c)


def work(case):
    """Row offsets, column indices and weights read once, the labels written
    (read, where they are scored) once; one addition per entry."""
    n, nnz = _size(case)
    entry = 8 if case["weights"] else 4
    offset = 8 if case.get("offsets64") else 4
    return {"bytes": nnz * entry + n * (offset + 4.0), "flops": nnz}
