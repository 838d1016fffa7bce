"""The calls whose speed this framework is judged by, with their inputs, their
minimum work and their values in 64-bit arithmetic.

A case is a dict of plain values; its "kind" names the public call it makes:

refine        tsgne_run on a small graph from an earlier layout (32 steps)
run           tsgne_run from a fresh layout: the first 32 steps under early exaggeration
step          one tsgne_step on caller-owned optimiser state
gradient      one tsgne_gradient (the loop of a caller with its own optimiser)
batch         tsgne_batch_run over many graphs (their first 16 steps)
serve         a burst of requests through a layout server
build_P       affinities of a new graph, exported to the host
knn           the neighbourhood graph G_knn,G
shortest_path the ShortestPath embedding
quality       KL, k-means, NMI and AQ of a finished layout
attraction    the sparse half of the gradient alone

Graphs are stochastic block models (communities of a size, 18 % of the edges
between them) or degree-corrected ones (power-law propensities), drawn on the
GPU from the seed, with node ids at random.  Layouts in progress are one
Gaussian blob per community with the density of a converged layout.

Runs stop at a few dozen steps and take a small learning rate: later layouts,
and early ones at the default rate, are chaotic functions of rounding, so that
nothing could be compared.  A step costs the same at any rate.
"""
from __future__ import annotations

import math

import torch

from paper_2310_11186_amd import tsgne

DEVICE = "cuda:0"
MIXING = 0.18          # share of the edges that leave their community
PERPLEXITY = 30.0
REFINE_STEPS = 32
RUN_STEPS = 32
BATCH_STEPS = 16


def listed():
    return [
        # the smallest graphs: a re-layout of 2,000 nodes, a few kernels of microseconds per step
        {"name": "refine_2000", "kind": "refine", "n": 2000, "degree": 10.5, "communities": 4},
        # a small graph of an odd size from scratch
        {"name": "run_9001", "kind": "run", "n": 9001, "degree": 6.0, "communities": 20},
        # a middling graph with hubs, the caller holding the optimiser state
        {"name": "step_31013", "kind": "step", "n": 31013, "degree": 8.0, "communities": 31, "gamma": 2.5},
        # the 100K-node configuration, under early exaggeration
        {"name": "gradient_100000", "kind": "gradient", "n": 100000, "degree": 8.0, "communities": 50, "gamma": 2.5,
         "alpha": 12.0},
        # the largest: the 300K-node, 1M-edge configuration, after early exaggeration
        {"name": "gradient_300000", "kind": "gradient", "n": 300000, "degree": 20 / 3, "communities": 200,
         "gamma": 2.3, "alpha": 1.0},
        # many independent graphs advanced together
        {"name": "batch_48", "kind": "batch", "count": 48, "n_min": 1000, "n_max": 20000, "degree": 5.5},
        # a burst of requests from host arrays to host layouts
        {"name": "serve_12", "kind": "serve", "count": 12, "n_min": 1000, "n_max": 30000, "degree": 5.0, "d": 64},
        # the start of every layout: affinities of a hub-heavy graph with a wide embedding
        {"name": "build_P_100003", "kind": "build_P", "n": 100003, "degree": 8.0, "communities": 50, "gamma": 2.5,
         "d": 128},
        # the literal neighbourhood of the method, k of 3 times the perplexity
        {"name": "knn_100000", "kind": "knn", "n": 100000, "degree": 8.0, "communities": 50, "gamma": 2.5, "k": 90},
        # the embedding for graphs that come without one
        {"name": "shortest_path_300000", "kind": "shortest_path", "n": 300000, "degree": 20 / 3, "communities": 200,
         "gamma": 2.3, "d": 128},
        # what is reported of a finished layout
        {"name": "quality_100003", "kind": "quality", "n": 100003, "degree": 8.0, "communities": 50, "gamma": 2.5},
        # gathers over a layout larger than a cache, ids at random
        {"name": "attraction_1000000", "kind": "attraction", "n": 1000000, "degree": 10.0, "communities": 100},
    ]


def draw(rng):
    """One more case of the listed ranges (sizes over their logarithm)."""
    def size(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    kind = rng.choice(["refine", "run", "step", "gradient", "gradient", "batch", "serve", "build_P", "knn",
                       "shortest_path", "quality", "attraction"])
    degree = round(rng.uniform(4.0, 9.0), 2)
    if kind == "batch":
        return {"kind": kind, "count": size(6, 48), "n_min": 1000, "n_max": size(2000, 20000), "degree": degree}
    if kind == "serve":
        return {"kind": kind, "count": size(3, 12), "n_min": 1000, "n_max": size(3000, 30000), "degree": degree,
                "d": rng.choice([64, 128])}
    n = size(*{"refine": (1500, 6000), "run": (2000, 20000), "step": (8000, 60000), "gradient": (3000, 290000),
               "build_P": (2000, 200000), "knn": (2000, 100000), "shortest_path": (2000, 300000),
               "quality": (2000, 100000), "attraction": (20000, 1000000)}[kind])
    case = {"kind": kind, "n": n, "degree": degree, "communities": max(4, n // 1000)}
    if kind not in ("refine", "run", "attraction"):
        case["gamma"] = round(rng.uniform(2.3, 2.8), 2)
    if kind == "gradient":
        case["alpha"] = rng.choice([1.0, 12.0])
    if kind == "build_P":
        case["d"] = rng.choice([8, 16, 64, 100, 128])
    if kind == "knn":
        case["k"] = rng.randint(10, 90)
    if kind == "shortest_path":
        case["d"] = rng.randint(16, 128)
    return case


# ---------------------------------------------------------------------------
# Inputs, from the seed alone
# ---------------------------------------------------------------------------

def _generator(seed):
    return torch.Generator(device=DEVICE).manual_seed(int(seed))


def _rand(g, *shape):
    return torch.rand(*shape, generator=g, device=DEVICE, dtype=torch.float64)


def _pick(cum, lo, hi, u):
    """Positions drawn in proportion to weights given by their running sum, inside (lo, hi] of it."""
    return torch.searchsorted(cum, lo + u * (hi - lo), right=True).clamp_(max=cum.numel() - 1)


def _graph(n, degree, communities, seed, gamma=None):
    """(communities of the nodes, row_ptr, col): canonical symmetric CSR (int32, device)."""
    g = _generator(seed)
    label = torch.randint(communities, (n,), generator=g, device=DEVICE).sort().values  # by rank; ids are shuffled below
    theta = torch.ones(n, dtype=torch.float64, device=DEVICE)
    if gamma:
        theta = torch.floor(2.0 * _rand(g, n) ** (-1.0 / (gamma - 1.0))).clamp_(max=math.floor(n ** (1.0 / (gamma - 1.0))))
    cum = torch.cumsum(theta, 0)
    end = torch.searchsorted(label, torch.arange(communities, device=DEVICE), right=True)
    hi = torch.where(end > 0, cum[(end - 1).clamp(min=0)], torch.zeros_like(cum[0]))
    lo = torch.cat([torch.zeros_like(hi[:1]), hi[:-1]])
    m = int(round(n * degree / 2))
    ids = torch.randperm(n, generator=g, device=DEVICE)
    pairs = torch.empty(0, dtype=torch.int64, device=DEVICE)
    while pairs.numel() < m:   # distinct unordered pairs, exactly m of them in the end
        k = 3 * m // 2 + 64
        u = _pick(cum, 0.0, cum[-1], _rand(g, k))
        inside = _rand(g, k) >= MIXING
        c, r = label[u], _rand(g, k)
        v = torch.where(inside, _pick(cum, lo[c], hi[c], r), _pick(cum, 0.0, cum[-1], r))
        u, v = ids[u], ids[v]
        key = torch.minimum(u, v) * n + torch.maximum(u, v)
        pairs = torch.unique(torch.cat([pairs, key[u != v]]))
    pairs = pairs[torch.randperm(pairs.numel(), generator=g, device=DEVICE)[:m]]
    u, v = pairs // n, pairs % n
    key = torch.cat([u * n + v, v * n + u]).sort().values
    row, col = key // n, (key % n).to(torch.int32)
    row_ptr = torch.searchsorted(row, torch.arange(n + 1, device=DEVICE)).to(torch.int32)
    community = torch.empty_like(label)
    community[ids] = label
    return community, row_ptr, col


def _embedding(community, communities, d, seed):
    g = _generator(seed + 1)
    centre = 2.0 * torch.randn(communities, d, generator=g, device=DEVICE)
    return (centre[community] + 0.5 * torch.randn(community.numel(), d, generator=g, device=DEVICE)).contiguous()


def _fresh_layout(n, seed):
    return 0.01 * torch.randn(n, 2, generator=_generator(seed + 2), device=DEVICE)


def _grown_layout(community, communities, seed):
    """One blob per community, on a spiral with room for each."""
    n = community.numel()
    k = torch.arange(communities, device=DEVICE, dtype=torch.float32)
    radius, angle = 0.36 * math.sqrt(n / communities) * torch.sqrt(k + 0.5), 2.399963 * k
    centre = torch.stack([radius * torch.cos(angle), radius * torch.sin(angle)], 1)
    noise = torch.randn(n, 2, generator=_generator(seed + 2), device=DEVICE)
    return (centre[community] + 0.25 * math.sqrt(n / communities) * noise).contiguous()


def _rows(row_ptr):
    deg = (row_ptr[1:] - row_ptr[:-1]).long()
    return torch.repeat_interleave(torch.arange(deg.numel(), device=row_ptr.device), deg), deg


def _uniform_P(row_ptr, col):
    """Joint affinities whose rows are uniform (what rows of at most `perplexity` neighbours get), float32."""
    row, deg = _rows(row_ptr)
    w = 1.0 / deg.clamp(min=1).double()
    return ((w[row] + w[col.long()]) / (2.0 * int((deg > 0).sum()))).float()


def _parts(case):
    return case["n"], case["degree"], case["communities"]


def _many(case, seed):
    """(nodes, average degree, communities, seed) of each graph of a batch or a burst."""
    lo, hi, last = math.log(case["n_min"]), math.log(case["n_max"]), max(1, case["count"] - 1)
    return [(int(round(math.exp(lo + (hi - lo) * k / last))), case["degree"] * (0.7 + 0.6 * (0.618 * k % 1)),
             4 + int(36 * (0.414 * k % 1)), seed * 1000 + k) for k in range(case["count"])]


def _inputs(case, seed):
    """Everything but the library's own handles."""
    kind = case["kind"]
    if kind == "batch":
        out = []
        for n, degree, communities, s in _many(case, seed):
            _, row_ptr, col = _graph(n, degree, communities, s)
            out.append({"row_ptr": row_ptr, "col": col, "P": _uniform_P(row_ptr, col), "Y0": _fresh_layout(n, s)})
        return out
    if kind == "serve":
        out = []
        for n, degree, communities, s in _many(case, seed):
            community, row_ptr, col = _graph(n, degree, communities, s)
            row, _ = _rows(row_ptr)
            edges = torch.stack([row, col.long()], 1)[row < col].to(torch.int32)
            out.append({"row_ptr": row_ptr, "col": col, "edges": edges.cpu().numpy(),
                        "X": _embedding(community, communities, case["d"], s).cpu().numpy(),
                        "Y0": _fresh_layout(n, s).cpu().numpy()})
        return out
    n, degree, communities = _parts(case)
    community, row_ptr, col = _graph(n, degree, communities, seed, case.get("gamma"))
    s = {"row_ptr": row_ptr, "col": col}
    if kind == "build_P":
        s["X"] = _embedding(community, communities, case["d"], seed)
    elif kind == "shortest_path":
        s["targets"] = torch.randperm(n, generator=_generator(seed + 3), device=DEVICE)[:case["d"]].to(torch.int32)
    elif kind != "knn":
        s["P"] = _uniform_P(row_ptr, col)
        s["Y"] = _fresh_layout(n, seed) if kind == "run" else _grown_layout(community, communities, seed)
    if kind == "step":
        g = _generator(seed + 3)
        s["U"] = 0.1 * torch.randn(n, 2, generator=g, device=DEVICE)
        s["G"] = 0.5 + torch.rand(n, 2, generator=g, device=DEVICE)
    if kind == "knn":       # one buffer for the lists, as long as they can get
        s["lists"] = torch.zeros(2 * n * case["k"], dtype=torch.int32, device=DEVICE)
    if kind == "quality":
        s["labels"] = community.to(torch.int32)
        s["seeds"] = torch.randperm(n, generator=_generator(seed + 3), device=DEVICE)[:communities].to(torch.int32)
    return s


def _handle(s):
    return tsgne.tsgne_graph_from_host_P(s["row_ptr"].cpu().numpy(), s["col"].cpu().numpy(), s["P"].cpu().numpy())


def _params(kind):
    if kind == "refine":   # an earlier layout is kept: no exaggeration, a small learning rate
        return tsgne.tsgne_params_default(exaggeration_iters=0, learning_rate=2.0)
    if kind in ("run", "batch", "serve"):
        return tsgne.tsgne_params_default(learning_rate=5.0)
    return tsgne.tsgne_params_default()


def prepare(case, seed):
    kind = case["kind"]
    s = {"kind": kind, "case": case, "params": _params(kind)}
    if kind == "batch":
        s["graphs"] = _inputs(case, seed)
        s["handles"] = [_handle(g) for g in s["graphs"]]
    elif kind == "serve":
        s["requests"] = [{k: r[k] for k in ("edges", "X", "Y0")} for r in _inputs(case, seed)]
        s["server"] = tsgne.Server(params=s["params"])
    else:
        s.update(_inputs(case, seed))
        if "P" in s:
            s["handle"] = _handle(s)
    return s


# ---------------------------------------------------------------------------
# One pass
# ---------------------------------------------------------------------------

def run(s):
    kind, case, p = s["kind"], s["case"], s["params"]
    if kind in ("refine", "run"):
        Y = s["Y"].clone()
        tsgne.tsgne_run(s["handle"], Y, REFINE_STEPS if kind == "refine" else RUN_STEPS, p)
        return Y
    if kind == "step":
        grad, Z = torch.empty_like(s["Y"]), torch.empty(1, dtype=torch.float64, device=DEVICE)
        tsgne.tsgne_step(s["handle"], s["Y"], s["U"], s["G"], 300, p, grad, Z)
        return {"Y": s["Y"], "U": s["U"], "G": s["G"], "grad": grad, "Z": Z}
    if kind == "gradient":
        grad, Z = tsgne.tsgne_gradient(s["handle"], s["Y"], case["alpha"], p)
        return {"grad": grad, "Z": Z}
    if kind == "batch":
        Ys = [g["Y0"].clone() for g in s["graphs"]]
        tsgne.tsgne_batch_run(s["handles"], Ys, [BATCH_STEPS] * len(Ys), p)
        return Ys
    if kind == "serve":
        srv = s["server"]
        tickets = [srv.submit(r["Y0"].shape[0], r["edges"], r["X"], r["Y0"], PERPLEXITY, RUN_STEPS)
                   for r in s["requests"]]
        done = [srv.wait(t) for t in tickets]
        for t in tickets:
            srv.release(t)
        return {"status": [st for st, _ in done], "Y": [Y for _, Y in done]}
    if kind == "build_P":
        g = tsgne.tsgne_build_P(s["row_ptr"], s["col"], s["X"], PERPLEXITY)
        out = g.export()
        g.close()
        return out
    if kind == "knn":
        row_ptr, col = tsgne.tsgne_knn_graph(s["row_ptr"], s["col"], case["k"])
        s["lists"][:col.numel()] = col
        return {"row_ptr": row_ptr, "col": s["lists"]}
    if kind == "shortest_path":
        return tsgne.tsgne_shortest_path_embedding(s["row_ptr"], s["col"], s["targets"])[0]
    if kind == "quality":
        k = case["communities"]
        kl = tsgne.tsgne_kl(s["handle"], s["Y"])
        clusters, passes = tsgne.tsgne_kmeans(s["Y"], s["seeds"])
        nmi = tsgne.tsgne_nmi(s["labels"], k, clusters, k)
        return {"kl": kl, "clusters": clusters, "passes": passes, "nmi": nmi,
                "aq": tsgne.tsgne_aq(s["Y"], s["labels"], k, 20, 0.5)}
    if kind == "attraction":
        return tsgne.tsgne_attraction(s["handle"], s["Y"])
    raise KeyError(kind)


# ---------------------------------------------------------------------------
# The least a pass can do
# ---------------------------------------------------------------------------

def _pairs(n):
    """Flops of all pairs, each unordered pair once: 2 subtractions, 2 FMAs for 1 + d^2, a reciprocal, an
    addition into Z, a product for w^2 and 4 FMAs into the two forces."""
    return 17.0 * n * (n - 1) / 2


def work(case):
    kind = case["kind"]
    if kind in ("batch", "serve"):
        sizes = [(n, n * degree) for n, degree, _, _ in _many(case, 0)]
        steps = BATCH_STEPS if kind == "batch" else RUN_STEPS
        nbytes = sum(16.0 * n + 8.0 * nnz for n, nnz in sizes)
        if kind == "serve":
            nbytes += sum(4.0 * n * case["d"] for n, _ in sizes)
        return {"bytes": nbytes, "flops": steps * sum(_pairs(n) + 12.0 * nnz for n, nnz in sizes)}
    n, degree, _ = _parts(case)
    nnz = n * degree
    csr = 4.0 * n + 4.0 * nnz
    if kind in ("refine", "run"):
        steps = REFINE_STEPS if kind == "refine" else RUN_STEPS
        return {"bytes": csr + 4.0 * nnz + 16.0 * n, "flops": steps * (_pairs(n) + 12.0 * nnz)}
    if kind in ("step", "gradient"):
        return {"bytes": csr + 4.0 * nnz + (56.0 if kind == "step" else 16.0) * n, "flops": _pairs(n) + 12.0 * nnz}
    if kind == "attraction":
        return {"bytes": csr + 4.0 * nnz + 24.0 * n, "flops": 12.0 * nnz}
    if kind == "build_P":   # in: CSR and X; out, on the host: row_ptr, col, mirror, P, beta
        return {"bytes": csr + 4.0 * n * case["d"] + 12.0 * n + 12.0 * nnz, "flops": 3.0 * nnz * case["d"] + 20.0 * nnz}
    if kind == "knn":       # the lists of a row hold k entries, most of them in one direction only
        return {"bytes": csr + 4.0 * n + 4.0 * 1.5 * n * case["k"], "flops": 0.0}
    if kind == "shortest_path":
        return {"bytes": csr + 4.0 * n * case["d"], "flops": 0.0}
    # quality: Z needs the weights only (7 flops a pair), k-means at least two passes over the centres
    return {"bytes": csr + 4.0 * nnz + 16.0 * n, "flops": 3.5 * n * (n - 1) + 2.0 * 5.0 * n * case["communities"]}


# ---------------------------------------------------------------------------
# The same values in 64 bits
# ---------------------------------------------------------------------------

def _repulsion64(Y, forces=True):
    """(sum_j w_ij^2 (y_i - y_j), Z) over all pairs."""
    n = Y.shape[0]
    x, y = Y[:, 0].contiguous(), Y[:, 1].contiguous()
    R, Z = torch.zeros_like(Y), torch.zeros((), dtype=Y.dtype, device=Y.device)
    step = max(1, min(n, 100_000_000 // n))
    for a in range(0, n, step):
        dx, dy = x[a:a + step, None] - x, y[a:a + step, None] - y
        w = (dx * dx).addcmul_(dy, dy).add_(1.0).reciprocal_()
        Z += w.sum() - w.shape[0]   # i = j: weight 1, no force
        if forces:
            w.square_()
            R[a:a + step, 0] = dx.mul_(w).sum(1)
            R[a:a + step, 1] = dy.mul_(w).sum(1)
    return R, Z


def _attraction64(row, col, P, Y):
    d = Y[row] - Y[col]
    return torch.zeros_like(Y).index_add_(0, row, (P / (1.0 + (d * d).sum(1)))[:, None] * d)


def _gradient64(row, col, P, Y, alpha):
    R, Z = _repulsion64(Y)
    return 4.0 * (alpha * _attraction64(row, col, P, Y) - R / Z), Z


def _update64(Y, U, G, grad, momentum, eta, min_gain):
    G = torch.where(grad * U < 0, G + 0.2, G * 0.8).clamp_(min=min_gain)
    U = momentum * U - eta * G * grad
    return Y + U, U, G


def _run64(row, col, P, Y, steps, p):
    U, G = torch.zeros_like(Y), torch.ones_like(Y)
    eta = p.learning_rate if p.learning_rate > 0 else max(Y.shape[0] / (4.0 * p.early_exaggeration), 50.0)
    for t in range(steps):
        early = t < p.exaggeration_iters
        grad, _ = _gradient64(row, col, P, Y, p.early_exaggeration if early else 1.0)
        Y, U, G = _update64(Y, U, G, grad, p.momentum_early if early else p.momentum_late, eta, p.min_gain)
    return Y


def _build64(row_ptr, col, X):
    """(P, beta) over the graph's neighbours: each row's bandwidth by bisection to the perplexity."""
    row, deg = _rows(row_ptr)
    n, col = deg.numel(), col.long()
    X = X.double()
    D = torch.cat([(X[r] - X[c]).square_().sum(1) for r, c in zip(row.split(1 << 20), col.split(1 << 20))])

    def total(v):
        return torch.zeros(n, dtype=torch.float64, device=D.device).index_add_(0, row, v)

    near = torch.full((n,), math.inf, dtype=torch.float64, device=D.device).scatter_reduce_(0, row, D, "amin")
    D = D - near[row]
    wide = deg > PERPLEXITY
    beta = torch.where(wide, deg / total(D).clamp(min=1e-300), torch.zeros_like(near))

    def entropy(b):
        e = torch.exp(-b[row] * D)
        S = total(e)
        return torch.log(S) + b * total(D * e) / S

    target = math.log(PERPLEXITY)
    lo, hi = beta.clone(), beta.clone()
    while bool((up := wide & (entropy(hi) > target)).any()):
        hi = torch.where(up, 2 * hi, hi)
    while bool((down := wide & (entropy(lo) <= target)).any()):
        lo = torch.where(down, lo / 2, lo)
    for _ in range(100):
        mid = 0.5 * (lo + hi)
        high = entropy(mid) > target
        lo, hi = torch.where(high, mid, lo), torch.where(high, hi, mid)
    beta = torch.where(wide, 0.5 * (lo + hi), torch.zeros_like(lo))
    e = torch.exp(-beta[row] * D)
    p = e / total(e)[row]
    key = row * n + col
    mirror = torch.searchsorted(key, col * n + row)
    return (p + p[mirror]) / (2.0 * int((deg > 0).sum())), beta


def _quality64(s, communities):
    n, Y, labels = s["Y"].shape[0], s["Y"].double(), s["labels"].long()
    row, _ = _rows(s["row_ptr"])
    P, d = s["P"].double(), Y[row] - Y[s["col"].long()]
    _, Z = _repulsion64(Y, forces=False)
    kl = float((P * (torch.log(P) + torch.log(Z) + torch.log1p((d * d).sum(1)))).sum())
    lo, hi = Y.min(0).values, Y.max(0).values
    q = torch.floor((Y - lo) / (hi - lo) * 2.0 ** 24).clamp_(max=2.0 ** 24 - 1)
    centre, clusters = q[s["seeds"].long()], torch.full((n,), -1, device=Y.device)
    for _ in range(300):
        dist = (q[:, None, 0] - centre[:, 0]).square_() + (q[:, None, 1] - centre[:, 1]).square_()
        new = dist.argmin(1)
        if torch.equal(new, clusters):
            break
        clusters = new
        size = torch.bincount(clusters, minlength=communities)
        mean = torch.zeros_like(centre).index_add_(0, clusters, q) / size.clamp(min=1)[:, None]
        centre = torch.where((size > 0)[:, None], mean, centre)
    joint = torch.bincount(labels * communities + clusters, minlength=communities ** 2).double().view(communities, -1) / n
    a, b = joint.sum(1), joint.sum(0)
    h = [float(-(v[v > 0] * torch.log(v[v > 0])).sum()) for v in (a, b)]
    some = joint > 0
    mutual = float((joint[some] * torch.log(joint[some] / (a[:, None] * b)[some])).sum())
    cell = torch.floor((Y - lo) / ((hi - lo) / 20)).clamp_(max=19).long()
    count = torch.bincount((cell[:, 0] * 20 + cell[:, 1]) * communities + labels, minlength=400 * communities).view(400, -1)
    good = (count.max(1).values.double() > 0.5 * count.sum(1)) & (count.sum(1) > 0)
    return {"kl": kl, "clusters": None, "passes": None, "nmi": 2.0 * mutual / (h[0] + h[1]),
            "aq": float(good.sum()) / 400.0}


def exact(case, seed):
    kind, p = case["kind"], _params(case["kind"])
    s = _inputs(case, seed)
    if kind == "batch":
        return [_run64(_rows(g["row_ptr"])[0], g["col"].long(), g["P"].double(), g["Y0"].double(), BATCH_STEPS, p)
                for g in s]
    if kind == "serve":
        Ys = []
        for r in s:
            X, Y0 = (torch.from_numpy(r[k]).to(DEVICE) for k in ("X", "Y0"))
            P, _ = _build64(r["row_ptr"], r["col"], X)
            Ys.append(_run64(_rows(r["row_ptr"])[0], r["col"].long(), P, Y0.double(), RUN_STEPS, p))
        return {"status": [None] * len(Ys), "Y": Ys}
    if kind == "knn":       # whole numbers only
        return None
    if kind == "build_P":
        P, beta = _build64(s["row_ptr"], s["col"], s["X"])
        return {"row_ptr": None, "col": None, "mirror": None, "P": P, "beta": beta}
    row, _ = _rows(s["row_ptr"])
    col = s["col"].long()
    if kind == "shortest_path":
        n, d = case["n"], case["d"]
        limit = int(math.sqrt(col.numel() / 2))
        X = torch.full((n, d), math.sqrt(col.numel() / 2) + 1, dtype=torch.float64, device=DEVICE)
        front = torch.zeros(n, d, dtype=torch.uint8, device=DEVICE)
        front[s["targets"].long(), torch.arange(d, device=DEVICE)] = 1
        X[front.bool()] = 0.0
        seen, level = front.clone(), 0
        while level < limit and bool(front.any()):
            level += 1
            reach = torch.zeros(n, d, device=DEVICE)
            for r, c in zip(row.split(1 << 18), col.split(1 << 18)):
                reach.index_add_(0, r, front[c].float())
            front = (reach > 0).to(torch.uint8) & (1 - seen)
            seen |= front
            X[front.bool()] = level
        return X
    if kind == "quality":
        return _quality64(s, case["communities"])
    P, Y = s["P"].double(), s["Y"].double()
    if kind in ("refine", "run"):
        return _run64(row, col, P, Y, REFINE_STEPS if kind == "refine" else RUN_STEPS, p)
    if kind == "attraction":
        return _attraction64(row, col, P, Y)
    if kind == "gradient":
        grad, Z = _gradient64(row, col, P, Y, case["alpha"])
        return {"grad": grad, "Z": Z.view(1)}
    grad, Z = _gradient64(row, col, P, Y, 1.0)   # step 300 of the default schedule: past early exaggeration
    Y, U, G = _update64(Y, s["U"].double(), s["G"].double(), grad, p.momentum_late, max(case["n"] / 48.0, 50.0), p.min_gain)
    return {"Y": Y, "U": U, "G": G, "grad": grad, "Z": Z.view(1)}
