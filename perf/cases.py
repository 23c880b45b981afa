"""The work that users of this package have it do, as cases that can be timed
and checked: whole clusterings and their steps (affinity, power iteration,
kNN graph, 1-D k-means) over every storage of W, from the smallest call,
where launches count, to the largest workloads of the repository.

listed() gives the cases, draw(rng) one more of the same ranges, prepare()
what a program holds before the call, run() one pass through the public
entry points, work() what a pass cannot do without, tolerance() how far
another correct implementation may be off, and exact() the outputs in 64
bits by plain torch.
"""
from __future__ import annotations

import math

import torch

import paper_1604_02700_amd as g

DEV = "cuda"


# ------------------------------------------------------------------ cases
def listed():
    return [
        # the smallest clustering: 1,000 points in the plane, to convergence
        # (three Gaussian blobs, sigma 1); latency and launches
        {"name": "job_dense_2d_1k", "kind": "dense_job", "data": "blobs", "n": 1000, "d": 2,
         "k": 3, "sigma": 1.0, "mode": "converge", "cap": 1000, "two_call": False},
        # an ordinary one: 10,000 points on three rings, about 60 updates
        {"name": "job_dense_rings_10k", "kind": "dense_job", "data": "rings", "n": 10000, "d": 2,
         "k": 3, "sigma": 0.3, "mode": "converge", "cap": 1000, "two_call": False},
        # the dense W of the headline workload (50,000 points in 16
        # dimensions, 10 GB of W), into a buffer that the program keeps
        {"name": "weights_16d_50k", "kind": "weights", "data": "blobs", "n": 50000, "d": 16,
         "k": 10, "sigma": 21.0, "form": "normalized"},
        # its power iteration, T = 50
        {"name": "iterate_dense_50k", "kind": "dense_iter", "data": "blobs", "n": 50000, "d": 16,
         "k": 10, "sigma": 21.0, "mode": "fixed", "cap": 50, "noalloc": False},
        # the largest experiment of the paper: two moons, cosine similarity,
        # at most three updates
        {"name": "job_cosine_moons_45k", "kind": "cosine_job", "data": "moons", "n": 45000,
         "d": 2, "k": 2, "mode": "converge", "cap": 3},
        # symmetric storage at an odd size, to convergence
        {"name": "job_sym_16d_20k", "kind": "sym_job", "data": "blobs", "n": 20011, "d": 16,
         "k": 10, "sigma": 21.0, "mode": "converge", "cap": 100},
        # W never stored, 200,000 points in 64 dimensions: ten of its updates
        {"name": "iterate_fused_64d_200k", "kind": "fused_iter", "data": "blobs", "n": 200000,
         "d": 64, "k": 20, "sigma": 4.0, "mode": "fixed", "cap": 10},
        # W never stored at few dimensions, odd sizes, a whole clustering
        {"name": "job_fused_5d_40k", "kind": "fused_job", "data": "blobs", "n": 40013, "d": 5,
         "k": 6, "sigma": 2.0, "mode": "fixed", "cap": 30},
        # the sparse workload: the 32-NN graph of 2,000,000 points in 8
        # dimensions, nodes in the builder's order ...
        {"name": "knn_8d_2m", "kind": "knn", "data": "blobs", "n": 2000000, "d": 8, "k": 50,
         "sigma": 1.0, "knn": 32, "local": True},
        # ... the power iteration over it, to convergence ...
        {"name": "iterate_csr_8d_2m", "kind": "csr_iter", "data": "blobs", "n": 2000000, "d": 8,
         "k": 50, "sigma": 1.0, "knn": 32, "local": True, "mode": "converge", "cap": 100},
        # ... and the k-means of the embedding that it ends with
        {"name": "kmeans_2m_50", "kind": "kmeans", "data": "blobs", "n": 2000000, "d": 8,
         "k": 50, "sigma": 1.0, "knn": 32},
        # a graph whose node order has no locality (the order the points came
        # in), a whole clustering over it
        {"name": "job_csr_6d_300k", "kind": "csr_job", "data": "blobs", "n": 300007, "d": 6,
         "k": 12, "sigma": 1.0, "knn": 20, "local": False, "mode": "converge", "cap": 100},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["dense_job", "dense_job", "weights", "dense_iter", "cosine_job",
                       "sym_job", "fused_iter", "fused_job", "knn", "csr_iter", "csr_job",
                       "kmeans"])
    c = {"kind": kind, "data": "blobs", "k": rng.randint(2, 24)}
    if kind in ("dense_job", "sym_job"):
        c.update(n=_log(rng, 500, 30000), d=rng.choice([2, 3, 6, 8, 16, 20, 33, 64, 100]),
                 mode=rng.choice(["converge", "fixed"]), cap=rng.randint(5, 60))
        c["sigma"] = _sigma_for(c["d"])
        if kind == "dense_job":
            c["two_call"] = rng.random() < 0.3
            if rng.random() < 0.3:
                c.update(data="rings", d=2, k=3, sigma=0.3)
    elif kind in ("weights", "dense_iter"):
        c.update(n=_log(rng, 1000, 48000), d=rng.choice([2, 3, 8, 16, 30, 64, 128]))
        c["sigma"] = _sigma_for(c["d"])
        if kind == "weights":
            c["form"] = rng.choice(["normalized", "affinity", "cosine"])
        else:
            c.update(mode="fixed", cap=rng.randint(5, 50), noalloc=rng.random() < 0.3)
    elif kind == "cosine_job":
        c.update(data=rng.choice(["moons", "circles"]), n=_log(rng, 2000, 44000), d=2,
                 mode="converge", cap=3)
        c["k"] = 2 if c["data"] == "moons" else 3
    elif kind in ("fused_iter", "fused_job"):
        c.update(n=_log(rng, 2000, 60000), d=rng.choice([2, 3, 5, 8, 12, 16, 25, 64, 96, 128]),
                 mode="fixed", cap=rng.randint(3, 12))
        c["sigma"] = _sigma_for(c["d"])
    else:
        c.update(n=_log(rng, 3000, 600000), d=rng.choice([2, 3, 5, 8, 8, 10, 16]),
                 knn=rng.choice([5, 10, 15, 32, 50]), sigma=1.0)
        if kind != "kmeans":
            c["local"] = rng.random() < 0.5
        if kind in ("csr_iter", "csr_job"):
            c.update(mode=rng.choice(["converge", "fixed"]), cap=rng.randint(10, 60))
    return c


def _sigma_for(d):
    """A width at which clusters are seen: about a cluster's own diameter."""
    return {2: 1.0, 3: 1.5}.get(d, round(2.0 * math.sqrt(d / 4.0), 3))


# ----------------------------------------------------------------- inputs
def _points(case, seed):
    """float32 points on the GPU, shuffled: the shapes of the repository's
    own workloads, from the seed alone."""
    n, d, data = case["n"], case["d"], case["data"]
    gen = torch.Generator(device=DEV).manual_seed(int(seed))
    f64 = dict(dtype=torch.float64, device=DEV, generator=gen)
    if data == "blobs":
        k = case["k"]
        if d <= 3:
            centres = torch.rand((k, d), **f64) * 20.0 - 10.0
        else:
            centres = (5.0 if d <= 16 and case["kind"] not in ("knn", "csr_iter", "csr_job",
                                                               "kmeans") else 4.0) * \
                torch.randn((k, d), **f64)
        which = torch.randint(k, (n,), device=DEV, generator=gen)
        X = centres[which] + torch.randn((n, d), **f64)
    elif data == "moons":
        t = torch.rand((n,), **f64) * math.pi
        lower = torch.arange(n, device=DEV) % 2 == 1
        X = torch.stack([torch.where(lower, 1.0 - torch.cos(t), torch.cos(t)),
                         torch.where(lower, 0.5 - torch.sin(t), torch.sin(t))], dim=1)
        X = X + 0.05 * torch.randn((n, 2), **f64)
        X = X[torch.randperm(n, device=DEV, generator=gen)]
    else:                                            # rings, circles
        radii, noise = ((1.0, 3.0, 5.0), 0.1) if data == "rings" else ((1.0, 2.0, 3.0), 0.05)
        r = torch.tensor(radii, dtype=torch.float64, device=DEV)
        r = r[torch.randint(3, (n,), device=DEV, generator=gen)] + noise * torch.randn((n,), **f64)
        t = torch.rand((n,), **f64) * (2.0 * math.pi)
        X = torch.stack([r * torch.cos(t), r * torch.sin(t)], dim=1)
    return X.float().contiguous()


def _graph(case, seed):
    """(X, row_ptr, col, val): the kNN graph of the points, from the builder."""
    X = _points(case, seed)
    if case.get("local", True):
        rp, col, val, _ = g.gpic_knn_graph_local(X, case["knn"], case["sigma"])
    else:
        rp, col, val = g.gpic_knn_graph(X, case["knn"], case["sigma"])
    return X, rp, col.clone(), val.clone()


def _eps(case):
    return 1e-5 / case["n"]


def prepare(case, seed):
    kind, n = case["kind"], case["n"]
    s = {"case": case}
    if kind in ("csr_iter", "csr_job", "kmeans"):
        _, s["rp"], s["col"], s["val"] = _graph(case, seed)
        if kind != "csr_job":
            s["val"], _, s["v0"], _ = g.gpic_degree_normalize_csr(s["rp"], s["col"], s["val"])
        if kind == "kmeans":
            v = s["v0"].clone()
            g.gpic_power_iterate_csr(s["rp"], s["col"], s["val"], v, None, "converge", 60,
                                     _eps(case))
            s = {"case": case, "v": v}
        return s
    s["X"] = _points(case, seed)
    ld = g.padded_ld(n)
    if kind in ("weights", "dense_job", "cosine_job"):
        s["W"] = torch.empty((n, ld), dtype=torch.float32, device=DEV)
    elif kind == "dense_iter":
        s["W"], _, s["v0"], _ = g.gpic_affinity_normalized(s["X"], case["sigma"])
    elif kind == "sym_job":
        s["As"] = torch.empty(g.sym_bytes(n) // 4, dtype=torch.float32, device=DEV)
    elif kind == "fused_iter":
        s["degree"], s["v0"], _ = g.gpic_degree_fused(s["X"], case["sigma"])
    return s


# ------------------------------------------------------------------- pass
def _job(o):
    return {"degree": o.degree, "v0": o.v0, "v": o.pi.v, "labels": o.km.labels,
            "centroids": o.km.centroids}


def _full(t, case):
    """A graph's array at its largest length, so that it has one shape
    whatever the number of edges."""
    return torch.nn.functional.pad(t, (0, 2 * case["n"] * case["knn"] - t.numel()))


def run(s):
    c = s["case"]
    kind, n = c["kind"], c["n"]
    if kind == "dense_job":
        return _job(g.pic_dense(s["X"], c["sigma"], c["k"], c["mode"], c["cap"], _eps(c),
                                A=s["W"], fused_normalize=not c["two_call"]))
    if kind == "cosine_job":
        return _job(g.pic_cosine(s["X"], c["k"], c["mode"], c["cap"], _eps(c), W=s["W"]))
    if kind == "sym_job":
        return _job(g.pic_sym(s["X"], c["sigma"], c["k"], c["mode"], c["cap"], _eps(c),
                              As=s["As"]))
    if kind == "fused_job":
        return _job(g.pic_fused(s["X"], c["sigma"], c["k"], c["mode"], c["cap"], _eps(c)))
    if kind == "csr_job":
        # the clustering scales the graph's weights in place: on a copy
        return _job(g.pic_csr(s["rp"], s["col"], s["val"].clone(), c["k"], c["mode"], c["cap"],
                              _eps(c)))
    if kind == "weights":
        if c["form"] == "normalized":
            W, degree, v0, _ = g.gpic_affinity_normalized(s["X"], c["sigma"], s["W"])
            return {"W": W[:, :n], "degree": degree, "v0": v0}
        if c["form"] == "affinity":
            A, degree = g.gpic_affinity(s["X"], c["sigma"], s["W"])
            return {"W": A[:, :n], "degree": degree}
        W, degree, v0, _ = g.gpic_affinity_cosine_normalized(s["X"], s["W"])
        return {"W": W[:, :n], "degree": degree, "v0": v0}
    if kind == "knn":
        if c["local"]:
            rp, col, val, perm = g.gpic_knn_graph_local(s["X"], c["knn"], c["sigma"])
            return {"row_ptr": rp, "col": _full(col, c), "val": _full(val, c), "perm": perm}
        rp, col, val = g.gpic_knn_graph(s["X"], c["knn"], c["sigma"])
        return {"row_ptr": rp, "col": _full(col, c), "val": _full(val, c)}
    if kind == "kmeans":
        o = g.gpic_kmeans1d(s["v"], c["k"])
        return {"labels": o.labels, "centroids": o.centroids, "cost": o.cost}
    v = s["v0"].clone()
    # the velocity after a fixed number of updates may be rounding alone: a
    # program that asks for it stops on it
    delta = s["v0"].clone() if c["mode"] == "converge" else None
    if kind == "dense_iter":
        f = g.gpic_power_iterate_dense_noalloc if c["noalloc"] else g.gpic_power_iterate_dense
        f(s["W"], v, delta, c["mode"], c["cap"], _eps(c), n=n)
    elif kind == "fused_iter":
        g.gpic_power_iterate_fused(s["X"], c["sigma"], s["degree"], v, delta, c["mode"], c["cap"],
                                   _eps(c))
    else:
        g.gpic_power_iterate_csr(s["rp"], s["col"], s["val"], v, delta, c["mode"], c["cap"],
                                 _eps(c))
    return _state(v, delta, c)


def _state(v, delta, c):
    return {"v": v, "delta": delta} if c["mode"] == "converge" else {"v": v}


# ------------------------------------------------------------------- work
def _updates(case):
    """Updates of a pass; to convergence, what these inputs typically take."""
    if case["mode"] == "fixed":
        return case["cap"]
    typical = {"rings": 60, "moons": 3, "circles": 3}.get(case["data"], 12)
    if case["kind"].startswith("csr"):
        typical = 38
    return min(typical, case["cap"])


def work(case):
    """Each input read once and each output written once, W (or A) written
    once and read once per update where the path stores it; flops: 2 d + 2
    per unordered pair for an affinity sweep, 2 per entry of a product."""
    kind, n, d = case["kind"], case["n"], case.get("d", 1)
    vec, pts = 8.0 * n, 4.0 * n * d
    pairs = 0.5 * n * n
    if kind == "weights":
        return {"bytes": pts + 4.0 * n * n + 2 * vec, "flops": (2 * d + 2) * pairs}
    if kind == "kmeans":
        return {"bytes": vec + 4.0 * n, "flops": 8.0 * n * case["k"]}
    if kind in ("knn", "csr_iter", "csr_job"):
        nnz = 1.4 * n * case["knn"]
        if kind == "knn":
            return {"bytes": pts + 8.0 * nnz + 12.0 * n, "flops": 2.0 * d * nnz}
        T = _updates(case)
        extra = 16.0 * nnz + 4.0 * n if kind == "csr_job" else 0.0
        return {"bytes": T * (8.0 * nnz + 24.0 * n) + extra, "flops": T * 2.0 * nnz}
    T = _updates(case)
    if kind in ("fused_iter", "fused_job"):
        sweeps = T + (1 if kind == "fused_job" else 0)
        return {"bytes": sweeps * (pts + 2 * vec), "flops": sweeps * (2 * d + 6) * pairs}
    if kind == "dense_iter":
        return {"bytes": T * (4.0 * n * n + 6 * vec), "flops": T * 2.0 * n * n}
    store = 2.0 * n * n if kind == "sym_job" else 4.0 * n * n
    return {"bytes": pts + store + T * (store + 6 * vec) + 4.0 * n,
            "flops": (2 * d + 2) * pairs + T * 2.0 * n * n}


def tolerance(case):
    """About four times the largest difference from exact() seen over the
    ranges."""
    kind = case["kind"]
    if kind == "weights":
        # float32 entries: the squared distance's rounding goes into the
        # exponent (1.4e-6 seen at 128 dimensions)
        return {"rel": 6e-6}
    if kind == "knn":
        return {"rel": 1e-7, "max": 1e-6, "differ": 0.0}
    if kind in ("dense_iter", "csr_iter"):
        # float64 sums over the same float32 W; the velocity is a difference
        # of iterates, about 1e-5 of them (1.8e-11 seen)
        return {"rel": 1e-10, "max": 1e-7}
    if kind == "kmeans":
        return {"rel": 1e-11, "max": 1e-10, "differ": 1e-5}
    # through float32 entries of A; a point at a cluster's end may change
    # sides with the last bits of v
    return {"rel": 6e-6, "differ": max(1e-3, 2.0 / case["n"])}


# ------------------------------------------------------------------ exact
_ROWS = 1 << 28                                      # entries of a block of rows


def _affinity_rows(P, sq, a, b, sigma, cosine):
    """Rows a .. b of the float64 affinity (zero diagonal)."""
    G = P[a:b] @ P.T
    if cosine:
        r = torch.rsqrt(sq)
        A = (0.5 + 0.5 * G * r[a:b, None] * r[None, :]).clamp_(min=0.0)
    else:
        A = torch.exp_(G.mul_(-2.0).add_(sq[a:b, None]).add_(sq[None, :]).clamp_(min=0.0)
                       .mul_(-0.5 / (sigma * sigma)))
    i = torch.arange(a, b, device=P.device)
    A[i - a, i] = 0.0
    return A


class _Operator:
    """W = D^-1 A in float64, stored when it fits, else row block by block."""

    def __init__(self, X, sigma, cosine=False):
        P = X.double()
        self.P = P if cosine else P - P.mean(0)
        self.sq = (self.P * self.P).sum(1)
        self.n, self.sigma, self.cosine = X.shape[0], float(sigma), cosine
        self.step = max(1, _ROWS // self.n)
        self.A = None
        if self.n <= 50000:
            self.A = torch.empty((self.n, self.n), dtype=torch.float64, device=X.device)
            for a in range(0, self.n, self.step):
                b = min(a + self.step, self.n)
                self.A[a:b] = self.rows(a, b)
        self.degree = self.product(torch.ones(self.n, dtype=torch.float64, device=X.device))

    def rows(self, a, b):
        return _affinity_rows(self.P, self.sq, a, b, self.sigma, self.cosine)

    def product(self, x):
        if self.A is not None:
            return self.A @ x
        return torch.cat([self.rows(a, min(a + self.step, self.n)) @ x
                          for a in range(0, self.n, self.step)])

    def __call__(self, x):
        y = self.product(x)
        return torch.where(self.degree == 0.0, torch.zeros_like(y), y / self.degree)


def _iterate(product, v0, case):
    """Algorithm 1's loop with the acceleration stop."""
    v, delta = v0, v0
    for _ in range(case["cap"]):
        y = product(v)
        new = y / y.abs().sum()
        dn = (new - v).abs()
        stat = float((dn - delta).abs().max())
        v, delta = new, dn
        if case["mode"] == "converge" and stat <= _eps(case):
            break
    return v, delta


def _kmeans(v, k):
    """The exact minimum within-cluster sum of squares partition of a vector:
    dynamic programme over prefix sums, each layer by divide and conquer over
    its rows, all rows of a depth at once.  Labels, centroids and cost."""
    x, order = torch.sort(v)
    n, dev = x.numel(), x.device
    u = x - x.mean()
    zero = torch.zeros(1, dtype=torch.float64, device=dev)
    S1, S2 = torch.cat([zero, u.cumsum(0)]), torch.cat([zero, (u * u).cumsum(0)])
    starts = torch.cat([torch.ones(1, dtype=torch.bool, device=dev), x[1:] != x[:-1]])
    k = min(k, int(starts.sum()))

    def cost(j, i):
        s = S1[i + 1] - S1[j]
        return (S2[i + 1] - S2[j] - s * s / (i - j + 1).double()).clamp_(min=0.0)

    rows = torch.arange(n, device=dev)
    D = cost(torch.zeros_like(rows), rows)
    back = []
    for _ in range(1, k):
        E = torch.full((n,), math.inf, dtype=torch.float64, device=dev)
        E[1:] = torch.where(starts[1:], D[:-1], E[1:])
        opt = torch.full((n + 1,), n - 1, dtype=torch.int64, device=dev)
        best = torch.full((n,), math.inf, dtype=torch.float64, device=dev)
        lo = torch.zeros(1, dtype=torch.int64, device=dev)
        hi = torch.full((1,), n - 1, dtype=torch.int64, device=dev)
        first = torch.ones(1, dtype=torch.int64, device=dev)
        last = torch.full((1,), n - 1, dtype=torch.int64, device=dev)
        while lo.numel():
            mid = (lo + hi) // 2
            count = (torch.minimum(last, mid) - first + 1).clamp_(min=1)
            seg = torch.repeat_interleave(torch.arange(mid.numel(), device=dev), count)
            begin = count.cumsum(0) - count
            j = first[seg] + torch.arange(seg.numel(), device=dev) - begin[seg]
            m = mid[seg]
            val = torch.where(j <= m, E[j.clamp(max=n - 1)] + cost(torch.minimum(j, m), m),
                              torch.full_like(m, math.inf, dtype=torch.float64))
            low = torch.full((mid.numel(),), math.inf, dtype=torch.float64, device=dev)
            low.scatter_reduce_(0, seg, val, "amin")
            arg = torch.full((mid.numel(),), n, dtype=torch.int64, device=dev)
            arg.scatter_reduce_(0, seg, torch.where(val == low[seg], j, n), "amin")
            arg = torch.where(torch.isinf(low), first, arg)
            best[mid], opt[mid] = low, arg
            left, right = lo < mid, mid < hi
            lo, hi, first, last = (torch.cat([lo[left], mid[right] + 1]),
                                   torch.cat([mid[left] - 1, hi[right]]),
                                   torch.cat([first[left], arg[right]]),
                                   torch.cat([arg[left], last[right]]))
        D = best
        back.append(opt)
    ends = [n]
    for opt in reversed(back):
        ends.append(int(opt[ends[-1] - 1]))
    ends.append(0)
    ends.reverse()
    centroids = torch.stack([x[a:b].mean() for a, b in zip(ends, ends[1:])])
    total = float(sum(((x[a:b] - x[a:b].mean()) ** 2).sum() for a, b in zip(ends, ends[1:])))
    labels = torch.empty(n, dtype=torch.int32, device=dev)
    of = torch.zeros(n, dtype=torch.int32, device=dev)
    for c, a in enumerate(ends[1:-1]):
        of[a:] = c + 1
    labels[order] = of
    return labels, centroids, total


def _exact_knn(X, case):
    n, k = case["n"], case["knn"]
    P = X.double()
    rows, cols = [], []
    step = max(1, (1 << 26) // n)
    for a in range(0, n, step):
        b = min(a + step, n)
        D2 = torch.zeros((b - a, n), dtype=torch.float64, device=X.device)
        for c in range(P.shape[1]):
            D2 += (P[a:b, c, None] - P[None, :, c]) ** 2
        i = torch.arange(a, b, device=X.device)
        D2[i - a, i] = math.inf
        rows.append(i.repeat_interleave(k))
        cols.append(torch.topk(D2, k, dim=1, largest=False).indices.reshape(-1))
    r, c = torch.cat(rows), torch.cat(cols)
    key = torch.unique(torch.cat([r * n + c, c * n + r]))
    r, c = key // n, key % n
    d2 = ((P[r] - P[c]) ** 2).sum(1)
    return torch.exp(-d2 / (2.0 * case["sigma"] ** 2))


def exact(case, seed):
    kind, n = case["kind"], case["n"]
    if kind == "knn":
        if case["local"] or n > 60000:
            return None
        return {"row_ptr": None, "col": None, "val": _full(_exact_knn(_points(case, seed), case), case)}
    s = prepare(case, seed)
    if kind == "kmeans":
        labels, centroids, cost = _kmeans(s["v"], case["k"])
        return {"labels": labels, "centroids": centroids, "cost": cost}
    if kind == "dense_iter":
        W = s["W"][:, :n].double()
        v, delta = _iterate(lambda x: W @ x, s["v0"], case)
        return _state(v, delta, case)
    if kind in ("csr_iter", "csr_job"):
        A = torch.sparse_csr_tensor(s["rp"], s["col"].long(), s["val"].double(), (n, n))
        if kind == "csr_iter":
            v, delta = _iterate(lambda x: A @ x, s["v0"], case)
            return _state(v, delta, case)
        degree = A @ torch.ones(n, dtype=torch.float64, device=DEV)
        v0 = degree / degree.sum()
        v, _ = _iterate(lambda x: (A @ x) / degree, v0, case)
    else:
        op = _Operator(s["X"], case.get("sigma", 1.0),
                       kind == "cosine_job" or case.get("form") == "cosine")
        degree = op.degree
        v0 = degree / degree.sum()
        if kind == "weights":
            if case["form"] == "affinity":
                return {"W": op.A, "degree": degree}
            return {"W": op.A.div_(degree[:, None]), "degree": degree, "v0": v0}
        if kind == "fused_iter":
            op.degree, v0 = s["degree"], s["v0"]
            v, delta = _iterate(op, v0, case)
            return _state(v, delta, case)
        v, _ = _iterate(op, v0, case)
    labels, centroids, _ = _kmeans(v, case["k"])
    return {"degree": degree, "v0": v0, "v": v, "labels": labels, "centroids": centroids}
