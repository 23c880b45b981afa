"""Every operation through the binding on buffers (workspaces and outputs)
full of zeros and full of a large finite value: the results must be the same
bits, on both sides of every change of route.  What a kernel reads it, or
one before it in the call, has written."""
import numpy as np
import pytest

from gpu_helpers import Filled

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
DEV = "cuda:0"


@pytest.fixture(scope="module")
def g():
    import paper_1604_02700_amd as g
    g.lib()
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    return g


def _points(n, d):
    rng = np.random.default_rng(n + d)
    C = 3.0 * rng.standard_normal((5, d))
    X = C[rng.integers(5, size=n)] + rng.standard_normal((n, d))
    return torch.from_numpy(X.astype(np.float32)).to(DEV)


def _vector(n):
    return torch.from_numpy(np.random.default_rng(n).uniform(0.5, 1.5, size=n)).to(DEV)


def _pi(out):
    return [out.v, out.delta, out.iterations, out.converged, out.stats]


def _affinity(g, n, d):
    A, deg = g.gpic_affinity(_points(n, d), 2.0)
    W, deg2, v0, nz = g.gpic_affinity_normalized(_points(n, d), 2.0)
    return [A[:, :n], deg, W[:, :n], deg2, v0, nz]


def _cosine(g, n, d):
    A, deg = g.gpic_affinity_cosine(_points(n, d))
    W, deg2, v0, nz = g.gpic_affinity_cosine_normalized(_points(n, d))
    return [A[:, :n], deg, W[:, :n], deg2, v0, nz]


def _normalize(g, n):
    A, _ = g.gpic_affinity(_points(n, 2), 2.0, want_degree=False)
    W, deg, v0, nz = g.gpic_degree_normalize(A, n)
    return [W[:, :n], deg, v0, nz]


def _dense(g, n, mode):
    W, _, v0, _ = g.gpic_affinity_normalized(_points(n, 2), 2.0)
    own = _pi(g.gpic_power_iterate_dense(W, v0.clone(), None, mode, 12, 1e-7 / n, n=n))
    kept = _pi(g.gpic_power_iterate_dense(W, v0.clone(), v0.clone(), mode, 12, 1e-7 / n, n=n))
    return own + kept + [g.gpic_matvec_dense(W, v0, n=n)]


def _host(g, n):
    W, _, v0, _ = g.gpic_affinity_normalized(_points(n, 2), 2.0)
    Wh = torch.empty((n, n), dtype=torch.float32, pin_memory=True)
    Wh.copy_(W[:, :n])
    small = 2 * 36 * ((n + 3) // 4 * 4) * 4 + g.workspace_bytes("pi_dense", n) + 1024
    return (_pi(g.gpic_power_iterate_dense_host(Wh, v0.clone(), None, "fixed", 5, n=n))
            + _pi(g.gpic_power_iterate_dense_host(Wh, v0.clone(), None, "fixed", 5, n=n,
                                                  ws_bytes=small)))


def _sym(g, n, d):
    As, deg, v0, nz = g.gpic_affinity_sym(_points(n, d), 2.0)
    out = g.gpic_power_iterate_sym(As, n, deg, v0.clone(), None, "converge", 12, 1e-7 / n)
    return [deg, v0, nz, g.gpic_matvec_sym(As, n, deg, _vector(n))] + _pi(out)


def _fused(g, n, d, mode):
    X = _points(n, d)
    deg, v0, nz = g.gpic_degree_fused(X, 2.0)
    own = _pi(g.gpic_power_iterate_fused(X, 2.0, deg, v0.clone(), None, mode, 6, 1e-7 / n))
    kept = _pi(g.gpic_power_iterate_fused(X, 2.0, deg, v0.clone(), v0.clone(), mode, 6, 1e-7 / n))
    return [deg, v0, nz, g.gpic_matvec_fused(X, 2.0, deg, _vector(n))] + own + kept


def _knn(g, n, d, k):
    X = _points(n, d)
    X[: n // 4] = X[torch.arange(n // 4, device=DEV) % 40]      # lists that overflow
    return list(g.gpic_knn_graph(X, k, 1.0)) + list(g.gpic_knn_graph_local(X, k, 1.0))


def _csr(g, n, per_row):
    """per_row entries a row at random ascending columns (n > 2^18: the
    column-blocked copy; more than 64 a row: the row product)."""
    gen = torch.Generator(device=DEV).manual_seed(n)
    col = torch.randint(n, (n, per_row), device=DEV, generator=gen).sort(1).values
    val = torch.rand((n, per_row), device=DEV, generator=gen)
    rp = torch.arange(0, n * per_row + 1, per_row, dtype=torch.int64, device=DEV)
    val, deg, v0, nz = g.gpic_degree_normalize_csr(rp, col.int().reshape(-1), val.reshape(-1))
    col = col.int().reshape(-1)
    out = g.gpic_power_iterate_csr(rp, col, val, v0.clone(), None, "converge", 20, 1e-7 / n)
    return [val, deg, v0, nz, g.gpic_matvec_csr(rp, col, val, v0)] + _pi(out)


def _kmeans(g, n, k, width):
    rng = np.random.default_rng(n + k)
    v = rng.random(k)[rng.integers(k, size=n)] + width * rng.standard_normal(n)
    o = g.gpic_kmeans1d(torch.from_numpy(v).to(DEV), k)
    return [o.labels, o.centroids, o.k_eff, o.cost]


CASES = (
    [(_affinity, n, d) for n, d in ((300, 2), (4096, 3), (4097, 16), (700, 64), (500, 140))]
    + [(_cosine, n, d) for n, d in ((300, 2), (4097, 20))]
    + [(_normalize, n) for n in (4096, 4097)]
    + [(_dense, n, m) for n in (1000, 2048, 2049) for m in ("fixed", "converge")]
    + [(_host, 1003)]
    + [(_sym, n, d) for n, d in ((255, 2), (1030, 16))]
    + [(_fused, n, d, m) for n, d in ((9999, 3), (10000, 3), (10241, 12), (383, 16), (3000, 100),
                                      (500, 140)) for m in ("fixed", "converge")]
    + [(_knn, n, d, k) for n, d, k in ((700, 2, 10), (17001, 8, 32), (9000, 16, 64))]
    + [(_csr, n, p) for n, p in ((5000, 12), (3000, 80), (270001, 8))]
    + [(_kmeans, n, k, w) for n, k, w in (
        (4096, 5, 1e-3), (4097, 5, 1e-3), (8191, 12, 1e-2), (8192, 12, 1e-2), (8192, 2, 1e-2),
        (65536, 16, 1e-2), (65537, 16, 1e-2), (131071, 9, 1e-2), (131072, 9, 1e-2),
        (262143, 24, 1e-2), (262144, 24, 1e-2), (262144, 24, 1e-12), (20000, 600, 1e-3))])


@pytest.mark.parametrize("case", CASES, ids=lambda c: "-".join([c[0].__name__[1:], *map(str, c[1:])]))
def test_results_do_not_depend_on_the_buffers(g, monkeypatch, case):
    runs = []
    for x in (0.0, 1e300):
        print(f"scratch {x}: {case[0].__name__} {case[1:]}", flush=True)
        with monkeypatch.context() as m:
            m.setattr(g, "torch", Filled(x))
            runs.append(case[0](g, *case[1:]))
        torch.cuda.synchronize()
    assert len(runs[0]) == len(runs[1])
    for a, b in zip(*runs):
        if isinstance(a, torch.Tensor):
            assert a.shape == b.shape and torch.equal(a, b)
        elif isinstance(a, np.ndarray):
            assert np.array_equal(a, b)
        else:
            assert a == b
