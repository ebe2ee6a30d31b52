"""Evaluations of small graphs in one workgroup: every split of rows over threads and its
edges, rows that take a wave, exhausted Krylov spaces, against the general path (which
profiling keeps) and the dense operator; errors stay what they were."""

import numpy as np
import pytest

import synth
from oracle import genfun, laplacian, walks
from synth.graphs import csr_from_edges

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def graph_of(name, n):
    if name == "er":
        return synth.erdos_renyi_gnm(n, min(4 * n, n * (n - 1) // 4), 3)
    if name == "hubs":  # rows of 31, 32, 33 and most of the graph; the last nodes isolated
        u, v = [], []
        for hub, d in ((0, 31), (1, 32), (2, 33), (3, max(4, n - 12))):
            k = min(d, n - 8)
            u += [hub] * k
            v += list(range(4, 4 + k))
        return csr_from_edges(n, u, v)
    return csr_from_edges(n, np.arange(n - 1), np.arange(1, n))  # a path


def both(lib, rp, ci, mu, kind, param, dtype, b, X, **kw):
    """The same call on the small and on the general path (a profiled context)."""
    out = []
    for profiled in (False, True):
        ctx = lib.Context(0)
        ctx.set_profiling(profiled)
        op = lib.Operator(lib.Graph(ctx, rp, ci), mu, kind, param, dtype=dtype, krylov_dim=40, **kw)
        Xd = torch.tensor(X, dtype=dtype, device="cuda")
        res = [op.fdeg(), op.apply_phi(Xd), op.apply_L(Xd)]
        if b == 1:
            res.append(op.expv(Xd, [0.7], outer_dim=20)[0][0])
        out.append([r.cpu().numpy().astype(np.float64) for r in res])
    return out


SIZES = [12, 63, 64, 65, 256, 257, 512, 513, 1024, 1025, 2048, 2049, 4096, 4097]


# FP64: 40 steps of rounding at 1e-16 on O(1) values; FP32: the library's 2e-5 for products, 1e-4
# for the diffusion
@pytest.mark.parametrize("n", SIZES)
@pytest.mark.parametrize("name", ["er", "hubs", "path"])
def test_small_equals_general(lib, name, n):
    rp, ci = graph_of(name, n)
    d = np.diff(rp)
    lam = max(np.sqrt(d.max()), d.max() if name != "hubs" else np.sqrt(d.max()) * 3)  # at least the largest eigenvalue
    for dtype, tol in ((torch.float64, 1e-11), (torch.float32, 2e-5)):
        for b in (1, 2, 3, 4):
            X = synth.gaussian_block(n, b, seed=n + b)
            for mu, kind, kw in ((0.5, "res", dict(rho_hint=lam, reorth=1)), (0.0, "res", dict(rho_hint=lam, reorth=0)),
                                 (0.25, "exp", {})):
                print(f"[gpu] {name} n={n} b={b} {dtype} mu={mu} {kind}", flush=True)
                small, general = both(lib, rp, ci, mu, kind, 0.5 / lam, dtype, b, X, **kw)
                for i, (s, g) in enumerate(zip(small, general)):
                    scale = max(np.linalg.norm(g), np.linalg.norm(X) if i else 0.0)
                    assert np.linalg.norm(s - g) <= (tol if i < 3 else 5 * tol) * scale, (dtype, b, mu, kind, i)


@pytest.mark.parametrize("b", [1, 2, 4])
@pytest.mark.parametrize("dtype,tol", [(torch.float64, 1e-10), (torch.float32, 2e-5)], ids=["f64", "f32"])
def test_exhausted_spaces(lib, b, dtype, tol):
    """Unit and repeated columns on a graph of small components: the space ends after a few
    steps, zero and dependent columns deflate."""
    n = 300
    u = np.arange(0, n - 60, 3)
    rp, ci = csr_from_edges(n, np.concatenate([u, u]), np.concatenate([u + 1, u + 2]))
    A = walks.adjacency(n, rp, ci)
    X = np.zeros((n, b))
    X[0, 0] = 1.0
    if b > 1:
        X[:, 1] = X[:, 0]
    if b > 2:
        X[3, 3] = -2.0
    X = np.ascontiguousarray(X)
    lam = float(np.linalg.eigvalsh(A)[-1])
    op = lib.Operator(lib.Graph(lib.Context(0), rp, ci), 1.0, "res", 0.5 / lam, dtype=dtype, krylov_dim=40, rho_hint=lam)
    phi = genfun.phi(A, 1.0, "res", 0.5 / lam)
    Xd = torch.tensor(X, dtype=dtype, device="cuda")
    got = op.apply_L(Xd).cpu().numpy()
    assert np.linalg.norm(got - laplacian.apply_laplacian(phi, X)) <= tol * np.linalg.norm(X)
    zero = op.apply_phi(torch.zeros_like(Xd)).cpu().numpy()
    assert np.all(zero == 0.0)


def test_errors_as_on_the_general_path(lib):
    n = 200
    rp, ci = synth.erdos_renyi_gnm(n, 800, 3)
    lam = float(np.linalg.eigvalsh(walks.adjacency(n, rp, ci))[-1])
    g = lib.Graph(lib.Context(0), rp, ci)
    x = torch.ones((n, 1), dtype=torch.float64, device="cuda")
    op = lib.Operator(g, 0.0, "res", 1.5 / lam, dtype=torch.float64, krylov_dim=20, rho_hint=0.5 * lam)
    with pytest.raises(lib.WLError, match="NOTSPD"):
        op.apply_phi(x)
    op = lib.Operator(g, 0.0, "res", 0.5 / lam, dtype=torch.float64, krylov_dim=20, rho_hint=lam)
    bad = x.clone()
    bad[3] = float("nan")
    with pytest.raises(lib.WLError, match="ENUMERIC"):
        op.apply_phi(bad)
    phi = genfun.phi(walks.adjacency(n, rp, ci), 0.0, "res", 0.5 / lam)
    assert np.linalg.norm(op.apply_phi(x).cpu().numpy()[:, 0] - phi @ np.ones(n)) <= 1e-10 * np.sqrt(n)
