"""Edge sizes of the learned part's kernels: sample tiles of the network, rounds beyond one
grid, neighbour sums on both sides of the long-row bound, and row sums of odd widths."""

import numpy as np
import pytest

import synth
from oracle import estimators, features, mlp
from synth.graphs import csr_from_edges

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def ctx(lib):
    return lib.Context(0)


# one tile, its edges, one workgroup's tiles, and one round of the largest grid (512
# workgroups of 4 waves of 8 tiles) with a remainder
@pytest.mark.parametrize("N", [1, 15, 16, 17, 65, 512 * 4 * 8 * 16 + 17])
def test_mlp_tiles(ctx, lib, N):
    p = np.asarray(synth.glorot_params(mlp.SIZES, 3), dtype=np.float32)
    rng = np.random.default_rng(N)
    X, t = rng.standard_normal((N, 8)).astype(np.float32), rng.standard_normal(N).astype(np.float32)
    net = lib.MLP(ctx, p)
    Xd, td = torch.tensor(X, device="cuda"), torch.tensor(t, device="cuda")
    p64, X64 = p.astype(np.float64), X.astype(np.float64)
    # 64-term FP32 sums of values below one: 64 * 2^-24 = 4e-6 of the largest output
    y_ref, _ = mlp.forward(p64, X64)
    y = net.forward(Xd).cpu().numpy().astype(np.float64)
    assert np.abs(y - y_ref).max() <= 1e-5 * max(1.0, np.abs(y_ref).max())
    L, g = net.loss_grad(Xd, td)
    L_ref, g_ref = mlp.loss_and_grad(p64, X64, t.astype(np.float64))
    assert abs(L - L_ref) <= 1e-5 * L_ref
    assert np.abs(g - g_ref).max() <= 2e-5 * np.abs(g_ref).max()
    assert net.loss_grad(Xd, td)[1].tolist() == g.tolist()  # fixed summation order


def hub_graph():
    """Hubs of 512, 513 and 514 neighbours (the long-row bound is 512) and isolated nodes."""
    u, v, at = [], [], 3
    for hub, d in enumerate((511, 511, 513)):
        u += [hub] * d
        v += range(at, at + d)
        at += d - 7  # some leaves are shared by two hubs: triangles with the edges below
    u += list(range(3, 60)) + [0, 1]
    v += list(range(4, 61)) + [1, 2]
    n = at + 40
    return (n,) + csr_from_edges(n, u, v)


def test_features_and_surrogate_at_the_long_row_bound(ctx, lib):
    n, rp, ci = hub_graph()
    g = lib.Graph(ctx, rp, ci, validate=True)
    f = g.features(0.05).cpu().numpy().astype(np.float64)
    ref = features.features(n, rp, ci, 0.05)
    np.testing.assert_allclose(f, ref, rtol=2.0 ** -23, atol=1e-30)  # FP64 values rounded to FP32
    A = np.zeros((n, n))
    A[np.repeat(np.arange(n), np.diff(rp)), ci] = 1.0
    op = lib.Operator(g, 0.5, "exp", 0.02, dtype=torch.float64)
    base, scale = op.surrogate_diag()
    rb, rs = features.surrogate_terms(A, 0.5, "exp", 0.02)
    np.testing.assert_allclose(base.cpu().numpy(), rb, rtol=1e-13)
    np.testing.assert_allclose(scale.cpu().numpy(), rs, rtol=1e-13)


@pytest.mark.parametrize("n,M", [(1, 1), (17, 15), (33, 16), (50, 17), (300, 64)])
def test_row_sums(ctx, lib, n, M):
    rng = np.random.default_rng(n)
    Om, Y, cv = rng.standard_normal((n, M)), rng.standard_normal((n, M)), rng.standard_normal(n)
    to = lambda a: torch.tensor(a, device="cuda")  # noqa: E731
    d = lib.estimate(ctx, to(Om), to(Y))[0].cpu().numpy()
    c = lib.estimate(ctx, to(Om), to(Y), cv=to(cv))[0].cpu().numpy()
    scale = np.abs(Om * Y).sum(1) / M + np.abs(cv) * (1 + (Om * Om).sum(1) / M)
    assert np.all(np.abs(d - estimators.hutchinson_diag(Om, Y)) <= 1e-14 * scale)
    assert np.all(np.abs(c - estimators.cv_diag(Om, Y, cv)) <= 1e-14 * scale)
