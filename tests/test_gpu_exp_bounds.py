"""exp(-t T) of the projected walk Laplacian where its spectrum is not [0, ||T||]: results far
below the start block, and projections with negative eigenvalues."""

import numpy as np
import pytest

import synth
from oracle import krylov, sparse
from synth.graphs import csr_from_edges

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def cliques(sizes):
    u, v, at = [], [], 0
    for s in sizes:
        i, j = np.triu_indices(s, 1)
        u.append(at + i)
        v.append(at + j)
        at += s
    return csr_from_edges(at, np.concatenate(u), np.concatenate(v))


def mean_free(sizes, b, seed):
    """Integer columns that sum to zero on every clique (exactly)."""
    rng = np.random.default_rng(seed)
    R = [rng.integers(-4, 5, (s, b)) for s in sizes]
    return np.concatenate([r - np.roll(r, 1, axis=0) for r in R]).astype(np.float64)


def clique_rates(sizes, beta):
    """Eigenvalue of L on the mean-free vectors of a clique of s nodes, mu = 0, exp(beta A)."""
    return [np.exp(beta * (s - 1)) - np.exp(-beta) for s in sizes]


# On cliques of 8 sizes L has 8 eigenvalues on mean-free blocks, so 8 steps are exact; exp(-t L) X
# is 3e-5 to 1e-22 of X.  Relative errors: t lambda = 50 times the products' 1e-8.
@pytest.mark.parametrize("t", [13.0, 36.0, 63.0])
@pytest.mark.parametrize("b", [8, 16, 32])  # 64 rows on the host, 128 and 256 on the device
def test_expv_far_below_the_start(lib, b, t):
    sizes = [40, 44, 48, 52, 56, 60, 64, 68]
    beta = 1.0 / 68
    rp, ci = cliques(sizes)
    X = mean_free(sizes, b, 5)
    op = lib.Operator(lib.Graph(lib.Context(0), rp, ci), 0.0, "exp", beta, dtype=torch.float64)
    outs, _ = op.expv(torch.tensor(X, device="cuda"), [0.5, t], outer_dim=8)
    rate = np.repeat(clique_rates(sizes, beta), sizes)[:, None]
    for s, o in zip([0.5, t], outs):
        ref = np.exp(-s * rate) * X
        assert np.linalg.norm(o.cpu().numpy() - ref) <= 5e-7 * np.linalg.norm(ref), s


# FP32: rates good to a few 6e-8, times t lambda <= 60
@pytest.mark.parametrize("b", [2, 8])
def test_batch_far_below_the_start(lib, b):
    sizes, ctx = [64, 50, 129, 64], lib.Context(0)
    tl = [0.0, 20.0, 45.0, 60.0]
    graphs, descs, U, refs, ts = [], [], [], [], []
    for i, (s, x) in enumerate(zip(sizes, tl)):
        graphs.append(lib.Graph(ctx, *cliques([s])))
        descs.append(dict(mu=0.0, func="exp", param=1.0 / s))
        U.append(mean_free([s], b, i))
        rate = clique_rates([s], 1.0 / s)[0]
        ts.append(x / rate)
        refs.append(np.exp(-x) * U[-1])
    batch = lib.Batch(ctx, graphs, descs)
    Y, _, _ = batch.expv(batch.pack([torch.tensor(u, dtype=torch.float32, device="cuda") for u in U]), ts, outer_dim=10)
    for ref, x, y in zip(refs, tl, batch.unpack(Y)):
        assert np.linalg.norm(y.cpu().numpy() - ref) <= 1e-4 * np.linalg.norm(ref), x


# phi by 5 inner steps is not entrywise positive: T has an eigenvalue -4e-3.  The reference is the
# same process in 64 bits.
@pytest.mark.parametrize("b,dim", [(10, 8), (20, 8)])  # 80 and 160 rows
def test_expv_of_an_indefinite_projection(lib, b, dim):
    n, inner = 400, 5
    rp, ci = synth.barabasi_albert(n, 4, 2)
    A = sparse.adjacency(n, rp, ci)
    alpha = 0.97 / sparse.lambda_max(A)
    op = lib.Operator(lib.Graph(lib.Context(0), rp, ci), 0.0, "res", alpha, dtype=torch.float64, krylov_dim=inner,
                      rho_hint=sparse.lambda_max(A))
    U = synth.gaussian_block(n, b, seed=1)
    ts = [0.1, 4.0, 600.0]
    outs, err = op.expv(torch.tensor(U, device="cuda"), ts, outer_dim=dim)
    phi = lambda X: krylov.phi_resolvent_lanczos(A, 0.0, alpha, X, inner)
    w = phi(np.ones((n, 1)))[:, 0]
    refs, rerr = krylov.expv_lanczos(phi, w, U, ts, dim)
    for t, o, r, e, re in zip(ts, outs, refs, err, rerr):
        assert np.linalg.norm(o.cpu().numpy() - r) <= 1e-8 * max(np.linalg.norm(r), np.linalg.norm(U)), t
        assert abs(e - re) <= 1e-7 * max(re, np.linalg.norm(U)), t
