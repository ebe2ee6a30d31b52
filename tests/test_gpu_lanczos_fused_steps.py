"""Block Lanczos at the sizes where a step's launches are joined or not: Grams summed by the
factorisation that needs them (32768 values in partial sums, 131072 for the second pass) and
projections formed inside the update, for well and badly conditioned start blocks; against the
truncated series in float64."""

import math

import numpy as np
import pytest
import scipy.sparse as sp
import scipy.sparse.linalg  # noqa: F401

import synth

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def reference(A, X, mu, beta, K=24):
    """sum_k beta^k q_k X / k!; the tail at beta lambda_max = 0.6 is below 1e-24 of the first terms."""
    D = np.asarray(A.sum(1))
    P2, P1 = X, A @ X
    S = P2 + beta * P1
    for k in range(2, K + 1):
        P = A @ P1 + (-mu * D * P2 if k == 2 else mu * (mu - D) * P2)
        S = S + beta ** k / math.factorial(k) * P
        P2, P1 = P1, P
    return S


# (columns, nodes): both sides of 128 partials of 16 x 16 (12 and 16 columns) and of 32 of
# 32 x 32 (24 and 32), and of 512 x 32 x 32 for the second pass; 5, 8: always joined
CASES = [(5, 700), (8, 40000), (12, 8192), (12, 8300), (16, 32700), (16, 33100), (24, 2048), (24, 2100), (32, 8192),
         (32, 33000), (40, 3000), (3, 2000), (4, 2000), (1, 6000), (2, 30000), (3, 30000), (4, 30000)]


@pytest.mark.parametrize("b,n", CASES)
@pytest.mark.parametrize("block", ["gaussian", "near", "dependent"])
def test_steps(lib, b, n, block):
    rp, ci = synth.barabasi_albert(n, 3, b)
    A = sp.csr_matrix((np.ones(len(ci)), ci, rp), shape=(n, n))
    lam = float(sp.linalg.eigsh(A, k=1, return_eigenvectors=False)[0])
    X = synth.gaussian_block(n, b, seed=n)
    if block == "near" and b > 1:  # condition about 1e3: the second factorisation runs
        X[:, 1] = X[:, 0] + 1e-3 * X[:, 1]
    if block == "dependent" and b > 1:  # a column deflates
        X[:, b - 1] = X[:, 0] - X[:, 1]
    beta = 0.6 / lam
    ref = reference(A, X, 0.0, beta)
    g = lib.Graph(lib.Context(0), rp, ci)
    for dtype, tol in ((torch.float64, 1e-8), (torch.float32, 1e-4)):  # the library's parity contract
        op = lib.Operator(g, 0.0, "exp", beta, dtype=dtype, krylov_dim=14, method="lanczos")
        Y = op.apply_phi(torch.tensor(X, dtype=dtype, device="cuda"))
        assert np.linalg.norm(Y.double().cpu().numpy() - ref) <= tol * np.linalg.norm(ref), dtype


@pytest.mark.parametrize("n", [700, 5000, 40000])
@pytest.mark.parametrize("block", ["gaussian", "near", "dependent"])
def test_operators_in_lock_step(lib, n, block):
    b, rp_ci = 16, synth.barabasi_albert(n, 3, 1)
    rp, ci = rp_ci
    A = sp.csr_matrix((np.ones(len(ci)), ci, rp), shape=(n, n))
    lam = float(sp.linalg.eigsh(A, k=1, return_eigenvectors=False)[0])
    X = synth.gaussian_block(n, b, seed=n)
    if block == "near":
        X[:, 1] = X[:, 0] + 1e-3 * X[:, 1]
    if block == "dependent":
        X[:, b - 1] = X[:, 0] - X[:, 1]
    g = lib.Graph(lib.Context(0), rp, ci)
    betas = [0.6 / lam, 0.3 / lam, 0.1 / lam]
    m = lib.Multi([lib.Operator(g, 0.0, "exp", be, krylov_dim=14, method="lanczos") for be in betas])
    Xd = torch.tensor(X, dtype=torch.float32, device="cuda")
    Y = m.apply_phi(Xd)
    Yf, W = m.apply_fdeg(Xd, laplacian=False)
    for q, be in enumerate(betas):
        ref = reference(A, X, 0.0, be)
        w = reference(A, np.ones((n, 1)), 0.0, be)
        for out in (Y, Yf):
            got = out[:, q * b:(q + 1) * b].double().cpu().numpy()
            assert np.linalg.norm(got - ref) <= 1e-4 * np.linalg.norm(ref), q
        assert np.linalg.norm(W[:, q:q + 1].double().cpu().numpy() - w) <= 1e-4 * np.linalg.norm(w), q
