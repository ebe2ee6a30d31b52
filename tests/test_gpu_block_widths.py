"""Block widths on both sides of every kernel size (8, 16, 32, 64 columns; multiples of 4
and of 2; odd), full rank and rank deficient, against the dense operator."""

import numpy as np
import pytest

import synth
from oracle import genfun, laplacian, walks

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

N = 701  # no multiple of a row tile


@pytest.fixture(scope="module")
def setup(lib):
    rp, ci = synth.barabasi_albert(N, 3, 5)
    A = walks.adjacency(N, rp, ci)
    lam = float(np.linalg.eigvalsh(A)[-1])
    return lib.Graph(lib.Context(0), rp, ci, validate=True), A, lam


WIDTHS = [1, 2, 3, 5, 7, 8, 9, 12, 15, 16, 17, 18, 24, 30, 31, 32, 33, 48, 62, 63, 64]


def block(b, rank, dtype):
    X = synth.gaussian_block(N, b, seed=b)
    if rank < b:
        X[:, rank:] = X[:, :rank] @ synth.gaussian_block(rank, b - rank, seed=1)
    return torch.tensor(X, dtype=dtype, device="cuda")


def check(op, X, phi, tol):
    Xh = X.cpu().numpy().astype(np.float64)
    got = op.apply_L(X).cpu().numpy().astype(np.float64)
    w = laplacian.walk_degree(phi)
    scale = np.linalg.norm(w[:, None] * Xh) + np.linalg.norm(phi @ Xh)
    assert np.linalg.norm(got - laplacian.apply_laplacian(phi, Xh)) <= tol * scale


# FP64: 1e-11 (thirty steps of FP64 rounding on O(1) values); FP32: the library's 2e-5
@pytest.mark.parametrize("b", WIDTHS)
@pytest.mark.parametrize("dtype,tol", [(torch.float64, 1e-11), (torch.float32, 2e-5)], ids=["f64", "f32"])
def test_lanczos_widths(lib, setup, b, dtype, tol):
    g, A, lam = setup
    op = lib.Operator(g, 0.5, "res", 0.5 / lam, dtype=dtype, krylov_dim=30, rho_hint=lam)
    phi = genfun.phi(A, 0.5, "res", 0.5 / lam)
    check(op, block(b, b, dtype), phi, tol)
    if b >= 5:
        check(op, block(b, 3, dtype), phi, tol)


@pytest.mark.parametrize("b", WIDTHS)
@pytest.mark.parametrize("dtype,tol", [(torch.float64, 1e-12), (torch.float32, 2e-5)], ids=["f64", "f32"])
def test_series_widths(lib, setup, b, dtype, tol):
    g, A, lam = setup
    op = lib.Operator(g, 0.25, "exp", 1.0 / lam, dtype=dtype, krylov_dim=20)
    check(op, block(b, b, dtype), genfun.phi(A, 0.25, "exp", 1.0 / lam), tol)
