"""Multigrid CG over block widths: the coarsest solve in one launch, column sums of widths that
are no power of two, rows of the coarse matrices longer than one batch of loads."""

import numpy as np
import pytest

import synth
from oracle import genfun, walks

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("name", ["er", "road"])
@pytest.mark.parametrize("b", [1, 3, 16, 33, 64])
def test_amg_widths(lib, name, b):
    rp, ci = synth.erdos_renyi_gnm(900, 4000, 3) if name == "er" else synth.road_grid(33, 31, 0.8, seed=3)
    n = len(rp) - 1
    A = walks.adjacency(n, rp, ci)
    rho = walks.spectral_radius(walks.linearisation(A, 1.0))
    g = lib.Graph(lib.Context(0), rp, ci, validate=True)
    op = lib.Operator(g, 1.0, "res", 0.9 / rho, dtype=torch.float64, method="amg", tol=1e-11, rho_hint=rho)
    assert op.amg_info()["levels"] >= 2
    X = synth.gaussian_block(n, b, seed=b)
    got = op.apply_phi(torch.tensor(X, dtype=torch.float64, device="cuda")).cpu().numpy()
    ref = genfun.phi(A, 1.0, "res", 0.9 / rho) @ X
    assert np.linalg.norm(got - ref) <= 1e-8 * np.linalg.norm(ref)  # residual 1e-11 times the condition (< 100)
