"""Batched diffusion at the block widths and graph sizes where the segmented Gram changes its
form: up to 8 columns and above, graphs below one round of rows, at the end of a reduction
unit and just past it; against the dense exponential's action."""

import numpy as np
import pytest
from scipy.sparse.linalg import expm_multiply

import synth
from oracle import genfun, laplacian, walks

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

SIZES, TIMES = [5, 64, 100, 130, 2048, 2050, 2120], [0.5, 1.0, 0.2, 0.7, 1.0, 0.4, 0.8]


@pytest.fixture(scope="module")
def parts():
    out = []
    for i, n in enumerate(SIZES):
        rp, ci = synth.barabasi_albert(n, 3, i)
        A = walks.adjacency(n, rp, ci)
        param = 1.0 / float(np.linalg.eigvalsh(A)[-1])
        ph = genfun.phi(A, 0.25, "exp", param)
        out.append((rp, ci, param, np.diag(laplacian.walk_degree(ph)) - ph))
    return out


@pytest.mark.parametrize("b", [2, 3, 7, 8, 9, 15, 16])
def test_widths(lib, parts, b):
    ctx = lib.Context(0)
    graphs = [lib.Graph(ctx, rp, ci) for rp, ci, _, _ in parts]
    batch = lib.Batch(ctx, graphs, [dict(mu=0.25, func="exp", param=p) for _, _, p, _ in parts])
    U = [synth.gaussian_block(n, b, seed=n + b) for n in SIZES]
    X = batch.pack([torch.tensor(u, dtype=torch.float32, device="cuda") for u in U])
    Y, _, _ = batch.expv(X, TIMES, outer_dim=min(20, 3840 // (b * b)))  # 5 dim b^2 doubles on chip
    for u, t, (_, _, _, L), y in zip(U, TIMES, parts, batch.unpack(Y)):
        ref = expm_multiply(-t * L, u)
        assert np.linalg.norm(y.cpu().numpy() - ref) <= 1e-4 * np.linalg.norm(u), len(u)  # FP32 parity contract
