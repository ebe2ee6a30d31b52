"""exp(-t T) of the projected walk Laplacian by Chebyshev series: a single graph on both sides
of the size where the series runs on the device, and batches up to several substeps,
against the dense exponential."""

import numpy as np
import pytest
from scipy.linalg import expm

import synth
from oracle import genfun, laplacian, walks

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def dense(n, m, seed, mu, kind):
    rp, ci = synth.barabasi_albert(n, m, seed)
    A = walks.adjacency(n, rp, ci)
    lam = float(np.linalg.eigvalsh(A)[-1])
    param = (0.5 if kind == "res" else 1.0) / lam
    ph = genfun.phi(A, mu, kind, param)
    return rp, ci, param, lam, np.diag(laplacian.walk_degree(ph)) - ph


# (block width, steps): 3 x 30 = 90 rows on the host, 5 x 30 and more on the device; 40 x 20
# exceeds what the work block of 700 rows holds in FP64 (host again); rank: columns that span
# the start block (the others are combinations, so basis columns deflate)
@pytest.mark.parametrize("b,dim,rank", [(3, 30, 3), (5, 30, 5), (8, 40, 8), (8, 40, 3), (20, 30, 20), (40, 20, 40)])
@pytest.mark.parametrize("mu,kind", [(0.5, "exp"), (1.0, "res")])
def test_expv_series(lib, b, dim, rank, mu, kind):
    n = 700
    rp, ci, param, lam, L = dense(n, 3, 9, mu, kind)
    U = synth.gaussian_block(n, b, seed=b)
    U[:, rank:] = U[:, :rank] @ synth.gaussian_block(rank, b - rank, seed=2) if rank < b else U[:, rank:]
    ts = [0.0, 1e-3, 1.0, 10.0]
    g = lib.Graph(lib.Context(0), rp, ci)
    for dtype, tol in ((torch.float64, 1e-8), (torch.float32, 1e-4)):  # the library's parity contract
        op = lib.Operator(g, mu, kind, param, dtype=dtype, krylov_dim=40, rho_hint=lam if kind == "res" else 0.0)
        outs, err = op.expv(torch.tensor(U, dtype=dtype, device="cuda"), ts, outer_dim=dim)
        for t, o in zip(ts, outs):
            ref = expm(-t * L) @ U
            assert np.linalg.norm(o.cpu().numpy() - ref) <= tol * np.linalg.norm(U), (dtype, t)
        assert all(np.isfinite(err)) and err[0] <= 1e-6


@pytest.mark.parametrize("b", [2, 5, 8])
def test_batch_series_substeps(lib, b):
    # times from 0 to beyond one substep (t ||T|| / 2 > 2000)
    sizes, ts = [150, 333, 64, 200], [0.0, 0.3, 20.0, 3000.0]
    ctx, graphs, descs, Ls = lib.Context(0), [], [], []
    for i, n in enumerate(sizes):
        rp, ci, param, lam, L = dense(n, 3, i, 0.25, "exp")
        graphs.append(lib.Graph(ctx, rp, ci))
        descs.append(dict(mu=0.25, func="exp", param=param))
        Ls.append(L)
    batch = lib.Batch(ctx, graphs, descs)
    U = [synth.gaussian_block(n, b, seed=n) for n in sizes]
    Y, _, _ = batch.expv(batch.pack([torch.tensor(u, dtype=torch.float32, device="cuda") for u in U]), ts, outer_dim=30)
    for u, L, t, y in zip(U, Ls, ts, batch.unpack(Y)):
        ref = expm(-t * L) @ u
        assert np.linalg.norm(y.cpu().numpy() - ref) <= 1e-4 * np.linalg.norm(u), t
