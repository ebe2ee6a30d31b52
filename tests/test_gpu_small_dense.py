"""Small dense graphs on both sides of the counts of long rows up to which one workgroup evaluates
them, against the general path (which profiling keeps)."""

import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def ring(n, longs):
    """32 neighbours a node, 33 for the first `longs` (an even number)."""
    i = np.arange(n)
    src = np.concatenate([i] * 16 + [np.arange(longs // 2)])
    dst = np.concatenate([(i + k) % n for k in range(1, 17)] + [np.arange(longs // 2) + longs // 2])
    return synth.csr_from_edges(n, src, dst)


@pytest.mark.parametrize("kind,n,longs,b", [
    ("exp", 350, 40, 1), ("exp", 350, 42, 3), ("exp", 350, 80, 1), ("exp", 350, 82, 4),
    ("res", 600, 400, 1), ("res", 600, 402, 1), ("res", 600, 500, 1), ("res", 600, 502, 1),
    ("res", 600, 100, 2), ("res", 600, 102, 2), ("res", 600, 200, 2), ("res", 600, 202, 2),
    ("res", 600, 50, 4), ("res", 600, 52, 4), ("res", 600, 100, 4), ("res", 600, 102, 4)])
def test_small_equals_general(lib, kind, n, longs, b):
    rp, ci = ring(n, longs)
    assert (np.diff(rp) > 32).sum() == longs
    X = synth.gaussian_block(n, b, seed=b)
    for dtype, tol in ((torch.float64, 1e-11), (torch.float32, 2e-5)):
        out = []
        for profiled in (False, True):
            ctx = lib.Context(0)
            ctx.set_profiling(profiled)
            kw = dict(rho_hint=33.0) if kind == "res" else {}
            op = lib.Operator(lib.Graph(ctx, rp, ci), 0.5, kind, 0.5 / 33, dtype=dtype, krylov_dim=30, **kw)
            out.append(op.apply_phi(torch.tensor(X, dtype=dtype, device="cuda")).cpu().numpy().astype(np.float64))
        assert np.linalg.norm(out[0] - out[1]) <= tol * np.linalg.norm(out[1])
