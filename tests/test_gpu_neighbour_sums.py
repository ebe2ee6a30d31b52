"""Features and surrogate terms where the work per row changes: one lane or 16 a row (number of
nodes, mean degree), a workgroup for the longest."""

import numpy as np
import pytest

import synth
from oracle import features

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

N = 1 << 15  # one lane a row from here on, in sparse graphs
HUBS = [1, 63, 64, 65, 66, 511, 512, 513, 3000]


def edges(mean_deg):
    rng = np.random.default_rng(7)
    m = mean_deg * N // 2
    src = np.r_[np.repeat(np.arange(len(HUBS)), HUBS), rng.integers(4000, N - 1, m)]
    dst = np.r_[np.concatenate([20 + np.arange(d) for d in HUBS]), rng.integers(4000, N - 1, m)]
    keep = src != dst
    return src[keep], dst[keep]


@pytest.mark.parametrize("mean_deg", [0, 2, 7, 9, 13, 15])
def test_same_at_any_width(lib, mean_deg):
    """A last node without edges moves the graph to the other rule; the sums are whole numbers, so
    nothing else may change."""
    src, dst = edges(mean_deg)
    out = []
    for n in (N - 1, N):
        rp, ci = synth.csr_from_edges(n, src, dst)
        g = lib.Graph(lib.Context(0), rp, ci)
        op = lib.Operator(g, 0.5, "exp", 0.02, dtype=torch.float64)
        out.append([t[:N - 1].cpu() for t in (g.features(0.05), *op.surrogate_diag())])
        ref = features.features(n, rp, ci, 0.05)
        # one rounding to FP32 and those of FP64 log1p
        np.testing.assert_allclose(g.features(0.05).cpu().numpy(), ref, rtol=2.0**-23, atol=0)
    assert all(torch.equal(a, b) for a, b in zip(*out))
