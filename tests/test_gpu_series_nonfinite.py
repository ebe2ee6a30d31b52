"""An infinite entry stays on the nodes its walks reach: an isolated node's row of phi X is the
row of X, whatever it holds, and the rows that no walk from it reaches are untouched."""

import numpy as np
import pytest

import synth
from synth.graphs import csr_from_edges

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64], ids=["f32", "f64"])
@pytest.mark.parametrize("b", [1, 2, 3, 4, 16])
@pytest.mark.parametrize("beta", [0.05, 0.1, 0.15, 0.2, 0.25])
def test_infinite_row_of_an_isolated_node(lib, dtype, b, beta):
    n = 3000  # beyond the one-workgroup evaluations
    i = np.arange(n - 2)
    rp, ci = csr_from_edges(n, np.concatenate([i[:-1], i[:-7]]), np.concatenate([i[1:], i[7:]]))
    op = lib.Operator(lib.Graph(lib.Context(0), rp, ci), 0.0, "exp", beta, dtype=dtype)
    X = synth.gaussian_block(n, b, seed=1)
    clean = op.apply_phi(torch.tensor(X, dtype=dtype, device="cuda")).cpu().numpy()
    X[n - 1, 0] = np.inf
    got = op.apply_phi(torch.tensor(X, dtype=dtype, device="cuda")).cpu().numpy()
    clean[n - 1, 0] = np.inf
    assert np.array_equal(got, clean)
