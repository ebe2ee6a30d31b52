"""Row counts around the 2^32 threads that one launch may have: nearly edgeless graphs with a
small graph on their last nodes, against the small graph alone."""

import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

TAIL = 700


def tail_graph(lib, ctx, n, hub=False):
    """(graph on n nodes whose last TAIL carry the edges, the same TAIL nodes alone)"""
    if hub:  # one row beyond the 16-lane groups
        rp, ci = synth.csr_from_edges(TAIL, np.r_[np.zeros(600, int), np.arange(50)], np.r_[np.arange(1, 601), np.arange(2, 52)])
    else:
        rp, ci = synth.erdos_renyi_gnm(TAIL, 2000, 3)
    big = torch.zeros(n + 1, dtype=torch.int32, device="cuda")
    big[n - TAIL:] = torch.tensor(rp, dtype=torch.int32, device="cuda")
    return lib.Graph(ctx, big, np.asarray(ci) + (n - TAIL)), lib.Graph(ctx, rp, ci)


def test_features_and_surrogate(lib):
    n = (1 << 28) + 37
    ctx = lib.Context(0)
    g, small = tail_graph(lib, ctx, n, hub=True)
    f = g.features(0.2)
    assert torch.equal(f[n - TAIL:], small.features(0.2))
    assert not f[:n - TAIL].any()
    del f
    kw = dict(dtype=torch.float32, krylov_dim=4)
    base, scale = lib.Operator(g, 0.5, "linear", 0.1, **kw).surrogate_diag()
    b0, s0 = lib.Operator(small, 0.5, "linear", 0.1, **kw).surrogate_diag()
    assert torch.equal(base[n - TAIL:], b0) and torch.equal(scale[n - TAIL:], s0)
    assert bool((base[:n - TAIL] == 1).all()) and not scale[:n - TAIL].any()


# widths whose row segment is 32 lanes below 2^27 rows
@pytest.mark.parametrize("b,dtype", [(17, torch.float32), (34, torch.float32), (17, torch.float64)], ids=str)
def test_products(lib, b, dtype):
    n = (1 << 27) + 5
    g, small = tail_graph(lib, lib.Context(0), n)
    X = torch.zeros((n, b), dtype=dtype, device="cuda")
    X[n - TAIL:] = torch.tensor(synth.gaussian_block(TAIL, b, 1), dtype=dtype, device="cuda")
    Y = g.spmm(X)
    ref = small.spmm(X[n - TAIL:].contiguous())
    tol = 1e-5 if dtype == torch.float32 else 1e-13  # sums of about 6 neighbours in another order
    assert (Y[n - TAIL:] - ref).abs().max() <= tol * ref.abs().max()
    assert not Y[:n - TAIL].any()
