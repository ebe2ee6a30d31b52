"""The error of a batch's return probability where a graph's Nystrom cores have no spectrum (NaN in
its block): not a certainty of zero, and the other graphs keep theirs."""

import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("b", [2, 8])
def test_error_without_a_spectrum(lib, b):
    ctx = lib.Context(0)
    graphs = [lib.Graph(ctx, *synth.barabasi_albert(n, 3, i)) for i, n in enumerate((120, 200))]
    batch = lib.Batch(ctx, graphs, [dict(mu=0.5, func="exp", param=0.1)] * 2)
    U = [synth.gaussian_block(n, b, seed=n) for n in (120, 200)]

    def run():
        packed = batch.pack([torch.tensor(u, dtype=torch.float32, device="cuda") for u in U])
        _, p, e = batch.expv(packed, [0.3, 0.3], outer_dim=20)
        return np.asarray(p, dtype=float), np.asarray(e, dtype=float)

    p, e = run()
    assert np.all(np.isfinite(p)) and np.all(e > 0)
    U[0][5, 1] = np.nan
    pn, en = run()
    assert np.isnan(en[0]) and np.isnan(pn[0])
    assert pn[1] == p[1] and en[1] == e[1]
