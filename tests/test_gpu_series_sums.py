"""Truncated series of every short degree: the running sum takes its terms two at a time, in an
order that depends on the degree modulo four, for single operators, operators of mixed degrees
side by side and batches of graphs of mixed degrees; against the recurrence in float64."""

import math

import numpy as np
import pytest

import synth
from oracle import walks

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

# A row sums at most a few hundred neighbours and a result at most 9 + 1 terms: in FP32 every
# term carries at most sqrt(deg) + 4 k roundings of 6e-8, under 4e-6 of the sum of magnitudes.
TOL = {torch.float32: 1e-5, torch.float64: 1e-13}


def terms(A, X, mu, kind, param, K):
    """The terms c_k q_k X, k = 0..K."""
    D = A.sum(1)[:, None]
    P, c = [X], [1.0]
    for k in range(1, K + 1):
        Y = A @ P[-1]
        if k == 2:
            Y = Y - mu * D * P[-2]
        elif k > 2:
            Y = Y + mu * (mu - D) * P[-2]
        P.append(Y)
        c.append(param ** k / (math.factorial(k) if kind == "exp" else 1.0))
    return [ck * p for ck, p in zip(c, P)]


def phi(A, X, mu, kind, param, K):
    ts = terms(A, X, mu, kind, param, K)
    return sum(ts), sum(np.abs(t) for t in ts)


def close(got, ref, mag, dtype):
    assert np.linalg.norm(got.double().cpu().numpy() - ref) <= TOL[dtype] * np.linalg.norm(mag)


def graph(n, seed):
    rp, ci = synth.barabasi_albert(n, 6, seed)
    A = walks.adjacency(n, rp, ci)
    return rp, ci, A, float(np.linalg.eigvalsh(A)[-1])


@pytest.mark.parametrize("mu,kind", [(0.0, "res"), (0.5, "exp"), (1.0, "res")])
@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
def test_single_degrees(lib, mu, kind, dtype):
    n = 1800  # over 12000 nonzeros: not the one-workgroup series
    rp, ci, A, lam = graph(n, 3)
    param = 0.6 / lam
    g = lib.Graph(lib.Context(0), rp, ci)
    for K in range(1, 10):
        op = lib.Operator(g, mu, kind, param, dtype=dtype, krylov_dim=K, method="recurrence", rho_hint=lam)
        for b in (1, 3, 6, 16):
            X = synth.gaussian_block(n, b, seed=K)
            ref, mag = phi(A, X, mu, kind, param, K)
            Xd = torch.tensor(X, dtype=dtype, device="cuda")
            out = torch.full_like(Xd, float("nan"))  # nothing of the target is read before it is written
            close(op.apply_phi(Xd, out=out), ref, mag, dtype)
            w, wm = phi(A, np.ones((n, 1)), mu, kind, param, K)
            close(op.apply_L(Xd, out=out.fill_(float("nan"))), w * X - ref, wm * np.abs(X) + mag, dtype)


@pytest.mark.parametrize("b", [1, 4, 6, 16])
@pytest.mark.parametrize("degrees", [(1, 2, 3), (4, 4, 4), (5, 8, 7), (9, 1, 6), (2, 2, 10)])
def test_operators_of_mixed_degrees(lib, b, degrees):
    n = 1800
    rp, ci, A, lam = graph(n, 4)
    g = lib.Graph(lib.Context(0), rp, ci)
    par = [(0.0, "exp"), (0.5, "exp"), (1.0, "res")]
    ops = [lib.Operator(g, mu, kind, 0.6 / lam, krylov_dim=K, method="recurrence", rho_hint=lam)
           for (mu, kind), K in zip(par, degrees)]
    X = synth.gaussian_block(n, b, seed=b)
    Xd = torch.tensor(X, dtype=torch.float32, device="cuda")
    m = lib.Multi(ops)
    nan = torch.full((n, 3 * b), float("nan"), device="cuda")
    Yp = m.apply_phi(Xd, out=nan.clone())
    Yl = m.apply_L(Xd, out=nan.clone())
    Yf, W = m.apply_fdeg(Xd, out=nan.clone())
    for q, ((mu, kind), K) in enumerate(zip(par, degrees)):
        ref, mag = phi(A, X, mu, kind, 0.6 / lam, K)
        w, wm = phi(A, np.ones((n, 1)), mu, kind, 0.6 / lam, K)
        cols = slice(q * b, (q + 1) * b)
        close(Yp[:, cols], ref, mag, torch.float32)
        close(W[:, q:q + 1], w, wm, torch.float32)
        for Y in (Yl, Yf):
            close(Y[:, cols], w * X - ref, wm * np.abs(X) + mag, torch.float32)


@pytest.mark.parametrize("b", [1, 3, 8])
def test_batch_of_mixed_degrees(lib, b):
    sizes, degrees = [150, 64, 333, 97, 210, 128, 65, 500, 80], [1, 2, 3, 4, 5, 6, 7, 8, 9]
    ctx, graphs, descs, mats = lib.Context(0), [], [], []
    for i, (n, K) in enumerate(zip(sizes, degrees)):
        rp, ci, A, lam = graph(n, i)
        graphs.append(lib.Graph(ctx, rp, ci))
        descs.append(dict(mu=(0.0, 0.5, 1.0)[i % 3], func="exp" if i % 2 else "res", param=0.6 / lam, krylov_dim=K,
                          rho_hint=lam))
        mats.append(A)
    batch = lib.Batch(ctx, graphs, descs)
    U = [synth.gaussian_block(n, b, seed=n) for n in sizes]
    X = batch.pack([torch.tensor(u, dtype=torch.float32, device="cuda") for u in U])
    Y = batch.apply_L(X, out=torch.full_like(X, float("nan")))
    for u, A, d, K, y in zip(U, mats, descs, degrees, batch.unpack(Y)):
        ref, mag = phi(A, u, d["mu"], d["func"], d["param"], K)
        w, wm = phi(A, np.ones((len(u), 1)), d["mu"], d["func"], d["param"], K)
        close(y, w * u - ref, wm * np.abs(u) + mag, torch.float32)
