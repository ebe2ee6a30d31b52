"""The planned workspace at sizes where the number of partial sums is rounded or falls
between two block counts: the call on a caller's region equals the allocating call."""

import pytest

import synth
from oracle import sparse

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def operator(lib, n, dtype, reorth, K, mu=0.5):
    rp, ci = synth.erdos_renyi_gnm(n, 4 * n, 3)
    lam = sparse.lambda_max(sparse.adjacency(n, rp, ci))
    return lambda: lib.Operator(lib.Graph(lib.Context(0), rp, ci), mu, "res", 0.4 / lam, dtype=dtype, krylov_dim=K,
                                reorth=reorth, rho_hint=lam)


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64], ids=["f32", "f64"])
@pytest.mark.parametrize("n,b,K", [(100, 16, 30), (100, 5, 30), (1000, 16, 30), (1500, 32, 12), (3000, 64, 8)])
def test_full_reorthogonalisation(lib, n, b, K, dtype):
    make = operator(lib, n, dtype, 2, K)
    X = torch.tensor(synth.gaussian_block(n, b, 1), dtype=dtype, device="cuda")
    ref = make().apply_phi(X)
    op = make()
    nbytes = op.workspace_size("apply_phi", b)
    work = torch.empty(nbytes, dtype=torch.uint8, device="cuda")
    assert torch.equal(op.apply_phi_ws(X, work), ref)


@pytest.mark.parametrize("n,b,dim,dtype", [(27000, 32, 40, torch.float32), (20000, 64, 30, torch.float64),
                                           (5000, 17, 33, torch.float32)])
def test_expv(lib, n, b, dim, dtype):
    make = operator(lib, n, dtype, 1, 4)
    X = torch.tensor(synth.gaussian_block(n, b, 1), dtype=dtype, device="cuda")
    (ref,), e_ref = make().expv(X, [1.0], outer_dim=dim)
    op = make()
    work = torch.empty(op.workspace_size("expv", b, dim), dtype=torch.uint8, device="cuda")
    (got,), e = op.expv_ws(X, [1.0], work, outer_dim=dim)
    assert torch.equal(got, ref) and e == e_ref
