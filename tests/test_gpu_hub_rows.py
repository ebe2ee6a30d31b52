"""Products on graphs whose longest rows set the time (narrower column tiles, whole batches of
gathers in long rows) and on graphs where they do not: integer blocks, so every sum is exact."""

import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

# batches of a long row: 16 gathers on each of 256 / lanes slots (lanes 2 .. 32 a column tile)
DEGREES = [65, 127, 128, 129, 255, 256, 257, 511, 512, 513, 1023, 1024, 1025, 2047, 2048, 2049, 4999]


def graph(filler):
    rng = np.random.default_rng(5)
    n = 6000
    hubs = np.repeat(np.arange(len(DEGREES)), DEGREES)
    leaves = np.concatenate([len(DEGREES) + rng.permutation(n - len(DEGREES))[:d] for d in DEGREES])
    if filler:  # enough edges elsewhere that no row stands out
        n = 400000
        hubs = np.r_[hubs, rng.integers(6000, n, 4 * n)]
        leaves = np.r_[leaves, rng.integers(6000, n, 4 * n)]
    keep = hubs != leaves
    return synth.csr_from_edges(n, hubs[keep], leaves[keep])


@pytest.fixture(scope="module", params=["hubs", "filled", 1023, 1024])
def case(request, lib):
    if isinstance(request.param, int):
        rp, ci = synth.erdos_renyi_gnm(request.param, 20 * request.param, 3)
    else:
        rp, ci = graph(request.param == "filled")
    return lib.Graph(lib.Context(0), rp, ci), torch.tensor(rp).cuda(), torch.tensor(ci).long().cuda()


@pytest.mark.parametrize("b", [1, 2, 3, 4, 5, 6, 7, 8, 9, 13, 16, 17, 25, 30, 33, 34, 48, 50, 65, 66, 96, 100])
@pytest.mark.parametrize("dtype", [torch.float32, torch.float64], ids=["fp32", "fp64"])
def test_products_are_exact(case, b, dtype):
    g, rp, ci = case
    n = len(rp) - 1
    X = torch.randint(-50, 51, (n, b), device="cuda").to(dtype)
    Y = torch.empty_like(X)
    g.spmm(X, Y)
    d = (rp[1:] - rp[:-1]).long()
    rows = torch.repeat_interleave(torch.arange(n, device="cuda"), d)
    want = torch.zeros_like(X).index_add_(0, rows, X[ci])  # integers below 2^24: exact in any order
    assert torch.equal(Y, want)


def test_nonfinite_column_stays_in_its_column(case):
    g, rp, _ = case
    X = torch.ones(len(rp) - 1, 13, device="cuda")
    X[:, 0] = float("nan")
    X[:, 12] = float("inf")
    Y = torch.empty_like(X)
    g.spmm(X, Y)
    assert bool((Y[:, 1:12] == (rp[1:] - rp[:-1])[:, None]).all())
