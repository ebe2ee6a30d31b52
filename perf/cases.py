"""Cases for timing the walk-Laplacian library through its public entry points.

Every case is a dict of plain values.  `prepare` draws the graph and the blocks of one
case on the GPU from a seed and makes the handles a program keeps (graph, operator,
network); `run` is one pass; `exact` gives the same outputs in 64 bits from plain torch.

The kinds of work (field "kind"):
  call   one operator from end to end: walk degrees, L X and exp(-t L) U0
  apply  L X of one operator (block Lanczos for the resolvent, series for the exponential)
  multi  five exponential operators side by side, L X and walk degrees in one evaluation
  expv   exp(-t L) U0 for three times from one Krylov basis
  batch  diffusion on many graphs of uneven size in one call
  rprob  average return probabilities by the rational Krylov method
  amg    phi X by multigrid-preconditioned conjugate gradients in double precision
  diag   the control-variate diagonal estimator: features, network, probe products, estimate
  train  loss and gradients of the control-variate network on a training set
"""

import math

import numpy as np
import torch

import paper_2601_11338_amd as wl

MUS = (0.0, 0.25, 0.5, 0.75, 1.0)
TIMES = (0.1, 1.0, 10.0)
SHAPES = ((64, 8), (64,), (64, 64), (64,), (1, 64), (1,))  # the network's parameters, in order


# ------------------------------------------------------------------ the cases
def listed():
    return [
        # the smallest call: an Erdos-Renyi graph of 1000 nodes in double precision, one
        # vector at a time (latency and launches)
        dict(name="er1k-call-fp64", kind="call", graph="er", n=1000, deg=8, b=1, f64=True, func="res", mu=0.0, steps=40),
        # a small network, an odd block width
        dict(name="ba5k-res-b5", kind="apply", graph="ba", n=5000, deg=5, b=5, f64=False, func="res", mu=0.5, steps=30),
        # the headline graph: one nonbacktracking resolvent operator on 16 columns
        dict(name="ba1m-res-b16", kind="apply", graph="ba", n=1000000, deg=5, b=16, f64=False, func="res", mu=1.0,
             steps=30),
        # the headline graph: the five exponential operators and their walk degrees
        dict(name="ba1m-exp5-b16", kind="multi", graph="ba", n=1000000, deg=5, b=16, steps=30),
        # double precision on a medium network (the library's tightest tolerance)
        dict(name="ba200k-res-fp64-b8", kind="apply", graph="ba", n=200000, deg=5, b=8, f64=True, func="res", mu=0.5,
             steps=30),
        # 30 probe columns (the paper's number) on an odd number of nodes: a width that is no
        # power of two
        dict(name="er100k-res-b30", kind="apply", graph="er", n=100003, deg=10, b=30, f64=False, func="res", mu=0.25,
             steps=30),
        # diffusion of 32 sparse initial conditions for three times
        dict(name="rmat18-expv-b32", kind="expv", graph="rmat", n=1 << 18, deg=16, b=32, f64=False, func="exp", mu=0.5,
             steps=11, dim=40),
        # many graphs of uneven size, mixed variants and times, 8 probes each
        dict(name="batch64-b8", kind="batch", count=64, n=50000, deg=10, b=8, dim=30),
        # average return probabilities on a road-like lattice, 30 probes, 90 times
        dict(name="road400-rprob-m30", kind="rprob", graph="road", n=400 * 400, b=30, times=90),
        # the resolvent close to its radius of convergence, by multigrid-preconditioned CG
        dict(name="road700-amg-b16", kind="amg", graph="road", n=700 * 700, b=16, frac=0.9),
        # the learned control variate: one evaluation on a new graph's probes
        dict(name="rmat19-diag-m64", kind="diag", graph="rmat", n=1 << 19, deg=16, b=64, f64=False, func="exp", mu=0.5,
             steps=12),
        # one full-batch pass of the network's training
        dict(name="mlp-train-200k", kind="train", n=204800),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(("call", "apply", "apply", "apply", "multi", "expv", "batch", "rprob", "amg", "diag", "train"))
    mu = rng.choice(MUS)
    if kind == "call":
        return dict(kind=kind, graph=rng.choice(("er", "ba")), n=_log(rng, 300, 20000), deg=rng.choice((3, 5, 8)),
                    b=rng.choice((1, 1, 2, 3, 4)), f64=True, func=rng.choice(("res", "exp")), mu=mu, steps=40)
    if kind == "apply":
        n, f64 = _log(rng, 1000, 1000000), rng.random() < 0.4
        b = min(_log(rng, 1, 64), max(1, (8000000 if f64 else 16000000) // n))
        func = rng.choice(("res", "res", "exp"))
        graph = rng.choice(("ba", "er", "rmat") if func == "exp" else ("ba", "er"))
        return dict(kind=kind, graph=graph, n=n, deg=5 if graph == "ba" else 10, b=b, f64=f64, func=func, mu=mu, steps=30)
    if kind == "multi":
        n = _log(rng, 20000, 1000000)
        return dict(kind=kind, graph="ba", n=n, deg=5, b=rng.choice((4, 8, 12, 16)), steps=rng.choice((12, 20, 30)))
    if kind == "expv":
        n = _log(rng, 5000, 1 << 17)
        return dict(kind=kind, graph=rng.choice(("rmat", "ba")), n=n, deg=8, b=rng.choice((3, 8, 16, 20, 32)), f64=False,
                    func="exp", mu=mu, steps=11, dim=40)
    if kind == "batch":
        return dict(kind=kind, count=rng.randint(16, 64), n=_log(rng, 4000, 50000), deg=10, b=rng.choice((4, 6, 8)), dim=30)
    if kind == "rprob":
        side = _log(rng, 60, 400)
        return dict(kind=kind, graph="road", n=side * side, b=rng.choice((10, 16, 20, 30)), times=90)
    if kind == "amg":
        side = _log(rng, 60, 700)
        return dict(kind=kind, graph="road", n=side * side, b=rng.choice((1, 4, 8, 16)), frac=rng.choice((0.3, 0.6, 0.9)))
    if kind == "diag":
        return dict(kind=kind, graph="rmat", n=_log(rng, 5000, 1 << 19), deg=rng.choice((8, 16)), b=rng.choice((16, 24, 64)),
                    f64=False, func="exp", mu=mu, steps=12)
    return dict(kind="train", n=_log(rng, 2000, 204800))


# ------------------------------------------------------------------ graphs
def _csr(n, u, v):
    """Symmetric CSR of an undirected edge list, loops and duplicates dropped."""
    keep = u != v
    u, v = u[keep], v[keep]
    lo, hi = torch.minimum(u, v), torch.maximum(u, v)
    key = torch.unique(lo * n + hi)
    lo, hi = key // n, key % n
    key, _ = torch.sort(torch.cat([lo * n + hi, hi * n + lo]))
    rowptr = torch.zeros(n + 1, dtype=torch.int64, device=key.device)
    rowptr[1:] = torch.cumsum(torch.bincount(key // n, minlength=n), 0)
    return rowptr.to(torch.int32), (key % n).to(torch.int32)


def _uniform(n, edges, gen):
    """Erdos-Renyi: `edges` uniform node pairs."""
    u, v = torch.randint(0, n, (2, edges), generator=gen, device="cuda")
    return _csr(n, u, v)


def _attach(n, m, gen):
    """Barabasi-Albert: a clique of m + 1 nodes, then m links per node to the endpoint found
    at a uniform place of the list of all earlier endpoints (chains of links followed by
    pointer jumping)."""
    m0 = m + 1
    cu, cv = torch.triu_indices(m0, m0, 1, device="cuda")
    first = 2 * cu.numel()
    t = torch.arange(m0, n, device="cuda").repeat_interleave(m)
    place = (torch.rand(t.numel(), generator=gen, device="cuda", dtype=torch.float64) * (first + 2 * m * (t - m0))).long()
    ends = torch.stack([cu, cv], 1).flatten()
    q = (place - first) // 2
    new = place >= first
    linked = new & ((place - first) % 2 == 1)
    node = torch.where(new, m0 + torch.div(q.clamp(min=0), m, rounding_mode="floor"), ends[place.clamp(max=first - 1)])
    link = torch.where(linked, q, torch.arange(t.numel(), device="cuda"))
    for _ in range(64):
        nxt = link[link]
        if torch.equal(nxt, link):
            break
        link = nxt
    return _csr(n, torch.cat([cu, t]), torch.cat([cv, node[link]]))


def _rmat(n, edges, gen):
    """R-MAT (a, b, c = 0.57, 0.19, 0.19) folded onto n nodes and relabelled."""
    scale = max(1, math.ceil(math.log2(n)))
    u = torch.zeros(edges, dtype=torch.int64, device="cuda")
    v = torch.zeros_like(u)
    for _ in range(scale):
        r = torch.rand(edges, generator=gen, device="cuda")
        u = 2 * u + (r >= 0.76)
        v = 2 * v + (((r >= 0.57) & (r < 0.76)) | (r >= 0.95))
    perm = torch.randperm(1 << scale, generator=gen, device="cuda") % n
    return _csr(n, perm[u], perm[v])


def _road(n, gen):
    """Square lattice with each edge kept with probability 0.7."""
    side = math.isqrt(n)
    at = torch.arange(side * side, device="cuda").view(side, side)
    u = torch.cat([at[:, :-1].flatten(), at[:-1].flatten()])
    v = torch.cat([at[:, 1:].flatten(), at[1:].flatten()])
    keep = torch.rand(u.numel(), generator=gen, device="cuda") < 0.7
    return _csr(side * side, u[keep], v[keep])


def _blocks(n, deg, gen, k):
    """Stochastic block model: k equal blocks, edges 20 times likelier inside a block."""
    edges = n * deg // 2
    u, v = torch.randint(0, n, (2, edges), generator=gen, device="cuda")
    inside = torch.rand(edges, generator=gen, device="cuda") < 20.0 / (20.0 + k - 1)
    size = n // k
    w = (u // size * size + v % size).clamp(max=n - 1)
    return _csr(n, u, torch.where(inside, w, v))


def _powerlaw(n, gen):
    """Configuration model: degrees with exponent 2.5 between 2 and sqrt(n)."""
    d = 2.0 * (1.0 - torch.rand(n, generator=gen, device="cuda")) ** (-1.0 / 1.5)
    d = d.clamp(max=math.sqrt(n)).long()
    stubs = torch.arange(n, device="cuda").repeat_interleave(d)
    stubs = stubs[torch.randperm(stubs.numel(), generator=gen, device="cuda")]
    half = stubs.numel() // 2
    return _csr(n, stubs[:half], stubs[half:2 * half])


def _draw_graph(case, gen):
    n = case["n"]
    if case["graph"] == "er":
        return _uniform(n, n * case["deg"] // 2, gen)
    if case["graph"] == "ba":
        return _attach(n, case["deg"], gen)
    if case["graph"] == "rmat":
        return _rmat(n, n * case["deg"], gen)
    return _road(n, gen)


def _adjacency(rp, ci):
    ones = torch.ones(ci.numel(), dtype=torch.float64, device="cuda")
    return torch.sparse_csr_tensor(rp.long(), ci.long(), ones, (rp.numel() - 1, rp.numel() - 1))


def _scale(rp, ci):
    """The adjacency's largest eigenvalue to a few per cent, by power iterations (six digits
    kept, so that the parameter is a plain number)."""
    A, x = _adjacency(rp, ci), torch.ones((rp.numel() - 1, 1), dtype=torch.float64, device="cuda")
    for _ in range(20):
        x = x / x.norm()
        y = A @ x
        lam, x = float((x * y).sum()), y
    return float("%.6g" % lam)


def _param(case, rp, ci):
    """(weight parameter, bound on the spectral radius) of the case's operator."""
    if case["graph"] == "road":  # degrees up to 4: rho(Z_1) <= 3
        return (0.285 if case["kind"] == "rprob" else case["frac"] / 3.0), 3.0
    lam = _scale(rp, ci)
    return (0.5 if case.get("func") == "res" else 1.0) / lam, 1.5 * lam


def _gen(seed, salt=0):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(1000003 * seed + salt)
    return gen


def _normal(n, b, gen, dtype):
    return torch.randn((n, b), generator=gen, device="cuda", dtype=torch.float64).to(dtype)


def _signs(n, b, gen, dtype):
    return torch.randint(0, 2, (n, b), generator=gen, device="cuda").to(dtype) * 2 - 1


def _spots(n, b, gen, dtype):
    """b distributions of 16 random nodes each."""
    U = torch.zeros((n, b), dtype=dtype, device="cuda")
    for j in range(b):
        U[torch.randperm(n, generator=gen, device="cuda")[:16], j] = 1.0 / 16
    return U


def _members(case, gen):
    """The batch's graphs: sizes log-uniform from 1000 to n, block models and power laws."""
    sizes = [int(1000 * (case["n"] / 1000.0) ** ((0.5 + 0.6180339887 * i) % 1.0)) for i in range(case["count"])]
    csrs = [_blocks(n, case["deg"], gen, 4 + 7 * i % 29) if i % 2 == 0 else _powerlaw(n, gen) for i, n in enumerate(sizes)]
    descs, ts = [], []
    for i, (rp, ci) in enumerate(csrs):
        res = (i // 5) % 2 == 1
        lam = _scale(rp, ci)
        descs.append(dict(mu=MUS[i % 5], func="res" if res else "exp", param=(0.5 if res else 1.0) / lam,
                          krylov_dim=25 if res else 11, rho_hint=1.5 * lam))
        ts.append(TIMES[i % 3])
    return csrs, descs, ts


def _network(gen):
    """Glorot-initialised parameters, flat in the library's order."""
    out = []
    for s in SHAPES:
        w = torch.randn(s, generator=gen, device="cuda") * math.sqrt(2.0 / sum(s)) if len(s) == 2 else torch.zeros(s, device="cuda")
        out.append(w.flatten())
    return torch.cat(out).cpu().numpy().astype(np.float32)


def _inputs(case, seed):
    """What a case draws from its seed: CSR arrays and blocks."""
    gen = _gen(seed)
    if case["kind"] == "train":
        F = torch.rand((case["n"], 8), generator=gen, device="cuda")
        T = torch.tanh(F.sum(1) - 4.0) * 0.5 + 0.05 * torch.randn(case["n"], generator=gen, device="cuda")
        return dict(F=F, T=T, theta=_network(gen))
    if case["kind"] == "batch":
        csrs, descs, ts = _members(case, gen)
        return dict(csrs=csrs, descs=descs, ts=ts, blocks=[_normal(rp.numel() - 1, case["b"], gen, torch.float32) for rp, _ in csrs])
    rp, ci = _draw_graph(case, gen)
    n, b = rp.numel() - 1, case["b"]
    dtype = torch.float64 if case.get("f64") or case["kind"] == "amg" else torch.float32
    d = dict(rp=rp, ci=ci, dtype=dtype)
    if case["kind"] in ("apply", "multi", "diag"):
        d["X"] = _signs(n, b, gen, dtype)
    elif case["kind"] == "expv":
        d["X"] = _spots(n, b, gen, dtype)
    else:
        d["X"] = _normal(n, b, gen, dtype)
    if case["kind"] == "call":
        d["U"] = torch.zeros((n, b), dtype=dtype, device="cuda")
        d["U"][torch.arange(b, device="cuda") * 7 % n, torch.arange(b, device="cuda")] = 1.0
    if case["kind"] == "diag":
        d["theta"] = _network(gen)
    return d


# ------------------------------------------------------------------ passes
def prepare(case, seed):
    s = dict(case=case, **_inputs(case, seed))
    ctx = s["ctx"] = wl.Context(0)
    kind = case["kind"]
    if kind == "train":
        s["net"] = wl.MLP(ctx, s["theta"])
        return s
    if kind == "batch":
        s["graphs"] = [wl.Graph(ctx, rp, ci) for rp, ci in s["csrs"]]
        s["batch"] = wl.Batch(ctx, s["graphs"], s["descs"])
        s["U"] = s["batch"].pack(s["blocks"])
        return s
    g = s["graph"] = wl.Graph(ctx, s["rp"], s["ci"])
    param, bound = _param(case, s["rp"], s["ci"])
    s["param"] = param
    if kind == "multi":
        s["ops"] = [wl.Operator(g, mu, "exp", param, dtype=s["dtype"], krylov_dim=case["steps"]) for mu in MUS]
        s["multi"] = wl.Multi(s["ops"])
    elif kind == "rprob":
        s["op"] = wl.Operator(g, 1.0, "res", param, dtype=s["dtype"], tol=1e-7, rho_hint=bound)
        s["ts"] = np.linspace(0.0, 100.0, case["times"])
    elif kind == "amg":
        s["op"] = wl.Operator(g, 1.0, "res", param, dtype=s["dtype"], method="amg", rho_hint=bound)
    else:
        s["op"] = wl.Operator(g, case["mu"], case["func"], param, dtype=s["dtype"], krylov_dim=case["steps"],
                              rho_hint=bound if case["func"] == "res" else 0.0)
    if kind == "diag":
        s["net"] = wl.MLP(ctx, s["theta"])
    return s


def run(s):
    case, kind = s["case"], s["case"]["kind"]
    if kind == "call":
        return dict(w=s["op"].fdeg(), LX=s["op"].apply_L(s["X"]), U=s["op"].expv(s["U"], [1.0])[0][0])
    if kind == "apply":
        return s["op"].apply_L(s["X"])
    if kind == "multi":
        return s["multi"].apply_fdeg(s["X"])
    if kind == "expv":
        return s["op"].expv(s["X"], TIMES, outer_dim=case["dim"])[0]
    if kind == "batch":
        Y, p, _ = s["batch"].expv(s["U"], s["ts"], outer_dim=case["dim"])
        return dict(Y=s["batch"].unpack(Y)[:60], p=p.astype(np.float32))  # (blocks in 32 bits, so their traces too)
    if kind == "rprob":
        p, _, _, _ = s["op"].return_prob(s["X"], s["ts"], 100.0)
        return p.astype(np.float32)  # from probe blocks in 32 bits
    if kind == "amg":
        return s["op"].apply_phi(s["X"])
    if kind == "diag":
        base, scale = s["op"].surrogate_diag()
        feat = s["graph"].features(s["param"])
        cv = s["net"].predict(feat, base, scale)
        Y = s["op"].apply_phi(s["X"])
        diag, trace, _ = wl.estimate(s["ctx"], s["X"], Y, cv=cv)
        return dict(features=feat, cv=cv, Y=Y, diag=diag, trace=np.float32(trace))
    loss, grad = s["net"].loss_grad(s["F"], s["T"])
    return dict(loss=np.float32(loss), grad=grad.astype(np.float32))  # the network computes in 32 bits


# ------------------------------------------------------------------ what a pass cannot do without
def work(case):
    kind, n = case["kind"], case["n"]
    if kind == "train":
        return dict(bytes=36.0 * n, flops=3 * 2.0 * n * (8 * 64 + 64 * 64 + 64))
    b, size = case["b"], 8 if case.get("f64") or kind == "amg" else 4
    if kind == "batch":  # mean of a log-uniform size, 10 neighbours
        n = case["count"] * (n - 1000) / math.log(n / 1000.0)
        nnz, products = 8.0 * n, case["dim"] * 18
    else:
        nnz = n * dict(er=case.get("deg", 0), ba=2 * case.get("deg", 0), rmat=1.8 * case.get("deg", 0), road=2.8)[case["graph"]]
        products = dict(call=2 + 30, apply=1, multi=1, expv=case.get("dim", 0), rprob=600.0 / 27, amg=10.0 / 27, diag=1)[kind]
        products *= case.get("steps", 27)
    width = b * 5 + 5 if kind == "multi" else b
    one = 4.0 * nnz + 4.0 * n + 2.0 * size * n * width  # the graph, the block read and the block written
    return dict(bytes=products * one, flops=2.0 * products * nnz * width)


# ------------------------------------------------------------------ 64-bit values
class _Walk:
    """phi and L of one operator, or of a block-diagonal union with weights per row, in
    double precision: q_{k+1} = A q_k + mu (mu - D) q_{k-1}, phi = sum_k c_k q_k."""

    def __init__(self, rp, ci, mu, param, exp):
        rp, ci = rp.long(), ci.long()
        self.n = rp.numel() - 1
        self.A = _adjacency(rp, ci)
        row = lambda v: torch.as_tensor(v, dtype=torch.float64, device="cuda").reshape(-1, 1)  # noqa: E731
        self.deg, self.mu, self.s, self.exp = (rp[1:] - rp[:-1]).double().view(-1, 1), row(mu), row(param), row(exp)
        self.w = self.phi(torch.ones((self.n, 1), dtype=torch.float64, device="cuda"))

    def phi(self, X):
        P0, P1, S, c = X, self.s * (self.A @ X), X.clone(), torch.ones_like(self.exp)
        for k in range(1, 400):
            c = torch.where(self.exp > 0, c / k, c)
            S += c * P1
            if float((c * P1).abs().max()) <= 1e-17 * float(S.abs().max()):
                break
            P2 = self.s * (self.A @ P1) - self.s ** 2 * self.mu * self.deg * P0
            if k > 1:
                P2 += self.s ** 2 * self.mu ** 2 * P0
            P0, P1 = P1, P2
        return S

    def lap(self, X):
        return self.w * X - self.phi(X)

    def diffuse(self, U, ts, group=None):
        """exp(-t L) U by Chebyshev polynomials on [0, 2 max w]; `ts`: the times (one output
        each), or with `group` (graph of each row) one time per graph and one output."""
        if group is None:
            top = torch.full((1,), 2.0 * float(self.w.max()), dtype=torch.float64, device="cuda")
        else:
            top = torch.zeros(len(ts), dtype=torch.float64, device="cuda").scatter_reduce(0, group, 2.0 * self.w[:, 0], "amax")
        tops = top.tolist() if group is not None else top.tolist() * len(ts)
        nodes = int(8 + max(2.0 * math.sqrt(25.0 * t * r) + t * r / 8 for t, r in zip(ts, tops)))
        th = (np.arange(nodes) + 0.5) * math.pi / nodes
        co = np.array([[2.0 / nodes * np.sum(np.exp(-t * r / 2 * (np.cos(th) + 1)) * np.cos(k * th)) for k in range(nodes)]
                       for t, r in zip(ts, tops)])
        co[:, 0] /= 2
        last = int(np.nonzero(np.abs(co).max(0) > 1e-17)[0][-1]) + 1
        two = (2.0 / top[group if group is not None else 0]).reshape(-1, 1)
        C = torch.as_tensor(co, device="cuda")
        pick = (lambda k: [C[group, k].view(-1, 1)]) if group is not None else (lambda k: [C[i, k] for i in range(len(ts))])
        T0, T1 = U, two * self.lap(U) - U
        out = [c0 * T0 + c1 * T1 for c0, c1 in zip(pick(0), pick(1))]
        for k in range(2, last):
            T0, T1 = T1, 2.0 * (two * self.lap(T1) - T1) - T0
            for o, c in zip(out, pick(k)):
                o += c * T1
        return out


def _exact_batch(d):
    sizes = [rp.numel() - 1 for rp, _ in d["csrs"]]
    off = np.cumsum([0] + sizes)
    nz = np.cumsum([0] + [ci.numel() for _, ci in d["csrs"]])
    rp = torch.cat([d["csrs"][0][0][:1].long()] + [r[1:].long() + int(z) for (r, _), z in zip(d["csrs"], nz)])
    ci = torch.cat([c.long() + int(o) for (_, c), o in zip(d["csrs"], off)])
    group = torch.arange(len(sizes), device="cuda").repeat_interleave(torch.tensor(sizes, device="cuda"))
    per = lambda f: torch.tensor([f(x) for x in d["descs"]], dtype=torch.float64, device="cuda")[group]  # noqa: E731
    walk = _Walk(rp, ci, per(lambda x: x["mu"]), per(lambda x: x["param"]), per(lambda x: x["func"] == "exp"))
    Y = walk.diffuse(torch.cat(d["blocks"]).double(), d["ts"], group)[0]
    return dict(Y=[Y[a:b] for a, b in zip(off[:-1], off[1:])][:60], p=None)


def _exact_train(d):
    th, at, P = torch.as_tensor(d["theta"], device="cuda").double(), 0, []
    th.requires_grad_(True)
    for s in SHAPES:
        size = math.prod(s)
        P.append(th[at:at + size].view(s))
        at += size
    h = torch.tanh(d["F"].double() @ P[0].T + P[1])
    h = torch.tanh(h @ P[2].T + P[3])
    loss = ((h @ P[4].T + P[5])[:, 0] - d["T"].double()).square().mean()
    loss.backward()
    return dict(loss=float(loss), grad=th.grad)


def exact(case, seed):
    d, kind = _inputs(case, seed), case["kind"]
    if kind == "train":
        return _exact_train(d)
    if kind == "batch":
        return _exact_batch(d)
    if kind == "rprob":  # a quotient of leave-one-out traces of an approximate exponential
        return None
    if kind == "multi":
        param, X = _param(case, d["rp"], d["ci"])[0], d["X"].double()
        walks = [_Walk(d["rp"], d["ci"], mu, param, 1.0) for mu in MUS]
        return torch.cat([k.lap(X) for k in walks], 1), torch.cat([k.w for k in walks], 1)
    X = d["X"].double()
    walk = _Walk(d["rp"], d["ci"], case.get("mu", 1.0), _param(case, d["rp"], d["ci"])[0], float(case.get("func") == "exp"))
    if kind == "amg" or kind == "diag":  # phi of the resolvent is (1 - mu^2 a^2) A_mu(a)^-1 = sum a^k q_k
        Y = walk.phi(X)
        return Y if kind == "amg" else dict(features=None, cv=None, Y=Y, diag=None, trace=None)
    if kind == "apply":
        return walk.lap(X)
    if kind == "call":
        return dict(w=walk.w[:, 0], LX=walk.lap(X), U=walk.diffuse(d["U"].double(), [1.0])[0])
    return walk.diffuse(X, TIMES)
