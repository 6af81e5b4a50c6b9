"""Performance cases of the framework's public entry points.

Each case is one pass of work that a program using this package has it do:
solve calls on one problem (resident, launch-bound and large, orthant and
Lorentz cones, FP64 and mixed precision), many small problems in one launch,
a parametric family, the standard-ADMM baseline, and the learned warm start's
basis fit and training.  Problems follow the repository's generators (k
nonzeros per column at distinct uniform rows, or a uniform density; b and c
from a primal-dual pair), drawn on the GPU from the seed alone.

The stopping tolerance is zero throughout, so that a pass is a fixed number
of iterations with a check every ten, as in a run that has not converged yet.
Results of the mixed-precision forms are single-precision results and are
handed on in that type.
"""
import math

import numpy as np
import torch

from paper_2203_05027_amd import learn
from paper_2203_05027_amd import solver as S

DEV = "cuda"


# ---------------------------------------------------------------------------
# The cases
# ---------------------------------------------------------------------------
def listed():
    return [
        # a small LP solved in one call that allocates nothing: the latency of a serving loop whose A, b and c are new each time
        dict(name="one call 150x331", kind="call", m=150, n=331, k=5, precision="fp64", iters=100),
        # the small LP of the repository's benchmark: a kept handle, iterations held in one compute unit
        dict(name="lp 500x1000", kind="lp", m=500, n=1000, k=5, precision="fp64", iters=1000),
        # an ordinary LP, too big for one compute unit and small enough that launches count; mixed precision
        dict(name="lp 6007x12011 mixed", kind="lp", m=6007, n=12011, k=7, precision="mixed", iters=1000),
        # the benchmark's headline: the 1e6 x 2e6 LP in FP64
        dict(name="lp 1e6x2e6", kind="lp", m=1_000_000, n=2_000_000, k=10, precision="fp64", iters=400),
        # a large LP in mixed precision at sizes that are no multiples of anything
        dict(name="lp 600011x1350007 mixed", kind="lp", m=600_011, n=1_350_007, k=9, precision="mixed", iters=400),
        # the SOCP workload: 1e5 Lorentz cones of sizes 3 to 50
        dict(name="socp 1e5 cones", kind="socp", cones=100_000, orth=0, k=8, precision="fp64", iters=150),
        # the experiments' own generator at 0.5 % density: long rows, vectors that fit the caches
        dict(name="paper lp 0.5%", kind="paper", m=20_000, n=100_000, density=0.005, cone="lp", precision="fp64", iters=400),
        # many LPs of mixed sizes in one persistent launch
        dict(name="batch 1024", kind="batch", count=1024, lo=50, hi=5000, k=6, precision="mixed", iters=1000),
        # one A, 256 right-hand sides, started from predicted points on the device
        dict(name="family 256", kind="family", m=50_000, n=100_000, k=8, B=256, nb=256, precision="mixed", iters=100),
        # the baseline: standard ADMM with two warm-started CG steps per iteration
        dict(name="standard cg 400kx800k", kind="standard", m=400_000, n=800_000, k=10, cg=2, iters=60),
        # training the warm start's network: eight Adam steps and the weights afterwards
        dict(name="mlp train 64-512-512-256", kind="mlp", din=64, hid=512, layers=3, dout=256, batch=256, iters=8),
        # the warm start's basis: a PCA fit of solutions, their coefficients and their reconstruction
        dict(name="pca 2000x30000", kind="pca", N=2000, D=30_000, k=96),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["call", "lp", "lp", "lp", "socp", "paper", "batch", "family", "standard", "mlp", "pca"])
    precision = rng.choice(["fp64", "mixed"])
    if kind == "call":
        m = _log(rng, 20, 300)
        return dict(kind=kind, m=m, n=int(m * rng.uniform(1.3, 2.2)), k=rng.randint(3, 6), precision=precision,
                    iters=rng.randint(20, 400))
    if kind == "lp":  # the range is wide: from one compute unit to the whole chip
        m = _log(rng, 100, 900_000)
        return dict(kind=kind, m=m, n=int(m * rng.uniform(1.3, 2.2)), k=rng.randint(4, 10), precision=precision,
                    iters=rng.randint(100, 400) if m > 50_000 else rng.randint(200, 1000))
    if kind == "socp":
        return dict(kind=kind, cones=_log(rng, 500, 90_000), orth=rng.choice([0, 0, _log(rng, 100, 100_000)]),
                    k=rng.randint(4, 8), precision=precision, iters=rng.randint(50, 150))
    if kind == "paper":
        m = _log(rng, 2000, 20_000)
        return dict(kind=kind, m=m, n=4 * (m * rng.randint(3, 5) // 4), density=rng.choice([0.001, 0.005, 0.01]) *
                    (0.9 if m > 14_000 else 1.0), cone=rng.choice(["lp", "socp"]), precision=precision,
                    iters=rng.randint(100, 300))
    if kind == "batch":
        lo = _log(rng, 20, 500)
        return dict(kind=kind, count=_log(rng, 32, 1000), lo=lo, hi=rng.randint(lo, 5000), k=rng.randint(3, 6),
                    precision=precision, iters=rng.randint(200, 900))
    if kind == "family":
        m, B = _log(rng, 2000, 50_000), 64 * rng.randint(1, 4)
        return dict(kind=kind, m=m, n=int(m * rng.uniform(1.5, 2.0)), k=rng.randint(4, 8), B=B,
                    nb=rng.randint(B // 2 + 1, B), precision=precision, iters=rng.randint(30, 80))
    if kind == "standard":
        m = _log(rng, 2000, 400_000)
        return dict(kind=kind, m=m, n=int(m * rng.uniform(1.9, 2.2)), k=rng.randint(5, 10), cg=rng.randint(1, 3),
                    iters=rng.randint(20, 60))
    if kind == "mlp":
        return dict(kind=kind, din=16 * rng.randint(2, 8), hid=16 * _log(rng, 8, 64), layers=rng.randint(2, 4),
                    dout=16 * _log(rng, 4, 32), batch=16 * _log(rng, 4, 32), iters=rng.randint(4, 10))
    return dict(kind=kind, N=_log(rng, 300, 2000), D=_log(rng, 3000, 30_000), k=rng.randint(16, 96))


# ---------------------------------------------------------------------------
# Problems, drawn on the GPU
# ---------------------------------------------------------------------------
def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed))
    return g


def _randn(g, *shape):
    return torch.randn(*shape, generator=g, device=DEV, dtype=torch.float64)


def _rand(g, *shape):
    return torch.rand(*shape, generator=g, device=DEV, dtype=torch.float64)


def _distinct(g, size, k):
    """k distinct sorted row numbers in [0, size[j]) for each column j."""
    size = size[:, None]

    def new(shape_like):
        return (_rand(g, *shape_like.shape) * size).long().clamp_(max=size - 1)

    rows = new(torch.empty(size.shape[0], k)).sort(1).values
    while True:
        dup = torch.zeros_like(rows, dtype=torch.bool)
        dup[:, 1:] = rows[:, 1:] == rows[:, :-1]
        if not bool(dup.any()):
            return rows
        rows = torch.where(dup, new(rows), rows).sort(1).values


class _Sparse:
    """A in coordinate form, sorted by row and then column, on the GPU."""

    def __init__(self, m, n, row, col, val):
        key = row * n + col
        key, at = key.sort()
        self.m, self.n, self.val = m, n, val[at]
        self.row, self.col = key // n, key % n
        self.ptr = torch.zeros(m + 1, dtype=torch.int64, device=DEV)
        self.ptr[1:] = torch.bincount(self.row, minlength=m).cumsum(0)

    def forms(self):
        """Padded row and column forms (indices, values), for plain products."""
        rows = _padded(self.m, self.row, self.col, self.val)
        at = (self.col * self.m + self.row).argsort()
        return rows, _padded(self.n, self.col[at], self.row[at], self.val[at])

    def host(self):
        return self.ptr.cpu().numpy(), self.col.int().cpu().numpy(), self.val.cpu().numpy()


def _padded(count, seg, idx, val):
    cnt = torch.bincount(seg, minlength=count)
    first = cnt.cumsum(0) - cnt
    w = max(int(cnt.max()), 1)
    at = seg * w + (torch.arange(seg.numel(), device=DEV) - first[seg])
    i = torch.zeros(count * w, dtype=torch.int64, device=DEV)
    v = torch.zeros(count * w, dtype=torch.float64, device=DEV)
    i[at], v[at] = idx, val
    return i.view(count, w), v.view(count, w)


def _times(form, vec):
    """The product of a padded form with a vector, or with a matrix of columns."""
    i, v = form
    if vec.dim() == 1:
        return (v * vec[i]).sum(1)
    out = torch.zeros(i.shape[0], vec.shape[1], dtype=torch.float64, device=DEV)
    for t in range(i.shape[1]):
        out += v[:, t, None] * vec[i[:, t]]
    return out


def _tail_norms(v, off, sizes):
    """Norms of the cones' tails (cones of at most 50 coordinates), always added in the same order."""
    t = torch.arange(1, 50, device=DEV)
    inside = t < sizes[:, None]
    return torch.where(inside, v[(off[:, None] + t).clamp_max(v.numel() - 1)], 0.0).square().sum(1).sqrt()


def _problem(case, seed):
    """The problem of a single-problem case: (A, b, c, n_orth, cone sizes)."""
    g = _gen(seed)
    kind = case["kind"]
    sizes = torch.zeros(0, dtype=torch.int64, device=DEV)
    if kind == "socp":
        sizes = torch.randint(3, 51, (case["cones"],), generator=_gen(case["cones"]), device=DEV)  # the case's own, whatever the seed
        n_orth = case["orth"]
        n = n_orth + int(sizes.sum())
        m = n // 2
    else:
        m, n = case["m"], case["n"]
        n_orth = n
        if kind == "paper" and case["cone"] == "socp":
            n_orth, sizes = 0, torch.full((n // 4,), 4, dtype=torch.int64, device=DEV)
    if kind == "paper":
        pos = torch.randint(0, m * n, (int(case["density"] * m * n),), generator=g, device=DEV).unique()
        row, col = pos // n, pos % n
    else:
        row = _distinct(g, torch.full((n,), m, dtype=torch.int64, device=DEV), case["k"]).reshape(-1)
        col = torch.arange(n, device=DEV).repeat_interleave(case["k"])
    A = _Sparse(m, n, row, col, _randn(g, row.numel()))
    if kind == "lp" and m > 100_000:  # the large LP has unit rows
        A.val /= _padded(m, A.row, A.col, A.val)[1].square().sum(1).clamp_min(1e-30).sqrt()[A.row]
    rows, cols = A.forms()
    x0 = torch.zeros(n, dtype=torch.float64, device=DEV)
    s0 = torch.zeros_like(x0)
    x0[:n_orth] = _randn(g, n_orth).clamp_min(0.0)
    s0[:n_orth] = torch.where(x0[:n_orth] == 0.0, _rand(g, n_orth), 0.0)
    if sizes.numel():
        off = sizes.cumsum(0) - sizes
        for v in (x0, s0):  # strictly inside each cone
            w = _randn(g, n - n_orth)
            w[off] = _tail_norms(w, off, sizes) + 0.1 + 0.9 * _rand(g, sizes.numel())
            v[n_orth:] = w
    b = _times(rows, x0)
    c = _randn(g, n) if kind == "paper" else _times(cols, _randn(g, m)) + s0
    return A, rows, cols, b, c, n_orth, sizes


def _dict(A, b, c, n_orth, sizes):
    ptr, col, val = A.host()
    return dict(m=A.m, n=A.n, row_ptr=ptr, col_idx=col, val=val, b=b.cpu().numpy(), c=c.cpu().numpy(), n_orth=n_orth,
                soc_sizes=sizes.int().cpu().numpy())


def _batch_sizes(case):
    u = _rand(_gen(case["count"]), case["count"])  # the case's own, whatever the seed
    return (case["lo"] * (case["hi"] / case["lo"]) ** u).round().long()


def _batch_problem(case, seed):
    """All instances as one block-diagonal problem: (A, rows, cols, b, c, row and column offsets)."""
    g = _gen(seed)
    ms = _batch_sizes(case)
    ns = 2 * ms
    roff, coff = ms.cumsum(0) - ms, ns.cumsum(0) - ns
    of = torch.arange(ms.numel(), device=DEV).repeat_interleave(ns)
    row = (_distinct(g, ms[of], case["k"]) + roff[of][:, None]).reshape(-1)
    col = torch.arange(int(ns.sum()), device=DEV).repeat_interleave(case["k"])
    A = _Sparse(int(ms.sum()), int(ns.sum()), row, col, _randn(g, row.numel()))
    rows, cols = A.forms()
    x0 = _randn(g, A.n).clamp_min(0.0)
    c = _times(cols, _randn(g, A.m)) + torch.where(x0 == 0.0, _rand(g, A.n), 0.0)
    return A, rows, cols, _times(rows, x0), c, roff, coff


def _batch_instances(A, b, c, roff, coff):
    ptr, col, val = A.host()
    b, c = b.cpu().numpy(), c.cpu().numpy()
    ro = np.append(roff.cpu().numpy(), A.m)
    co = np.append(coff.cpu().numpy(), A.n)
    out = []
    for r0, r1, c0, c1 in zip(ro[:-1], ro[1:], co[:-1], co[1:]):
        k0, k1 = ptr[r0], ptr[r1]
        out.append(dict(m=int(r1 - r0), n=int(c1 - c0), row_ptr=ptr[r0:r1 + 1] - k0,
                        col_idx=(col[k0:k1] - c0).astype(np.int32), val=val[k0:k1], b=b[r0:r1], c=c[c0:c1]))
    return out


def _family_problem(case, seed):
    """One A and c, the members' right-hand sides and their predicted starts [x ; lambda]."""
    g = _gen(seed)
    m, n, nb = case["m"], case["n"], case["nb"]
    row = _distinct(g, torch.full((n,), m, dtype=torch.int64, device=DEV), case["k"]).reshape(-1)
    A = _Sparse(m, n, row, torch.arange(n, device=DEV).repeat_interleave(case["k"]), _randn(g, row.numel()))
    rows, cols = A.forms()
    y = _randn(g, m)
    c = _times(cols, y) + torch.where(_rand(g, n) < 0.5, _rand(g, n), 0.0)
    X = (_randn(g, n, nb) + _randn(g, n, 1)).clamp_min(0.0)
    b = _times(rows, X)
    start = torch.cat([X + 0.3 * _randn(g, n, nb), 0.3 * _randn(g, m, nb) - y[:, None]]).float().t().contiguous()
    return A, rows, cols, b, c, start


def _mlp_problem(case, seed):
    g = _gen(seed)
    dims = [case["din"]] + [case["hid"]] * (case["layers"] - 1) + [case["dout"]]
    ws = [((2 * _rand(g, a, b) - 1) * math.sqrt(6.0 / a)).float() for a, b in zip(dims[:-1], dims[1:])]
    bs = [(0.2 * _rand(g, b) - 0.1).float() for b in dims[1:]]
    xs = [_randn(g, case["batch"], dims[0]).float() for _ in range(case["iters"])]
    ts = [_randn(g, case["batch"], dims[-1]).float() for _ in range(case["iters"])]
    return dims, ws, bs, xs, ts


def _pca_samples(case, seed):
    """Samples around a k-dimensional subspace, as solutions of a smooth family are, with noise in every direction."""
    g = _gen(seed)
    N, D, k = case["N"], case["D"], case["k"]
    scale = torch.logspace(0.0, -0.5, k, dtype=torch.float64, device=DEV)
    Y = ((_randn(g, N, k) * scale) @ _randn(g, k, D)).float()
    Y += 0.25 * torch.randn(N, D, generator=g, device=DEV)
    return Y + torch.randn(D, generator=g, device=DEV)


# ---------------------------------------------------------------------------
# prepare and run
# ---------------------------------------------------------------------------
def prepare(case, seed):
    kind = case["kind"]
    st = dict(case=case)
    if kind in ("call", "lp", "socp", "paper"):
        A, _, _, b, c, n_orth, sizes = _problem(case, seed)
        inst = _dict(A, b, c, n_orth, sizes)
        if kind == "call":
            st["inst"] = inst
        else:
            st["h"] = S.Solver.from_instance(inst, precision=case["precision"], eps=0.0)
    elif kind == "batch":
        A, _, _, b, c, roff, coff = _batch_problem(case, seed)
        st["h"] = S.Batch(_batch_instances(A, b, c, roff, coff), precision=case["precision"], eps=0.0)
    elif kind == "family":
        A, _, _, b, c, st["start"] = _family_problem(case, seed)
        ptr, col, val = A.host()
        st["h"] = S.Family(A.m, A.n, ptr, col, val, c.cpu().numpy(), case["B"], precision=case["precision"], eps=0.0)
        st["h"].set_rhs(b.t().cpu().numpy())
        st["out"] = torch.empty(case["nb"], A.n + A.m, dtype=torch.float32, device=DEV)
    elif kind == "standard":
        A, _, _, b, c, n_orth, sizes = _problem(case, seed)
        st["h"] = S.Standard.from_instance(_dict(A, b, c, n_orth, sizes), cg_iters=case["cg"], eps=0.0)
    elif kind == "mlp":
        dims, ws, bs, st["xs"], st["ts"] = _mlp_problem(case, seed)
        st["h"] = learn.MLP(dims, max_batch=case["batch"])
        st["h"].set_params(*[np.concatenate([t.cpu().numpy().reshape(-1) for t in v]) for v in (ws, bs)])
    else:
        st["Y"] = _pca_samples(case, seed)
    torch.cuda.synchronize()
    return st


def _values(case, res):
    """The residuals and objectives; in mixed precision the vectors alone stand for the result (the values are their cancellations)."""
    return [res[k] for k in ("r_prim", "r_dual", "pobj", "dobj")] if case["precision"] == "fp64" else []


def _typed(case, sol):
    if case["precision"] == "mixed":
        return {k: v.astype(np.float32) for k, v in sol.items()}
    return sol


def run(st):
    case = st["case"]
    kind = case["kind"]
    if kind == "call":
        _, sol, res = S.solve(st["inst"], case["iters"], noalloc=True, precision=case["precision"], eps=0.0)
        return [_typed(case, sol), _values(case, res)]
    if kind in ("lp", "socp", "paper"):
        h = st["h"]
        h.set_start()
        h.iterate(case["iters"])
        res = h.residuals()
        return [_typed(case, h.solution()), _values(case, res)]
    if kind == "batch":  # goes on from where the last pass left the instances
        h = st["h"]
        h.iterate(case["iters"])
        sols = [h.solution(i) for i in range(h.count)]
        return _typed(case, {k: np.concatenate([s[k] for s in sols]) for k in sols[0]})
    if kind == "family":
        h = st["h"]
        h.set_start_predicted(st["start"].data_ptr(), st["start"].shape[1])
        h.iterate(case["iters"])
        h.solution_device(st["out"].data_ptr(), st["out"].shape[1])
        return st["out"]
    if kind == "standard":
        h = st["h"]
        h.set_state()
        h.iterate(case["iters"])
        return h.solution()
    if kind == "mlp":  # goes on training from the weights it has
        h = st["h"]
        losses = [h.train_step(x, t, lr=1e-3) for x, t in zip(st["xs"], st["ts"])]
        return [list(h.params()), losses]
    Y = st["Y"].clone()  # the fit centers its samples in place
    mean, basis, sv = learn.pca_fit(Y, case["k"])
    coef = learn.gemm(Y, basis, transB=True)
    back = learn.gemm(coef, basis)
    learn.add_row_vector(back, mean)
    return [mean, sv, back]


# ---------------------------------------------------------------------------
# What a pass cannot do without
# ---------------------------------------------------------------------------
def _entries(case):
    if case["kind"] == "socp":
        n = case["orth"] + 26.5 * case["cones"]
        return n / 2, n, n * case["k"]
    if case["kind"] == "paper":
        return case["m"], case["n"], case["density"] * case["m"] * case["n"]
    if case["kind"] == "batch":
        lo, hi = case["lo"], case["hi"]
        m = case["count"] * ((hi - lo) / math.log(hi / lo) if hi > lo else lo)
        return m, 2 * m, 2 * m * case["k"]
    return case["m"], case["n"], case["n"] * case["k"]


def work(case):
    kind = case["kind"]
    if kind == "mlp":
        dims = [case["din"]] + [case["hid"]] * (case["layers"] - 1) + [case["dout"]]
        w, B = sum(a * b for a, b in zip(dims[:-1], dims[1:])), case["batch"]
        return dict(bytes=case["iters"] * (4 * B * (dims[0] + dims[-1])) + 24 * w,
                    flops=case["iters"] * 2 * B * (3 * w - dims[0] * dims[1]))
    if kind == "pca":
        N, D, k = case["N"], case["D"], case["k"]
        l = min(k + 32, N)
        return dict(bytes=4 * (2 * N * D + k * D), flops=2 * N * D * (6 * l + 2 * k))
    m, n, nnz = _entries(case)
    it = case["iters"]
    t = 4 if case.get("precision") == "mixed" else 8
    if kind == "family":  # the entries once per iteration, the members' vectors read and written
        B = case["nb"]
        return dict(bytes=it * ((8 + 2 * t) * nnz + B * ((2 * t + 16) * n + t * n + (2 * t + 16) * m + t * m)),
                    flops=it * 4.0 * nnz * B)
    once = (4 + 8) * nnz + 8 * (4 * n + 2 * m)
    if kind == "call" or 24 * nnz < 16e6:  # small enough to stay on the chip for the whole pass
        return dict(bytes=once, flops=it * 4.0 * nnz)
    if kind == "standard":
        return dict(bytes=it * ((1 + 2 * case["cg"]) * (12 * nnz + 8 * (m + n)) + 8 * (8 * n + 4 * m)),
                    flops=it * 2.0 * (1 + 2 * case["cg"]) * nnz)
    if kind == "batch":  # two-byte local numbers
        return dict(bytes=it * (2 * (2 + t) * nnz + (16 + 2 * t) * (m + n)), flops=it * 4.0 * nnz)
    return dict(bytes=it * (2 * (4 + t) * nnz + (20 + 4 * t) * m + (20 + 6 * t) * n), flops=it * 4.0 * nnz)


# ---------------------------------------------------------------------------
# The same results in 64 bits by plain torch
# ---------------------------------------------------------------------------
def _admm(rows, cols, b, c, iters, project, x=None, z=None, d=None, lam=None):
    """Algorithm 1 of the paper (mu = 1) in its reduced form, on vectors or on matrices of columns."""
    count = (cols[1] != 0.0).sum(1).double()
    fu = 1.0 / (1.0 + (rows[1] * rows[1]).sum(1))
    if b.dim() == 2:
        count, fu, c = count[:, None], fu[:, None], c[:, None]
    if x is None:
        x, lam = torch.zeros_like(c), torch.zeros_like(b)
        z, d = torch.zeros_like(c), torch.zeros_like(c)
    u = -lam
    for _ in range(iters):
        x = (count * x + _times(cols, u) + z + d - c) / (1.0 + count)
        z = project(x - d)
        d = d + (z - x)
        e = fu * (b - _times(rows, x))
        lam = lam - e
        u = e - lam
    return x, z, d, lam


def _projection(n_orth, sizes):
    if not sizes.numel():
        return lambda v: v.clamp_min(0.0)
    off = sizes.cumsum(0) - sizes
    cone_of = torch.arange(sizes.numel(), device=DEV).repeat_interleave(sizes)

    def project(v):
        out = v.clamp_min(0.0)
        w = v[n_orth:]
        head = w[off]
        tail = _tail_norms(w, off, sizes)
        zero, keep = tail <= -head, tail <= head
        h = torch.where(zero, 0.0, torch.where(keep, head, 0.5 * (head + tail)))
        s = torch.where(zero, 0.0, torch.where(keep, 1.0, 0.5 * (1.0 + head / tail.clamp_min(1e-300))))
        w = s[cone_of] * w
        w[off] = h
        out[n_orth:] = w
        return out

    return project


def _residuals(rows, cols, b, c, z, d, lam):
    cz, bl = float(c @ z), float(b @ lam)
    return [float((_times(rows, z) - b).norm()) / (1.0 + float(b.norm())),
            float((_times(cols, lam) + c - d).norm()) / (1.0 + float(c.norm())),
            cz, -bl]


def _named(x, z, d, lam):
    return {"x": x, "z": z, "delta": d, "lambda": lam}


def _exact_standard(case, rows, cols, b, c):
    """Standard ADMM (mu = 1): the block system by conjugate gradients on A A' from the last multiplier."""
    x2, lam, nu = torch.zeros_like(c), torch.zeros_like(c), torch.zeros_like(b)
    for _ in range(case["iters"]):
        x1 = (x2 - lam).clamp_min(0.0)
        delta = lam + (x1 - x2)
        v = x1 + lam - c
        r = _times(rows, v - _times(cols, nu)) - b
        p, rr = r, r @ r
        for _ in range(case["cg"]):
            q = _times(rows, _times(cols, p))
            pq = p @ q
            if not (rr > 0.0 and pq > 0.0):
                break
            a = rr / pq
            nu = nu + a * p
            r = r - a * q
            rn = r @ r
            p, rr = r + (rn / rr) * p, rn
        x2 = v - _times(cols, nu)
        lam = lam + (x1 - x2)
    return {"x1": x1, "x2": x2, "lam": lam, "nu": nu, "delta": delta}


def _exact_mlp(case, seed):
    dims, ws, bs, xs, ts = _mlp_problem(case, seed)
    ps = [t.double().requires_grad_(True) for t in ws + bs]
    m1, m2 = [torch.zeros_like(p) for p in ps], [torch.zeros_like(p) for p in ps]
    L, losses = len(ws), []
    for s, (x, t) in enumerate(zip(xs, ts), 1):
        h = x.double()
        for i in range(L):
            h = h @ ps[i] + ps[L + i]
            h = h.relu() if i < L - 1 else h
        loss = ((h - t.double()) ** 2).mean()
        losses.append(float(loss))
        grads = torch.autograd.grad(loss, ps)
        with torch.no_grad():
            for i, gr in enumerate(grads):
                m1[i] = 0.9 * m1[i] + 0.1 * gr
                m2[i] = 0.999 * m2[i] + 0.001 * gr * gr
                ps[i] -= 1e-3 * (m1[i] / (1 - 0.9 ** s)) / ((m2[i] / (1 - 0.999 ** s)).sqrt() + 1e-8)
    flat = [torch.cat([p.detach().reshape(-1) for p in v]) for v in (ps[:L], ps[L:])]
    return [flat, losses]


def exact(case, seed):
    kind = case["kind"]
    if kind in ("call", "lp", "socp", "paper"):
        _, rows, cols, b, c, n_orth, sizes = _problem(case, seed)
        x, z, d, lam = _admm(rows, cols, b, c, case["iters"], _projection(n_orth, sizes))
        return [_named(x, z, d, lam), _residuals(rows, cols, b, c, z, d, lam) if case["precision"] == "fp64" else []]
    if kind == "batch":
        _, rows, cols, b, c, _, _ = _batch_problem(case, seed)
        return _named(*_admm(rows, cols, b, c, case["iters"], lambda v: v.clamp_min(0.0)))
    if kind == "family":
        A, rows, cols, b, c, start = _family_problem(case, seed)
        start = start.double().t()
        x, lam = start[: A.n], start[A.n:]
        d = (c[:, None] + _times(cols, lam.contiguous())).clamp_min(0.0)
        _, z, _, lam = _admm(rows, cols, b, c, case["iters"], lambda v: v.clamp_min(0.0), x, x.clamp_min(0.0), d, lam)
        return torch.cat([z, lam]).t().contiguous()
    if kind == "standard":
        _, rows, cols, b, c, _, _ = _problem(case, seed)
        return _exact_standard(case, rows, cols, b, c)
    if kind == "mlp":
        return _exact_mlp(case, seed)
    Y = _pca_samples(case, seed).double()
    mean = Y.mean(0)
    Y -= mean
    w, V = torch.linalg.eigh((Y @ Y.t()).cpu())
    U = V.flip(1)[:, : case["k"]].contiguous().to(DEV)
    return [mean, w.flip(0)[: case["k"]].clamp_min(0.0).sqrt(), U @ (U.t() @ Y) + mean]
