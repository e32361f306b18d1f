"""What a user of this framework has it do, as cases that can be timed and checked.

Every case is one call sequence through the public drivers (paper_2605_08793_amd.driver) on seeded synthetic
problems of the recipes in paper_2605_08793_amd.workloads.  The solver these kernels serve starts with a number of
Sinkhorn sweeps, evaluates the dual objective and gradient at every trial point of its line search, takes the
threshold-sparsified plan from the same pass, renews the pattern by the top-k rule every few iterations, rebuilds
the sparse term H_Omega from it and solves for the quasi-Newton direction; `kind` says which of these a case is.
Everything is fp64, as the library is.
"""
import math

import torch

from paper_2605_08793_amd import workloads as W
from paper_2605_08793_amd.driver import DirectionSolver, DualPass, PatternRefresh, SparseTerm, TopK

_CHUNK = 1 << 27      # entries of M worked on at a time by the torch code below
_POINT_SWEEPS = 8     # Sinkhorn sweeps (in torch) that lead to the dual point a case is evaluated at
_SAMPLE = 1 << 22     # entries of T looked at for a threshold

_OUTPUTS = ("obj", "grad_alpha", "grad_beta", "row_sum", "col_sum")


def listed():
    return [
        # one evaluation with the pattern at 1000 x 1000, the smallest configuration: a handful of launches
        dict(name="fused_small", kind="fused", recipe="c1", n=1000, m=1000),
        # the start of a solve at the paper's synthetic size, eta = 0.001: ten sweeps, the matrix stays in cache
        dict(name="sweeps_small", kind="sweeps", recipe="syn1_diff", n=1600, m=1200, sweeps=10),
        # objective and gradient at a trial point of the line search; odd sizes, so rows start at odd multiples of 8 bytes
        dict(name="eval_ragged", kind="eval", recipe="c5", n=4999, m=3001),
        # the start of a solve at an odd size
        dict(name="sweeps_ragged", kind="sweeps", recipe="c5", n=7001, m=4999, sweeps=3),
        # candidate iterates: a few sweeps at 10000 x 10000, eta = 0.01
        dict(name="sweeps_mid", kind="sweeps", recipe="c2", n=10000, m=10000, sweeps=4),
        # a new pattern by the top-k rule together with the evaluation, at 10000 x 10000
        dict(name="refresh_mid", kind="refresh", recipe="c2", n=10000, m=10000),
        # the headline call: objective, gradient and pattern at 20000 x 20000, eta = 0.001
        dict(name="fused_flagship", kind="fused", recipe="c3", n=20000, m=20000),
        # candidate iterates at the same size
        dict(name="sweeps_flagship", kind="sweeps", recipe="c3", n=20000, m=20000, sweeps=4),
        # the threshold alone, for a caller that sets its own capacity: a tall matrix, 40000 x 10000
        dict(name="topk_tall", kind="topk", recipe="c4", n=40000, m=10000),
        # a new pattern becomes the sparse term: by columns, values, lower triangle for a Cholesky solver (2e6 entries)
        dict(name="pattern_flagship", kind="pattern", recipe="c3", n=20000, m=20000),
        # the quasi-Newton direction with the rank-two term: product, two solves, combination (2e6 entries)
        dict(name="direction_flagship", kind="direction", recipe="c3", n=20000, m=20000),
        # the largest configuration, 50000 x 50000 (20 GB)
        dict(name="fused_largest", kind="fused", recipe="c5", n=50000, m=50000),
    ]


def _log_between(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["fused", "fused", "eval", "sweeps", "sweeps", "sweeps", "refresh", "topk", "pattern", "direction"])
    recipe = rng.choice(["c2", "c3", "c5", "syn1_diff"])
    lo, hi = {"pattern": (1000, 20000), "direction": (1000, 20000), "refresh": (1200, 40000),
              "topk": (1200, 40000)}.get(kind, (600, 50000))
    n, m = _log_between(rng, lo, hi), _log_between(rng, lo, hi)
    case = dict(kind=kind, recipe=recipe, n=n, m=m)
    if kind == "sweeps":
        case["sweeps"] = max(1, min(rng.randint(2, 10), int(2.4e9 / (n * m))))
    return case


# ------------------------------------------------------------------ the same things in plain torch

def _rows(M):
    step = max(1, _CHUNK // M.shape[1])
    return [(r, min(M.shape[0], r + step)) for r in range(0, M.shape[0], step)]


def _torch_sweeps(M, a, b, eta, sweeps):
    """Log-domain Sinkhorn sweeps from zero: alpha half-step, then beta half-step."""
    alpha, beta = torch.zeros_like(a), torch.zeros_like(b)
    for _ in range(sweeps):
        for r0, r1 in _rows(M):
            alpha[r0:r1] = eta * torch.log(a[r0:r1]) - eta * torch.logsumexp((beta - M[r0:r1]) / eta, dim=1)
        total = torch.full_like(b, -math.inf)
        for r0, r1 in _rows(M):
            total = torch.logaddexp(total, torch.logsumexp((alpha[r0:r1, None] - M[r0:r1]) / eta, dim=0))
        beta = eta * torch.log(b) - eta * total
    return alpha, beta


def _plan(M, alpha, beta, eta, r0, r1):
    return torch.exp(((alpha[r0:r1, None] + beta) - M[r0:r1]) / eta)


def _threshold(M, alpha, beta, eta, keep):
    """A threshold that keeps about `keep` entries of T: between two neighbouring values of an evenly spread sample."""
    n, m = M.shape
    count = min(n * m, _SAMPLE)
    at = (torch.arange(count, device=M.device, dtype=torch.float64) * (n * m / count)).long()
    i, j = at // m, at % m
    T = torch.exp(((alpha[i] + beta[j]) - M[i, j]) / eta).sort(descending=True).values
    k = min(max(1, round(keep * count / (n * m))), count - 1)
    return float(torch.sqrt(T[k - 1] * T[k]))


def _sums(M, alpha, beta, eta):
    rs, cs = torch.empty_like(alpha), torch.zeros_like(beta)
    for r0, r1 in _rows(M):
        T = _plan(M, alpha, beta, eta, r0, r1)
        rs[r0:r1] = T.sum(1)
        cs += T.sum(0)
    return rs, cs


def _csr(M, alpha, beta, eta, delta):
    counts, cols, vals = [], [], []
    for r0, r1 in _rows(M):
        T = _plan(M, alpha, beta, eta, r0, r1)
        hit = T >= delta
        counts.append(hit.sum(1))
        cols.append(hit.nonzero()[:, 1].to(torch.int32))
        vals.append(T[hit])
    row_ptr = torch.zeros(M.shape[0] + 1, dtype=torch.int64, device=M.device)
    row_ptr[1:] = torch.cumsum(torch.cat(counts), 0)
    return row_ptr, torch.cat(cols), torch.cat(vals)


def _largest(M, alpha, beta, eta, k):
    """The s_ij of a little more than the k largest entries of T, in descending order."""
    floor = 0.8 * _threshold(M, alpha, beta, eta, 1.05 * k)
    found = []
    for r0, r1 in _rows(M):
        s = (alpha[r0:r1, None] + beta) - M[r0:r1]
        found.append(s[torch.exp(s / eta) >= floor])
    return torch.cat(found).sort(descending=True).values


def _by_row(row_ptr):
    return torch.repeat_interleave(torch.arange(row_ptr.numel() - 1, device=row_ptr.device), row_ptr.diff())


class _Hessian:
    """H_Omega + tau I on n + m - 1 unknowns: diagonal blocks from the full sums, pattern entries of column m - 1 left out."""

    def __init__(self, row_ptr, col_idx, val, rs, cs, eta, tau):
        n, m = rs.numel(), cs.numel()
        rows, cols = _by_row(row_ptr), col_idx.long()
        keep = cols < m - 1
        self.n, self.rows, self.cols, self.val = n, rows[keep], cols[keep], val[keep] / eta
        self.diag = torch.cat([rs, cs[:-1]]) / eta + tau

    def __call__(self, x):
        y = self.diag * x
        y.index_add_(0, self.rows, self.val * x[self.n + self.cols])
        y.index_add_(0, self.n + self.cols, self.val * x[self.rows])
        return y

    def solve(self, rhs):
        x, r = torch.zeros_like(rhs), rhs.clone()
        z = r / self.diag
        p, rz, stop = z.clone(), torch.dot(r, z), 1e-14 * float(rhs.norm())
        for _ in range(400):
            Ap = self(p)
            step = rz / torch.dot(p, Ap)
            x += step * p
            r -= step * Ap
            if float(r.norm()) <= stop:
                break
            z = r / self.diag
            rz, old = torch.dot(r, z), rz
            p = z + (rz / old) * p
        return x


def _problem(case, seed):
    """(problem, dual point): a, b > 0 that sum to 1, M / max(M), alpha and beta after a few sweeps."""
    p = W.make_problem(case["recipe"], device="cuda", n=case["n"], m=case["m"], seed=seed)
    if case["kind"] == "sweeps":
        return p, None, None
    alpha, beta = _torch_sweeps(p.M, p.a, p.b, p.eta, _POINT_SWEEPS)
    # a trial point of the solver, a fraction of eta away from the last Sinkhorn iterate
    g = torch.Generator(device="cuda").manual_seed(seed)
    alpha += 0.1 * p.eta * torch.randn(p.n, generator=g, device="cuda", dtype=torch.float64)
    beta += 0.1 * p.eta * torch.randn(p.m, generator=g, device="cuda", dtype=torch.float64)
    return p, alpha, beta


def _capacity(p):
    k = p.k_keep()
    return k + k // 16 + 4096


def _direction_inputs(p, alpha, beta, seed):
    """Pattern, sums, gradient and the previous step of a quasi-Newton iteration."""
    k = p.k_keep()
    v = _largest(p.M, alpha, beta, p.eta, k)
    delta = float(torch.exp(0.5 * (v[k - 1] + v[k]) / p.eta))      # keeps exactly k entries
    row_ptr, col_idx, val = _csr(p.M, alpha, beta, p.eta, delta)
    rs, cs = _sums(p.M, alpha, beta, p.eta)
    g = torch.cat([rs - p.a, (cs - p.b)[:-1]])
    tau = min(1e-3, float(g.norm()))
    H = _Hessian(row_ptr, col_idx, val, rs, cs, p.eta, tau)
    gen = torch.Generator(device="cuda").manual_seed(seed + 1)
    s_prev = 0.1 * p.eta * torch.randn(g.numel(), generator=gen, device="cuda", dtype=torch.float64)
    y_prev = H(s_prev) * (1.0 + 0.2 * torch.rand(g.numel(), generator=gen, device="cuda", dtype=torch.float64))
    return dict(row_ptr=row_ptr, col_idx=col_idx, val=val, rs=rs, cs=cs, g=g, tau=tau, H=H, s_prev=s_prev, y_prev=y_prev)


# ------------------------------------------------------------------ the calls

def prepare(case, seed):
    kind = case["kind"]
    p, alpha, beta = _problem(case, seed)
    st = dict(case=case, kind=kind, p=p, alpha=alpha, beta=beta)
    if kind in ("eval", "sweeps"):
        st["dp"] = DualPass(p.n, p.m)
    elif kind == "fused":
        st["delta"] = _threshold(p.M, alpha, beta, p.eta, p.k_keep())
        st["dp"] = DualPass(p.n, p.m, capacity=_capacity(p))
    elif kind == "refresh":
        st["dp"] = PatternRefresh(p.n, p.m, p.k_keep())
    elif kind == "topk":
        st["tk"] = TopK(p.n, p.m, p.k_keep())
    else:
        d = _direction_inputs(p, alpha, beta, seed)
        for name in ("row_ptr", "col_idx", "rs", "cs", "g", "tau", "s_prev", "y_prev"):
            st[name] = d[name]
        if kind == "direction":
            term = SparseTerm(p.n, p.m, d["row_ptr"], d["col_idx"], d["col_idx"].numel())
            term.refresh(p.M, alpha, beta, p.eta)
            st["solver"] = DirectionSolver(term)
            del st["p"].M      # a direction needs the stored pattern only
    return st


def run(state):
    kind, p, alpha, beta = state["kind"], state["p"], state["alpha"], state["beta"]
    if kind == "sweeps":
        return state["dp"].sinkhorn_sweeps(p.M, p.a, p.b, p.eta, state["case"]["sweeps"])
    if kind == "topk":
        tk = state["tk"]
        tk.threshold(p.M, alpha, beta, p.eta)
        return dict(delta=tk.delta, s_k=tk.s_k, info=tk.info)
    if kind == "pattern":
        term = SparseTerm(p.n, p.m, state["row_ptr"], state["col_idx"], state["col_idx"].numel())
        term.refresh(p.M, alpha, beta, p.eta)
        term.lower_csc(p.eta, state["tau"], state["rs"], state["cs"])
        return dict(val=term.val, val_csc=term.val_csc, col_ptr=term.col_ptr, row_idx=term.row_idx, csc_pos=term.csc_pos,
                    h_col_ptr=term.h_col_ptr, h_row_idx=term.h_row_idx, h_val=term.h_val, h_info=term.h_info)
    if kind == "direction":
        s = state["solver"]
        s.direction(p.config.eta, state["tau"], state["rs"], state["cs"], state["g"], state["s_prev"], state["y_prev"])
        return dict(d=s.d, p=s.p, q=s.q)
    dp = state["dp"]
    if kind == "eval":
        dp.dual_eval(p.M, p.a, p.b, alpha, beta, p.eta)
        return {name: getattr(dp, name) for name in _OUTPUTS}
    if kind == "fused":
        dp.dual_eval_sparsify(p.M, p.a, p.b, alpha, beta, p.eta, state["delta"])
    else:
        dp.refresh(p.M, p.a, p.b, alpha, beta, p.eta)
    out = {name: getattr(dp, name) for name in _OUTPUTS + ("row_ptr", "col_idx", "val", "info")}
    if kind == "refresh":
        out["delta"] = dp.delta
    return out


def work(case):
    """Bytes and operations of one pass: M is 8 n m bytes; an entry of the plan is about 24 operations (two adds, the
    exponential, the sums).  A sweep needs every row's sum before any column's, and every column's before the next
    sweep's rows: a matrix beyond the 256 MB of on-chip cache has to be read once per sweep."""
    kind, n, m = case["kind"], case["n"], case["m"]
    frac = W.CONFIGS[case["recipe"]].frac
    nnz = max(1, round(frac * n * m))
    matrix, vectors = 8.0 * n * m, 8.0 * (n + m)
    if kind == "sweeps":
        reads = case["sweeps"] if matrix > 256e6 else 1
        return {"bytes": reads * matrix + 2 * vectors, "flops": 24.0 * n * m * case["sweeps"]}
    if kind == "topk":
        return {"bytes": matrix + vectors, "flops": 3.0 * n * m}
    if kind == "pattern":
        # the pattern in (columns), every entry of M it names, then by columns (rows, positions), values twice, the triangle
        return {"bytes": 4.0 * nnz + 8.0 * nnz + 12.0 * nnz + 16.0 * nnz + 12.0 * (nnz + n + m) + 5 * vectors, "flops": 24.0 * nnz}
    if kind == "direction":
        # about 15 iterations of a pair of systems, each reading the pattern by rows and by columns; the pattern of a
        # usual size stays in cache, so it is counted once
        return {"bytes": 24.0 * nnz + 10 * vectors, "flops": 15.0 * 2 * 4 * nnz}
    out = {"eval": 4.0 * vectors, "fused": 4.0 * vectors + 12.0 * nnz + 8.0 * n, "refresh": 4.0 * vectors + 12.0 * nnz + 8.0 * n}[kind]
    return {"bytes": matrix + 2 * vectors + out, "flops": 24.0 * n * m}


def tolerance(case):
    """fp64 throughout.  Against exact() the calls of this library show up to 1e-15 in sums, duals and plan entries and
    5e-15 in the gradient, which is a difference of two nearly equal numbers (a drawn case may magnify that a little
    more); single entries are a few hundred times as far off as the norm is, since the rounding of s counts 1 / eta-fold
    in exp(s / eta).  A direction stops at a residual of 1e-8 of its right-hand side: 7e-8 seen.  Whole numbers are exact."""
    if case["kind"] == "direction":
        return {"rel": 3e-7, "max": 3e-5}
    return {"rel": 4e-14, "max": 4e-12}


def exact(case, seed):
    kind = case["kind"]
    p, alpha, beta = _problem(case, seed)
    M, a, b, eta, k = p.M, p.a, p.b, p.eta, p.k_keep()
    if kind == "sweeps":
        return _torch_sweeps(M, a, b, eta, case["sweeps"])
    if kind == "topk":
        s_k = _largest(M, alpha, beta, eta, k)[k - 1]
        return dict(delta=torch.exp(s_k / eta).reshape(1), s_k=s_k.reshape(1), info=None)
    if kind in ("pattern", "direction"):
        d = _direction_inputs(p, alpha, beta, seed)
        n, m, H = p.n, p.m, d["H"]
        if kind == "direction":
            q, r = H.solve(d["g"]), H.solve(d["y_prev"])
            g, s, y = d["g"], d["s_prev"], d["y_prev"]
            v, ys = H(s), torch.dot(y, s)
            if not float(ys) > 1e-6 * float(torch.dot(y, y)):
                return dict(d=-q, p=q, q=r)
            # B = A + U C U^T, U = [y, v], C = diag(1 / y.s, -1 / v.s); A^-1 U = [r, s]
            U, AU = torch.stack([y, v], 1), torch.stack([r, s], 1)
            C_inv = torch.diag(torch.stack([ys, -torch.dot(v, s)]))
            small = (C_inv + U.T.contiguous() @ AU).cpu()
            coef = torch.linalg.solve(small, (U.T.contiguous() @ q).cpu()).cuda()
            return dict(d=-(q - AU @ coef), p=q, q=r)
        rows, cols, val = _by_row(d["row_ptr"]), d["col_idx"].long(), d["val"]
        by_col = torch.argsort(cols, stable=True)
        keep = cols < m - 1
        column = torch.cat([torch.arange(n + m - 1, device="cuda"), rows[keep]])
        place = torch.cat([torch.full((n + m - 1,), -1, device="cuda"), cols[keep]])
        h = torch.cat([H.diag, H.val])[torch.argsort(column * (m + 1) + place + 1)]
        pad = torch.zeros(n + m - 1 + val.numel() - h.numel(), dtype=torch.float64, device="cuda")
        return dict(val=val, val_csc=val[by_col], col_ptr=None, row_idx=None, csc_pos=None, h_col_ptr=None, h_row_idx=None,
                    h_val=torch.cat([h, pad]), h_info=None)
    rs, cs = _sums(M, alpha, beta, eta)
    obj = -eta * rs.sum() + (torch.dot(alpha, a) + torch.dot(beta, b))
    out = dict(obj=obj.reshape(1), grad_alpha=a - rs, grad_beta=b - cs, row_sum=rs, col_sum=cs)
    if kind == "eval":
        return out
    if kind == "fused":
        delta, capacity = _threshold(M, alpha, beta, eta, k), _capacity(p)
    else:
        v = _largest(M, alpha, beta, eta, k)
        out["delta"], capacity = torch.exp(v[k - 1] / eta).reshape(1), k + 4096
        delta = float(torch.exp(0.5 * (v[k - 1] + v[k]) / eta))
    _, _, val = _csr(M, alpha, beta, eta, delta)
    out.update(row_ptr=None, col_idx=None, info=None, val=torch.cat([val, torch.zeros(capacity - val.numel(), dtype=torch.float64, device="cuda")]))
    return out
