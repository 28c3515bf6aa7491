"""Performance cases: the work that users of the library have it do, through
the package's public entry points, from the smallest calls to the largest.

A case names a kind of matrix (the three kinds of ``workloads/generators.py``,
drawn here on the GPU so that inputs are made quickly), its size and column
partition, what is done with it (``op``) and the options of the handle:

* ``once``          setup, solve and close: one least-squares problem (or one
                    batch of them) from the CSR arrays to x;
* ``solve``         another right-hand side on a handle that is kept;
* ``gradient``      forward and backward through ``lstsq`` on a kept handle;
* ``precondition``  z = M r on a kept handle (an outer iteration of the user's own);
* ``products``      y = A x and x = A^T y on a kept handle;
* ``transpose``     A^T of a CSR matrix by the stand-alone entry point.
"""
import math

import numpy as np
import torch

import paper_2107_09006_amd as L

DEVICE = "cuda:0"
VARIANTS = {"additive": L.ADDITIVE, "one_level": L.ONE_LEVEL, "balanced": L.BALANCED,
            "ras": L.RAS, "deflated": L.DEFLATED}
KRYLOV = {"pcg": L.PCG, "lsqr": L.LSQR, "gmres": L.GMRES}
PRECISION = {"fp64": L.FP64, "mixed": L.MIXED}
FACTOR = {"cholesky": L.FACTOR_CHOLESKY, "qr": L.FACTOR_QR}


def case(op, kind, n, parts, *, instances=1, precision="fp64", variant="additive", krylov="pcg",
         factor="cholesky", tol=1e-8, **name):
    """n: columns (per instance the upper end of the range for a batch); for a
    grid, its side, and parts the patches along a side."""
    return {**name, "op": op, "kind": kind, "n": n, "parts": parts, "instances": instances,
            "precision": precision, "variant": variant, "krylov": krylov, "factor": factor,
            "tol": tol}


def listed():
    return [
        # the smallest whole call: a plain problem of 1,000 columns, where launches and host work count
        case("once", "banded", 1000, 8, name="banded_1000"),
        # the smallest single call: one preconditioner application inside a user's own iteration
        case("precondition", "grid", 40, 4, name="grid_40_precondition"),
        # an ordinary single problem with the factors taken from thin QR instead of the normal matrix
        case("once", "banded", 30011, 32, factor="qr", name="banded_30k_qr"),
        # a serving loop: right-hand side after right-hand side on a kept batch, FP32 factors
        case("solve", "banded", 50000, 64, instances=16, precision="mixed", tol=1e-10,
             name="banded_batch_16_mixed"),
        # training through the solve: x, dL/db and dL/dvals on the 500 x 500 grid
        case("gradient", "grid", 500, 16, tol=1e-10, name="grid_500_gradient"),
        # the pairings of the paper's experiments: LSQR with the balanced form on an irregular matrix
        case("solve", "irregular", 200003, 128, variant="balanced", krylov="lsqr",
             name="irregular_200k_lsqr"),
        # and GMRES with the deflated form on a grid that no tile size divides
        case("solve", "grid", 301, 10, variant="deflated", krylov="gmres",
             name="grid_301_gmres"),
        # matrix products of both directions on a matrix above the last-level cache
        case("products", "irregular", 1000000, 512, name="irregular_1m_products"),
        # the transpose of the same matrix on its own
        case("transpose", "irregular", 1000000, 512, name="irregular_1m_transpose"),
        # one ill-scaled irregular problem of a million columns, FP32 factors
        case("once", "irregular", 1000000, 512, precision="mixed", tol=1e-10, name="irregular_1m_mixed"),
        # one ill-conditioned grid of a million columns (large coarse space)
        case("once", "grid", 1000, 16, name="grid_1000"),
        # a batch of 64 independent problems, 5,000 to 200,000 columns each
        case("once", "banded", 200000, 128, instances=64, name="banded_batch_64"),
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _draw_shape(rng, kind, top):
    """(n, parts) of a single matrix of up to ``top`` columns."""
    if kind == "grid":
        side = _log_uniform(rng, 24, math.isqrt(top))
        return side, max(2, min(16, side // rng.randint(12, 48)))
    n = _log_uniform(rng, 1000 if kind == "banded" else 6000, top)
    lo, hi = (125, 4000) if kind == "banded" else (1000, 3000)
    return n, max(2, min(512, n // _log_uniform(rng, lo, hi)))


def draw(rng):
    """One more case of the same ranges."""
    op = rng.choice(["once", "once", "once", "solve", "solve", "solve", "gradient", "precondition",
                     "products", "transpose"])
    kind = rng.choice(["banded", "grid", "irregular"])
    if op in ("products", "transpose"):
        n, parts = _draw_shape(rng, kind, 1000000)
        return case(op, kind, n, parts)
    if op == "precondition":
        n, parts = _draw_shape(rng, kind, 500000)
        return case(op, kind, n, parts,
                    variant=rng.choice(["additive", "additive", "one_level", "balanced", "deflated"]))
    # FP32 factors with a tolerance that needs the double-precision recurrences
    # (not on the grids, whose condition number is near 1e10)
    precision = rng.choice(["fp64", "mixed"]) if kind != "grid" else "fp64"
    if op == "gradient":
        n, parts = _draw_shape(rng, kind, 250000)
        return case(op, kind, n, parts, precision=precision, tol=1e-10)
    tol = 1e-10 if precision == "mixed" else 1e-8
    if kind == "banded" and rng.random() < 0.5:
        return case(op, kind, _log_uniform(rng, 10000, 200000), 128, instances=rng.randint(2, 48),
                    precision=precision, tol=tol)
    how = rng.choice(["pcg", "pcg", "qr", "lsqr", "gmres"])
    if how == "qr":
        n, parts = _draw_shape(rng, kind, 60000)
        return case(op, kind, n, parts, factor="qr")
    if how == "lsqr":
        n, parts = _draw_shape(rng, kind, 400000)
        return case(op, kind, n, parts, krylov="lsqr", variant=rng.choice(["additive", "balanced"]))
    if how == "gmres":
        n, parts = _draw_shape(rng, kind, 400000)
        return case(op, kind, n, parts, krylov="gmres", variant=rng.choice(["additive", "deflated"]))
    n, parts = _draw_shape(rng, kind, 1000000)
    return case(op, kind, n, parts, precision=precision, tol=tol)


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------

def _sizes(c):
    """[(n, parts)] of the instances of a case (fixed by the case alone)."""
    if c["kind"] == "grid":
        return [(c["n"] ** 2, c["parts"] ** 2)]
    if c["instances"] == 1:
        return [(c["n"], c["parts"])]
    out = []
    for j in range(c["instances"]):       # as the batched workload: n and parts log-uniform
        rng = np.random.default_rng(3000 + j)
        n = int(round(math.exp(rng.uniform(math.log(5e3), math.log(c["n"])))))
        out.append((n, int(round(math.exp(rng.uniform(math.log(8), math.log(c["parts"])))))))
    return out


def _reg(kind):
    return {"banded": 0.1, "grid": 1e-3, "irregular": 1e-4}[kind]


def _tau(c):
    return 0.05 if c["kind"] == "irregular" else 0.1


def _stack(rows, cols, vals, m_rows, n, reg):
    """CSR (int64 row pointers) of entries sorted by row, with the n rows
    reg e_j after them."""
    dev = rows.device
    j = torch.arange(n, device=dev)
    counts = torch.ones(m_rows + n, dtype=torch.int64, device=dev)
    counts[:m_rows] = torch.bincount(rows, minlength=m_rows)
    rowptr = torch.zeros(m_rows + n + 1, dtype=torch.int64, device=dev)
    torch.cumsum(counts, 0, out=rowptr[1:])
    return (rowptr, torch.cat([cols, j]).to(torch.int32),
            torch.cat([vals, torch.full((n,), reg, dtype=torch.float64, device=dev)]))


def _contiguous(n, parts):
    bounds = (np.arange(parts + 1, dtype=np.int64) * n) // parts
    return np.repeat(np.arange(parts, dtype=np.int32), np.diff(bounds))


def _banded(n, parts, g):
    """2 n rows of 4 distinct columns within 20 of the diagonal, N(0, 1)."""
    m = 2 * n
    width = min(41, n)
    base = (torch.arange(m, device=DEVICE) // 2 - 20).clamp(0, n - width)
    cols = torch.empty(m, 4, dtype=torch.int64, device=DEVICE)
    for i in range(4):                    # Floyd's sampling without replacement
        top = width - 4 + i
        pick = torch.randint(0, top + 1, (m,), generator=g, device=DEVICE)
        seen = (cols[:, :i] == pick[:, None]).any(1)
        cols[:, i] = torch.where(seen, top, pick)
    cols = (cols.sort(1).values + base[:, None]).reshape(-1)
    vals = torch.randn(4 * m, generator=g, device=DEVICE, dtype=torch.float64)
    rows = torch.arange(m, device=DEVICE).repeat_interleave(4)
    return _stack(rows, cols, vals, m, n, _reg("banded")), _contiguous(n, parts)


def _grid(side, patches, g):
    """Forward differences with weights 10^U(-2, 2) along both directions."""
    node = torch.arange(side * side, device=DEVICE).reshape(side, side)
    tail = torch.cat([node[:, :-1].reshape(-1), node[:-1].reshape(-1)])
    head = torch.cat([node[:, 1:].reshape(-1), node[1:].reshape(-1)])
    w = 10.0 ** (4.0 * torch.rand(tail.numel(), generator=g, device=DEVICE, dtype=torch.float64) - 2.0)
    rows = torch.arange(tail.numel(), device=DEVICE).repeat_interleave(2)
    csr = _stack(rows, torch.stack([tail, head], 1).reshape(-1), torch.stack([-w, w], 1).reshape(-1),
                 tail.numel(), side * side, _reg("grid"))
    band = _contiguous(side, patches)
    return csr, (band[:, None] * patches + band[None, :]).reshape(-1).astype(np.int32)


def _irregular(n, parts, g):
    """3 n rows of 1 + geometric(0.2) entries (at most 64) around a centre,
    N(0, 1) values, columns scaled by 10^U(-3, 3); parts of uneven size with
    ragged edges."""
    m = 3 * n
    u = (torch.arange(m, device=DEVICE, dtype=torch.float64) + 0.5) / m     # quantiles: the same
    length = (2 + torch.floor(torch.log1p(-u) / math.log(0.8))).clamp(max=64).to(torch.int64)
    length = length[torch.randperm(m, generator=g, device=DEVICE)]           # entries in every draw
    rows = torch.arange(m, device=DEVICE).repeat_interleave(length)
    centre = torch.randint(0, n, (m,), generator=g, device=DEVICE)
    off = torch.randn(rows.numel(), generator=g, device=DEVICE) * math.sqrt(2000.0)
    span = 1 << 10                                                           # |off| stays below span / 2
    key = (rows * span + off.round().to(torch.int64) + span // 2).sort().values
    rank = torch.arange(rows.numel(), device=DEVICE) - (length.cumsum(0) - length)[rows]
    off = key % span - span // 2 + rank - length[rows] // 2                  # strictly increasing
    cols = (rows * n + (centre[rows] + off) % n).sort().values % n
    scale = 10.0 ** (6.0 * torch.rand(n, generator=g, device=DEVICE, dtype=torch.float64) - 3.0)
    vals = torch.randn(rows.numel(), generator=g, device=DEVICE, dtype=torch.float64) * scale[cols]
    size = 500.0 + 2500.0 * torch.rand(parts, generator=g, device=DEVICE, dtype=torch.float64)
    edge = (size.cumsum(0) / size.sum() * n)[:-1].contiguous()
    at = torch.arange(n, device=DEVICE, dtype=torch.float64)
    at += 20.0 * torch.randn(n, generator=g, device=DEVICE, dtype=torch.float64).clamp(-3, 3)
    part = torch.bucketize(at, edge).to(torch.int32).cpu().numpy()
    return _stack(rows, cols, vals, m, n, _reg("irregular")), part


def _problems(c, seed):
    """[(rowptr, colind, vals, part, nparts, m, n)] and the generator left over."""
    g = torch.Generator(device=DEVICE).manual_seed(seed)
    out = []
    for n, parts in _sizes(c):
        if c["kind"] == "grid":
            (rp, ci, va), part = _grid(c["n"], c["parts"], g)
        else:
            (rp, ci, va), part = (_banded if c["kind"] == "banded" else _irregular)(n, parts, g)
        out.append((rp, ci, va, part, parts, rp.numel() - 1, n))
    return out, g


def _solver(c, problems):
    opts = dict(tol=c["tol"], precision=PRECISION[c["precision"]], variant=VARIANTS[c["variant"]],
                krylov=KRYLOV[c["krylov"]], local_factor=FACTOR[c["factor"]],
                flexible=int(c["precision"] == "mixed" and c["variant"] == "balanced"
                             and c["krylov"] == "pcg"))
    if c["instances"] > 1:
        return L.Solver.batched(problems, _tau(c), device=DEVICE, **opts)
    rp, ci, va, part, parts, m, n = problems[0]
    return L.Solver(rp, ci, va, part, parts, m, n, _tau(c), device=DEVICE, **opts)


def _right_hand_side(c, problems, g):
    """The vectors of the call: b, or what the op takes in its place."""
    m, n = sum(p[5] for p in problems), sum(p[6] for p in problems)
    long = torch.randn(m, generator=g, device=DEVICE, dtype=torch.float64)
    short = torch.randn(n, generator=g, device=DEVICE, dtype=torch.float64)
    return long, short


def prepare(c, seed):
    problems, g = _problems(c, seed)
    b, v = _right_hand_side(c, problems, g)
    state = {"case": c, "problems": problems, "b": b, "v": v}
    if c["op"] == "transpose":
        rp, ci, va, _, _, m, n = problems[0]
        state["csr"] = (m, n, rp.to(torch.int32), ci, va)
    elif c["op"] != "once":
        state["solver"] = _solver(c, problems)
    if c["op"] == "gradient":
        state["vals"] = problems[0][2].clone().requires_grad_(True)
        state["b"] = b.requires_grad_(True)
    return state


def run(state):
    c, op = state["case"], state["case"]["op"]
    if op == "once":
        s = _solver(c, state["problems"])
        x, _, _ = s.solve(state["b"])
        s.close()
        return x
    if op == "transpose":
        m, n, rp, ci, va = state["csr"]
        return L.transpose(m, n, rp, ci, va, device=DEVICE)
    s = state["solver"]
    if op == "solve":
        return s.solve(state["b"])[0]
    if op == "gradient":
        x = L.lstsq(state["vals"], state["b"], s)
        loss = 0.5 * (x - state["v"]).square().sum()
        dvals, db = torch.autograd.grad(loss, (state["vals"], state["b"]))
        return {"x": x.detach(), "dLdb": db, "dLdvals": dvals}
    if op == "precondition":
        return s.apply_preconditioner(state["v"])
    return s.spmv(state["v"]), s.spmv(state["b"], trans=True)


def _size(c):
    """(m, n, entries) over the instances (entries of the irregular kind: the mean)."""
    m = n = nnz = 0
    for k, _ in _sizes(c):
        edges = 2 * c["n"] * (c["n"] - 1) if c["kind"] == "grid" else 0
        rows, entries = {"banded": (2 * k, 8 * k), "grid": (edges, 2 * edges),
                         "irregular": (3 * k, 18 * k)}[c["kind"]]
        m, n, nnz = m + rows + k, n + k, nnz + entries + k
    return m, n, nnz


def work(c):
    """The matrix and the vectors read once and the results written once; one
    product with A and A^T where there is a right-hand side to check."""
    m, n, nnz = _size(c)
    matrix = 12 * nnz
    vectors = 8 * (m + n)
    rows, part = 8 * (m + 1), 4 * n
    return {"once": {"bytes": matrix + rows + part + vectors, "flops": 4 * nnz},
            "solve": {"bytes": matrix + 4 * m + vectors, "flops": 4 * nnz},
            "gradient": {"bytes": matrix + 4 * m + 2 * vectors + 8 * nnz, "flops": 12 * nnz},
            "precondition": {"bytes": matrix + 4 * m + 16 * n, "flops": 4 * nnz},
            "products": {"bytes": 2 * matrix + 4 * (m + n) + 2 * vectors, "flops": 4 * nnz},
            "transpose": {"bytes": 2 * matrix + 4 * nnz + 4 * (m + n), "flops": 0}}[c["op"]]


# ---------------------------------------------------------------------------
# the same in plain torch, 64 bits
# ---------------------------------------------------------------------------

class _Normal:
    """C = A^T A of the whole case: products, and a solve that is refined until
    it has converged."""

    def __init__(self, c, problems):
        self.kind, self.side = c["kind"], c["n"]
        r0 = c0 = 0
        rows, cols, vals = [], [], []
        for rp, ci, va, _, _, m, n in problems:
            rows.append(torch.arange(m, device=DEVICE).repeat_interleave(rp.diff()) + r0)
            cols.append(ci.to(torch.int64) + c0)
            vals.append(va)
            r0, c0 = r0 + m, c0 + n
        self.m, self.n = r0, c0
        self.rows, self.cols, self.vals = torch.cat(rows), torch.cat(cols), torch.cat(vals)
        order = torch.sort(self.cols, stable=True).indices
        self.A = self._csr(self.rows, self.cols, self.vals, r0, c0)
        self.AT = self._csr(self.cols[order], self.rows[order], self.vals[order], c0, r0)

    @staticmethod
    def _csr(rows, cols, vals, m, n):
        ptr = torch.zeros(m + 1, dtype=torch.int64, device=DEVICE)
        torch.cumsum(torch.bincount(rows, minlength=m), 0, out=ptr[1:])
        return torch.sparse_csr_tensor(ptr, cols, vals, size=(m, n))

    def a(self, x):
        return torch.mv(self.A, x)

    def at(self, y):
        return torch.mv(self.AT, y)

    def _jacobi_cg(self, rhs):
        diag = torch.zeros(self.n, dtype=torch.float64, device=DEVICE)
        diag.index_add_(0, self.cols, self.vals.square())
        x, r = torch.zeros_like(rhs), rhs.clone()
        z = r / diag
        p, rho = z.clone(), torch.dot(r, z)
        stop = 1e-24 * float(rho)
        for k in range(4000):
            q = self.at(self.a(p))
            alpha = rho / torch.dot(p, q)
            x += alpha * p
            r -= alpha * q
            z = r / diag
            old, rho = rho, torch.dot(r, z)
            if k % 20 == 0 and float(rho) <= stop:
                break
            p = z + (rho / old) * p
        return x

    def _grid_factors(self):
        """Block Cholesky of the grid's C: one block per grid row, coupled by a
        diagonal block to the next."""
        G = self.side
        edges = G * (G - 1)
        w2 = self.vals[:4 * edges].reshape(-1, 2)[:, 1].square()
        h, v = w2[:edges].reshape(G, G - 1), w2[edges:].reshape(G - 1, G)
        diag = torch.full((G, G), _reg("grid") ** 2, dtype=torch.float64, device=DEVICE)
        diag[:, :-1] += h
        diag[:, 1:] += h
        diag[:-1] += v
        diag[1:] += v
        factors, last = [], None
        for r in range(G):
            D = torch.diag(diag[r]) - torch.diag(h[r], 1) - torch.diag(h[r], -1)
            if r:
                inv = torch.cholesky_inverse(last)
                D -= v[r - 1][:, None] * inv * v[r - 1][None, :]
            last = torch.linalg.cholesky(D)
            factors.append(last)
        return factors, v

    def _grid_solve(self, rhs):
        G = self.side
        if not hasattr(self, "_factors"):
            self._factors = self._grid_factors()
        factors, v = self._factors
        y = list(rhs.reshape(G, G).unbind(0))
        for r in range(1, G):
            y[r] = y[r] + v[r - 1] * torch.cholesky_solve(y[r - 1][:, None], factors[r - 1])[:, 0]
        x = [None] * G
        for r in range(G - 1, -1, -1):
            t = y[r] if r == G - 1 else y[r] + v[r] * x[r + 1]
            x[r] = torch.cholesky_solve(t[:, None], factors[r])[:, 0]
        return torch.cat(x)

    def solve(self, rhs=None, b=None):
        """C^{-1} rhs, or the least-squares solution for b."""
        x = torch.zeros(self.n, dtype=torch.float64, device=DEVICE)
        for _ in range(4):
            r = self.at(b - self.a(x)) if b is not None else rhs - self.at(self.a(x))
            x = x + (self._grid_solve(r) if self.kind == "grid" else self._jacobi_cg(r))
        return x


def _one_preconditioner(c, N, problem, r):
    """M r of eq. (two_level_schwarz), (one_level_schwarz), (balanced) or
    (deflated) with dense matrices: the coarse vectors of subdomain i span the
    eigenvectors of (C_I - C_IG Ct_GG^+ C_GI) x = mu C_I x with mu < tau."""
    part = torch.as_tensor(problem[3], device=DEVICE)
    A = N.A.to_dense()
    C = A.T @ A
    local, basis = [], []
    for i in range(problem[4]):
        inner = part == i
        xi = (A[:, inner] != 0).any(1)
        I = inner.nonzero()[:, 0]
        B = ((A[xi] != 0).any(0) & ~inner).nonzero()[:, 0]
        om = torch.cat([I, B])
        d = C[om, om].rsqrt()
        local.append((I, om, d, torch.linalg.cholesky(C[om][:, om] * d[:, None] * d[None, :])))
        if c["variant"] in ("one_level", "ras"):
            continue
        dI, dB = d[:I.numel()], d[I.numel():]
        AG = A[xi][:, B] * dB[None, :]
        LI = torch.linalg.cholesky(C[I][:, I] * dI[:, None] * dI[None, :])
        Q = torch.linalg.solve_triangular(LI, C[I][:, B] * dI[:, None] * dB[None, :], upper=False)
        lam, U = torch.linalg.eigh(AG.T @ AG)
        keep = lam > lam.max() * B.numel() * 2.3e-16
        K = Q @ (U[:, keep] * lam[keep].rsqrt()[None, :])
        U, sigma, _ = torch.linalg.svd(K, full_matrices=False)
        X = U[:, 1.0 - sigma.square() < _tau(c)]
        if X.shape[1]:
            R = torch.zeros(N.n, X.shape[1], dtype=torch.float64, device=DEVICE)
            R[I] = torch.linalg.solve_triangular(LI.T.contiguous(), X, upper=True) * dI[:, None]
            basis.append(R)
    R0 = torch.cat(basis, 1) if basis else None
    E = torch.linalg.cholesky((A @ R0).T @ (A @ R0)) if basis else None

    def q(v):
        return R0 @ torch.cholesky_solve((R0.T @ v)[:, None], E)[:, 0] if basis else torch.zeros_like(v)

    def first(v, restricted):
        z = torch.zeros_like(v)
        for I, om, d, F in local:
            y = d * torch.cholesky_solve((d * v[om])[:, None], F)[:, 0]
            if restricted:
                z[I] += y[:I.numel()]
            else:
                z[om] += y
        return z

    if c["variant"] == "balanced":
        y = first(r - C @ q(r), False)
        return y + q(r - C @ y)
    if c["variant"] == "deflated":
        u = q(r)
        return u + first(r - C @ u, True)
    return first(r, c["variant"] == "ras") + q(r)


def exact(c, seed):
    problems, g = _problems(c, seed)
    b, v = _right_hand_side(c, problems, g)
    if c["op"] == "precondition" and _size(c)[0] * _size(c)[1] > 1.5e8:
        return None                       # dense matrices of this size take too long
    N = _Normal(c, problems)
    if c["op"] in ("once", "solve"):
        return N.solve(b=b)
    if c["op"] == "gradient":
        x = N.solve(b=b)
        lam = N.solve(rhs=x - v)
        al, r = N.a(lam), b - N.a(x)
        return {"x": x, "dLdb": al, "dLdvals": r[N.rows] * lam[N.cols] - al[N.rows] * x[N.cols]}
    if c["op"] == "products":
        return N.a(v), N.at(b)
    if c["op"] == "transpose":
        return None, None, N.vals[torch.sort(N.cols, stable=True).indices], None
    return _one_preconditioner(c, N, problems[0], v)
