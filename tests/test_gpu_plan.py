"""The device planner (matrices of at least 131,072 entries) against the
definitions of the index sets, of the tile envelope and of the row order's
copy: contiguous, grown and scattered parts, shuffled rows, several instances,
one part, interfaces shared by many parts, and the two forms that are left to the
host planner (a long row that several parts share, many parts in every row).
The sets and counts are whole numbers and equal; the preconditioner, which reads
the overlap map and the pairs, is compared through its symmetry and through the
solution's normal-equation residual, with the solve's own tolerance."""
import numpy as np
import pytest

from workloads import generators as W

pytestmark = pytest.mark.gpu


def _problem(kind):
    rng = np.random.default_rng(11)
    if kind == "irregular":
        return W.irregular_clustered(12000, 24000, 9, seed=5)
    if kind == "grid":
        return W.grid_gradient(220, 6, seed=6)
    if kind == "many":
        p = W.random_banded(3000, 6600, 40, seed=8, k=20)
    else:
        p = W.random_banded(22000, 44000, 1 if kind == "one" else 13, seed=7)
    if kind == "shuffled":
        import scipy.sparse as sp
        A = p.scipy()[rng.permutation(p.m)].tocsr()
        A.sort_indices()
        p.indptr, p.indices, p.data = A.indptr.astype(np.int32), A.indices.astype(np.int32), A.data
    if kind in ("scattered", "many"):
        some = rng.random(p.n) < (0.002 if kind == "scattered" else 1.0)
        p.part = np.where(some, rng.integers(0, p.nparts, p.n), p.part).astype(np.int32)
    if kind == "dense_row":
        import scipy.sparse as sp
        row = sp.random(1, p.n, density=0.22, random_state=3, format="csr")
        A = sp.vstack([p.scipy(), 1e-3 * row]).tocsr()
        A.sort_indices()
        p.m = A.shape[0]
        p.indptr, p.indices, p.data = A.indptr.astype(np.int32), A.indices.astype(np.int32), A.data
        p.b = np.append(p.b, 1.0)
    return p


def _definitions(p):
    """(I, Xi, Gamma) of every part and the stored tiles of all envelopes."""
    A = p.scipy()
    row_of = np.repeat(np.arange(p.m), np.diff(p.indptr))
    sets, tiles = [], 0
    for i in range(p.nparts):
        I = np.flatnonzero(p.part == i)
        xi = np.unique(row_of[p.part[p.indices] == i])
        B = A[xi]
        cols = np.unique(B.indices)
        G = cols[p.part[cols] != i]
        sets.append((I, xi, G))
        nIp = -(-len(I) // 32) * 32
        nt = nIp // 32 + -(-len(G) // 32)
        pos = np.zeros(p.n, dtype=np.int64)
        pos[I] = np.arange(len(I))
        pos[G] = nIp + np.arange(len(G))
        at = pos[B.indices]
        least = np.minimum.reduceat(at, B.indptr[:-1])
        F = np.arange(nt)
        np.minimum.at(F, at // 32, np.repeat(least, np.diff(B.indptr)) // 32)
        tiles += int(np.sum(np.arange(nt) - F + 1))
    return sets, tiles


@pytest.mark.parametrize("kind", ["banded", "shuffled", "irregular", "grid", "scattered", "one", "many", "dense_row"])
def test_plan(kind):
    import torch
    import paper_2107_09006_amd as L
    p = _problem(kind)
    assert p.nnz >= 1 << 17
    wide = kind in ("many", "dense_row")     # interfaces above the selection's limit
    s = L.solver_from_problem(p, variant=L.ONE_LEVEL if wide else L.ADDITIVE)
    sets, tiles = _definitions(p)
    for i, (I, xi, G) in enumerate(sets):
        d = s.subdomain(i)
        assert np.array_equal(d["I"], I) and np.array_equal(d["Xi"], xi) and np.array_equal(d["G"], G)
    assert s.info()["split_tiles"] == tiles
    rng = np.random.default_rng(1)
    u, v = (torch.as_tensor(rng.standard_normal(p.n)).cuda() for _ in range(2))
    Mu, Mv = s.apply_preconditioner(u), s.apply_preconditioner(v)
    a, b = float(u @ Mv), float(v @ Mu)
    assert abs(a - b) <= 1e-9 * float(u.norm() * Mv.norm())
    x = s.solve(torch.as_tensor(p.b).cuda())[0].cpu().numpy()
    A = p.scipy()
    assert np.linalg.norm(A.T @ (p.b - A @ x)) <= 10 * p.tol * np.linalg.norm(A.T @ p.b)
    s.close()


def test_plan_of_a_batch():
    import torch
    import paper_2107_09006_amd as L
    ps = [W.random_banded(9000 + 777 * k, 20000, 4 + k, seed=k) for k in range(3)]
    assert sum(q.nnz for q in ps) >= 1 << 17
    s = L.Solver.batched([(q.indptr, q.indices, q.data, q.part, q.nparts, q.m, q.n) for q in ps], 0.1)
    part = row = col = total = 0
    for q in ps:
        sets, tiles = _definitions(q)
        for i, (I, xi, G) in enumerate(sets):
            d = s.subdomain(part + i)
            assert np.array_equal(d["I"], I + col) and np.array_equal(d["Xi"], xi + row)
            assert np.array_equal(d["G"], G + col)
        part, row, col, total = part + q.nparts, row + q.m, col + q.n, total + tiles
    assert s.info()["split_tiles"] == total
    xs, _, _ = s.solve_batched([torch.as_tensor(q.b).cuda() for q in ps])
    for q, x in zip(ps, xs):
        A, x = q.scipy(), x.cpu().numpy()
        assert np.linalg.norm(A.T @ (q.b - A @ x)) <= 10 * q.tol * np.linalg.norm(A.T @ q.b)
    s.close()
