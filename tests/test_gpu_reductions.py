"""The reductions of the Krylov methods where their cut changes: one chunk
(1,024 columns), several, more than one group of 16 counted chunks, and
segments of different lengths in a batch.  A wrong sum shows as a residual
that does not reach the tolerance, or as a reported one that is not the true
one: the reported ||A^T (b - A x)|| / ||A^T b|| is a sum of n squares in
double, recomputed here from x, so both agree to the rounding of the residual
itself, eps ||A||^2 ||x|| / ||A^T b|| (below 1e-13 for these matrices)."""
import numpy as np
import pytest

from workloads import generators as W

pytestmark = pytest.mark.gpu
TOL = 1e-9


def _check(p, x, info):
    A = p.scipy()
    rel = np.linalg.norm(A.T @ (p.b - A @ x)) / np.linalg.norm(A.T @ p.b)
    assert rel <= TOL * (1 + 1e-6)
    assert abs(rel - info["relres"]) <= 1e-12


@pytest.mark.parametrize("krylov", ["PCG", "LSQR", "GMRES"])
@pytest.mark.parametrize("sizes", [(1024,), (1025,), (16 * 1024,), (16 * 1024 + 1,), (33, 20000, 1024)])
def test_reductions(krylov, sizes):
    import torch
    import paper_2107_09006_amd as L
    probs = [W.random_banded(n, 2 * n, 2 + n // 2000, seed=n) for n in sizes]
    # LSQR stops on its own estimate: a tenth of TOL leaves the residual below TOL
    opts = dict(tol=TOL / 10 if krylov == "LSQR" else TOL, krylov=getattr(L, krylov))
    args = [(p.indptr, p.indices, p.data, p.part, p.nparts, p.m, p.n) for p in probs]
    s = L.Solver.batched(args, 0.1, **opts)
    b = torch.as_tensor(np.concatenate([p.b for p in probs])).cuda()
    x, info, _ = s.solve(b)
    x = x.cpu().numpy()
    at = 0
    for p, i in zip(probs, info):
        _check(p, x[at:at + p.n], i)
        at += p.n
    s.close()
