"""A long instance beside many short ones: every instance converges with its own
true residual, and the long one's vectors get their workgroups whatever lies
beside it.  4,200 instances of 32 columns add an eighth to the columns of the one of
1,000,000; an iteration may take four times as long as without them (1.6 times was
measured for PCG and LSQR; where the workgroups were shared out evenly over the
instances it took nine times as long)."""
import time

import numpy as np
import pytest

from workloads import generators as W

pytestmark = pytest.mark.gpu
COUNT = 4200
TOL = 1e-8


def _iteration(args, b, krylov):
    """Seconds per iteration, the solution and its report."""
    import torch
    import paper_2107_09006_amd as L
    s = L.Solver.batched(args, 0.1, krylov=getattr(L, krylov), tol=TOL / 10 if krylov == "LSQR" else TOL)
    best = np.inf
    for _ in range(4):
        torch.cuda.synchronize()
        t = time.perf_counter()
        x, info, _ = s.solve(b)
        torch.cuda.synchronize()
        best = min(best, time.perf_counter() - t)
    s.close()
    return best / max(i["iterations"] for i in info), x.cpu().numpy(), info


@pytest.mark.parametrize("krylov", ["PCG", "LSQR"])
def test_long_beside_short(krylov):
    import torch
    long = W.random_banded(1000000, 2000000, 500, seed=1)
    short = W.random_banded(32, 64, 1, seed=2)

    def arg(p):
        return (torch.as_tensor(p.indptr.astype(np.int32)).cuda(), torch.as_tensor(p.indices).cuda(),
                torch.as_tensor(p.data).cuda(), p.part, p.nparts, p.m, p.n)

    al, ash = arg(long), arg(short)
    bl, bs = torch.as_tensor(long.b).cuda(), torch.as_tensor(short.b).cuda()
    alone, _, _ = _iteration([al], bl, krylov)
    half = COUNT // 2
    beside, x, info = _iteration([ash] * half + [al] + [ash] * half, torch.cat([bs] * half + [bl] + [bs] * half), krylov)
    at = 0
    for k, i in enumerate(info):
        p = long if k == half else short
        if k in (0, half - 1, half, half + 1, COUNT):
            A = p.scipy()
            rel = np.linalg.norm(A.T @ (p.b - A @ x[at:at + p.n])) / np.linalg.norm(A.T @ p.b)
            assert rel <= TOL * (1 + 1e-6) and abs(rel - i["relres"]) <= 1e-12
        assert i["relres"] <= TOL
        at += p.n
    assert beside <= 4 * alone
