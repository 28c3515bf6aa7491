"""The assembly of the C_ii where its two forms change course: short and long
rows of A, tile columns with fewer and with more stored tiles than one pass
holds, one tile, padding, more interface columns than fit LDS (1,024) and more
tile rows than the direct slot table (4,096).  With one level the preconditioner
is sum_i R_i^T C_ii^{-1} R_i, compared with scipy's sparse LU; a solve from
correctly assembled matrices is accurate to about u kappa of the equilibrated
C_ii (1-norm estimate), the bound is ten times that."""
import numpy as np
import pytest

from workloads import generators as W

pytestmark = pytest.mark.gpu


def _inverse(C, r):
    import scipy.sparse as sp
    import scipy.sparse.linalg as sla
    s = sp.diags(1.0 / np.sqrt(C.diagonal()))
    E = (s @ C @ s).tocsc()
    lu = sla.splu(E)
    inv = sla.LinearOperator(E.shape, matvec=lu.solve, rmatvec=lambda v: lu.solve(v, "T"), dtype=float)
    return s @ lu.solve(s @ r), sla.norm(E, 1) * sla.onenormest(inv)


@pytest.mark.parametrize("k", [4, 12])
@pytest.mark.parametrize("n,parts,half", [(31, 1, 20), (33, 2, 20), (700, 3, 60), (1600, 1, 1600),
                                          (2600, 2, 2600), (131200, 1, 20)])
def test_local_matrices(n, parts, half, k):
    import torch
    import paper_2107_09006_amd as L
    p = W.random_banded(n, 2 * n, parts, seed=n + k, k=k, half_width=half)
    s = L.solver_from_problem(p, variant=L.ONE_LEVEL)
    r = np.random.default_rng(n).standard_normal(n)
    z = s.apply_preconditioner(torch.as_tensor(r).cuda()).cpu().numpy()
    A = p.scipy().tocsc()
    ref, kappa = np.zeros(n), 1.0
    for i in range(parts):
        d = s.subdomain(i)
        om = np.concatenate([d["I"], d["G"]])
        B = A[:, om]
        zi, ki = _inverse((B.T @ B).tocsc(), r[om])
        ref[om] += zi
        kappa = max(kappa, ki)
    s.close()
    assert np.linalg.norm(z - ref) <= 10 * 2.0 ** -53 * kappa * np.linalg.norm(ref)


@pytest.mark.parametrize("kind", ["grid", "irregular"])
def test_setups_agree_to_the_bit(kind):
    """The products of a column are added in a fixed order: two handles of the
    same matrix apply the same preconditioner, bit for bit."""
    import torch
    import paper_2107_09006_amd as L
    p = W.grid_gradient(60, 3, seed=2) if kind == "grid" else W.irregular_clustered(9000, 18000, 6, seed=2)
    r = torch.as_tensor(np.random.default_rng(5).standard_normal(p.n)).cuda()
    z = []
    for _ in range(2):
        s = L.solver_from_problem(p)
        z.append(s.apply_preconditioner(r).cpu().numpy())
        s.close()
    assert np.array_equal(z[0], z[1])
