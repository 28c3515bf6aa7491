"""The streaming local solve where its layout changes: one, two and three tile
rows, padding, narrow and wide envelopes (the slabs of a step on no helper, on
one or two, on all six), the largest subdomain held in LDS (18,944 unknowns)
and the first one solved in global memory, in both orders and precisions.  With
one part the preconditioner is C^{-1}, with several and one level it is
sum_i R_i^T C_ii^{-1} R_i; both are compared with scipy's sparse LU.  A factored
solve in precision u is accurate to about u kappa of the equilibrated matrix
(1-norm estimate here); the bound is ten times that, as for the other tests of
M r."""
import numpy as np
import pytest

from workloads import generators as W

pytestmark = pytest.mark.gpu


def _oracle(C, r):
    """C^{-1} r and the 1-norm condition estimate of the equilibrated C."""
    import scipy.sparse as sp
    import scipy.sparse.linalg as sla
    s = sp.diags(1.0 / np.sqrt(C.diagonal()))
    E = (s @ C @ s).tocsc()
    lu = sla.splu(E)
    inv = sla.LinearOperator(E.shape, matvec=lu.solve, rmatvec=lambda v: lu.solve(v, "T"), dtype=float)
    return s @ lu.solve(s @ r), sla.norm(E, 1) * sla.onenormest(inv)


def _check(p, precision, order):
    import torch
    import paper_2107_09006_amd as L
    s = L.solver_from_problem(p, precision=precision, solve_order=order, variant=L.ONE_LEVEL)
    r = np.random.default_rng(p.n).standard_normal(p.n)
    z = s.apply_preconditioner(torch.as_tensor(r).cuda()).cpu().numpy()
    A = p.scipy().tocsc()
    ref, kappa = np.zeros(p.n), 1.0
    for i in range(p.nparts):
        d = s.subdomain(i)
        om = np.concatenate([d["I"], d["G"]])
        B = A[:, om]
        zi, k = _oracle((B.T @ B).tocsc(), r[om])
        ref[om] += zi
        kappa = max(kappa, k)
    s.close()
    u = 2.0 ** -53 if precision == L.FP64 else 2.0 ** -24
    assert np.linalg.norm(z - ref) <= 10 * u * kappa * np.linalg.norm(ref)


@pytest.mark.parametrize("mixed", [False, True])
@pytest.mark.parametrize("split", [False, True])
@pytest.mark.parametrize("n", [31, 32, 33, 64, 65, 97, 1000, 18944, 18945])
def test_one_subdomain(n, split, mixed):
    import paper_2107_09006_amd as L
    _check(W.random_banded(n, 2 * n, 1, seed=n), L.MIXED if mixed else L.FP64,
           L.ORDER_SPLIT if split else L.ORDER_GLOBAL)


@pytest.mark.parametrize("mixed", [False, True])
@pytest.mark.parametrize("split", [False, True])
@pytest.mark.parametrize("kind", ["banded", "wide", "irregular"])
def test_several_subdomains(kind, split, mixed):
    import paper_2107_09006_amd as L
    p = {"banded": lambda: W.random_banded(3001, 6002, 7, seed=3),
         "wide": lambda: W.random_banded(2000, 4000, 3, seed=4, half_width=150),
         "irregular": lambda: W.small_config("irregular")}[kind]()
    _check(p, L.MIXED if mixed else L.FP64, L.ORDER_SPLIT if split else L.ORDER_GLOBAL)
