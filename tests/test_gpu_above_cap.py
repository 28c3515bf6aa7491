"""A subdomain of 19,500 columns, beyond the streams of the local solves (18,944
unknowns), beside one of 2,000: y of the large one in global memory, the small one
through the streams, with Cholesky and QR factors, in both orders and precisions.
z = M r against the oracle within ten times unit roundoff times the condition of the
equilibrated C_ii, and the solve within 1e-8 (FP32 factors: 1e-6), as for the
sizes that the streams hold."""
import numpy as np
import pytest

import oracle as O
from tests.test_gpu_parity import L, _np, _t, assert_close  # noqa: F401
from workloads import generators as W

pytestmark = pytest.mark.gpu
SIZES = (19500, 2000)
U = {"fp64": float(np.finfo(np.float64).eps), "mixed": float(np.finfo(np.float32).eps)}


@pytest.fixture(scope="module")
def above_cap():
    import scipy.sparse as sp
    import scipy.sparse.linalg as spla
    n = sum(SIZES)
    p = W.random_banded(n, 2 * n, 2, seed=94, tau=0.1, half_width=20, name="above_cap")
    p.part = np.repeat(np.arange(2, dtype=np.int32), SIZES)
    orc = O.Oracle(p.scipy(), p.part, 2, p.tau, variant="one_level").setup()
    A, kappa = p.scipy(), 1.0
    for st in orc.sets:
        Ac = A[:, st.Omega]
        C = (Ac.T @ Ac).tocsc()
        d = sp.diags(1.0 / np.sqrt(C.diagonal()))
        Cs = (d @ C @ d).tocsc()
        hi = spla.eigsh(Cs, k=1, which="LA", return_eigenvectors=False)[0]
        lo = spla.eigsh(Cs, k=1, sigma=0.0, which="LM", return_eigenvectors=False)[0]
        kappa = max(kappa, hi / lo)
    r = np.random.default_rng(13).standard_normal(p.n)
    return p, kappa, r, orc.apply(r), orc.solve(p.b, tol=1e-10)["x"]


@pytest.mark.parametrize("order", ["split", "global"])
@pytest.mark.parametrize("precision,factor", [("fp64", "cholesky"), ("mixed", "cholesky"), ("fp64", "qr"), ("mixed", "qr")])
def test_above_the_streams(L, above_cap, order, precision, factor):  # noqa: F811
    p, kappa, r, z, x = above_cap
    s = L.Solver(p.indptr, p.indices, p.data, p.part, 2, p.m, p.n, p.tau, variant=L.ONE_LEVEL, tol=1e-10,
                 precision=L.FP64 if precision == "fp64" else L.MIXED,
                 local_factor=L.FACTOR_QR if factor == "qr" else L.FACTOR_CHOLESKY,
                 solve_order=L.ORDER_SPLIT if order == "split" else L.ORDER_GLOBAL)
    assert s.info()["max_ni"] > 18944
    assert_close(_np(s.apply_preconditioner(_t(r))), z, 10 * U[precision] * kappa)
    got, info, _ = s.solve(_t(p.b))
    assert info[0]["relres"] <= 1e-10
    assert_close(_np(got), x, 1e-8 if precision == "fp64" else 1e-6)
    s.close()
