"""FP32 factors on subdomains above 12,544 local unknowns: the local solve keeps
its vector and its sums in double.  With one part and one level M r = S y, where
S = 1 / ||A(:, c)|| and y is the solver's vector: a vector held in single
precision would give y = M r / S within 2^-50 of a single-precision number in
every entry, one held in double lies that close in about one of 2^24."""
import numpy as np
import pytest

from workloads import generators as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("order", ["split", "global"])
@pytest.mark.parametrize("n", [12545, 18944])
def test_vector_in_double(n, order):
    import torch
    import paper_2107_09006_amd as L
    p = W.random_banded(n, 2 * n, 1, seed=n)
    s = L.solver_from_problem(p, precision=L.MIXED, variant=L.ONE_LEVEL,
                              solve_order=L.ORDER_SPLIT if order == "split" else L.ORDER_GLOBAL)
    r = np.random.default_rng(n).standard_normal(n)
    z = s.apply_preconditioner(torch.as_tensor(r).cuda()).cpu().numpy()
    s.close()
    A = p.scipy()
    y = z * np.sqrt(np.asarray(A.multiply(A).sum(0)).ravel())
    near = np.abs(y - y.astype(np.float32)) <= 2.0 ** -45 * np.abs(y)
    assert near.mean() < 1e-3
