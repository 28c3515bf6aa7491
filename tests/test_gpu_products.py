"""A x and A^T y of matrices whose rows start at unrelated columns, which run on
the row-permuted copy with the m-vector placed or gathered: rows in random
order, empty rows, a row above the LDS block (4,096 entries and more), the other
launch shapes, and a matrix that keeps its order.  Against scipy; a sum of k
products is off by at most about k u times the sum of their magnitudes."""
import numpy as np
import pytest

from workloads import generators as W

pytestmark = pytest.mark.gpu


def _matrix(kind, m, n):
    import scipy.sparse as sp
    p = W.random_banded(n, m - n, 4, seed=m)
    A = p.scipy()
    rng = np.random.default_rng(n)
    if kind != "sorted":
        A = A[rng.permutation(m)]
    if kind == "long_row":
        A = sp.vstack([A[:100], 1e-3 * sp.random(1, n, density=6000 / n, random_state=1, format="csr"), A[100:]])
    if kind == "empty_rows":
        A = sp.vstack([sp.csr_matrix((3, n)), A[:7000], sp.csr_matrix((500, n)), A[7000:], sp.csr_matrix((1, n))])
    A = A.tocsr()
    A.sort_indices()
    return A, p


@pytest.mark.parametrize("shape", [None, (4, 8), (0, 16)])
@pytest.mark.parametrize("kind", ["sorted", "shuffled", "long_row", "empty_rows"])
def test_products(kind, shape):
    import torch
    import paper_2107_09006_amd as L
    A, p = _matrix(kind, 66001, 20011)
    s = L.Solver(A.indptr, A.indices, A.data, p.part, p.nparts, A.shape[0], A.shape[1], p.tau,
                 variant=L.ONE_LEVEL)
    if shape:
        s.autotune(reps=0, shapes=shape)
    rng = np.random.default_rng(0)
    for trans, B in ((False, A), (True, A.T.tocsr())):
        x = rng.standard_normal(B.shape[1])
        y = s.spmv(torch.as_tensor(x).cuda(), trans=trans).cpu().numpy()
        k = max(1, int(np.diff(B.indptr).max()))
        assert np.all(np.abs(y - B @ x) <= 2 * k * 2.0 ** -53 * (abs(B) @ abs(x)))
    s.close()
