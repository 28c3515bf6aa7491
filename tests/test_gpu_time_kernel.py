"""Bytes that ``time_kernel`` reports for the local solves, where a subdomain
lies beyond the streaming kernel's largest one (18,944 local unknowns).  Such a
subdomain is priced by its stored tiles, read in both sweeps, and 40 bytes per
(padded) unknown for the gather and the result; uncoupled parts add up.  All are
whole numbers below 2^53 and equal."""
import numpy as np
import pytest

from workloads import generators as W

pytestmark = pytest.mark.gpu
N_BIG, N_SMALL = 19500, 2000


def _bytes(p, **opts):
    import paper_2107_09006_amd as L
    s = L.solver_from_problem(p, variant=L.ONE_LEVEL, **opts)
    ms, by = s.time_kernel(2, reps=1)
    tiles = s.info()["factor_tiles"]
    s.close()
    assert ms > 0
    return by, tiles


@pytest.mark.parametrize("order", ["split", "global"])
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_bytes_beyond_the_streams(order, precision):
    import scipy.sparse as sp
    import paper_2107_09006_amd as L
    opts = dict(precision=L.FP64 if precision == "fp64" else L.MIXED,
                solve_order=L.ORDER_SPLIT if order == "split" else L.ORDER_GLOBAL)
    big = W.random_banded(N_BIG, 2 * N_BIG, 1, seed=5)
    small = W.random_banded(N_SMALL, 2 * N_SMALL, 1, seed=6)
    by_big, tiles = _bytes(big, **opts)
    entry = 8 if precision == "fp64" else 4
    assert by_big == 2 * entry * 1024 * tiles + 40 * (-(-N_BIG // 32) * 32)
    by_small, _ = _bytes(small, **opts)
    both = W.random_banded(N_BIG + N_SMALL, 2 * (N_BIG + N_SMALL), 2, seed=7)
    A = sp.block_diag([big.scipy(), small.scipy()]).tocsr()
    A.sort_indices()
    both.indptr, both.indices, both.data = A.indptr.astype(np.int32), A.indices.astype(np.int32), A.data
    both.part = np.repeat(np.array([0, 1], np.int32), [N_BIG, N_SMALL])
    assert _bytes(both, **opts)[0] == by_big + by_small
