"""The radix sort behind the transpose at the edges of its tiles (8,192
entries), of its digits (2^11 and 2^22 columns) and of the row table (64
entries per line), against numpy's stable sort: integers and values exact."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("noalloc", [False, True])
@pytest.mark.parametrize("n, nnz", [(1, 70), (2, 1), (2048, 8191), (2049, 8192), (2049, 8193),
                                    (1 << 22, 40001), ((1 << 22) + 1, 40001), (300, 100000)])
def test_transpose_edges(n, nnz, noalloc):
    import torch
    import paper_2107_09006_amd as L
    rng = np.random.default_rng(n + nnz)
    m = max(1, nnz // 3)
    cuts = np.sort(rng.integers(0, nnz + 1, size=m - 1))     # ragged and empty rows
    rowptr = np.concatenate([[0], cuts, [nnz]]).astype(np.int32)
    cols = rng.integers(0, n, size=nnz).astype(np.int32)
    cols[0], cols[-1] = n - 1, 0
    vals = rng.standard_normal(nnz)
    trp, tr, tv, tp = L.transpose(m, n, rowptr, cols, vals, noalloc=noalloc)
    torch.cuda.synchronize()
    perm = np.argsort(cols, kind="stable")
    rows = np.repeat(np.arange(m), np.diff(rowptr))
    assert np.array_equal(tp.cpu().numpy(), perm)
    assert np.array_equal(tr.cpu().numpy(), rows[perm])
    assert np.array_equal(tv.cpu().numpy(), vals[perm])
    assert np.array_equal(trp.cpu().numpy(), np.searchsorted(cols[perm], np.arange(n + 1)))
