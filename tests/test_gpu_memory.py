"""Calls with little device memory left: what needs less than that is still
answered, with the results that it has with plenty.  The rest of the card is
held by tensors meanwhile."""
import contextlib
import ctypes

import numpy as np
import pytest

pytestmark = pytest.mark.gpu
MiB = 1 << 20


@contextlib.contextmanager
def _left(nbytes):
    """About nbytes of device memory free, and nothing cached."""
    import torch
    import paper_2107_09006_amd as L
    L.load_library().lsq2l_release_cache()
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    hold = []
    while (free := torch.cuda.mem_get_info()[0]) > nbytes + 4 * MiB:   # the first reading is low
        hold.append(torch.empty(free - nbytes, dtype=torch.uint8, device="cuda"))
    try:
        yield
    finally:
        del hold
        torch.cuda.empty_cache()


def test_transpose_with_little_memory():
    """2^25 entries: the sort that carries rows and values takes 768 MiB, the
    one that gathers them 256 (and 8 per entry less without values)."""
    import torch
    import paper_2107_09006_amd as L
    m, n, k = 1 << 21, 1 << 20, 16
    nnz = m * k
    g = torch.Generator(device="cuda").manual_seed(1)
    base = torch.randint(0, n - 64, (m, 1), generator=g, device="cuda")
    col = (base + 4 * torch.arange(k, device="cuda")).to(torch.int32).reshape(-1)
    ptr = torch.arange(0, nnz + 1, k, device="cuda", dtype=torch.int32)
    val = torch.randn(nnz, generator=g, device="cuda", dtype=torch.float64)

    def transpose(out):
        lib = L.load_library()
        p = [ctypes.c_void_p(t.data_ptr()) for t in (ptr, col, val, *out)]
        s = lib.lsq2l_transpose(m, n, nnz, *p, None)
        assert s == L.OK, lib.lsq2l_last_error()

    def outputs():
        return (torch.empty(n + 1, dtype=torch.int32, device="cuda"), torch.empty(nnz, dtype=torch.int32, device="cuda"),
                torch.empty(nnz, dtype=torch.float64, device="cuda"), torch.empty(nnz, dtype=torch.int32, device="cuda"))

    full, short = outputs(), outputs()
    transpose(full)
    with _left(512 * MiB):
        transpose(short)
    for a, b in zip(full, short):
        assert torch.equal(a, b)


def test_handle_keeps_no_work_space():
    """A handle with 2^24 entries on 4,096 columns: A and A^T take 28 bytes per
    entry (blocks are up to an eighth larger), all the rest comes from one chunk of
    256 MiB; the sort's 24 bytes per entry do not stay."""
    import torch
    import paper_2107_09006_amd as L
    from workloads import generators as W
    p = W.random_banded(1 << 12, 1 << 17, 4, seed=3, k=128, half_width=200)
    assert p.nnz >= 1 << 24
    lib = L.load_library()
    lib.lsq2l_release_cache()
    before = torch.cuda.mem_get_info()[0]
    s = L.solver_from_problem(p, variant=L.ONE_LEVEL)
    lib.lsq2l_release_cache()
    held = before - torch.cuda.mem_get_info()[0]
    s.close()
    assert held <= 28 * p.nnz * 9 / 8 + (256 + 64) * MiB


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_handle_keeps_one_copy_of_the_factors(precision):
    """What the local solves read (two sweeps of at most factor_tiles tiles each;
    blocks are up to an eighth larger) and A stay; the factors that they are laid
    out from do not.  512 MiB: two chunks for the arrays of up to 64 MiB."""
    import torch
    import paper_2107_09006_amd as L
    from workloads import generators as W
    p = W.random_banded(160000, 320000, 40, seed=9, half_width=200)
    lib = L.load_library()
    lib.lsq2l_release_cache()
    before = torch.cuda.mem_get_info()[0]
    s = L.solver_from_problem(p, variant=L.ONE_LEVEL, precision=L.FP64 if precision == "fp64" else L.MIXED)
    lib.lsq2l_release_cache()
    held = before - torch.cuda.mem_get_info()[0]
    tile = 1024 * (8 if precision == "fp64" else 4)
    two = 2 * tile * s.info()["factor_tiles"]
    assert two > 512 * MiB
    s.close()
    assert held <= (two + 28 * p.nnz) * 9 / 8 + 512 * MiB


def _problem(kind):
    from workloads import generators as W
    if kind == "wide":            # up to four entries per row
        return W.random_banded(160000, 320000, 40, seed=9, half_width=200)
    if kind == "qr":
        return W.random_banded(80000, 160000, 40, seed=9, half_width=200)
    return W.irregular_clustered(100000, 300000, 50, seed=5)      # more, and a row-permuted copy


# MiB free: enough for the least setup, with room for the streams of the local
# solves in the finished handle (3100, 2000) or without (2600, 1450); a setup with
# plenty takes 4,780 and 2,580 (qr: 1850, without streams; 2,580)
@pytest.mark.parametrize("kind,precision,mib", [("wide", "fp64", 3100), ("wide", "fp64", 2600), ("wide", "mixed", 2900),
                                                ("irregular", "fp64", 2000), ("irregular", "fp64", 1450),
                                                ("qr", "fp64", 1850)])
def test_setup_with_little_memory(kind, precision, mib):
    """Products against scipy to rounding (n eps of the sum of magnitudes), and the
    solve's true residual with its own tolerance."""
    import torch
    import paper_2107_09006_amd as L
    p = _problem(kind)
    A = p.scipy()
    dev = [torch.as_tensor(a).cuda() for a in (p.indptr.astype(np.int32), p.indices, p.data)]
    b = torch.as_tensor(p.b).cuda()
    v = torch.as_tensor(np.random.default_rng(2).standard_normal(p.n)).cuda()
    with _left(mib * MiB):
        s = L.Solver(*dev, p.part, p.nparts, p.m, p.n, p.tau,
                     local_factor=L.FACTOR_QR if kind == "qr" else L.FACTOR_CHOLESKY, precision=L.FP64 if precision == "fp64" else L.MIXED)
        x, info, _ = s.solve(b)
        Av, Ab = s.spmv(v), s.spmv(b, True)
        s.close()
    eps = np.finfo(float).eps
    for got, M, u in ((Av, A, v), (Ab, A.T.tocsr(), b)):
        u = u.cpu().numpy()
        assert np.all(np.abs(got.cpu().numpy() - M @ u) <= M.shape[1] * eps * (abs(M) @ np.abs(u)))
    x = x.cpu().numpy()
    assert np.linalg.norm(A.T @ (p.b - A @ x)) <= 10 * p.tol * np.linalg.norm(A.T @ p.b)
