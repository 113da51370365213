"""The one-pass prefix sum of the setups, through the AMG hierarchy and the
assembly at sizes around its tiles (4096 counts) and its look-back window (64
tiles): row pointers against the oracle's, repeated calls and calls from two
host threads on streams of their own giving the same bits."""
import threading

import numpy as np
import pytest

import bo_casegen as cg
from tests.gpu_util import to_host

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    from paper_1606_00556_amd import bo
    bo.lib()
    return bo


def stencil_rowptr(nx, ny, nz):
    g = np.arange(nx * ny * nz)
    i, j, k = g % nx, (g // nx) % ny, g // (nx * ny)
    c = 1 + (i > 0) + (i < nx - 1) + (j > 0) + (j < ny - 1) + (k > 0) + (k < nz - 1)
    return np.concatenate([[0], np.cumsum(c)])


def assemble(B, case, stream=None):
    import torch
    p = B.problem_from_case(case)
    x = torch.from_numpy(case.x_old).cuda()
    return B.bo_jacobian_bsr(p, x, x, case.dt)


@pytest.mark.parametrize("shape", [(1, 1, 1), (3, 1, 1), (64, 64, 1), (17, 241, 1), (4097, 1, 1), (64, 64, 65),
                                   (128, 64, 33), (90, 91, 64)])
def test_row_pointers_at_tile_edges(B, shape):
    nx, ny, nz = shape
    case = cg.tiny_case(nx, ny, nz, seed=3, wells=[cg.Well(0, 0, 0, nz - 1, "inj", "bhp", 3500.0)])
    ref = stencil_rowptr(nx, ny, nz)
    for _ in range(3):
        J, _ = assemble(B, case)
        assert np.array_equal(to_host(J.rowptr), ref)


def test_scans_from_two_threads(B):
    import torch
    cases = [cg.tiny_case(40, 41, 9, seed=5), cg.tiny_case(64, 64, 33, seed=6)]
    refs = [stencil_rowptr(c.nx, c.ny, c.nz) for c in cases]
    bad = []

    def work(q):
        c = cases[q]
        s = torch.cuda.Stream()
        with torch.cuda.stream(s):
            for _ in range(10):
                J, _ = assemble(B, c)
                pc = B.bo_cpr_setup(J, (c.nx, c.ny, c.nz))
                s.synchronize()
                if not np.array_equal(J.rowptr.cpu().numpy(), refs[q]):
                    bad.append(q)
                pc.close()

    th = [threading.Thread(target=work, args=(q,)) for q in range(2)]
    for t in th:
        t.start()
    for t in th:
        t.join()
    assert not bad


@pytest.mark.parametrize("shape", [(1, 1, 1), (31, 33, 1), (32, 32, 1), (25, 41, 1), (64, 2, 127), (32, 32, 16),
                                   (5, 29, 113)])
def test_row_pointers_without_a_read(B, shape):
    """The sums whose total is not read back (bo_jacobian_bsr_noalloc): one
    workgroup up to 16384 counts, three launches above."""
    import torch
    nx, ny, nz = shape
    case = cg.tiny_case(nx, ny, nz, seed=8, step=0.01, wells=[])
    p = B.problem_from_case(case)
    n, nnzb = B.bo_jacobian_bsr_size(p)
    J = B.DeviceBsr(torch.full((n + 1,), -7, dtype=torch.int32, device="cuda"),
                    torch.full((nnzb,), 123456, dtype=torch.int32, device="cuda"),
                    torch.zeros(9 * nnzb, dtype=torch.float64, device="cuda"))
    b = torch.zeros(3 * n, dtype=torch.float64, device="cuda")
    x = torch.from_numpy(case.x_old).cuda()
    B.bo_jacobian_bsr_noalloc(p, x, x, case.dt, J, b)
    assert np.array_equal(to_host(J.rowptr), stencil_rowptr(nx, ny, nz))
