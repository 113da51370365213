"""The BSR products of the caller's matrices on rows of every length."""
import numpy as np
import pytest

from tests.gpu_util import to_dev, to_host

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    from paper_1606_00556_amd import bo
    bo.lib()
    return bo


@pytest.mark.parametrize("rows", [1, 63, 64, 65, 200])
@pytest.mark.parametrize("bs", [2, 3])
@pytest.mark.parametrize("shift", [0, 1])
def test_bsr_spmv_rows_of_every_length(B, bs, rows, shift):
    """Block rows of 0 to 40 blocks and one of 1500 (several chunks of the
    kernel's staging) around its 64-row workgroups, values on a 16-byte boundary
    and off one, beta zero and not: bit for bit the row sums in stored order on
    integer data, to 1e-14 of each sum's own magnitude on random data."""
    import torch
    rng = np.random.default_rng(100 * bs + rows + shift)
    ln = rng.integers(0, 41, rows)
    ln[rows // 2] = 1500
    nc = 2000
    rp = np.concatenate([[0], np.cumsum(ln)]).astype(np.int32)
    ci = np.concatenate([np.sort(rng.choice(nc, m, replace=False)) for m in ln]).astype(np.int32)
    for integer in (True, False):
        draw = (lambda *s: rng.integers(-8, 9, s).astype(np.float64)) if integer else (lambda *s: rng.standard_normal(s))
        val, x, y0 = draw(int(rp[-1]), bs, bs), draw(nc, bs), draw(rows, bs)
        buf = torch.zeros(val.size + 1, dtype=torch.float64, device="cuda")
        buf[shift:shift + val.size] = to_dev(val.reshape(-1))
        A = (B.DeviceBsr2 if bs == 2 else B.DeviceBsr)(to_dev(rp), to_dev(ci), buf[shift:shift + val.size])
        prod = np.einsum("eij,ej->ei", val, x[ci])
        mag = np.einsum("eij,ej->ei", np.abs(val), np.abs(x[ci]))
        at = np.repeat(np.arange(rows), ln)
        ax, am = np.zeros((rows, bs)), np.zeros((rows, bs))
        np.add.at(ax, at, prod)
        np.add.at(am, at, mag)
        for alpha, beta in ((-1.0, 1.0), (2.0, 0.0)):
            y = to_dev(y0.reshape(-1).copy())
            (B.bo_bsr2_spmv if bs == 2 else B.bo_bsr_spmv)(A, alpha, to_dev(x.reshape(-1)), beta, y)
            got, ref = to_host(y).reshape(rows, bs), alpha * ax + beta * y0
            if integer:
                assert np.array_equal(got, ref)
            else:
                # a sum of m terms: at most m eps of the terms' magnitudes
                assert np.all(np.abs(got - ref) <= 4500 * 2.3e-16 * (2.0 * am + np.abs(y0)))


def test_bsr2_spmv_of_as_many_rows_and_blocks_as_an_index_holds(B):
    """2^31 - 1 rows of one block each: row and block numbers up to the largest
    32-bit index (119 GB of operands)."""
    import torch
    n = 2**31 - 1
    dev = "cuda"
    A = B.DeviceBsr2(torch.arange(n + 1, dtype=torch.int32, device=dev),
                     torch.zeros(n, dtype=torch.int32, device=dev),
                     torch.ones(4 * n, dtype=torch.float64, device=dev))
    x = torch.tensor([1.0, 2.0], dtype=torch.float64, device=dev)
    y = torch.full((2 * n,), float("nan"), dtype=torch.float64, device=dev)
    B.bo_bsr2_spmv(A, 2.0, x, 0.0, y)
    try:
        assert all(bool((c == 6.0).all()) for c in y.split(1 << 28))
    finally:
        del A, y
        torch.cuda.empty_cache()


@pytest.mark.parametrize("shift", [0, 1])
@pytest.mark.parametrize("bs", [2, 3])
@pytest.mark.parametrize("rows,lengths", [(24576, (6, 8)), (24577, (6, 8)), (131073, (2, 8))])
def test_bsr_spmv_staged_rows(B, bs, rows, lengths, shift):
    """The products whose blocks are staged: the first size that is staged of 7-point
    and of shorter rows (long ones first, so that some workgroups fill their chunk),
    with rows of 600 blocks, empty rows and a ragged last workgroup."""
    import torch
    rng = np.random.default_rng(7 * bs + rows + shift)
    lo, hi = lengths
    ln = rng.integers(lo, hi, rows)
    if lo == 2:
        ln[:rows // 2], ln[rows // 2:] = 8, 2
    ln[1000:1100] = 0
    ln[[70, 71, rows - 1]] = 600
    rp = np.concatenate([[0], np.cumsum(ln)]).astype(np.int32)
    assert 4 * rows <= rp[-1] < 8 * rows and (rp[-1] > 6 * rows) == (lo == 6)
    ci = rng.integers(0, rows, rp[-1]).astype(np.int32)
    val = rng.integers(-8, 9, (int(rp[-1]), bs, bs)).astype(np.float64)
    x, y0 = rng.integers(-8, 9, (rows, bs)).astype(np.float64), rng.integers(-8, 9, (rows, bs)).astype(np.float64)
    buf = torch.zeros(val.size + 1, dtype=torch.float64, device="cuda")
    buf[shift:shift + val.size] = to_dev(val.reshape(-1))
    A = (B.DeviceBsr2 if bs == 2 else B.DeviceBsr)(to_dev(rp), to_dev(ci), buf[shift:shift + val.size])
    ax = np.zeros((rows, bs))
    np.add.at(ax, np.repeat(np.arange(rows), ln), np.einsum("eij,ej->ei", val, x[ci]))
    for alpha, beta in ((-1.0, 1.0), (2.0, 0.0)):
        y = to_dev(y0.reshape(-1).copy())
        (B.bo_bsr2_spmv if bs == 2 else B.bo_bsr_spmv)(A, alpha, to_dev(x.reshape(-1)), beta, y)
        assert np.array_equal(to_host(y).reshape(rows, bs), alpha * ax + beta * y0)
