"""What the one-pass import of a grid's matrix refuses, and values off a 16-byte
boundary (3x3 and 2x2 blocks)."""
import numpy as np
import pytest

import bo_casegen as cg
from tests import test_gpu_twophase as T2
from tests.gpu_util import device_bsr, oracle_system, ragged_case, run_stage, to_dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    from paper_1606_00556_amd import bo
    bo.lib()
    return bo


@pytest.fixture(scope="module")
def O():
    from oracle import oracle
    oracle.lib()
    return oracle


def system(B, O, bs):
    """(grid, rowptr, colind, values, matrix maker, setup) of a ragged grid's system"""
    if bs == 3:
        case = ragged_case()
        P, rp, ci, val, b = oracle_system(O, case)
        return (case.nx, case.ny, case.nz), rp, ci, val, B.DeviceBsr, B.bo_cpr_setup
    case = T2.ragged2()
    P, rp, ci, val, b = T2.oracle_system(O, case)
    return (case.nx, case.ny, case.nz), rp, ci, val, B.DeviceBsr2, B.bo_cpr2_setup


def matrix(cls, rp, ci, val):
    return cls(to_dev(np.asarray(rp, np.int32)), to_dev(np.asarray(ci, np.int32)),
               to_dev(np.ascontiguousarray(val, np.float64).reshape(-1)))


@pytest.mark.parametrize("bs", [3, 2])
def test_values_off_a_16_byte_boundary(B, O, bs):
    import torch
    g, rp, ci, val, cls, setup = system(B, O, bs)
    n = g[0] * g[1] * g[2]
    flat = np.ascontiguousarray(val, np.float64).reshape(-1)
    buf = torch.zeros(flat.size + 1, dtype=torch.float64, device="cuda")
    buf[1:] = to_dev(flat)
    shifted = cls(to_dev(rp.astype(np.int32)), to_dev(ci.astype(np.int32)), buf[1:])
    assert shifted.val.data_ptr() % 16 == 8
    a, s = setup(matrix(cls, rp, ci, val), g), setup(shifted, g)
    v = np.random.default_rng(61).standard_normal(bs * n)
    assert np.array_equal(B.bo_cpr_copy_weights(a), B.bo_cpr_copy_weights(s))
    assert np.array_equal(run_stage(B, a, B.bo_cpr_apply, v, bs * n), run_stage(B, s, B.bo_cpr_apply, v, bs * n))


@pytest.mark.parametrize("bs", [3, 2])
def test_refusals_and_their_order(B, O, bs):
    """A value that is not finite comes before a wrong pattern, wherever it stands:
    in the rows, in a row whose pattern is wrong, or behind the last row."""
    g, rp, ci, val, cls, setup = system(B, O, bs)
    wrong = ci.copy()
    e = rp[40]
    wrong[e] = ci[e] + 1 if ci[e] + 1 < ci[e + 1] else ci[e] - 1  # not the row's first neighbour
    bad_row = val.copy()
    bad_row[e, 0, 0] = np.nan
    bad_end = val.copy()
    bad_end[-1, -1, -1] = np.inf
    one = np.ones((1, bs, bs))

    def status(ci_, val_):
        with pytest.raises(B.BoError) as err:
            setup(matrix(cls, rp, ci_, val_), g)
        return err.value.status

    assert status(wrong, val) == B.BO_ERR_UNSUPPORTED
    assert status(wrong, bad_row) == B.BO_ERR_NONFINITE
    assert status(wrong, bad_end) == B.BO_ERR_NONFINITE
    assert status(ci, bad_end) == B.BO_ERR_NONFINITE
    # one block more than the rows hold: accepted when it is finite
    longer = np.concatenate([ci, [0]])
    setup(matrix(cls, rp, longer, np.concatenate([val, one])), g)
    assert status(longer, np.concatenate([val, np.nan * one])) == B.BO_ERR_NONFINITE
