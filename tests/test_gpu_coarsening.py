"""The coarsening against the oracle's at the sizes where its kernels change
form: level 0 of a plain grid from its slot arrays (lines, plates, grids below
and above a workgroup), coarsest matrices on both sides of the register
elimination's thread counts, and rows of the general form on both sides of what
a wavefront holds in one, two, four and eight registers (a rate well through
many layers)."""
import dataclasses

import numpy as np
import pytest

import bo_casegen as cg
from tests.gpu_util import device_bsr, rel_err, run_stage, setup_both

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


def check_levels(B, opc, gpc):
    nl = opc.nlevels()
    assert B.bo_cpr_levels(gpc) == nl
    for l in range(nl):
        ol, gl = opc.level(l), B.bo_cpr_level_copy(gpc, l)
        assert gl["n"] == ol["n"] and gl["nnz"] == ol["nnz"]
        assert np.array_equal(gl["rowptr"], ol["rowptr"]) and np.array_equal(gl["colind"], ol["colind"])
        assert rel_err(gl["val"], ol["val"]) <= 1e-12
        if l < nl - 1:
            assert np.array_equal(gl["agg"], ol["agg"]) and np.array_equal(gl["root"], ol["root"])
            assert np.array_equal(gl["p_rowptr"], ol["p_rowptr"])
            assert np.array_equal(gl["p_colind"], ol["p_colind"])
            assert rel_err(gl["p_val"], ol["p_val"]) <= 1e-12
            assert gl["omega"] == pytest.approx(ol["omega"], rel=1e-14)
    return nl


@pytest.mark.parametrize("dims", [(300, 1, 1), (1, 1, 70), (1, 40, 9), (37, 1, 11), (16, 16, 1), (23, 12, 5)])
def test_level0_from_slots(B, O, dims):
    case = cg.tiny_case(*dims, seed=61, step=0.01)
    _, _, _, _, _, opc, gpc = setup_both(B, O, case, coarse_max=10)
    assert check_levels(B, opc, gpc) >= 2
    r = np.random.default_rng(3).standard_normal(case.n)
    assert rel_err(run_stage(B, gpc, B.bo_cpr_vcycle, r, case.n), opc.vcycle(r)) <= 1e-10


@pytest.mark.parametrize("n", [1, 2, 16, 31, 32, 33, 64, 65, 96, 97, 128, 129, 160, 161, 192])
def test_coarsest_inverse_sizes(B, O, n):
    """A grid of n cells that is its own coarsest level: the cycle applies the
    dense inverse."""
    case = cg.tiny_case(n, 1, 1, seed=62, step=0.01)
    _, _, _, _, _, opc, gpc = setup_both(B, O, case, coarse_max=192)
    assert check_levels(B, opc, gpc) == 1
    r = np.random.default_rng(4).standard_normal(n)
    assert rel_err(run_stage(B, gpc, B.bo_cpr_vcycle, r, n), opc.vcycle(r)) <= 1e-10


@pytest.mark.parametrize("nz", [15, 16, 62, 63, 64, 127, 128, 255, 256, 511, 512])
def test_long_prolongator_rows(B, O, nz):
    """A rate well through nz layers: a pressure row of nz + 1 entries."""
    case = cg.tiny_case(3, 3, nz, seed=63, step=0.01, wells=[cg.Well(1, 1, 0, nz - 1, "prod", "lrat", 500.0)])
    case = dataclasses.replace(case, x_old=np.concatenate([case.x_old, [2800.0, 0.0, 0.0]]),
                               x_new=np.concatenate([case.x_new, [2800.0, 0.0, 0.0]]))
    P = O.Problem(case)
    rp, ci, val, _ = O.jacobian(P)
    assert rp[-1] - rp[-2] == nz + 1
    opc = O.Cpr(P, rp, ci, val, ftype=O.F_BJ, smoother=O.SMOOTH_L1, npr=P.rows, coarse_max=20)
    opts = B.bo_cpr_default_opts(ftype=B.BO_F_BJ, smoother=B.BO_SMOOTH_L1, npr=P.rows, coarse_max=20)
    gpc = B.bo_cpr_setup(device_bsr(B, rp, ci, val), None, opts)
    assert check_levels(B, opc, gpc) >= 2
    r = np.random.default_rng(5).standard_normal(P.rows)
    assert rel_err(run_stage(B, gpc, B.bo_cpr_vcycle, r, P.rows), opc.vcycle(r)) <= 1e-10
