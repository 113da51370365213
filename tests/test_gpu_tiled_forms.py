"""The tiled ILU's sweeps against the oracle at every line of their dispatch: up to
1024 tiles and beyond, factors that the 256 MB last-level cache holds and larger
ones, finished layers staged through LDS and (tile_x + tile_y - 1 > 21) not.

Tolerances as for the stages elsewhere: 1e-10 per unknown in FP64, 1e-5 (FP32) and
2^-7 (BF16) of the oracle's emulation of the same form."""
import numpy as np
import pytest

import bo_casegen as cg
from tests import test_gpu_twophase as T2
from tests.gpu_util import rel_err_parts, run_stage, setup_both

pytestmark = pytest.mark.gpu

TOL = {"fp64": 1e-10, "fp32": 1e-5, "bf16": 2.0**-7}


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


def case_of(shape, seed):
    nx, ny, nz = shape
    return cg.tiny_case(nx, ny, nz, seed=seed, step=0.01,
                        wells=[cg.Well(0, 0, 0, nz - 1, "inj", "bhp", 3500.0),
                               cg.Well(nx - 1, ny - 1, 0, nz - 1, "prod", "bhp", 2500.0)])


# (grid, tile, precision): tiles and megabytes that the sweeps read of their factors
# (forward, backward)
FORMS = [
    ((132, 132, 1), (4, 4), "fp64"),     # 1089 tiles, 19 and 24 MB
    ((100, 100, 50), (4, 4), "fp64"),    # 625 tiles, 115 and 148 MB (of 480 and 617 stored)
    ((530, 530, 1), (8, 8), "fp64"),     # 4489 tiles, 491 and 631 MB
    ((530, 530, 1), (8, 8), "fp32"),     # 4489 tiles, 316 MB
    ((700, 700, 1), (8, 8), "bf16"),     # 7744 tiles, 306 MB
    ((265, 265, 3), (8, 8), "fp32"),     # 1156 tiles, 102 MB
    ((265, 265, 3), (8, 8), "bf16"),     # 1156 tiles, 56 MB
    ((256, 256, 12), (8, 8), "fp64"),    # 1024 tiles, 266 and 342 MB
    ((256, 256, 22), (8, 8), "fp32"),    # 1024 tiles, 261 MB
    ((1600, 100, 1), (64, 1), "fp64"),   # 2500 tiles, 273 and 352 MB, not staged
    ((2560, 100, 1), (64, 1), "fp32"),   # 4000 tiles, 281 MB, not staged
    ((600, 30, 2), (1, 24), "fp64"),     # 1200 tiles, 55 and 71 MB, not staged
    ((600, 30, 2), (1, 24), "bf16"),     # 1200 tiles, 34 MB, not staged
]


@pytest.mark.parametrize("shape,tile,prec", FORMS, ids=lambda v: "x".join(map(str, v)) if isinstance(v, tuple) else v)
def test_sweeps_at_every_line_of_the_dispatch(B, O, shape, tile, prec):
    case = case_of(shape, 71)
    v = np.random.default_rng(72).standard_normal(3 * case.n)
    for fpf in (0, 1):  # 1: the last F stage is added to z
        _, _, _, _, _, opc, gpc = setup_both(B, O, case, tile=tile, precision=prec, use_amg=0, fpf=fpf)
        got = run_stage(B, gpc, B.bo_cpr_apply, v, 3 * case.n)
        assert rel_err_parts(got, opc.apply(v)) <= TOL[prec]


@pytest.mark.parametrize("prec", ["fp64", "fp32", "bf16"])
@pytest.mark.parametrize("shape,tile", [((5, 4), (1, 1)), ((33, 32), (1, 1)), ((6, 4), (3, 2))])
def test_sweeps_of_few_steps(B, O, shape, tile, prec):
    """Tiles of one step (four with 3x2 columns) up to four rounds of the sweeps'
    rings of loads and every remainder, few tiles and more than 1024."""
    v = np.random.default_rng(77)
    for nz in range(1, 14):
        case = case_of((*shape, nz), 78)
        r = v.standard_normal(3 * case.n)
        for fpf in (0, 1):
            _, _, _, _, _, opc, gpc = setup_both(B, O, case, tile=tile, precision=prec, use_amg=0, fpf=fpf)
            got = run_stage(B, gpc, B.bo_cpr_apply, r, 3 * case.n)
            assert rel_err_parts(got, opc.apply(r)) <= TOL[prec], nz


@pytest.mark.parametrize("prec", ["fp64", "fp32", "bf16"])
@pytest.mark.parametrize("tile", [(32, 2), (1, 64), (21, 1), (22, 1)])
def test_sweeps_around_the_staging_limit(B, O, tile, prec):
    """Tiles of 21 layers in flight (the last that are staged) and more, with the
    pressure correction added (PF) and all of it added to z (FPF)."""
    case = case_of((70, 66, 5), 73)
    v = np.random.default_rng(74).standard_normal(3 * case.n)
    for fpf in (0, 1):
        _, _, _, _, _, opc, gpc = setup_both(B, O, case, tile=tile, precision=prec, coarse_max=40, fpf=fpf)
        got = run_stage(B, gpc, B.bo_cpr_apply, v, 3 * case.n)
        assert rel_err_parts(got, opc.apply(v)) <= TOL[prec]


@pytest.mark.parametrize("shape,tile", [((530, 530, 1), (8, 8)), ((375, 375, 2), (3, 2))])
def test_two_phase_sweeps_of_many_tiles(B, O, shape, tile):
    """4489 tiles that read 281 MB of factors a sweep, and 23500 of five steps that
    read 115 MB."""
    case = cg.two_phase(case_of(shape, 75))
    v = np.random.default_rng(76).standard_normal(2 * case.n)
    for kw in (dict(use_amg=0), dict(use_amg=0, fpf=1), dict(coarse_max=40)):
        _, _, _, _, _, opc, gpc = T2.setup_both2(B, O, case, tile=tile, **kw)
        got = T2.run(B, gpc, B.bo_cpr_apply, v, 2 * case.n)
        assert rel_err_parts(got, opc.apply(v), parts=2) <= 1e-10
