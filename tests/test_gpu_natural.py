"""GPU parity of the natural-order block ILU(0) F stage (BO_F_ILU_NATURAL:
Section 3.2's ILU(0) over the whole system, no coupling dropped, applied by
level scheduling over the grid's hyperplanes) against the oracle's IKJ block
ILU(0) in natural order:

  - the F stage per unknown (Po, Sw, Sg separately) to 1e-10 on a plain grid
    (several hyperplane lengths, ragged x and y), on a grid with fixed-rate
    well rows (cell-well couplings inside the factorisation) and on the
    condensed dual-porosity form's reduced system;
  - CPR (PF and FPF) built on it to 1e-10, and FGMRES: true residual <= 1e-6
    with an iteration count within max(1, ceil(0.1 * oracle)) of the
    oracle's;
  - bo_cpr_update gives the bits of a fresh setup; the forms it does not
    take are refused."""
import math

import numpy as np
import pytest

import bo_casegen as cg
from tests.gpu_util import device_bsr, rel_err_parts, run_stage, to_dev, to_host

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


def plain_case():
    return cg.tiny_case(19, 13, 6, seed=31, step=0.01,
                        wells=[cg.Well(0, 0, 0, 5, "inj", "bhp", 3500.0),
                               cg.Well(18, 12, 0, 5, "prod", "bhp", 2500.0)])


def rate_case():
    # two vertical fixed-rate wells: their rows follow the cells, and each
    # perforated cell's block towards its well is updated by the elimination
    # of the perforation above it
    return cg.tiny_case(19, 13, 6, seed=32, step=0.01,
                        wells=[cg.Well(0, 0, 0, 5, "inj", "wrat", 800.0),
                               cg.Well(18, 12, 0, 5, "prod", "lrat", 600.0),
                               cg.Well(9, 6, 1, 4, "prod", "bhp", 2600.0)])


def dual_rate_case():
    nx, ny, nz = 19, 13, 5
    wells = [cg.Well(0, 0, 0, nz - 1, "inj", "wrat", 900.0), cg.Well(nx - 1, ny - 1, 0, nz - 1, "prod", "lrat", 700.0),
             cg.Well(nx // 2, ny // 2, 1, nz - 2, "prod", "bhp", 2500.0)]
    return cg.make_dual_case(nx, ny, nz, seed=17, wells=wells)


def with_rate_unknowns(case):
    """Appends the fixed-rate wells' unknowns (p_h, 0, 0) to the state."""
    import dataclasses
    if case.dual or not case.nrate:
        return case
    extra = np.tile(np.array([3000.0, 0.0, 0.0]), case.nrate)
    return dataclasses.replace(case, x_old=np.concatenate([case.x_old, extra]),
                               x_new=np.concatenate([case.x_new, extra]))


def build(B, O, case, fpf=0, condensed=False, coarse_max=40):
    case = with_rate_unknowns(case)
    P = O.Problem(case)
    rp, ci, val, R = O.jacobian(P)
    A = device_bsr(B, rp, ci, val)
    if condensed:
        sm_o = O.SMOOTH_L1 if case.nrate else O.SMOOTH_GS
        opc = O.Condensed(P, rp, ci, val, ftype=O.F_ILU_NATURAL, smoother=sm_o, fpf=fpf, coarse_max=coarse_max)
        opts = B.bo_cpr_default_opts(condense=1, fpf=fpf, ftype=B.BO_F_ILU_NATURAL, smoother=B.BO_SMOOTH_L1,
                                     coarse_max=coarse_max)
        gpc = B.bo_cpr_setup(A, (case.nx, case.ny, case.nz, 1), opts)
    elif case.nrate:
        opc = O.Cpr(P, rp, ci, val, ftype=O.F_ILU_NATURAL, smoother=O.SMOOTH_L1, fpf=fpf, coarse_max=coarse_max)
        opts = B.bo_cpr_default_opts(ftype=B.BO_F_ILU_NATURAL, smoother=B.BO_SMOOTH_L1, fpf=fpf,
                                     coarse_max=coarse_max)
        gpc = B.bo_cpr_setup(A, (case.nx, case.ny, case.nz), opts)
    else:
        opc = O.Cpr(P, rp, ci, val, ftype=O.F_ILU_NATURAL, fpf=fpf, coarse_max=coarse_max)
        opts = B.bo_cpr_default_opts(ftype=B.BO_F_ILU_NATURAL, fpf=fpf, coarse_max=coarse_max)
        gpc = B.bo_cpr_setup(A, (case.nx, case.ny, case.nz), opts)
    return case, P, rp, ci, val, -R, opc, gpc


CASES = {"plain": (plain_case, False), "rate_wells": (rate_case, False), "condensed": (dual_rate_case, True),
         "condensed_cfg4_twin8": (lambda: cg.make_cfg4(1, scale=8), True)}


@pytest.mark.parametrize("name", list(CASES))
def test_natural_fstage_matches_oracle(B, O, name):
    make, condensed = CASES[name]
    case, P, rp, ci, val, b, opc, gpc = build(B, O, make(), condensed=condensed)
    rng = np.random.default_rng(5)
    if condensed:
        nr = case.n + case.nrate
        vr = opc.reduce(rng.standard_normal(3 * P.rows))
        got = run_stage(B, gpc, B.bo_cpr_fstage, vr, 3 * nr)
        assert rel_err_parts(got, opc.cpr.fstage(vr)) <= 1e-10
    else:
        for v in (rng.standard_normal(3 * P.rows), b):
            got = run_stage(B, gpc, B.bo_cpr_fstage, v, 3 * P.rows)
            assert rel_err_parts(got, opc.fstage(v)) <= 1e-10


def test_natural_unit_responses(B, O):
    """Unit vectors at a corner cell, an interior cell, a perforated cell and
    a well row: the response spreads through every later hyperplane in the
    forward sweep and every earlier one in the backward sweep."""
    case, P, rp, ci, val, b, opc, gpc = build(B, O, rate_case())
    N = case.n
    for row in (0, 7 + 19 * 5 + 19 * 13 * 3, N - 1, 19 * 13 * 2, N, P.rows - 1):
        for q in range(3):
            v = np.zeros(3 * P.rows)
            v[3 * row + q] = 1.0
            got = run_stage(B, gpc, B.bo_cpr_fstage, v, 3 * P.rows)
            assert rel_err_parts(got, opc.fstage(v)) <= 1e-10, (row, q)


@pytest.mark.parametrize("name", list(CASES))
@pytest.mark.parametrize("fpf", [0, 1])
def test_natural_cpr_apply_matches_oracle(B, O, name, fpf):
    make, condensed = CASES[name]
    case, P, rp, ci, val, b, opc, gpc = build(B, O, make(), fpf=fpf, condensed=condensed)
    v = np.random.default_rng(6).standard_normal(3 * P.rows)
    for vec in (v, b):
        assert rel_err_parts(run_stage(B, gpc, B.bo_cpr_apply, vec, 3 * P.rows), opc.apply(vec)) <= 1e-10


@pytest.mark.parametrize("name", list(CASES))
def test_natural_solve_matches_oracle(B, O, name):
    import torch
    make, condensed = CASES[name]
    case, P, rp, ci, val, b, opc, gpc = build(B, O, make(), fpf=1, condensed=condensed)
    if condensed:
        xo, oinfo = O.condensed_fgmres(rp, ci, val, b, opc)
    else:
        xo, oinfo = O.fgmres(rp, ci, val, b, opc)
    x = torch.zeros(3 * P.rows, dtype=torch.float64, device="cuda")
    info = B.bo_fgmres_solve(gpc, gpc.A, to_dev(b), x)
    xg = to_host(x)
    true_rel = np.linalg.norm(b - O.bsr_spmv(rp, ci, val, xg)) / np.linalg.norm(b)
    print(f"{name}: iterations gpu {info['iterations']} oracle {oinfo['iterations']}, true rel {true_rel:.2e}")
    assert info["converged"] and true_rel <= 1e-6
    io = oinfo["iterations"]
    assert abs(info["iterations"] - io) <= max(1, math.ceil(0.1 * io))


def test_natural_update_equals_fresh_setup(B, O):
    import torch
    c1 = with_rate_unknowns(rate_case())
    c2 = with_rate_unknowns(cg.tiny_case(19, 13, 6, seed=33, step=0.02, wells=rate_case().wells))
    opts = B.bo_cpr_default_opts(ftype=B.BO_F_ILU_NATURAL, smoother=B.BO_SMOOTH_L1, fpf=1, coarse_max=40)
    grid = (c1.nx, c1.ny, c1.nz)
    mats = []
    for c in (c1, c2):
        rp, ci, val, R = O.jacobian(O.Problem(c))
        mats.append(device_bsr(B, rp, ci, val))
    pc = B.bo_cpr_setup(mats[0], grid, opts)
    B.bo_cpr_update(pc, mats[1])
    fresh = B.bo_cpr_setup(mats[1], grid, opts)
    v = to_dev(np.random.default_rng(7).standard_normal(3 * (c1.n + c1.nrate)))
    z1 = torch.zeros_like(v)
    z2 = torch.zeros_like(v)
    B.bo_cpr_apply(pc, v, z1)
    B.bo_cpr_apply(fresh, v, z2)
    assert torch.equal(z1, z2)


def test_natural_refusals(B, O):
    case = with_rate_unknowns(rate_case())
    rp, ci, val, R = O.jacobian(O.Problem(case))
    A = device_bsr(B, rp, ci, val)
    grid = (case.nx, case.ny, case.nz)
    for prec in (B.BO_PREC_FP32, B.BO_PREC_FP32_BF16):
        with pytest.raises(B.BoError):
            B.bo_cpr_setup(A, grid, B.bo_cpr_default_opts(ftype=B.BO_F_ILU_NATURAL, smoother=B.BO_SMOOTH_L1,
                                                          precision=prec))
    with pytest.raises(B.BoError):  # no grid
        B.bo_cpr_setup(A, None, B.bo_cpr_default_opts(ftype=B.BO_F_ILU_NATURAL, smoother=B.BO_SMOOTH_L1))
    d = dual_rate_case()
    drp, dci, dval, _ = O.jacobian(O.Problem(d))
    with pytest.raises(B.BoError):  # the extended form: matrix cells
        B.bo_cpr_setup(device_bsr(B, drp, dci, dval), (d.nx, d.ny, d.nz, 1),
                       B.bo_cpr_default_opts(ftype=B.BO_F_ILU_NATURAL, smoother=B.BO_SMOOTH_L1))


@pytest.mark.parametrize("shape", [(1, 1, 7), (8, 8, 3), (9, 17, 1), (17, 3, 4), (33, 25, 9), (403, 405, 2)])
def test_natural_tiles_hand_over_every_edge(B, O, shape):
    """The plain grid's sweeps run tile by tile (8x8 columns) with the edge
    values handed over: one column, one full tile, single columns past a tile's
    edge, several tiles each way, and 2601 tiles (more than the chip holds at
    once); repeated applications, also through a captured graph's replay in a
    solve, give the same bits, and a rebuilt handle those of a fresh one."""
    import torch
    nx, ny, nz = shape
    mats = []
    for seed in (41, 42):
        case = cg.tiny_case(nx, ny, nz, seed=seed, step=0.01, wells=[cg.Well(0, 0, 0, nz - 1, "inj", "bhp", 3500.0)])
        P = O.Problem(case)
        rp, ci, val, R = O.jacobian(P)
        mats.append((P, rp, ci, val, device_bsr(B, rp, ci, val)))
    P, rp, ci, val, A = mats[0]
    opc = O.Cpr(P, rp, ci, val, ftype=O.F_ILU_NATURAL, use_amg=0)
    opts = B.bo_cpr_default_opts(ftype=B.BO_F_ILU_NATURAL, use_amg=0)
    gpc = B.bo_cpr_setup(A, (nx, ny, nz), opts)
    v = np.random.default_rng(8).standard_normal(3 * case.n)
    ref = opc.fstage(v)
    first = None
    for _ in range(3):
        got = run_stage(B, gpc, B.bo_cpr_fstage, v, 3 * case.n)
        assert rel_err_parts(got, ref) <= 1e-10
        first = got if first is None else first
        assert np.array_equal(got, first)
    xs = []
    for graph in (0, 1):
        x = torch.zeros(3 * case.n, dtype=torch.float64, device="cuda")
        B.bo_fgmres_solve(gpc, A, to_dev(v), x, B.bo_fgmres_default_opts(graph=graph, maxit=5))
        xs.append(to_host(x))
    assert np.array_equal(xs[0], xs[1])
    B.bo_cpr_update(gpc, mats[1][4])
    fresh = B.bo_cpr_setup(mats[1][4], (nx, ny, nz), opts)
    assert np.array_equal(run_stage(B, gpc, B.bo_cpr_fstage, v, 3 * case.n),
                          run_stage(B, fresh, B.bo_cpr_fstage, v, 3 * case.n))


@pytest.mark.parametrize("shape", [(1, 1, 1), (70, 1, 1), (1, 37, 2), (65, 66, 1), (9, 1, 40), (24, 16, 2)])
def test_natural_thin_grids(B, O, shape):
    """Grids of one layer, one column or one cell: fewer rows than the steps in
    flight, tiles of one column and of one row of columns."""
    nx, ny, nz = shape
    case = cg.tiny_case(nx, ny, nz, seed=43, step=0.01, wells=[cg.Well(0, 0, 0, nz - 1, "inj", "bhp", 3500.0)])
    P = O.Problem(case)
    rp, ci, val, R = O.jacobian(P)
    opc = O.Cpr(P, rp, ci, val, ftype=O.F_ILU_NATURAL, use_amg=0)
    gpc = B.bo_cpr_setup(device_bsr(B, rp, ci, val), shape,
                         B.bo_cpr_default_opts(ftype=B.BO_F_ILU_NATURAL, use_amg=0))
    v = np.random.default_rng(9).standard_normal(3 * case.n)
    for _ in range(2):
        got = run_stage(B, gpc, B.bo_cpr_fstage, v, 3 * case.n)
        assert rel_err_parts(got, opc.fstage(v)) <= 1e-10


@pytest.mark.parametrize("shape", [(256, 256, 1), (2048, 8, 2), (64, 64, 16)])
def test_natural_storage_per_cell(B, O, shape):
    """The factors take one slot a cell (51 pairs of doubles), whatever the
    number of layers, and the edge places a row a layer: measured through a
    caller's allocator against the block-Jacobi handle (9 doubles a cell)."""
    import torch
    nx, ny, nz = shape
    case = cg.tiny_case(nx, ny, nz, seed=44, step=0.01, wells=[cg.Well(0, 0, 0, nz - 1, "inj", "bhp", 3500.0)])
    rp, ci, val, R = O.jacobian(O.Problem(case))
    A = device_bsr(B, rp, ci, val)

    def bytes_of(ftype):
        live = {}

        def alloc(nbytes, stream):
            t = torch.empty(max(nbytes, 1), dtype=torch.uint8, device="cuda")
            live[t.data_ptr()] = t
            return t.data_ptr()

        pc = B.bo_cpr_setup(A, shape, B.bo_cpr_default_opts(ftype=ftype, use_amg=0),
                            allocator=(alloc, lambda ptr, stream: live.pop(ptr)))
        total = sum(t.numel() for t in live.values())
        pc.close()
        return total

    tiles = -(-nx // 8) * -(-ny // 8)
    places = tiles * (nz + 1) * 3 * 64 * 8
    extra = bytes_of(B.BO_F_ILU_NATURAL) - bytes_of(B.BO_F_BJ) + 72 * case.n
    assert extra <= 51 * 16 * case.n + places + (1 << 17), extra / case.n


def test_natural_expired_wait_is_reported(B, O):
    """With no looks allowed beyond the first the waits for neighbouring tiles run
    out (every kernel still ends): applications give NaN, both solvers and a
    rebuild say so, and a rebuild with the default limit is as good as new."""
    import torch
    shape = (104, 104, 3)
    case = cg.tiny_case(*shape, seed=45, step=0.01, wells=[cg.Well(0, 0, 0, 2, "inj", "bhp", 3500.0)])
    P = O.Problem(case)
    rp, ci, val, R = O.jacobian(P)
    A = device_bsr(B, rp, ci, val)
    opts = B.bo_cpr_default_opts(ftype=B.BO_F_ILU_NATURAL, use_amg=0)
    pc = B.bo_cpr_setup(A, shape, opts)
    v = np.random.default_rng(10).standard_normal(3 * case.n)
    good = run_stage(B, pc, B.bo_cpr_fstage, v, 3 * case.n)
    assert np.isfinite(good).all()
    with pytest.raises(B.BoError) as e:
        B.bo_cpr_wait_limit(pc, -1)
    assert e.value.status == B.BO_ERR_INVALID_ARG
    B.bo_fgmres_solve(pc, A, to_dev(v), torch.zeros(3 * case.n, dtype=torch.float64, device="cuda"),
                      B.bo_fgmres_default_opts(graph=1, maxit=2))  # (a captured graph holds the old limit)
    B.bo_cpr_wait_limit(pc, 0)
    solves = [lambda x: B.bo_fgmres_solve(pc, A, to_dev(v), x, B.bo_fgmres_default_opts(graph=1)),
              lambda x: B.bo_fgmres_solve(pc, A, to_dev(v), x, B.bo_fgmres_default_opts(orth=1)),
              lambda x: B.bo_bicgstab_solve(pc, A, to_dev(v), x)]
    for solve in solves:
        with pytest.raises(B.BoError) as e:
            solve(torch.zeros(3 * case.n, dtype=torch.float64, device="cuda"))
        assert e.value.status == B.BO_ERR_HIP and "wait" in str(e.value)
    assert np.isnan(run_stage(B, pc, B.bo_cpr_fstage, v, 3 * case.n)).any()
    with pytest.raises(B.BoError) as e:
        B.bo_cpr_update(pc, A)
    assert e.value.status == B.BO_ERR_HIP and "wait" in str(e.value)
    B.bo_cpr_wait_limit(pc, 1 << 21)
    B.bo_cpr_update(pc, A)
    assert np.array_equal(run_stage(B, pc, B.bo_cpr_fstage, v, 3 * case.n), good)
