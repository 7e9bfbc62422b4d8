"""GPU test of the wall rules in the launches of several applications: every
meeting of two wall types at a corner and beside periodic sides, with random
boundary data, against the FP64 oracle, at sizes where a wall falls on, next to
and a tile's remainder away from a tile edge."""
import sys

import numpy as np
import pytest

from conftest import oracle_threads
from gpu_helpers import rel
from oracle.oracle import Oracle
from paper_2409_11382_amd import problem as P

pytestmark = pytest.mark.gpu

BIG = 1 << 40
EL = {"P": P.EL_PERIODIC, "D": P.EL_DIRICHLET, "T": P.EL_TRACTION, "S": P.EL_SYMMETRY}
FLOW = {"P": P.FLOW_PERIODIC, "D": P.FLOW_NOFLOW, "T": P.FLOW_DIRICHLET, "S": P.FLOW_SYMMETRY}


@pytest.fixture(scope="module")
def lbm():
    import torch

    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2409_11382_amd import lbm as L

    L.load_library()
    return L


def _problem(walls, nx, ny):
    """walls: types of left, right, bottom, top; random displacements,
    tractions and pressures on them, uniform permeability"""
    lam, mu = P.plane_stress_lame(1.0, 0.3)
    sides = [P.Side.uniform(ny if k < 2 else nx, EL[c], FLOW[c]) for k, c in enumerate(walls)]
    h = 1.0 / max(nx, ny)
    p = P.Problem(nx=nx, ny=ny, dx=h, dt=h * h / 4, lam=lam, mu=mu, c0=1.0, alpha=0.8, kappa=1.0, sides=sides,
                  K=4, ne_fixed=2, name="walls_" + walls)
    return P.with_random_boundary_data(p, seed=11, scale=1e-2)


@pytest.mark.parametrize("walls", ["DTSD", "SDTS", "TSDT", "SSDT", "DDTT", "TDSS", "PPDT", "PPSS", "TDPP", "SSPP"])
@pytest.mark.parametrize("nx,ny", [(112, 48), (58, 50)])
def test_wall_types_in_multi_application_launches(lbm, walls, nx, ny):
    p = _problem(walls, nx, ny)
    o = Oracle(p, threads=oracle_threads())
    o.step(2)
    B = o.fields()
    pairs = dict(quad_max_cells=0, tall_max_cells=0)
    for prec, tol in (("fp64", 1e-10), ("fp32_shifted", 1e-5)):
        for bounds in (pairs, dict(quad_max_cells=0, tall_max_cells=BIG), dict(quad_max_cells=BIG),
                       dict(quad_max_cells=BIG, quad_res_narrow_max_cells=0)):
            s = lbm.Solver(p, prec)
            s.set_tuning(bounds)
            s.step(2)
            A = s.fields()
            s.close()
            e = {k: rel(A[k], B[k]) for k in ("eta", "p")}
            print(walls, nx, ny, prec, bounds, e, flush=True)
            sys.stdout.flush()
            assert max(e.values()) <= tol  # no data on periodic and symmetry sides: the fields stay zero there
            if prec == "fp64":
                assert float(np.abs(A["eta"] - B["eta"]).max()) <= tol * float(np.abs(B["eta"]).max())


@pytest.mark.parametrize("shape", [(4, 4, 1), (4, 4, 2), (8, 8, 2), (8, 8, 3), (16, 16, 4), (8, 2, 1), (12, 12, 3),
                                   (20, 20, 3), (40, 24, 4)])
@pytest.mark.parametrize("walls", ["SSST", "PPDT", "DTSD"])
@pytest.mark.parametrize("sweeps", [0, 6])
def test_smallest_levels_as_a_matrix(lbm, shape, walls, sweeps):
    """The V-cycle's levels of at most 16 cells run as one matrix: the coarse
    cycle from zero on the coarse tail's top level (which the matrix covers
    whole, in part or not at all here) and time steps against the oracle."""
    nx, ny, L = shape
    if walls[0] != "P" and nx >> (L - 1) < 2:
        pytest.skip("fewer than two cells across on the coarsest level")
    p = _problem(walls, 2 * nx, 2 * ny).replace(levels=L + 1, coarse_sweeps=sweeps)
    o = Oracle(p, threads=oracle_threads())
    rng = np.random.default_rng(5)
    s = lbm.Solver(p, "fp64")
    lnx, lny = s.level_shape(L)
    r = rng.standard_normal((8, lny, lnx)) * 1e-3
    z = np.zeros_like(r)
    e = rel(s.mg_cycle(L, z, r=r), o.mg_cycle(L, z, r=r))
    s.close()
    o = Oracle(p, threads=oracle_threads())
    o.step(3)
    B = o.fields()
    errs = []
    for prec, tol in (("fp64", 1e-10), ("fp32_shifted", 1e-5)):
        s = lbm.Solver(p, prec)
        s.step(3)
        A = s.fields()
        s.close()
        errs.append((max(rel(A[k], B[k]) for k in ("eta", "p")), tol))
    print(shape, walls, sweeps, e, errs, flush=True)
    assert e < 1e-11
    assert all(v < tol for v, tol in errs)


@pytest.mark.parametrize("prec,tol", [("fp64", 1e-10), ("fp32_shifted", 1e-5)])
@pytest.mark.parametrize("nx,ny", [(256, 128), (272, 128), (512, 250), (530, 250), (640, 400)])
def test_regions_chosen_by_their_rounds(lbm, nx, ny, prec, tol):
    """Sizes at the lines between launch shapes: 256 low and 512 blocks of four
    applications and more, one and two rounds of the pairs' regions; the
    chosen shapes and the pairs' default regions against the oracle."""
    p = _problem("DTSD", nx, ny)
    o = Oracle(p, threads=oracle_threads())
    o.step(1)
    B = o.fields()
    for bounds in ({}, dict(quad_max_cells=0, tall_max_cells=0, quad_res_narrow_max_cells=0)):
        s = lbm.Solver(p, prec)
        if bounds:
            s.set_tuning(bounds)
        s.step(1)
        A = s.fields()
        s.close()
        e = {k: rel(A[k], B[k]) for k in ("eta", "p")}
        assert max(e.values()) <= tol, (nx, ny, prec, bounds, e)


@pytest.mark.parametrize("walls", ["DTSD", "TSDT", "PPDT", "SDPP"])
@pytest.mark.parametrize("nx,ny", [(5, 3), (62, 14), (63, 15), (125, 29)])
def test_flow_tiles(lbm, walls, nx, ny):
    """The flow step's tiles (62 x 14 outputs): smaller than, exactly and one
    more than a tile, and a ragged last tile, on every wall type; the step
    counter and norms follow from its last block over several steps."""
    p = _problem(walls, nx, ny).replace(levels=1)
    o = Oracle(p, threads=oracle_threads())
    o.step(4)
    B = o.fields()
    for prec, tol in (("fp64", 1e-10), ("fp32_shifted", 1e-5)):
        s = lbm.Solver(p, prec)
        s.step(4)
        A = s.fields()
        n = s.stats()["step"]
        s.close()
        e = {k: rel(A[k], B[k]) for k in ("eta", "p")}
        assert n == 4 and max(e.values()) <= tol, (walls, nx, ny, prec, e)
