"""GPU test of the wall rules in the launches of several applications under a
body force and a fluid source, which leave no field zero where the sides carry
no data (symmetry walls beside periodic sides and each other): displacement,
pressure and stress against the FP64 oracle.  A mirror rule of the bottom and top
walls that forgets its column moves the displacement of PPSS by 0.7%."""
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


def _problem(walls, nx, ny):
    """walls: types of left, right, bottom, top; loads without a mean (a mean
    force has no answer where the sides hold nothing)"""
    lam, mu = P.plane_stress_lame(1.0, 0.3)
    sides = [P.Side.uniform(ny if k < 2 else nx, EL[c], FLOW[c]) for k, c in enumerate(walls)]
    h = 1.0 / max(nx, ny)
    rng = np.random.default_rng(7)
    f, s = rng.standard_normal((2, ny, nx)), rng.standard_normal((ny, nx))
    f -= f.mean(axis=(1, 2), keepdims=True)
    s -= s.mean()
    p = P.Problem(nx=nx, ny=ny, dx=h, dt=h * h / 4, lam=lam, mu=mu, c0=1.0, alpha=0.8, kappa=1.0, sides=sides,
                  K=4, ne_fixed=2, body_f=f, source_s=s, name="loaded_walls_" + walls)
    return P.with_random_boundary_data(p, seed=11, scale=1e-2)


@pytest.mark.parametrize("walls", ["PPSS", "SSPP", "SSSS", "SSDT", "TDSS", "PPDT", "DTSD"])
@pytest.mark.parametrize("nx,ny", [(112, 48), (58, 50)])
def test_walls_under_loads(walls, nx, ny):
    from paper_2409_11382_amd import lbm

    p = _problem(walls, nx, ny)
    o = Oracle(p, threads=oracle_threads())
    o.step(2)
    B = o.fields()
    assert all(np.abs(B[k]).max() > 0 for k in ("eta", "p", "sigma"))
    # FP32: the stress is a difference of neighbouring offsets, which loses a
    # factor of the grid size against displacement and pressure
    for prec, tol in (("fp64", dict(eta=1e-10, p=1e-10, sigma=1e-10)),
                      ("fp32_shifted", dict(eta=1e-5, p=1e-5, sigma=1e-4))):
        for bounds in (dict(quad_max_cells=0, tall_max_cells=0), dict(quad_max_cells=0, tall_max_cells=BIG),
                       dict(quad_max_cells=BIG), dict(quad_max_cells=BIG, quad_res_narrow_max_cells=0)):
            s = lbm.Solver(p, prec)
            s.set_tuning(bounds)
            s.step(2)
            A = s.fields()
            s.close()
            e = {k: rel(A[k], B[k]) for k in ("eta", "p", "sigma")}
            print(walls, nx, ny, prec, bounds, e, flush=True)
            assert all(e[k] <= tol[k] for k in e), (walls, nx, ny, prec, bounds, e)
