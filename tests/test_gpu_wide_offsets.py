"""GPU test of the pairs that planes of 4 GiB and more take, whose cells lie
beyond a 32-bit offset, with the line moved down by the environment: still
pairs, the same values as within the line, on walled, ragged and periodic
grids."""
import numpy as np
import pytest

from gpu_helpers import mixed_walls, rel
from paper_2409_11382_amd import problem as P

pytestmark = pytest.mark.gpu

PAIRS = dict(quad_max_cells=0, tall_max_cells=0)


def _run(p, prec, steps):
    from paper_2409_11382_amd import lbm

    s = lbm.Solver(p, prec)
    s.set_tuning(PAIRS)
    s.step(steps)
    names = {r["name"] for r in s.profile_step(1) if r["depth"] == 0}
    _, nbytes = s.time_kernel(4, 2)
    F = s.fields()
    s.close()
    return F, names, nbytes


@pytest.mark.parametrize("prec,ref64", [("fp64", 0), ("fp32", 0), ("fp64_shifted", 0), ("fp32_shifted", 0),
                                        ("fp32_shifted", 1)])
@pytest.mark.parametrize("name", ["mixed", "strip", "periodic"])
def test_pairs_with_wide_offsets(monkeypatch, name, prec, ref64):
    if name == "mixed":
        p = mixed_walls(124, 68, seed=4).replace(K=4, ne_fixed=3)
    elif name == "strip":  # periodic in x
        p = P.loaded_strip(n=130, ny=72, alpha=1.0, K=2, ne_fixed=2)
    else:
        M = P.Manufactured(64, alpha=0.9, r=0.5, K=2, ne_fixed=2)
        f, src = M.loads(0.2)
        p = M.problem.replace(body_f=f, source_s=src)
    monkeypatch.setenv("BIOT_REF64", str(ref64))
    A, na, ba = _run(p, prec, 3)
    monkeypatch.setenv("BIOT_OFFSET32_BYTES", "1")
    B, nb, bb = _run(p, prec, 3)
    assert any(k.startswith("pair ") for k in nb) and any(k.startswith("pair+restrict ") for k in nb), nb
    assert na == nb and ba == bb
    assert np.abs(A["eta"]).max() > 0 and np.abs(A["p"]).max() > 0
    for k in ("eta", "p", "sigma"):
        if prec == "fp32_shifted" and not ref64:
            # wall terms formed in FP64 there; the stress is a difference of
            # neighbouring offsets, which loses a factor of the grid size
            assert rel(B[k], A[k]) < (1e-4 if k == "sigma" else 1e-5), k
        else:
            assert np.array_equal(A[k], B[k]), k
