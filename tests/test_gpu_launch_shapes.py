"""GPU tests of the launch shapes that the schedule picks, where no bound is
given and where one is: the profile names the region of each launch."""
import pytest

from paper_2409_11382_amd import problem as P

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lbm():
    import torch

    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2409_11382_amd import lbm as L

    L.load_library()
    return L


def _finest(solver):
    """names of the finest level's launches"""
    return {r["name"] for r in solver.profile_step(1) if r["depth"] == 0}


@pytest.mark.parametrize("n,tall", [(512, True), (640, False), (736, True), (896, False), (1024, False),
                                    (1216, False), (1280, False), (1376, False), (1408, False), (1536, False)])
def test_tall_pairs_where_they_are_faster(lbm, n, tall):
    """Pairs in FP32 shifted storage: tall regions in one round of blocks, or in
    two where the default region takes two as well."""
    s = lbm.Solver(P.loaded_strip(n=n, ne_fixed=2), "fp32_shifted")
    names = _finest(s)
    s.close()
    assert ("pair alt shift f32" in names) == tall, names
    assert ("pair shift f32" in names) != tall, names


@pytest.mark.parametrize("n,bound,cells,shape", [(736, "tall_max_cells", 512 * 512, "pair alt"),
                                                 (320, "quad_max_cells", 256 * 256, "quad")])
def test_every_given_bound_is_literal(lbm, n, bound, cells, shape):
    """A bound below the finest level's cells keeps it from the launch that the
    rule takes there, whatever the bound's value; the reported bounds applied
    to another solver give the same launches, by rule or by bound."""
    p = P.loaded_strip(n=n, ne_fixed=2)
    s = lbm.Solver(p, "fp32_shifted")
    assert s.tuning()[bound] == lbm.TUNING_BY_RULE
    by_rule = _finest(s)
    assert any(shape in k for k in by_rule)
    t = lbm.Solver(p, "fp32_shifted")
    t.set_tuning(s.tuning())
    assert _finest(t) == by_rule
    s.set_tuning({bound: cells})
    assert s.tuning()[bound] == cells
    assert not any(shape in k for k in _finest(s))
    t.set_tuning(s.tuning())
    assert _finest(t) == _finest(s)
    s.set_tuning({bound: lbm.TUNING_BY_RULE})
    assert _finest(s) == by_rule
    for bad in (-1, lbm.TUNING_BY_RULE + 1):
        with pytest.raises(lbm.BiotError):
            s.set_tuning({bound: bad})
    s.close()
    t.close()


@pytest.mark.parametrize("cycle", [P.CYCLE_V, P.CYCLE_W])
@pytest.mark.parametrize("prec,size", [("fp32_shifted", 4), ("fp64", 8)])
def test_bytes_of_the_coarse_tail(lbm, prec, size, cycle):
    """The profile charges a tail the sweeps it runs (2K + 1 a level, populations
    in and out and the right-hand side, the coarsest level in FP64 with its own
    number) and, in a V-cycle, the matrix in place of its levels of at most 16
    cells: 64^2, tail of 32^2 and below."""
    K = 3
    s = lbm.Solver(P.loaded_strip(n=64, K=K, ne_fixed=2).replace(cycle=cycle), prec)
    row = [r for r in s.profile_step(1) if r["name"].startswith("tail")][0]
    s.close()
    sweep = lambda n, apps, v: n * n * apps * 24 * v
    want = sum(sweep(n, 2 * K + 1, size) for n in (32, 16, 8))
    if cycle == P.CYCLE_V:
        want += (8 * 16) ** 2 * 8
    else:
        want += sweep(4, 2 * K + 1, size) + sweep(2, 2 * K, 8)
    assert row["bytes_per_step"] == row["launches"] * want
