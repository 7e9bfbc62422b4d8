"""GPU test of the launch shapes that the schedule picks where no bound is
given: the profile names the region of each launch."""
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
