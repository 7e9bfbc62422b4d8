"""GPU test of time steps while the caller captures the solver's stream: the
library's own step graphs are no stream work that the runtime records, so after
one step outside (which captures them) the steps run at once, whatever their
number."""
import ctypes as C

import numpy as np
import pytest

from paper_2409_11382_amd import problem as P

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("steps", [1, 4, 6])
def test_steps_while_the_caller_captures(steps):
    import torch

    from paper_2409_11382_amd import lbm

    hip = C.CDLL("libamdhip64.so")
    p = P.loaded_strip(n=64, alpha=0.9, ne_fixed=2)
    s = lbm.Solver(p, "fp64")
    ref = lbm.Solver(p, "fp64")
    st = C.c_void_p(s.stream.cuda_stream)
    s.step(1)
    torch.cuda.synchronize()
    graph = C.c_void_p(0)
    assert hip.hipStreamBeginCapture(st, C.c_int(1)) == 0  # thread local
    try:
        s.step(steps)
    finally:
        rc = hip.hipStreamEndCapture(st, C.byref(graph))
        if graph.value:
            hip.hipGraphDestroy(graph)
    assert rc == 0
    s.step(5)  # and outside again
    ref.step(1 + steps + 5)
    A, B = s.fields(), ref.fields()
    s.close()
    ref.close()
    assert A["step"] == B["step"]
    for k in ("eta", "p", "sigma"):
        assert np.array_equal(A[k], B[k]), (steps, k)
