"""The backward pass on both sides of the step count from which it replays a
graph of its first step: 31 and 33 recorded steps with checkpoints in between,
against the eager pass, 1e-13 of the largest gradient entry (the same launches
on the same addresses)."""
import numpy as np
import pytest

from paper_2210_03763_amd import ttn as T
from paper_2210_03763_amd import workload as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", [T.PREC_FP64, T.PREC_FP32])
@pytest.mark.parametrize("steps", [31, 33])
def test_long_backward_passes_match_eager(steps, precision):
    w = W.make_random_drive(4, 2, 3, 8, steps, 0.05, 4, 7, plus_sites=tuple(range(8)), eps=5e-2, precision=precision)
    out = []
    for graphs in (True, False):
        g = T.TTN(w)
        g.set_graphs(graphs)
        g.record(steps, 10)
        g.step(steps)
        out.append(g.backward())
        g.close()
    (go1, gd1), (go0, gd0) = out
    scale = max(np.abs(go0).max(), np.abs(gd0).max())
    err = max(np.abs(go1 - go0).max(), np.abs(gd1 - gd0).max()) / scale
    print(f"[adjoint] {steps} steps, precision {precision}: max|g| {scale:.3e}, err {err:.3e}", flush=True)
    assert scale > 0 and err <= 1e-13
