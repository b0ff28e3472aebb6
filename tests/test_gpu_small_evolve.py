"""One-workgroup evolution of small operators at the edges of its forms: dense
(up to 96 entries: the bottom nodes of d = 4, chi = 6, and every smaller bond),
basis in registers (up to 256) and in LDS (above), against the oracle on the
same inputs: 1e-10, the bar of the FP64 path."""
import pytest

from paper_2210_03763_amd import workload as W
from test_gpu_parity import compare

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,chi", [(3, 2), (3, 3), (3, 4), (3, 5), (4, 6), (4, 7), (4, 16)])
def test_small_operators(d, chi):
    w = W.make_random_drive(4, 4, d, chi, 2, 0.01, 2, 31 + chi, plus_sites=tuple(range(16)), eps=5e-2)
    print(f"[small] d={d} chi={chi}", flush=True)
    compare(w, tol=1e-10, tolC=1e-10)
