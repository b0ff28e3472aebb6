"""Gauge moves whose second factorization is near the identity and ones where it
is not: states of a product state plus eps of noise have legs of condition
about 1 / eps, so |G - I| after the first pass runs from rounding (first-order
factor) to past the threshold (full factorization), over bond dimensions that
are and are not multiples of 16, against the oracle's QR.

Tolerance: the FP64 bar of 1e-10, or the rounding of a leg of that condition
over the gauge moves of the run, 1e-13 / eps."""
import pytest

from paper_2210_03763_amd import workload as W
from test_gpu_parity import compare

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("eps", [1.0, 5e-2, 1e-2, 1e-3, 1e-4])
@pytest.mark.parametrize("d,chi", [(3, 7), (4, 16), (4, 40)])
def test_conditions(d, chi, eps):
    w = W.make_random_drive(4, 4, d, chi, 2, 0.01, 2, 5 + chi, plus_sites=tuple(range(16)), eps=eps)
    print(f"[gauge] d={d} chi={chi} eps={eps}", flush=True)
    tol = max(1e-10, 1e-13 / eps)
    compare(w, tol=tol, tolC=tol)


@pytest.mark.parametrize("d,chi", [(3, 2), (3, 8), (3, 9), (3, 13), (3, 16), (3, 17), (4, 15), (4, 17)])
def test_one_workgroup_moves(d, chi):
    """Bonds on both sides of 16 and tensors on both sides of 256 rows: moves in
    one workgroup, with rows and columns padded to whole tiles, and beside them
    the ones that take a launch per product."""
    w = W.make_random_drive(4, 4, d, chi, 2, 0.01, 2, 3 + chi, plus_sites=tuple(range(16)), eps=5e-2)
    print(f"[gauge] d={d} chi={chi}", flush=True)
    compare(w, tol=1e-10, tolC=1e-10)
