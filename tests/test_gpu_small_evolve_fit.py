"""One-workgroup evolution of the operators that just fit its LDS: the (6, 6, 6)
nodes of 32 sites at chi = 6, the (16, 1, 16) bonds of 4x4 at chi = 16 and m = 16,
the (11, 1, 11) bonds of 32 sites at chi = 11 and m = 15 (the basis without padded
rows).  None of them may leave that kernel, which is FP64 in every precision
mode: the contraction matvecs of a step, over m, are those of a basis that fits
with room to spare.  Values: 1e-10 against the oracle, the bar of the FP64 path."""
import pytest

from paper_2210_03763_amd import ttn as T
from paper_2210_03763_amd import workload as W
from test_gpu_parity import compare

pytestmark = pytest.mark.gpu

# (Lx, Ly, d, chi, m)
EDGES = [(8, 4, 3, 6, 12), (4, 4, 3, 16, 16), (4, 2, 3, 16, 16), (8, 4, 4, 11, 15)]


def _drive(Lx, Ly, d, chi, m, prec):
    w = W.make_random_drive(Lx, Ly, d, chi, 2, 0.01, 2, 17 + chi, plus_sites=tuple(range(Lx * Ly)), eps=5e-2,
                            precision=prec)
    return w.copy(krylov_dim=m)


def _matvecs(w):
    g = T.TTN(w)
    g.profile_begin(timed=False)
    g.step(1)
    n = int(g.profile_end().matvecs)
    g.close()
    assert n % w.krylov_dim == 0
    return n // w.krylov_dim


@pytest.mark.parametrize("prec", [T.PREC_FP64, T.PREC_FP32])
@pytest.mark.parametrize("edge", EDGES)
def test_edges_stay_in_one_workgroup(edge, prec):
    print(f"[fit] {edge} prec={prec}", flush=True)
    assert _matvecs(_drive(*edge, prec)) == _matvecs(_drive(*edge[:4], 8, prec))


@pytest.mark.parametrize("edge", EDGES)
def test_edge_values(edge):
    print(f"[fit] {edge} values", flush=True)
    compare(_drive(*edge, T.PREC_FP64), tol=1e-10, tolC=1e-10)
