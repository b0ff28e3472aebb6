"""Sampling where the passes beside the contractions are folded into them:
column norms left by the contraction (left bonds of 64 and 128: one and two
row tiles a column), outer products formed while staging (bonds that are
multiples of 16), and the bonds that keep passes of their own, over shot
counts that end inside a tile, against the sampling oracle: the same shots
and, to 1e-12, their amplitudes."""
import numpy as np
import pytest

from oracle import sampling as S
from oracle import ttn_oracle as O
from paper_2210_03763_amd import ttn as T
from paper_2210_03763_amd import workload as W
from test_gpu_parity import gpu_state_as_oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,chi,n", [(3, 64, 33), (3, 64, 130), (3, 72, 70), (3, 80, 70), (4, 128, 65), (4, 128, 7)])
def test_shots_equal_the_oracle_sampler(d, chi, n):
    w = W.make_random_drive(4, 4, d, chi, 2, 0.01, 2, 9 + chi, plus_sites=tuple(range(16)), eps=0.5)
    print(f"[wide] d={d} chi={chi} n={n}", flush=True)
    g = T.TTN(w)
    g.step(1)
    st = gpu_state_as_oracle(g, O.build(w))
    cfg_g, amp_g = g.sample(n, 99)
    cfg_o, amp_o = S.sample(st, n, 99)
    same = (cfg_g == cfg_o).all(axis=1)
    print(f"[wide] {same.sum()} of {n} shots identical", flush=True)
    assert same.all()
    assert np.abs(amp_g - amp_o).max() < 1e-12
    g.close()
