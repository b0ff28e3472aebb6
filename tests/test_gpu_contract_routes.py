"""Contractions at the lines between the kernels' ranges, against real float64
products of the same inputs: FP32 1e-5, FP64 1e-12 of the largest output (the
bars of the other shapes)."""
import pytest
import torch

from paper_2210_03763_amd import ttn as T
from test_gpu_contract_range import _contract, _inputs

pytestmark = pytest.mark.gpu

# (DL, DR, DP, leg, n_ops, sum)
# FP32 above 1 Gflop with short inner extents, which the bf16-piece kernel would pad to 16 each
SHORT_INNER = [(8, 256, 256, 0, 33, 1), (256, 256, 20, 2, 5, 1), (20, 256, 128, 0, 33, 1), (31, 130, 130, 0, 9, 1)]


def _check(prec, case):
    print(f"[routes] {case} prec={prec}", flush=True)
    dt = torch.float64 if prec == T.PREC_FP64 else torch.float32
    o, x = (t.to(dt) for t in _inputs(case))
    got, ref = _contract(prec, case, o, x)
    err = ((got - ref).abs().max() / ref.abs().max()).item()
    print(f"[routes] err {err:.2e}", flush=True)
    assert err <= (1e-12 if prec == T.PREC_FP64 else 1e-5)


@pytest.mark.parametrize("case", SHORT_INNER)
def test_short_inner_extents(case):
    _check(T.PREC_FP32, case)


# tiles enough for one wave each, thin outputs beside long ones, and a long K over few tiles
WAVES = [(160, 36, 20, 2, 16, 0), (21, 73, 245, 0, 4, 0), (27, 64, 129, 0, 4, 0), (9, 208, 156, 1, 2, 0),
         (8, 256, 256, 0, 17, 1), (16, 33, 700, 1, 5, 1), (13, 200, 90, 1, 33, 1), (85, 9, 13, 0, 16, 1), (64, 8, 12, 0, 17, 1)]


@pytest.mark.parametrize("prec", [T.PREC_FP64, T.PREC_FP32])
@pytest.mark.parametrize("case", WAVES)
def test_wave_counts(case, prec):
    _check(prec, case)


# aligned tiles: 32 x 32 ones split into whole rounds, 64 x 64 ones around one round, a padded long K
ALIGNED = [(192, 16, 18, 0, 8, 1), (16, 72, 112, 2, 17, 1), (160, 12, 8, 0, 5, 1), (112, 27, 12, 0, 33, 1),
           (128, 48, 48, 2, 4, 0), (48, 64, 221, 0, 1, 0), (54, 36, 48, 2, 9, 0), (80, 32, 64, 2, 9, 0), (24, 64, 80, 1, 17, 1)]


@pytest.mark.parametrize("prec", [T.PREC_FP64, T.PREC_FP32])
@pytest.mark.parametrize("case", ALIGNED)
def test_aligned_plans(case, prec):
    _check(prec, case)
