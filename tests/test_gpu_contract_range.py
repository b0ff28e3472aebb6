"""The FP32 contraction at 1 Gflop and above outside the range in which its
bf16 pieces hold a number: operands near the ends of the FP32 range,
infinities and NaN, on whole and ragged tiles, against real float64 products
of the same inputs.  Finite outputs: 1e-5 of the largest (the bar of the mode);
non-finite ones where, and of the kind that, plain FP32 products give."""
import ctypes as C

import pytest
import torch

from paper_2210_03763_amd import ttn as T

pytestmark = pytest.mark.gpu


def _contract(prec, case, o, x):
    """Both operands [k][re / im][...]; returns the device result and the float64 one."""
    DL, DR, DP, leg, K, sm = case
    L = T.lib()
    L.ttn_leg_contract_noalloc.restype = C.c_int
    L.ttn_leg_contract_noalloc.argtypes = [C.c_int32] * 6 + [C.c_void_p, C.c_void_p, C.c_int32, C.c_void_p, C.c_int32,
                                                            C.c_int32, C.c_void_p]
    d_o, d_x = o.cuda(), x.cuda()
    d_y = torch.zeros((1 if sm else K, 2, DP, DR, DL), dtype=x.dtype, device="cuda")
    rc = L.ttn_leg_contract_noalloc(prec, leg, DL, DR, DP, K, d_o.data_ptr(), d_x.data_ptr(), sm, d_y.data_ptr(), sm,
                                    0, torch.cuda.current_stream().cuda_stream)
    assert rc == 0, L.ttn_last_error(None)
    eq = {0: "kba,kprb->kpra", 1: "kba,kpbl->kpal", 2: "kba,kbrl->karl"}[leg]
    od, xd = o.double(), x.double().expand(K, *x.shape[1:])
    p = lambda i, j: torch.einsum(eq, od[:, i], xd[:, j])
    y = torch.stack([p(0, 0) - p(1, 1), p(0, 1) + p(1, 0)], dim=1)
    return d_y.cpu().double(), y.sum(0, keepdim=True) if sm else y


def _inputs(case):
    DL, DR, DP, leg, K, sm = case
    D = (DL, DR, DP)[leg]
    g = torch.Generator().manual_seed(DL + DR + DP + leg)
    return torch.randn(K, 2, D, D, generator=g), torch.randn(K if sm else 1, 2, DP, DR, DL, generator=g)


CASES = [(128, 128, 128, 0, 1, 0), (128, 128, 128, 2, 2, 1), (100, 100, 130, 1, 2, 1), (70, 200, 128, 2, 2, 0)]


@pytest.mark.parametrize("so,sx", [(-120, 90), (90, -125), (-60, -50), (-115, 0), (60, 55)])
@pytest.mark.parametrize("case", CASES)
def test_scales(case, so, sx):
    o, x = _inputs(case)
    print(f"[range] {case} 2^{so} 2^{sx}", flush=True)
    got, ref = _contract(T.PREC_FP32, case, torch.ldexp(o, torch.tensor(so)), torch.ldexp(x, torch.tensor(sx)))
    assert ((got - ref).abs().max() / ref.abs().max()).item() <= 1e-5


@pytest.mark.parametrize("case", CASES)
def test_non_finite(case):
    o, x = _inputs(case)
    o[0, 0, 3, 5] = float("inf")
    o[0, 1, 9, 8] = float("nan")
    o[0, 0, 11, 17] = 3.4e38
    x *= 2.0 ** -20
    print(f"[range] {case} inf, nan, largest", flush=True)
    got, ref = _contract(T.PREC_FP32, case, o, x)
    assert torch.equal(torch.isnan(got), torch.isnan(ref))
    assert torch.equal(torch.isinf(got), torch.isinf(ref)) and torch.equal(got[torch.isinf(ref)], ref[torch.isinf(ref)])
    ok = torch.isfinite(ref)
    assert ((got - ref)[ok].abs().max() / ref[ok].abs().max()).item() <= 1e-5


# two-piece products on outputs that are not whole tiles (inner extent a multiple of 32)
@pytest.mark.parametrize("case", [(160, 192, 200, 0, 3, 0), (256, 160, 130, 1, 5, 1), (130, 200, 224, 2, 3, 1)])
def test_two_pieces_ragged(case):
    o, x = _inputs(case)
    print(f"[range] bf16x3 {case}", flush=True)
    got, ref = _contract(T.PREC_BF16X3, case, o, x)
    err = ((got - ref).abs().max() / ref.abs().max()).item()
    print(f"[range] err {err:.2e}", flush=True)
    assert err <= 1e-5
