"""The contraction launches of short, ragged and unaligned shapes: the
wave-sliced kernel (every wave count, its in-block reduction, its split over
blocks) at the edges of its 16 x 16 x 16 tiles, and the ragged form of the
LDS-tiled kernel (contraction extents that are not whole tiles, 32 and 64
wide tiles, split K), against a complex128 einsum on the same inputs.

Tolerances as for the aligned shapes: FP64 1e-12, FP32 1e-5 of the largest
output (rounding of K <= 8250 products accumulated in the arrays' precision).
"""
import ctypes as C

import pytest
import torch

from paper_2210_03763_amd import ttn as T

pytestmark = pytest.mark.gpu

# (DL, DR, DP, leg, n_ops, sum)
SHORT = [(1, 1, 1, 0, 1, 0), (3, 3, 9, 1, 2, 1), (15, 16, 17, 0, 3, 0), (17, 15, 16, 1, 2, 0), (16, 17, 15, 2, 4, 1),
         (9, 9, 64, 2, 5, 1), (9, 9, 64, 1, 3, 1), (27, 27, 64, 1, 5, 1), (17, 1, 33, 2, 33, 1), (16, 1, 16, 2, 64, 1),
         (12, 12, 144, 0, 9, 0), (130, 1, 130, 0, 9, 0)]
RAGGED = [(81, 81, 128, 1, 5, 1), (81, 81, 128, 0, 5, 0), (100, 100, 100, 0, 5, 0), (45, 45, 250, 2, 7, 1),
          (5, 20, 250, 2, 33, 1), (200, 65, 33, 0, 3, 1), (67, 67, 67, 1, 9, 0)]


def _planar(z, dtype):
    return torch.cat([z.real, z.imag], dim=-1).to(dtype).contiguous()


@pytest.mark.parametrize("accumulate", [0, 1])
@pytest.mark.parametrize("prec", [T.PREC_FP64, T.PREC_FP32, T.PREC_BF16X3])
@pytest.mark.parametrize("case", SHORT + RAGGED)
def test_leg_contract_shapes(case, prec, accumulate):
    DL, DR, DP, leg, K, sm = case
    print(f"[shapes] {case} prec={prec} acc={accumulate}", flush=True)
    L = T.lib()
    L.ttn_leg_contract_noalloc.restype = C.c_int
    L.ttn_leg_contract_noalloc.argtypes = [C.c_int32] * 6 + [C.c_void_p, C.c_void_p, C.c_int32, C.c_void_p, C.c_int32,
                                                            C.c_int32, C.c_void_p]
    g = torch.Generator().manual_seed(DL * 7 + DR * 5 + DP * 3 + leg)
    D, n = (DL, DR, DP)[leg], DL * DR * DP
    nx, ny = (K, 1) if sm else (1, K)
    dt = torch.float64 if prec == T.PREC_FP64 else torch.float32
    cplx = lambda *s: torch.complex(torch.randn(*s, generator=g, dtype=dt), torch.randn(*s, generator=g, dtype=dt))
    ops, xs, y0 = cplx(K, D, D), cplx(nx, DP, DR, DL), cplx(ny, DP, DR, DL)      # ops[k, b, a]: column-major
    d_ops, d_x, d_y = (_planar(t.reshape(t.shape[0], -1), dt).cuda() for t in (ops, xs, y0))
    rc = L.ttn_leg_contract_noalloc(prec, leg, DL, DR, DP, K, d_ops.data_ptr(), d_x.data_ptr(), sm, d_y.data_ptr(), sm,
                                    accumulate, torch.cuda.current_stream().cuda_stream)
    assert rc == 0, L.ttn_last_error(None)
    o, x = ops.to(torch.complex128), xs.to(torch.complex128)
    eq = {0: "kba,kprb->kpra", 1: "kba,kpbl->kpal", 2: "kba,kbrl->karl"}[leg]
    ref = torch.einsum(eq, o, x.expand(K, *x.shape[1:]))
    if sm:
        ref = ref.sum(0, keepdim=True)
    if accumulate:
        ref = ref + y0.to(torch.complex128)
    got = d_y.cpu().double()
    got = torch.complex(got[:, :n], got[:, n:]).reshape(ref.shape)
    err = ((got - ref).abs().max() / ref.abs().max()).item()
    print(f"[shapes] err/scale = {err:.2e}", flush=True)
    assert err <= (1e-12 if prec == T.PREC_FP64 else 1e-5)
