"""The aligned contraction tiles at the edges of their rule: 32 x 32 tiles with
one, two and four groups of waves on a tile (uneven shares of the k-tiles,
ragged outputs), the same with K split over the grid, 64 x 64 tiles without and
with a split (over many and over few outputs), 128 x 64 tiles, against a complex128 einsum on the same inputs.

Tolerances as for the other aligned shapes: FP64 1e-12, FP32 1e-5 of the
largest output.
"""
import ctypes as C

import pytest
import torch

from paper_2210_03763_amd import ttn as T

pytestmark = pytest.mark.gpu

# (DL, DR, DP, leg, n_ops, sum)
TILES = [(48, 50, 50, 0, 7, 1), (64, 64, 80, 0, 3, 1), (48, 100, 90, 1, 2, 0), (100, 48, 90, 1, 2, 1),
         (20, 20, 64, 2, 40, 1), (64, 150, 120, 0, 1, 0), (64, 128, 130, 0, 16, 1), (128, 130, 128, 0, 4, 1),
         (40, 33, 32, 2, 9, 0), (16, 67, 96, 2, 4, 1),
         (100, 1, 128, 2, 128, 1), (48, 64, 96, 1, 32, 1)]


def _planar(z, dtype):
    return torch.cat([z.real, z.imag], dim=-1).to(dtype).contiguous()


@pytest.mark.parametrize("accumulate", [0, 1])
@pytest.mark.parametrize("prec", [T.PREC_FP64, T.PREC_FP32])
@pytest.mark.parametrize("case", TILES)
def test_leg_contract_tiles(case, prec, accumulate):
    DL, DR, DP, leg, K, sm = case
    print(f"[tiles] {case} prec={prec} acc={accumulate}", flush=True)
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
    eq = {0: "ba,prb->pra", 1: "ba,pbl->pal", 2: "ba,brl->arl"}[leg]
    ref = torch.stack([torch.einsum(eq, o[k], x[k if sm else 0]) for k in range(K)])
    if sm:
        ref = ref.sum(0, keepdim=True)
    if accumulate:
        ref = ref + y0.to(torch.complex128)
    got = d_y.cpu().double()
    got = torch.complex(got[:, :n], got[:, n:]).reshape(ref.shape)
    err = ((got - ref).abs().max() / ref.abs().max()).item()
    print(f"[tiles] err/scale = {err:.2e}", flush=True)
    assert err <= (1e-12 if prec == T.PREC_FP64 else 1e-5)
