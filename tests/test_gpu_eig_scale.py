"""The Hermitian eigensolver (ttn_herm_eig) on matrices whose entries' squares
underflow or overflow: eigenvalues, residual and orthonormality at the bars of
matrices of order one, 1e-13 and 1e-12 of the largest eigenvalue, for every
form of the solver (one pair of blocks, several)."""
import ctypes as C

import numpy as np
import pytest
import torch

from paper_2210_03763_amd import ttn as T

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("exponent", [-700, -500, 500, 1000])
@pytest.mark.parametrize("n", [2, 16, 40, 100])
def test_eigensolver_scales(n, exponent):
    L = T.lib()
    L.ttn_herm_eig.restype = C.c_int
    L.ttn_herm_eig.argtypes = [C.c_int32] + [C.c_void_p] * 5
    rng = np.random.default_rng(n)
    A = rng.standard_normal((n, n)) + 1j * rng.standard_normal((n, n))
    A = 0.5 * (A + A.conj().T)
    dA = torch.tensor(np.ldexp(np.concatenate([A.real.ravel(order="F"), A.imag.ravel(order="F")]), exponent),
                      dtype=torch.float64, device="cuda")
    dV, dw = torch.zeros(2 * n * n, dtype=torch.float64, device="cuda"), torch.zeros(n, dtype=torch.float64, device="cuda")
    do = torch.zeros(n, dtype=torch.int32, device="cuda")
    print(f"[eig] n={n} 2^{exponent}", flush=True)
    assert L.ttn_herm_eig(n, dA.data_ptr(), dV.data_ptr(), dw.data_ptr(), do.data_ptr(),
                          torch.cuda.current_stream().cuda_stream) == 0
    w, order, v = np.ldexp(dw.cpu().numpy(), -exponent), do.cpu().numpy(), dV.cpu().numpy()
    V = (v[:n * n] + 1j * v[n * n:]).reshape(n, n, order="F")[:, order]
    ref = np.linalg.eigvalsh(A)[::-1]
    scale = abs(ref).max()
    assert sorted(order.tolist()) == list(range(n))
    assert np.abs(w - ref).max() <= 1e-13 * scale
    assert np.abs(A @ V - V * w).max() <= 1e-12 * scale
    assert np.abs(V.conj().T @ V - np.eye(n)).max() <= 1e-12


@pytest.mark.parametrize("n", [5, 20, 60])
def test_order_is_a_permutation_with_nan(n):
    """Callers gather columns by d_order: it has to stay in range whatever the matrix holds."""
    L = T.lib()
    L.ttn_herm_eig.restype = C.c_int
    L.ttn_herm_eig.argtypes = [C.c_int32] + [C.c_void_p] * 5
    dA = torch.eye(n, dtype=torch.float64, device="cuda").repeat(2, 1, 1)
    dA[1] = 0
    dA[0, n // 2, n // 2] = float("nan")
    dV, dw = torch.zeros(2 * n * n, dtype=torch.float64, device="cuda"), torch.zeros(n, dtype=torch.float64, device="cuda")
    do = torch.full((n,), -1, dtype=torch.int32, device="cuda")
    print(f"[eig] n={n} nan", flush=True)
    L.ttn_herm_eig(n, dA.data_ptr(), dV.data_ptr(), dw.data_ptr(), do.data_ptr(), torch.cuda.current_stream().cuda_stream)
    assert sorted(do.cpu().tolist()) == list(range(n))
