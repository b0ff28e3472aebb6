"""The block Jacobi eigensolver (ttn_herm_eig) at the edges of its 16-wide
blocks and 32-wide pairs, and on spectra that leave nothing to rotate or are
degenerate, against numpy.linalg.eigvalsh: eigenvalues within 1e-13 of the
largest, residual and orthonormality within 1e-12 (the bars of the solver's
other sizes)."""
import ctypes as C

import numpy as np
import pytest
import torch

from paper_2210_03763_amd import ttn as T

pytestmark = pytest.mark.gpu


def _matrix(n, kind):
    rng = np.random.default_rng(n)
    q, _ = np.linalg.qr(rng.standard_normal((n, n)) + 1j * rng.standard_normal((n, n)))
    if kind == "zero":
        return np.zeros((n, n), complex)
    d = {"graded": np.logspace(0, -14, n), "repeated": np.repeat([2.0, 1.0], [n // 2, n - n // 2]),
         "rank1": np.r_[1.0, np.zeros(n - 1)], "identity": np.ones(n)}[kind]
    a = (q * d) @ q.conj().T if kind != "identity" else np.diag(d).astype(complex)
    return 0.5 * (a + a.conj().T)


@pytest.mark.parametrize("n,kind", [(n, "graded") for n in (1, 2, 15, 17, 31, 32, 33, 48, 63, 65, 96, 97, 255)] +
                         [(48, "repeated"), (33, "rank1"), (40, "identity"), (40, "zero"), (16, "zero")])
def test_eigensolver_blocks(n, kind):
    L = T.lib()
    L.ttn_herm_eig.restype = C.c_int
    L.ttn_herm_eig.argtypes = [C.c_int32] + [C.c_void_p] * 5
    A = _matrix(n, kind)
    dA = torch.tensor(np.concatenate([A.real.ravel(order="F"), A.imag.ravel(order="F")]), dtype=torch.float64,
                      device="cuda")
    dV, dw = torch.zeros(2 * n * n, dtype=torch.float64, device="cuda"), torch.zeros(n, dtype=torch.float64, device="cuda")
    do = torch.zeros(n, dtype=torch.int32, device="cuda")
    print(f"[eig] n={n} {kind}", flush=True)
    assert L.ttn_herm_eig(n, dA.data_ptr(), dV.data_ptr(), dw.data_ptr(), do.data_ptr(),
                          torch.cuda.current_stream().cuda_stream) == 0
    w, order, v = dw.cpu().numpy(), do.cpu().numpy(), dV.cpu().numpy()
    V = (v[:n * n] + 1j * v[n * n:]).reshape(n, n, order="F")[:, order]
    ref = np.linalg.eigvalsh(A)[::-1]
    scale = max(abs(ref).max(), 1e-300)
    assert sorted(order.tolist()) == list(range(n)) and np.all(np.diff(w) <= 0)
    assert np.abs(w - ref).max() <= 1e-13 * scale
    assert np.abs(A @ V - V * w).max() <= 1e-12 * scale
    assert np.abs(V.conj().T @ V - np.eye(n)).max() <= 1e-12
