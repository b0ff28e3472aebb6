"""Accuracy of the Hermitian eigensolver (ttn_herm_eig) against extended
precision, on Gram matrices with a spectrum over six decades (those of a
two-site split): eigenvalues within 4 eps of the spectrum's norm, the projector
on the leading eigenvectors within 1e-14 of its norm -- eigenvectors rounded
entry by entry, a few eps in every product of two -- where the rounding of the
rotations alone leaves n eps over the gap, 1e-13 and more at these sizes; all
eigenvectors orthonormal to 1e-13, also of a matrix that is Hermitian to
rounding only."""
import ctypes as C

import numpy as np
import pytest
import torch

from paper_2210_03763_amd import ttn as T

pytestmark = pytest.mark.gpu


def _refined(a):
    """Eigenvalues (descending) and vectors in extended precision: numpy's, corrected to first order twice."""
    A, V = a.astype(np.clongdouble), np.linalg.eigh(a)[1].astype(np.clongdouble)
    for _ in range(2):
        R = np.eye(len(a)) - V.conj().T @ V
        S = V.conj().T @ (A @ V)
        lam = np.real(np.diag(S)) / (1 - np.real(np.diag(R)))
        gap = lam[None, :] - lam[:, None]
        np.fill_diagonal(gap, 1)
        E = (S + R * lam[None, :]) / gap
        np.fill_diagonal(E, np.diag(R) / 2)
        V = V + V @ E
    return lam[::-1], V[:, ::-1]


@pytest.mark.parametrize("n", [3, 4, 5, 8, 9, 12, 16, 17, 24, 25, 32, 33, 39, 40, 41, 48, 49, 70, 144, 200])
def test_leading_projector(n):
    L = T.lib()
    L.ttn_herm_eig.restype = C.c_int
    L.ttn_herm_eig.argtypes = [C.c_int32] + [C.c_void_p] * 5
    rng = np.random.default_rng(n)
    z = lambda *s: rng.standard_normal(s) + 1j * rng.standard_normal(s)
    m = (z(4 * n, n) * np.logspace(0, -3, n)) @ np.linalg.qr(z(n, n))[0] / np.sqrt(4 * n)
    a = m.conj().T @ m
    dA = torch.tensor(np.concatenate([a.real.ravel(order="F"), a.imag.ravel(order="F")]), dtype=torch.float64,
                      device="cuda")
    dV, dw = torch.zeros(2 * n * n, dtype=torch.float64, device="cuda"), torch.zeros(n, dtype=torch.float64, device="cuda")
    do = torch.zeros(n, dtype=torch.int32, device="cuda")
    print(f"[eig] n={n} accuracy", flush=True)
    assert L.ttn_herm_eig(n, dA.data_ptr(), dV.data_ptr(), dw.data_ptr(), do.data_ptr(),
                          torch.cuda.current_stream().cuda_stream) == 0
    w, order, v = dw.cpu().numpy(), do.cpu().numpy(), dV.cpu().numpy()
    k = max(1, n // 12)
    lam, X = _refined(a)
    V = (v[:n * n] + 1j * v[n * n:]).reshape(n, n, order="F")[:, order]
    assert np.abs(V.conj().T @ V - np.eye(n)).max() <= 1e-13
    V = V[:, :k].astype(np.clongdouble)
    norm = lambda d: float(np.sqrt(np.sum(np.abs(d) ** 2)))
    ew = norm(w - lam) / norm(lam)
    ep = norm(V @ V.conj().T - X[:, :k] @ X[:, :k].conj().T) / np.sqrt(k)
    print(f"[eig] eigenvalues {ew:.2e} projector {ep:.2e}", flush=True)
    assert ew <= 4 * np.finfo(float).eps
    assert ep <= 1e-14
