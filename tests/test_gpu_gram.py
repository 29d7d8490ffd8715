"""GPU: the kernel matrix of packed spectra and the training loss at the
edges of the 64 x 64 tiles, the 32-wide slabs and the feature split, against
float64.  The bounds are the worst case of a float sum: every entry is a sum
of F products (in parts, which only lowers it), so its error is at most
(F + 64) 2^-24 times the same sum of absolute values; the gradient adds the
error of D = K~ - Kref carried through the product over j and that product's
own (n + 8) 2^-24."""
from __future__ import annotations

import ctypes

import numpy as np
import pytest
import torch

import paper_2101_08814_amd as P
from paper_2101_08814_amd import _lib

pytestmark = pytest.mark.gpu

U = 2.0 ** -24


def weights_of(Q, lmax):
    iu = np.triu_indices(Q)
    return np.tile(np.where(iu[0] == iu[1], 1.0, 2.0), lmax + 1)


@pytest.mark.parametrize("n,Q,lmax", [(1, 1, 0), (3, 1, 12), (63, 5, 3), (64, 4, 0), (65, 12, 2), (130, 30, 4),
                                      (257, 9, 12), (70, 72, 6), (512, 8, 1)])
@pytest.mark.parametrize("split", [True, False])
def test_gram_and_loss_tiles(n, Q, lmax, split):
    rng = np.random.default_rng(n + Q + lmax)
    F = (lmax + 1) * Q * (Q + 1) // 2
    X = rng.normal(size=(n, F)).astype(np.float32)
    Kref = rng.normal(size=(n, n)).astype(np.float32) * F
    w = weights_of(Q, lmax)
    X64, R64 = X.astype(np.float64), Kref.astype(np.float64)
    K64 = (X64 * w) @ X64.T
    bound_K = (F + 64) * U * ((np.abs(X64) * w) @ np.abs(X64).T)
    Xd, Rd = torch.tensor(X, device="cuda"), torch.tensor(Kref, device="cuda")
    calc = P.Calculator(1, Q if Q <= 16 else 8, lmax, 5.0, 0.5)
    net = P.Compressor(calc, min(Q, 64), 4)
    if split:
        K = net.gram(Xd, Q)
    else:
        K = torch.empty((n, n), dtype=torch.float32, device="cuda")
        e = calc._exec()
        _lib.check(_lib.lib().soap_spectrum_gram(ctypes.byref(e), n, Q, lmax, Xd.data_ptr(), K.data_ptr()))
    err = np.abs(K.double().cpu().numpy() - K64)
    assert np.all(err <= bound_K), float((err / bound_K).max())
    assert torch.equal(K, K.T.contiguous())
    # loss and gradient
    gX = torch.empty_like(Xd)
    work = torch.empty(n * n + 1, dtype=torch.float32, device="cuda")
    loss = torch.empty(1, dtype=torch.float32, device="cuda")
    e, L, nb = calc._exec(), _lib.lib(), ctypes.c_size_t()
    args = (ctypes.byref(e), n, Q, lmax, Xd.data_ptr(), Rd.data_ptr(), work.data_ptr(), loss.data_ptr(), gX.data_ptr())
    if split:
        _lib.check(L.soap_spectrum_gram_workspace_size(n, Q, lmax, ctypes.byref(nb)))
        ws = torch.empty(nb.value, dtype=torch.uint8, device="cuda")
        _lib.check(L.soap_spectrum_kernel_loss_ws(*args, ws.data_ptr(), ws.numel()))
        assert L.soap_spectrum_kernel_loss_ws(*args, ws.data_ptr(), ws.numel() - 1) == _lib.SOAP_EINVAL
    else:
        _lib.check(L.soap_spectrum_kernel_loss(*args))
    D, n2 = K64 - R64, (R64 ** 2).sum()
    L64 = (D ** 2).sum() / n2
    # D's entries are off by bound_K, its square by twice that times |D|
    assert abs(float(loss) - L64) <= (2 * np.abs(D) * bound_K + bound_K ** 2).sum() / n2 + 4 * U * L64
    G64 = 4 / n2 * (D @ X64) * w
    bound_G = 4 / n2 * w * ((bound_K + U * np.abs(D)) @ np.abs(X64) + (n + 8) * U * (np.abs(D) @ np.abs(X64)))
    err = np.abs(gX.double().cpu().numpy() - G64)
    assert np.all(err <= bound_G), float((err / bound_G).max())
