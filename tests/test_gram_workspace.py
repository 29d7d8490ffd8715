"""The workspace of the kernel matrix and the training loss: a small part of
the matrix itself where its tiles already fill the chip, and the products in
that form on the GPU, over more tiles than there are work-groups to aim for."""
import ctypes

import numpy as np
import pytest
import torch

import paper_2101_08814_amd as P
from paper_2101_08814_amd import _lib

from test_gpu_gram import U, weights_of


def workspace(n, Q, lmax):
    nb = ctypes.c_size_t()
    _lib.check(_lib.lib().soap_spectrum_gram_workspace_size(n, Q, lmax, ctypes.byref(nb)))
    return nb.value


@pytest.mark.parametrize("n", [2048, 2900, 16384, 65536])
@pytest.mark.parametrize("Q,lmax", [(16, 6), (96, 8), (4096, 12)])
def test_small_beside_the_matrix(n, Q, lmax):
    assert workspace(n, Q, lmax) <= 4 * n * n // 100


@pytest.mark.gpu
def test_many_tiles():
    """n = 2113 (34 tile rows, the last of one row): bounds as in
    test_gpu_gram.py."""
    n, Q, lmax = 2113, 8, 3
    rng = np.random.default_rng(n)
    F = (lmax + 1) * Q * (Q + 1) // 2
    X = rng.normal(size=(n, F)).astype(np.float32)
    Kref = rng.normal(size=(n, n)).astype(np.float32) * F
    w = weights_of(Q, lmax)
    X64, R64 = X.astype(np.float64), Kref.astype(np.float64)
    K64 = (X64 * w) @ X64.T
    bound_K = (F + 64) * U * ((np.abs(X64) * w) @ np.abs(X64).T)
    calc = P.Calculator(1, Q, lmax, 5.0, 0.5)
    net = P.Compressor(calc, Q, 4)
    Xd = torch.tensor(X, device="cuda")
    K = net.gram(Xd, Q)
    assert np.all(np.abs(K.double().cpu().numpy() - K64) <= bound_K)
    loss, gX = net.kernel_loss(Xd, torch.tensor(Kref, device="cuda"))
    D, n2 = K64 - R64, (R64 ** 2).sum()
    L64 = (D ** 2).sum() / n2
    assert abs(float(loss) - L64) <= (2 * np.abs(D) * bound_K + bound_K ** 2).sum() / n2 + 4 * U * L64
    G64 = 4 / n2 * (D @ X64) * w
    bound_G = 4 / n2 * w * ((bound_K + U * np.abs(D)) @ np.abs(X64) + (n + 8) * U * (np.abs(D) @ np.abs(X64)))
    assert np.all(np.abs(gX.double().cpu().numpy() - G64) <= bound_G)


@pytest.mark.parametrize("n,Q,lmax", [(1, 8, 6), (256, 64, 6), (300, 48, 6), (64, 72, 6), (500, 32, 6), (700, 33, 12),
                                      (900, 20, 2)])
def test_slices_keep_to_the_xcds(n, Q, lmax):
    """Eight slices or more are a multiple of eight, so that work-groups
    that differ by eight (one XCD) take the same columns of X."""
    tiles = -(-n // 64) * (-(-n // 64) + 1) // 2
    bytes_ = workspace(n, Q, lmax)
    slices = (bytes_ - 64 * tiles) / (16384 * tiles) if bytes_ > 64 * tiles else 1
    assert slices == int(slices) and (slices < 8 or slices % 8 == 0)
