"""GPU: infinities and NaN in the inputs of the products on the matrix cores
stay where the sums have them (no padded row, column or step of a tile takes
part): the FP32 power spectrum by one, four and eight waves per centre and by
the VALU kernel, and the kernel matrix in one and in many slices, against the
same sums in float64."""
import numpy as np
import pytest
import torch

import paper_2101_08814_amd as P

from test_gpu_gram import weights_of

pytestmark = pytest.mark.gpu

BAD = (np.inf, -np.inf, np.nan)


def kinds(x):
    return np.isnan(x) * 1 + np.isposinf(x) * 2 + np.isneginf(x) * 4


@pytest.mark.parametrize("b", range(3))
@pytest.mark.parametrize("S,nmax,lmax,N", [(1, 5, 3, 4), (3, 8, 6, 9), (3, 9, 8, 1001), (5, 13, 4, 6), (8, 12, 8, 3),
                                           (6, 11, 3, 600)])
def test_spectrum(S, nmax, lmax, N, b):
    K = S * nmax
    calc = P.Calculator(S, nmax, lmax, 5.0, 0.5)
    c = np.random.default_rng(S + b).standard_normal((N, K, calc.L2)).astype(np.float32)
    c[N // 2, K - 1, calc.L2 - 1] = BAD[b]
    c[1, 0, 0] = BAD[(b + 1) % 3]
    p = calc.power_spectrum(torch.tensor(c.reshape(N, S, nmax, -1), device="cuda"), torch.float32).cpu().numpy()
    assert calc.device_status() == 0
    iu = np.triu_indices(K)
    at = sorted({0, 1, 2, N // 2, N - 1})
    for l in range(lmax + 1):
        x = c[at, :, l * l:(l + 1) ** 2].astype(np.float64)
        with np.errstate(invalid="ignore"):
            ref = (x[:, iu[0]] * x[:, iu[1]]).sum(2)
        assert np.array_equal(kinds(p[at, l]), kinds(ref)), l
    rest = np.setdiff1d(np.arange(N), [1, N // 2])
    assert np.isfinite(p[rest]).all()


@pytest.mark.parametrize("b", range(3))
@pytest.mark.parametrize("n,Q,lmax", [(5, 3, 2), (130, 30, 4), (300, 6, 1)])
def test_kernel_matrix(n, Q, lmax, b):
    calc = P.Calculator(1, 8, lmax, 5.0, 0.5)
    net = P.Compressor(calc, Q, 4)
    rng = np.random.default_rng(n + b)
    X = rng.standard_normal((n, (lmax + 1) * Q * (Q + 1) // 2)).astype(np.float32)
    X[n // 2, -1] = BAD[b]
    X[1, 1] = BAD[b]
    K = net.gram(torch.tensor(X, device="cuda"), Q).cpu().numpy()
    with np.errstate(invalid="ignore"):
        x = X.astype(np.float64)
        ref = np.stack([(x * weights_of(Q, lmax) * x[i]).sum(1) for i in range(n)])
    assert np.array_equal(kinds(K), kinds(ref))
