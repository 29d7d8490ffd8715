"""GPU: the FP32 power spectrum on the matrix cores for few centres (from 24
channels on it serves any number of them), at one centre, a partial
work-group, the edges of the row blocks and of the split of a centre over
four and eight waves (K <= 64 and above), against a float64 product.  Each
entry is a float sum of 2l+1 <= 25 products, so its error is at most 25 2^-24
times the sum of their absolute values."""
import numpy as np
import pytest
import torch

import paper_2101_08814_amd as P

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("S,nmax,lmax,N", [(3, 8, 6, 1), (2, 12, 0, 5), (3, 11, 12, 3), (3, 16, 8, 7), (7, 7, 2, 2),
                                           (4, 16, 5, 9), (5, 13, 5, 4), (8, 12, 8, 3), (8, 16, 12, 2), (8, 16, 1, 300)])
def test_few_centres(S, nmax, lmax, N):
    K, L2 = S * nmax, (lmax + 1) ** 2
    calc = P.Calculator(S, nmax, lmax, 5.0, 0.5)
    c = np.random.default_rng(K + lmax).standard_normal((N, K, L2)).astype(np.float32)
    p = calc.power_spectrum(torch.tensor(c, device="cuda").reshape(N, S, nmax, L2), torch.float32)
    assert calc.device_status() == 0
    iu = np.triu_indices(K)
    got = p.double().cpu().numpy()
    for l in range(lmax + 1):
        x = c[:, :, l * l:(l + 1) ** 2].astype(np.float64)
        ref = (x @ x.transpose(0, 2, 1))[:, iu[0], iu[1]]
        bound = 25 * 2.0 ** -24 * (np.abs(x) @ np.abs(x).transpose(0, 2, 1))[:, iu[0], iu[1]]
        assert np.all(np.abs(got[:, l] - ref) <= bound), l
