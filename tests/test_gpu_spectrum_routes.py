"""GPU: the power spectrum on both sides of the rules that pick its kernel: a
centre by four or eight waves above 64 channels (few and many centres, small
and large c), and in FP32 the VALU kernel where the channels fill little of
their 16-wide blocks, against a float64 product.  FP32: each entry is a float
sum of 2l+1 <= 25 products, so its error is at most 25 2^-24 times the sum of
their absolute values; bfloat16 hi/lo: 2e-3 relative Frobenius error and per
centre, as in test_gpu_bf16_shapes.py."""
import numpy as np
import pytest
import torch

import paper_2101_08814_amd as P

from test_gpu_parity import rel, worst_centre

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["f32", "bf16"])
@pytest.mark.parametrize("S,nmax,lmax,N", [(6, 11, 2, 512), (6, 11, 2, 513), (6, 11, 8, 514), (8, 12, 5, 600),
                                           (8, 12, 6, 515), (2, 12, 10, 999), (2, 12, 10, 1001), (3, 9, 8, 1003),
                                           (3, 10, 9, 1000), (3, 11, 6, 1000), (3, 11, 6, 1001), (4, 9, 8, 1002),
                                           (5, 10, 4, 1000), (5, 10, 8, 1000), (7, 7, 0, 1001)])
def test_routes(S, nmax, lmax, N, prec):
    K, L2 = S * nmax, (lmax + 1) ** 2
    calc = P.Calculator(S, nmax, lmax, 5.0, 0.5)
    c = np.random.default_rng(K + lmax + N).standard_normal((N, K, L2)).astype(np.float32)
    p = calc.power_spectrum(torch.tensor(c, device="cuda").reshape(N, S, nmax, L2), prec)
    assert calc.device_status() == 0
    iu = np.triu_indices(K)
    at = np.unique(np.concatenate([np.arange(5), np.arange(N - 5, N), np.arange(0, N, 37)]))
    got, ref, bound = p.double().cpu().numpy()[at], [], []
    for l in range(lmax + 1):
        x = c[at][:, :, l * l:(l + 1) ** 2].astype(np.float64)
        ref.append((x @ x.transpose(0, 2, 1))[:, iu[0], iu[1]])
        bound.append(25 * 2.0 ** -24 * (np.abs(x) @ np.abs(x).transpose(0, 2, 1))[:, iu[0], iu[1]])
    ref, bound = np.stack(ref, 1), np.stack(bound, 1)
    if prec == "f32":
        assert np.all(np.abs(got - ref) <= bound)
    else:
        assert rel(got, ref) <= 2e-3 and worst_centre(got, ref) <= 2e-3
    # every centre: the sum of all entries against the product's own
    tot = p.double().sum(dim=(1, 2)).cpu().numpy()
    full = c.astype(np.float64).reshape(N, K, L2)
    want = 0.5 * ((full.sum(1) ** 2).sum(1) + (full ** 2).sum(axis=(1, 2)))
    scale = 0.5 * ((np.abs(full).sum(1) ** 2).sum(1) + (full ** 2).sum(axis=(1, 2)))
    assert np.all(np.abs(tot - want) <= (25 * 2.0 ** -24 if prec == "f32" else 2e-3) * scale)
