"""GPU: the bfloat16 compression with the weights laid out in the workspace,
at every number of 32-wide steps over the channels, both numbers of hidden
tiles, one and two output tiles, ragged sizes and one and two tiles of m:
bit for bit the form without a workspace, and within the bounds of
test_gpu_compression.py of the oracle."""
import numpy as np
import pytest
import torch

import paper_2101_08814_amd as P
from oracle import compression as C

from test_gpu_compression import BF16_CT, BF16_PT, random_weights, rel

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("S,nmax,lmax,Q,H,n", [(1, 4, 7, 1, 4, 67), (4, 16, 12, 16, 64, 2), (8, 12, 5, 31, 60, 9),
                                               (10, 10, 3, 32, 68, 3), (8, 16, 8, 17, 128, 1), (8, 16, 12, 32, 124, 3),
                                               (3, 12, 1, 5, 100, 65)])
def test_shapes(S, nmax, lmax, Q, H, n):
    K, L2 = S * nmax, (lmax + 1) ** 2
    calc = P.Calculator(S, nmax, lmax, 5.0, 0.5)
    c = np.random.default_rng(K + H).standard_normal((n, K, L2)).astype(np.float32)
    cd = torch.tensor(c, device="cuda").reshape(n, S, nmax, L2)
    net = P.Compressor(calc, Q, H)
    w = random_weights(11, K, Q, H, lmax)
    net.weights.copy_(torch.tensor(w))
    ct, pt = net.forward(cd, precision="bf16", want_coeffs=True)
    ct_b, pt_b = net.forward_plain(cd, precision="bf16", want_coeffs=True)
    _, pt_alone = net.forward(cd, precision="bf16")
    assert calc.device_status() == 0
    assert torch.equal(ct, ct_b) and torch.equal(pt, pt_b) and torch.equal(pt, pt_alone)
    ref = C.compress(c.astype(np.float64), w.astype(np.float64), Q, H)
    assert rel(ct, ref) <= BF16_CT and rel(pt, C.power_spectrum(ref)) <= BF16_PT
