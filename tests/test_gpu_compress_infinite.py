"""GPU: an infinite coefficient in the bfloat16 compression, with and without
the laid-out weights: with positive weights c~ is +inf in that column m of its
degree and finite in the others, the other degrees and the other centres, as
in float, also where the hidden units fill only part of the tiles (32 and 96;
a padded unit's product with infinity must not reach the outputs)."""
import numpy as np
import pytest
import torch

import paper_2101_08814_amd as P

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("lmax,lm", [(3, 5), (8, 70)])
@pytest.mark.parametrize("H", [32, 64, 96, 128])
def test_infinite_coefficient(H, lmax, lm):
    S, nmax, Q, n = 4, 10, 8, 5
    calc = P.Calculator(S, nmax, lmax, 5.0, 0.5)
    net = P.Compressor(calc, Q, H)
    rng = np.random.default_rng(H + lmax)
    net.weights.copy_(torch.tensor(rng.uniform(0.05, 0.2, net.n_params).astype(np.float32)))
    c = torch.tensor(rng.uniform(0.1, 1.0, (n, S, nmax, calc.L2)).astype(np.float32), device="cuda")
    c[2, 1, 3, lm] = float("inf")
    want = torch.zeros((n, Q, calc.L2), dtype=torch.bool, device="cuda")
    want[2, :, lm] = True
    for ct in (net.forward(c, precision="bf16", want_coeffs=True)[0],
               net.forward_plain(c, precision="bf16", want_coeffs=True)[0],
               net.forward(c, want_coeffs=True)[0]):
        assert calc.device_status() == 0
        assert torch.equal(torch.isposinf(ct), want)
        assert torch.isfinite(ct[~want]).all()
