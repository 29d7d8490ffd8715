"""GPU: small float networks on both sides of the rule that gives them a
work-group per centre (from 1024 centres on, few products per column), against
the same network in float64 with autograd.  Bounds as in
test_gpu_train_shapes.py: twice the longest chain of float sums in front of a
result times 2^-24."""
import numpy as np
import pytest
import torch

import paper_2101_08814_amd as P

from test_gpu_train_shapes import network

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("S,nmax,lmax,Q,H,n", [(1, 2, 12, 4, 4, 1024), (1, 2, 12, 4, 4, 1023), (1, 8, 9, 4, 20, 1030),
                                               (2, 8, 4, 16, 12, 1025), (2, 8, 4, 16, 13, 1025), (4, 16, 2, 3, 5, 1100)])
def test_small_networks(S, nmax, lmax, Q, H, n):
    K, L2 = S * nmax, (lmax + 1) ** 2
    rng = np.random.default_rng(K + 3 * Q + 7 * H + n)
    calc = P.Calculator(S, nmax, lmax, 5.0, 0.5)
    net = P.Compressor(calc, Q, H)
    parts = []
    for _ in range(lmax + 1):
        parts += [rng.normal(size=H * K) / np.sqrt(K), rng.normal(size=Q * H) / np.sqrt(H), rng.normal(size=2 * H) * 0.5]
    w = np.concatenate(parts).astype(np.float32)
    c = rng.normal(size=(n, K, L2)).astype(np.float32)
    gp = rng.normal(size=(n, lmax + 1, Q * (Q + 1) // 2)).astype(np.float32)
    net.weights.copy_(torch.tensor(w))
    cd = torch.tensor(c.reshape(n, S, nmax, L2), device="cuda")
    ct, pt = net.forward(cd, want_coeffs=True)
    grad = net.backward(cd, torch.tensor(gp, device="cuda"))
    assert calc.device_status() == 0
    w64 = torch.tensor(w.astype(np.float64), requires_grad=True)
    r_ct, r_pt = network(w64, torch.tensor(c.astype(np.float64)), K, Q, H, lmax)
    (r_g,) = torch.autograd.grad((r_pt * torch.tensor(gp.astype(np.float64))).sum(), w64)
    rel = lambda a, b: float((a.double().cpu() - b).norm() / b.norm())  # noqa: E731
    u, M = 2.0 ** -24, 2 * lmax + 1
    e = rel(ct, r_ct.detach()), rel(pt, r_pt.detach()), rel(grad, r_g)
    print(f"[small K={K} Q={Q} H={H} lmax={lmax} n={n}] c~ {e[0]:.1e} p~ {e[1]:.1e} grad {e[2]:.1e}")
    assert e[0] <= 2 * (K + H + M) * u
    assert e[1] <= 2 * (2 * (K + H + M) + M) * u
    assert e[2] <= 2 * (2 * (K + H + M) + H + Q + n * M) * u
