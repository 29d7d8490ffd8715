"""GPU: forward pass and weight gradient of the compression network in float
at the edges of its tiles (16 channels, units and outputs; groups of 32
columns with up to eight centres), against the same network in float64 with
autograd.  The bound is the length of the longest chain of float sums in
front of each result times 2^-24, doubled for the gate's transcendentals:
K + H terms for c~ (twice for p~, which is quadratic), and for the gradient
another H + Q terms back and the n (2 lmax + 1) columns of the last product."""
from __future__ import annotations

import numpy as np
import pytest
import torch

import paper_2101_08814_amd as P

pytestmark = pytest.mark.gpu


def network(w, c, K, Q, H, lmax):
    """(c~, p~) in the precision of w and c [n, K, L2]."""
    iu = torch.triu_indices(Q, Q)
    o, ct, pt = 0, [], []
    for l in range(lmax + 1):
        W1, W2 = w[o:o + H * K].reshape(H, K), w[o + H * K:o + H * K + Q * H].reshape(Q, H)
        o += H * K + Q * H
        al, be = w[o:o + H], w[o + H:o + 2 * H]
        o += 2 * H
        h = torch.einsum("qk,ikm->iqm", W1, c[:, :, l * l:(l + 1) ** 2])
        s = torch.sigmoid(al[None] * h.pow(2).sum(2).sqrt() + be[None])
        x = torch.einsum("pq,iqm->ipm", W2, 2.0 * s[:, :, None] * h)
        ct.append(x)
        pt.append((x[:, iu[0]] * x[:, iu[1]]).sum(2))
    return torch.cat(ct, 2), torch.stack(pt, 1)


@pytest.mark.parametrize("S,nmax,lmax,Q,H,n", [(1, 1, 0, 1, 1, 1), (1, 5, 2, 7, 16, 9), (2, 16, 3, 16, 17, 33),
                                               (3, 11, 12, 17, 40, 5), (5, 16, 1, 32, 128, 70), (8, 9, 6, 32, 128, 130),
                                               (8, 12, 8, 12, 96, 40), (8, 16, 4, 31, 128, 17), (8, 16, 8, 16, 128, 3),
                                               (9, 15, 2, 8, 20, 6), (2, 4, 2, 33, 20, 6), (2, 4, 2, 8, 130, 6)])
def test_float_forward_and_gradient(S, nmax, lmax, Q, H, n):
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
    ct_only, _ = net.forward(cd, want_coeffs=True, want_p=False)
    grad = net.backward(cd, torch.tensor(gp, device="cuda")).clone()
    again = net.backward(cd, torch.tensor(gp, device="cuda"))
    assert calc.device_status() == 0
    w64 = torch.tensor(w.astype(np.float64), requires_grad=True)
    r_ct, r_pt = network(w64, torch.tensor(c.astype(np.float64)), K, Q, H, lmax)
    (r_g,) = torch.autograd.grad((r_pt * torch.tensor(gp.astype(np.float64))).sum(), w64)
    rel = lambda a, b: float((a.double().cpu() - b).norm() / b.norm())  # noqa: E731
    u, M = 2.0 ** -24, 2 * lmax + 1
    e = rel(ct, r_ct.detach()), rel(pt, r_pt.detach()), rel(grad, r_g)
    print(f"[train K={K} Q={Q} H={H} lmax={lmax} n={n}] c~ {e[0]:.1e} p~ {e[1]:.1e} grad {e[2]:.1e}")
    assert e[0] <= 2 * (K + H + M) * u
    assert e[1] <= 2 * (2 * (K + H + M) + M) * u
    assert e[2] <= 2 * (2 * (K + H + M) + H + Q + n * M) * u
    assert torch.equal(ct_only, ct) and torch.equal(again, grad)
