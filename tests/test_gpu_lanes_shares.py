"""GPU: c and p in one kernel (fewer than 4096 centres) where a pair's radial
values are shared by one, two or four lanes of a wave: at the edges of the
chunks and of the shares, nmax on both sides of multiples of four, against
the FP64 oracle.  Tolerances as in test_gpu_parity.py (relative Frobenius
error: FP64 <= 1e-7, FP32 <= 1e-6)."""
import numpy as np
import pytest
import torch

import oracle
import paper_2101_08814_amd as P
from synthetic.structures import _hypers

from test_gpu_lanes_split import _clusters
from test_gpu_parity import gpu_neighbors, rel

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dt", [torch.float32, torch.float64])
@pytest.mark.parametrize("nmax,lmax", [(1, 0), (4, 3), (5, 8), (3, 12), (13, 2)])
@pytest.mark.parametrize("sizes", [(1, 2, 16, 17, 18), (1, 2, 32, 33, 34, 64, 65, 66, 98) + 30 * (17,)])
def test_shares(sizes, nmax, lmax, dt):
    b = _clusters(sizes, _hypers(2, 6.5, 0.5, nmax, lmax))
    calc = P.Calculator.from_hypers(b.hypers)
    nl, pos, spc = gpu_neighbors(calc, b, dt)
    c, p = calc.features(nl, spc, dt)
    assert calc.device_status() == 0
    ref_c = oracle.expansion(b.hypers, b.species, oracle.neighbors(b))
    ref_p = oracle.power_spectrum(b.hypers, ref_c)
    tol = 1e-7 if dt == torch.float64 else 1e-6
    off = np.concatenate([[0], np.cumsum(sizes)])
    c, p = c.double().cpu().numpy(), p.double().cpu().numpy()
    for k, n in enumerate(sizes):
        s = slice(off[k], off[k + 1])
        assert rel(c[s], ref_c[s]) <= tol, n
        assert rel(p[s], ref_p[s]) <= 2 * tol, n
