"""GPU: the expansion's adjoint in the forms that a rule on the degree, nmax
and the number of centres picks: whole pairs with two waves a SIMD at lmax 9
in float (over 1024 centres, and one n at any number), one n above it, and
groups of two cubics or one in double up to lmax 5, with an even and an odd
last group.  Copies of a few open clusters, every copy per pair against the
FP64 oracle.  Tolerances as in test_gpu_parity.py (relative Frobenius error of
a gradient: FP64 <= 1e-7, FP32 <= 1e-5)."""
import numpy as np
import pytest
import torch

import oracle
import paper_2101_08814_amd as P
from synthetic.structures import _hypers

from test_gpu_lanes_split import _clusters
from test_gpu_parity import gpu_neighbors, rel

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dt,nmax,lmax,copies", [(torch.float32, 5, 9, 11), (torch.float32, 1, 9, 1),
                                                 (torch.float32, 1, 12, 1), (torch.float64, 1, 0, 1),
                                                 (torch.float64, 4, 2, 1), (torch.float64, 5, 4, 1),
                                                 (torch.float64, 3, 5, 1)])
def test_forms(dt, nmax, lmax, copies):
    sizes = (1, 2, 33, 65)
    one = _clusters(sizes, _hypers(2, 6.5, 0.5, nmax, lmax))
    b = _clusters(sizes * copies, one.hypers)
    b.positions, b.species = np.tile(one.positions, (copies, 1)), np.tile(one.species, copies)
    calc = P.Calculator.from_hypers(b.hypers)
    nl, pos, spc = gpu_neighbors(calc, b, dt)
    gc = np.random.default_rng(29).standard_normal((one.n_atoms, 2, nmax, (lmax + 1) ** 2))
    _, gpair = calc.spherical_expansion_backward(
        nl, spc, torch.tensor(np.tile(gc, (copies, 1, 1, 1)), dtype=dt, device="cuda"))
    assert calc.device_status() == 0
    ref_nl = oracle.neighbors(one)
    dc = oracle.gradients(one.hypers, one.species, ref_nl)[0]
    centre = np.repeat(np.arange(one.n_atoms), np.diff(ref_nl.pair_offsets))
    ref = np.einsum("qanm,qnm->qa", dc, gc[centre, one.species[ref_nl.pair_j]])
    got = gpair.double().cpu().numpy().reshape(copies, ref_nl.n_pairs, 3)
    for k in range(copies):
        assert rel(got[k], ref) <= (1e-7 if dt == torch.float64 else 1e-5), k
