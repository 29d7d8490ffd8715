"""GPU: the expansion's adjoint where a pair has two lanes (the degrees above
8 in float and 5 in double, a chunk of at most 32 pairs), at the edges of the
chunks and of the halves of nmax, per pair against the FP64 oracle.
Tolerances as in test_gpu_parity.py (relative Frobenius error of a gradient:
FP64 <= 1e-7, FP32 <= 1e-5)."""
import numpy as np
import pytest
import torch

import oracle
import paper_2101_08814_amd as P
from synthetic.structures import _hypers, _pack

from test_gpu_parity import gpu_neighbors, rel

pytestmark = pytest.mark.gpu


def _clusters(sizes, hypers):
    """Open clusters in which every atom is a neighbour of every other."""
    rng = np.random.default_rng(17)
    grid = np.stack(np.meshgrid(*[np.arange(5) * 0.75] * 3, indexing="ij"), -1).reshape(-1, 3)
    structs = []
    for n in sizes:
        pos = rng.permutation(grid)[:n] + rng.uniform(-0.1, 0.1, (n, 3))
        structs.append((pos, rng.integers(0, 2, n), np.eye(3) * 20.0, np.zeros(3, dtype=np.uint8)))
    return _pack(structs, hypers, "clusters")


@pytest.mark.parametrize("dt,nmax,lmax", [(torch.float32, 1, 9), (torch.float32, 5, 9), (torch.float32, 4, 10),
                                          (torch.float32, 3, 12), (torch.float64, 2, 6), (torch.float64, 5, 7),
                                          (torch.float64, 3, 10)])
def test_halves(dt, nmax, lmax):
    sizes = (1, 2, 33, 34, 65, 66, 97, 98)   # 0, 1, 32, 33, 64, 64 + 1, 64 + 32 and 64 + 33 pairs
    b = _clusters(sizes, _hypers(2, 6.5, 0.5, nmax, lmax))
    calc = P.Calculator.from_hypers(b.hypers)
    nl, pos, spc = gpu_neighbors(calc, b, dt)
    assert nl.count() == sum(n * (n - 1) for n in sizes)
    gc = np.random.default_rng(23).standard_normal((b.n_atoms, 2, nmax, (lmax + 1) ** 2))
    gpos, gpair = calc.spherical_expansion_backward(nl, spc, torch.tensor(gc, dtype=dt, device="cuda"))
    assert calc.device_status() == 0
    ref_nl = oracle.neighbors(b)
    dc = oracle.gradients(b.hypers, b.species, ref_nl)[0]
    centre = np.repeat(np.arange(b.n_atoms), np.diff(ref_nl.pair_offsets))
    sj = b.species[ref_nl.pair_j]
    ref = np.einsum("qanm,qnm->qa", dc, gc[centre, sj])
    tol = 1e-7 if dt == torch.float64 else 1e-5
    got = gpair[:ref_nl.n_pairs].double().cpu().numpy()
    for k in np.unique(np.diff(ref_nl.pair_offsets)):
        if k:
            at = np.diff(ref_nl.pair_offsets)[centre] == k
            assert rel(got[at], ref[at]) <= tol, k
