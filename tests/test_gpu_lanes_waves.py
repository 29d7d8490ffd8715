"""GPU: c and p in one kernel (fewer than 4096 centres) by one, two and four
waves per centre, centres of several chunks among them, with the pairs grouped
by species and in a random order (then the work-group's waves redo the centre
together, one species at a time).  The batch is copies of a few open clusters,
one copy compared with the FP64 oracle, the others with it.  Tolerances as in
test_gpu_lanes.py (relative Frobenius error: FP64 <= 1e-7, FP32 <= 1e-6 against
the oracle, twice that for p in FP32; 1e-12 and 1e-6 between the lists)."""
import numpy as np
import pytest
import torch

import oracle
import paper_2101_08814_amd as P
from paper_2101_08814_amd.soap import Neighbors
from synthetic.structures import _hypers

from test_gpu_lanes_split import _clusters
from test_gpu_parity import gpu_neighbors, rel

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dt", [torch.float32, torch.float64])
@pytest.mark.parametrize("nmax,lmax,n", [(5, 4, 100), (5, 4, 700), (9, 6, 600), (4, 2, 2600), (4, 3, 2499), (4, 3, 2500),
                                         (6, 4, 2600), (3, 8, 2600)])
def test_waves_per_centre(nmax, lmax, n, dt):
    sizes = (1, 2, 17, 34, 66)
    one = _clusters(sizes, _hypers(2, 6.5, 0.5, nmax, lmax))
    copies = -(-n // one.n_atoms)
    b = _clusters(sizes * copies, one.hypers)
    b.positions, b.species = np.tile(one.positions, (copies, 1)), np.tile(one.species, copies)
    calc = P.Calculator.from_hypers(b.hypers)
    nl, pos, spc = gpu_neighbors(calc, b, dt)
    c, p = (t.double().reshape(copies, -1) for t in calc.features(nl, spc, dt))
    assert calc.device_status() == 0
    ref_c = oracle.expansion(one.hypers, one.species, oracle.neighbors(one))
    ref_p = oracle.power_spectrum(one.hypers, ref_c)
    f64 = dt == torch.float64
    assert rel(c[0].cpu().numpy(), ref_c.reshape(-1)) <= (1e-7 if f64 else 1e-6)
    assert rel(p[0].cpu().numpy(), ref_p.reshape(-1)) <= 2 * (1e-7 if f64 else 1e-6)
    off = nl.pair_offsets.cpu().numpy()
    n_pairs = int(off[-1])
    centre = np.repeat(np.arange(b.n_atoms), np.diff(off))
    perm = torch.tensor(np.lexsort((np.random.default_rng(9).random(n_pairs), centre)), device="cuda")
    nl2 = Neighbors(nl.pair_offsets, nl.pair_j[perm].contiguous(), nl.pair_shift[perm].contiguous(),
                    nl.pair_vec[perm].contiguous(), None, n_pairs)
    c2, p2 = (t.double().reshape(copies, -1) for t in calc.features(nl2, spc, dt))
    assert calc.device_status() == 0
    same = 1e-12 if f64 else 1e-6
    for x, x2 in ((c, c2), (p, p2)):
        assert float(((x - x[0]).norm(dim=1) / x[0].norm()).max()) <= same
        assert float(((x2 - x).norm(dim=1) / x[0].norm()).max()) <= 2 * same
