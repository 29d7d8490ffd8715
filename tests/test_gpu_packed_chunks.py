"""GPU: c alone in chunks of 16 and of 32 pairs with one, two and four centres
per wave: centres of few and of many pairs around the chunk's length, every
number of quads of nmax, on both sides of what the chip holds at once.  The
batch is copies of a few open clusters, of which one copy is compared with the
FP64 oracle and the others with it; the same list with every centre's pairs in
a random order (not grouped by species) has the same sums in another order.
Tolerances as in test_gpu_packed.py (relative Frobenius error: FP64 <= 1e-7,
FP32 <= 1e-6 against the oracle, 1e-12 and 1e-6 between the forms)."""
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

SHORT = (1, 2, 5, 16, 17, 18)   # 14 pairs a centre on average
LONG = (33, 34, 17, 65)         # 44


@pytest.mark.parametrize("dt", [torch.float32, torch.float64])
@pytest.mark.parametrize("sizes,nmax,lmax,n", [(SHORT, 3, 2, 1), (SHORT, 3, 2, 5000), (SHORT, 4, 2, 9000),
                                               (LONG, 2, 0, 20000), (SHORT, 5, 3, 5000), (LONG, 6, 4, 4600),
                                               (SHORT, 8, 6, 17000), (LONG, 5, 3, 33000), (LONG, 9, 5, 3001),
                                               (LONG, 13, 8, 300), (LONG, 12, 8, 1500)])
def test_chunks_and_centres_per_wave(sizes, nmax, lmax, n, dt):
    one = _clusters(sizes, _hypers(2, 6.5, 0.5, nmax, lmax))
    copies = -(-n // one.n_atoms)
    b = _clusters(sizes, one.hypers)
    b.positions = np.tile(one.positions, (copies, 1))
    b.species = np.tile(one.species, copies)
    b.atom_offsets = np.concatenate([[0]] + [one.atom_offsets[1:] + k * one.n_atoms for k in range(copies)])
    b.cells, b.pbc = np.tile(one.cells, (copies, 1, 1)), np.tile(one.pbc, (copies, 1))
    calc = P.Calculator.from_hypers(b.hypers)
    nl, pos, spc = gpu_neighbors(calc, b, dt)
    c = calc.spherical_expansion(nl, spc, dt).double().reshape(copies, -1)
    assert calc.device_status() == 0
    ref = oracle.expansion(one.hypers, one.species, oracle.neighbors(one))
    f64 = dt == torch.float64
    assert rel(c[0].cpu().numpy(), ref.reshape(-1)) <= (1e-7 if f64 else 1e-6)
    same = 1e-12 if f64 else 1e-6
    assert float(((c - c[0]).norm(dim=1) / c[0].norm()).max()) <= same
    # the pairs of every centre in a random order
    off = nl.pair_offsets.cpu().numpy()
    n_pairs = int(off[-1])
    centre = np.repeat(np.arange(b.n_atoms), np.diff(off))
    perm = torch.tensor(np.lexsort((np.random.default_rng(9).random(n_pairs), centre)), device="cuda")
    nl2 = Neighbors(nl.pair_offsets, nl.pair_j[perm].contiguous(), nl.pair_shift[perm].contiguous(),
                    nl.pair_vec[perm].contiguous(), None, n_pairs)
    c2 = calc.spherical_expansion(nl2, spc, dt).double().reshape(copies, -1)
    assert calc.device_status() == 0
    assert float(((c2 - c).norm(dim=1) / c[0].norm()).max()) <= same
