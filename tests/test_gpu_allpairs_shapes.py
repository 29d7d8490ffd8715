"""GPU: the all-pairs neighbour list over many small structures, against the
oracle's list (identical pairs, order and shifts): empty structures and
single atoms between others, wide cells where the nearest image is taken by
rounding (diagonal and triclinic), thin cells with several images, mixed
periodicity, centres of more than 64 and more than 128 pairs (the counts by
species in registers, the records in LDS and in global memory), the searches
of one and of several levels over the structures, and 65,536 centres, from
which on a wave counts four."""
import numpy as np
import pytest
import torch

import oracle
import paper_2101_08814_amd as P
from synthetic.structures import _hypers, _pack

from test_gpu_parity import assert_same_list, gpu_neighbors

pytestmark = pytest.mark.gpu

WIDE = np.array([[11.0, 0, 0], [1.5, 10.5, 0], [-1.0, 2.0, 12.0]])


def _grid(rng, n, step, origin=0.0):
    m = int(np.ceil(n ** (1 / 3)))
    g = np.stack(np.meshgrid(*[np.arange(m) * step] * 3, indexing="ij"), -1).reshape(-1, 3)
    return rng.permutation(g)[:n] + rng.uniform(-0.2, 0.2, (n, 3)) + origin


def _mixed(n_structs, seed, S):
    rng = np.random.default_rng(seed)
    kinds = [
        lambda: (np.zeros((0, 3)), np.eye(3) * 9.0, (1, 1, 1)),
        lambda: (rng.uniform(-3, 3, (1, 3)), np.eye(3) * 3.1, (1, 1, 1)),
        lambda: (_grid(rng, 27, 3.0, -4.0), np.diag([9.0, 10.0, 9.5]), (1, 1, 1)),
        lambda: (_grid(rng, 30, 2.5, 20.0), WIDE, (1, 1, 1)),
        lambda: (_grid(rng, 17, 1.6), WIDE * 0.5, (1, 0, 1)),
        lambda: (_grid(rng, 64 + 5, 1.2), np.zeros((3, 3)), (0, 0, 0)),
        lambda: (_grid(rng, 150, 1.05), np.zeros((3, 3)), (0, 0, 0)),
        lambda: (_grid(rng, 9, 1.4), np.diag([4.5, 4.4, 40.0]), (1, 1, 0)),
    ]
    out = []
    for k in range(n_structs):
        pos, cell, pbc = kinds[(k * 5 + 3) % len(kinds)]()
        out.append((pos, rng.integers(0, S, len(pos)), cell, np.array(pbc, dtype=np.uint8)))
    return out


@pytest.mark.parametrize("dt", [torch.float32, torch.float64])
@pytest.mark.parametrize("n_structs,S", [(1, 1), (24, 3), (66, 8), (300, 4), (4200, 2)])
def test_mixed_structures(n_structs, S, dt):
    b = _pack(_mixed(n_structs, 100 + n_structs, S), _hypers(S, 4.0, 0.5, 4, 2), "mixed")
    calc = P.Calculator.from_hypers(b.hypers)
    nl, _, _ = gpu_neighbors(calc, b, dt)
    assert_same_list(nl, oracle.neighbors(b), b, dt == torch.float64)


@pytest.mark.parametrize("extra", [0, 3])
def test_four_centres_per_wave(extra):
    """65,536 + extra centres in structures of 1 to 23 atoms: groups of four
    consecutive centres cross structures, the last one is partial."""
    rng = np.random.default_rng(5)
    left, structs = 65536 + extra, []
    while left:
        n = int(min(left, rng.integers(1, 24)))
        cell, pbc = [(np.zeros((3, 3)), (0, 0, 0)), (WIDE, (1, 1, 1)), (np.diag([8.5, 9.0, 8.2]), (1, 1, 1))][n % 3]
        structs.append((_grid(rng, n, 2.0, -1.0), rng.integers(0, 3, n), cell, np.array(pbc, dtype=np.uint8)))
        left -= n
    b = _pack(structs, _hypers(3, 4.0, 0.5, 4, 2), "small")
    calc = P.Calculator.from_hypers(b.hypers)
    nl, _, _ = gpu_neighbors(calc, b)
    assert_same_list(nl, oracle.neighbors(b), b, False)
