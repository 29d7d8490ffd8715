"""GPU: the all-pairs neighbour list with more species than a fill wave counts
by (nine, and the largest number), where it ranks its pairs also when no
neighbour has several images: identical pairs, order and shifts as the
oracle's list."""
import pytest
import torch

import oracle
import paper_2101_08814_amd as P
from synthetic.structures import _hypers, _pack

from test_gpu_allpairs_shapes import _mixed
from test_gpu_parity import assert_same_list, gpu_neighbors

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_structs,S", [(24, 9), (66, 9), (300, 64)])
def test_many_species(n_structs, S):
    b = _pack(_mixed(n_structs, 200 + n_structs, S), _hypers(S, 4.0, 0.5, 2, 1), "mixed")
    calc = P.Calculator.from_hypers(b.hypers)
    nl, _, _ = gpu_neighbors(calc, b, torch.float64)
    assert_same_list(nl, oracle.neighbors(b), b, True)
