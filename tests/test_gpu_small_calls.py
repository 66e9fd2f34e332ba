"""Calls whose keys fit one block are sorted by one launch, and the bounding
box is reduced from the partial boxes of the point kernel's blocks: the lists
equal the oracle's exactly at the edges of both (4,096 keys per block, 256
points per partial box)."""
import pytest

import parity_cases as C
from gpu_helpers import gpu_neighbors, say
from paper_2510_18838_amd import synth

pytestmark = pytest.mark.gpu


class _Lists:
    def __init__(self, lbvh):
        self.lbvh = lbvh

    def neighbors(self, prob):
        return gpu_neighbors(prob, lbvh=self.lbvh)


@pytest.mark.parametrize("lbvh", [False, True])
@pytest.mark.parametrize("n_src", [1, 63, 255, 257, 4095, 4096, 4097, 70000])
@pytest.mark.parametrize("dim", [2, 3])
def test_lists_at_the_edges(dim, n_src, lbvh):
    r = min(1.0, (20.0 / (n_src * synth.unit_ball_volume(dim))) ** (1.0 / dim))
    n_tgt = {4095: 4097, 4097: 4095}.get(n_src, 300)
    p = synth.uniform_problem(17 + n_src, n_src, n_tgt, dim, 1, synth.FIXED, n_fields=1,
                              radius=r, k_cap=32)
    say(f"{dim}-D {n_src} sources {n_tgt} targets lbvh={lbvh}")
    C.check_lists(_Lists(lbvh), p, f"{dim}-D {n_src}")
