"""The lists of test_search_range.py and test_distant_targets.py on the GPU, whose
FP32 arithmetic (subnormals among it) the bounds rest on: one lane per target (the
targets repeated beyond 49,152), four, and the tree."""
import numpy as np
import pytest

import parity_cases as C
import test_distant_targets as distant
import test_search_range as ends
from gpu_helpers import gpu_neighbors, say
from paper_2510_18838_amd import synth

pytestmark = pytest.mark.gpu


class _Gpu:
    def __init__(self, copies=1, lbvh=False):
        self.copies, self.lbvh = copies, lbvh

    def neighbors(self, prob):
        n = len(prob.tgt)
        r = gpu_neighbors(prob, tgt=np.tile(prob.tgt, (self.copies, 1)), lbvh=self.lbvh)
        for key in ("n_kept", "n_found", "r2", "status"):
            assert np.array_equal(r[key], np.tile(r[key][:n], self.copies)), key
        return {k: v[:n] for k, v in r.items()}


BACKENDS = {"one": _Gpu(copies=2100), "four": _Gpu(), "tree": _Gpu(lbvh=True)}
MODES = [synth.FIXED, synth.KNN, synth.GROW]


@pytest.mark.parametrize("backend", list(BACKENDS))
@pytest.mark.parametrize("dim", [2, 3, 5])
@pytest.mark.parametrize("kind", list(ends.SCALES))
def test_ends_of_the_range(kind, dim, backend):
    for mode in MODES:
        where = f"{kind} {dim}-D mode {mode} ({backend})"
        say(where)
        C.check_lists(BACKENDS[backend], ends.problem(kind, dim, mode), where, brute=True)


@pytest.mark.parametrize("backend", list(BACKENDS))
@pytest.mark.parametrize("dim,box,far", [(1, 1e-12, 1000.0), (2, 1e-17, 1.0), (3, 2e-12, 1000.0),
                                         (5, 1e-15, 1.0)])
def test_distant(dim, box, far, backend):
    for mode in MODES:
        where = f"{dim}-D box {box} far {far} mode {mode} ({backend})"
        say(where)
        C.check_lists(BACKENDS[backend], distant.problem(dim, box, far, mode), where, brute=True)
