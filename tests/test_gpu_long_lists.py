"""Long lists leave a CU few waves of one lane per target, so larger calls take
four lanes for them too: the same targets repeated beyond 49,152 meet the
oracle's bars, on each side of the rule's lines (k_cap 80 | 96 in 5-D, 96 | 128
in 3-D, 32 | 64 for lists alone)."""
import numpy as np
import pytest

import parity_cases as C
from gpu_helpers import gpu_neighbors, gpu_transfer, say
from paper_2510_18838_amd import pcms, synth

pytestmark = pytest.mark.gpu

MANY = 49152 + 300


class _Repeated:
    """The targets over and over; every copy gives the first one's bits."""

    @staticmethod
    def _targets(prob):
        return np.resize(prob.tgt, (MANY, prob.dim))

    def neighbors(self, prob):
        n = len(prob.tgt)
        r = gpu_neighbors(prob, tgt=self._targets(prob))
        for key in ("n_kept", "n_found", "r2", "status"):
            assert np.array_equal(r[key], np.resize(r[key][:n], MANY)), key
        return {k: v[:n] for k, v in r.items()}

    def transfer(self, prob, precision, weight=0, lam=0.0, block=0):
        n = len(prob.tgt)
        out, st, _ = gpu_transfer(prob, precision, tgt=self._targets(prob), weight=weight,
                                  lam=lam, block=block)
        first = np.arange(MANY) % n
        assert np.array_equal(st, st[:n][first])
        assert np.array_equal(out, out[:, :n][:, first], equal_nan=True)
        return dict(out=out[:, :n], status=st[:n])


@pytest.mark.parametrize("dim,degree,k_cap", [(5, 1, 96), (5, 0, 96), (5, 1, 80), (5, 2, 96),
                                              (4, 1, 128), (3, 1, 128), (3, 1, 96), (2, 1, 64),
                                              (3, 1, 32)])
def test_long_lists(dim, degree, k_cap):
    n = 6000
    kbar = 0.75 * k_cap
    p = synth.uniform_problem(7 + k_cap, n, 400, dim, degree, synth.GROW, n_fields=3,
                              radius=(kbar / (n * synth.unit_ball_volume(dim))) ** (1.0 / dim),
                              n_min=k_cap // 2, k_cap=k_cap)
    where = f"{dim}-D degree {degree} k_cap {k_cap}"
    say(where)
    C.check_lists(_Repeated(), p, where)
    C.check_transfer(_Repeated(), p, where, precisions=(pcms.FP64, pcms.MIXED_REFINE))


@pytest.mark.parametrize("k", [56, 85, 100])
def test_long_nearest_lists(k):
    p = synth.uniform_problem(k, 6000, 400, 3, 1, synth.KNN, n_fields=1, k=k, k_cap=128)
    C.check_lists(_Repeated(), p, f"3-D k {k}")
