"""The longest lists, whose targets take the most LDS words: one lane per target
(more than 49,152 targets) and four, against the oracle."""
import pytest

import parity_cases as C
from gpu_helpers import gpu_neighbors, gpu_transfer, say
from paper_2510_18838_amd import pcms, synth
from test_gpu_long_lists import _Repeated

pytestmark = pytest.mark.gpu


class _Few:
    neighbors = staticmethod(gpu_neighbors)

    @staticmethod
    def transfer(prob, precision, weight=0, lam=0.0, block=0):
        out, st, _ = gpu_transfer(prob, precision, weight=weight, lam=lam, block=block)
        return dict(out=out, status=st)


@pytest.mark.parametrize("backend", [_Repeated(), _Few()], ids=["one", "four"])
@pytest.mark.parametrize("dim,k,k_cap", [(5, 247, 256), (5, 232, 256), (4, 233, 256), (3, 247, 256),
                                         (3, 256, 256)])
def test_longest(dim, k, k_cap, backend):
    p = synth.uniform_problem(dim + k, 6000, 300, dim, 1, synth.KNN, n_fields=1, k=k, k_cap=k_cap)
    where = f"{dim}-D k {k} k_cap {k_cap}"
    say(where)
    C.check_lists(backend, p, where)
    C.check_transfer(backend, p, where, precisions=(pcms.FP64, pcms.MIXED_REFINE))
