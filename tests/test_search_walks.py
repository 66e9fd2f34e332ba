"""The walks that a search takes (CPU emulation): a radius within the estimate's
window costs two, and a wave waits for its longest target."""
import re

import numpy as np
import pytest

import emu_driver
import parity_cases as C
from paper_2510_18838_amd import synth


@pytest.fixture(scope="module", autouse=True)
def _built():
    emu_driver.build()


def walks(p, lbvh=False, op=0):
    """(mean over the targets, mean over the waves of their longest target's)"""
    emu_driver.run(p, op, lbvh=lbvh)
    err = emu_driver.run.last_stderr
    return (float(re.search(r"target mean ([\d.]+)", err).group(1)),
            float(re.search(r"wave max walks ([\d.]+)", err).group(1)))


@pytest.mark.parametrize("lbvh", [False, True], ids=["grid", "tree"])
@pytest.mark.parametrize("dim,k,k_cap", [(2, 20, 32), (3, 24, 32), (4, 30, 48), (5, 40, 64)])
def test_nearest_in_the_windows_first_bin(dim, k, k_cap, lbvh):
    """A k-th distance in the first of the window's 64 bins lies in the window.
    Were it taken for one below, its target would take the general path (five
    walks or more).  Two walks where the estimate holds and four where the k-th
    is beside the window (4 % of these targets at most) keep the waves' mean of
    their longest target below three."""
    p = synth.uniform_problem(5, 20000, 2000, dim, 1, synth.KNN, n_fields=1, k=k, k_cap=k_cap)
    mean, longest = walks(p, lbvh)
    assert mean <= 2.08 and longest < 3.0, (mean, longest)


@pytest.mark.parametrize("dim,mode,lbvh,bar", [
    (2, synth.FIXED, True, 5.2), (3, synth.FIXED, False, 5.0), (4, synth.FIXED, False, 4.5),
    (5, synth.FIXED, False, 4.5), (2, synth.GROW, True, 3.1), (3, synth.GROW, True, 3.1)])
def test_capped_targets(dim, mode, lbvh, bar):
    """About 70 sources in the ball and a cap of 32.  One walk counts them: the
    list, which is selected afresh, costs no second one where it met the row
    table.  With a growing radius two more select the cap's nearest.  With a
    fixed one, whose words are the cap's alone, the selection gives up after its
    first walk and the general path takes two to four."""
    n = 8000
    r = (70 / (n * synth.unit_ball_volume(dim))) ** (1.0 / dim)
    p = synth.uniform_problem(5, n, 400, dim, 1, mode, n_fields=1, radius=r, n_min=8, k_cap=32)
    mean, _ = walks(p, lbvh)
    assert mean <= bar, mean


def test_1d_selection_is_exact():
    """In 1-D the selection reads FP64 records: far from the cloud's corner (a
    stray source lies a million cloud widths away) FP32 images tell nothing
    apart, and every capped target would take the general path of six walks
    instead of three (a bin too full for the words costs a few of them more)."""
    rng = np.random.default_rng(11)
    src = np.concatenate([rng.uniform(0.0, 1e-3, (3000, 1)), [[-1000.0]]])
    p = C.custom(src, rng.uniform(0.0, 1.0, (1, 3001)), rng.uniform(2e-4, 8e-4, (200, 1)), 1,
                 synth.GROW, radius=1e-5, n_min=8, k_cap=24)
    mean, _ = walks(p)
    assert mean < 4.0, mean
