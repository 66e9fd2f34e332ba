"""One lane per target and four give the same bits where a list meets the row
table beside it: tight caps, in the dimensions of many rows, over several
clouds (CPU emulation)."""
import numpy as np
import pytest

import emu_driver
from paper_2510_18838_amd import synth
from test_emulation import EmuBackend

MIXED_REFINE = 2


@pytest.fixture(scope="module", autouse=True)
def _built():
    emu_driver.build()


@pytest.mark.parametrize("dim,mode,k,n_min,k_cap,scale,seeds", [
    (3, synth.GROW, 0, 12, 16, 0.5, range(300, 303)), (3, synth.GROW, 0, 20, 24, 0.5, range(300, 306)),
    (3, synth.KNN, 12, 0, 64, 1.0, range(306, 309)), (3, synth.KNN, 60, 0, 62, 1.0, range(300, 302)),
    (4, synth.GROW, 0, 30, 36, 0.5, range(300, 303)), (4, synth.KNN, 34, 0, 46, 1.0, range(300, 302)),
    (5, synth.GROW, 0, 20, 24, 0.7, range(300, 303)), (5, synth.KNN, 60, 0, 60, 1.0, range(300, 302))])
def test_same_bits(dim, mode, k, n_min, k_cap, scale, seeds):
    r = scale * ((n_min or 1) / (2500 * synth.unit_ball_volume(dim))) ** (1.0 / dim)
    for seed in seeds:
        p = synth.uniform_problem(seed, 2500, 400, dim, 1, mode, n_fields=1, radius=r, k=k or 1,
                                  n_min=n_min or 1, k_cap=k_cap)
        a, b = (EmuBackend(g).transfer(p, MIXED_REFINE) for g in (1, 4))
        assert (a["status"] == b["status"]).all(), seed
        bad = np.nonzero(~((a["out"] == b["out"]) | np.isnan(a["out"])).all(axis=0))[0]
        assert bad.size == 0, (seed, bad, np.abs(a["out"] - b["out"])[:, bad])
