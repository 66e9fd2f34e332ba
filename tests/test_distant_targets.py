"""Targets at a distance of very many bucket widths: sources within a box of
1e-12 to 1e-17 and targets 1 to 1000 away, where a ball that reaches the
sources has a squared radius above 1e30 bucket widths.  Lists of the CPU
emulation against the oracle's brute force, bit for bit."""
import numpy as np
import pytest

import parity_cases as C
from paper_2510_18838_amd import synth
from test_emulation import EmuBackend

BACKENDS = {"one": EmuBackend(1), "four": EmuBackend(4), "tree": EmuBackend(1, lbvh=True)}


def problem(dim, box, far, mode):
    rng = np.random.default_rng([dim, int(-np.log10(box)), int(far), mode])
    n = 40
    # (a box of 1e-15 around 0.1 holds a few distinct coordinates)
    src = (0.1 if box < 1e-13 else 0.0) + box * rng.uniform(0.0, 1.0, (n, dim))
    tgt = far * rng.uniform(0.5, 1.0, (24, dim)) * np.sign(rng.uniform(-1.0, 1.0, (24, dim)))
    kw = {synth.KNN: dict(k=12), synth.FIXED: dict(radius=1.5 * far * dim ** 0.5),
          synth.GROW: dict(radius=0.2 * far, n_min=12)}[mode]
    return C.custom(src, rng.uniform(0.0, 1.0, (1, n)), tgt, 0, mode, k_cap=20, **kw)


@pytest.mark.parametrize("backend", list(BACKENDS))
@pytest.mark.parametrize("mode", [synth.KNN, synth.FIXED, synth.GROW])
@pytest.mark.parametrize("dim,box,far", [(1, 1e-12, 1000.0), (2, 1e-12, 1000.0), (2, 1e-17, 1.0),
                                         (3, 2e-12, 1000.0), (3, 1e-15, 1.0), (4, 1e-14, 30.0),
                                         (5, 1e-15, 1.0), (5, 3e-13, 500.0)])
def test_lists(dim, box, far, mode, backend):
    C.check_lists(BACKENDS[backend], problem(dim, box, far, mode),
                  f"{dim}-D box {box} far {far} mode {mode} ({backend})", brute=True)
