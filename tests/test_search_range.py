"""Clouds and metrics at the ends of the FP32 range, which the searches' FP32
images must not misjudge: differences of coordinates that overflow, coordinates
that are subnormal, metric factors that are subnormal or overflow.  Lists of the
CPU emulation against the oracle's, bit for bit."""
import numpy as np
import pytest

import parity_cases as C
from paper_2510_18838_amd import synth
from test_emulation import EmuBackend

BACKENDS = {"one": EmuBackend(1), "four": EmuBackend(4), "tree": EmuBackend(1, lbvh=True)}

# coordinates' scale, their offset, metric factor
SCALES = {"overflowing differences": (6e38, -3e38, 1e-38), "large and unit": (1e18, -5e17, 1.0),
          "subnormal factor": (1e37, 0.0, 1e-41), "overflowing factor": (1e-39, 0.0, 1e39),
          "subnormal coordinates": (2e-42, -1e-42, 1e37), "beyond the range": (1e60, 0.0, 1e-60)}


def problem(kind, dim, mode):
    scale, offset, g = SCALES[kind]
    rng = np.random.default_rng([dim, mode, len(kind)])
    n = 1500
    src = offset + scale * rng.uniform(0.0, 1.0, (n, dim))
    tgt = offset + scale * rng.uniform(-0.1, 1.1, (150, dim))
    tgt[:20] = src[:20]
    r = scale * g * (20 / (n * synth.unit_ball_volume(dim))) ** (1.0 / dim)
    return C.custom(src, rng.uniform(0.0, 1.0, (1, n)), tgt, 0, mode, k=16, radius=r, n_min=8,
                    k_cap=24, inv_scale=[g] * dim)


@pytest.mark.parametrize("backend", list(BACKENDS))
@pytest.mark.parametrize("mode", [synth.FIXED, synth.KNN, synth.GROW])
@pytest.mark.parametrize("dim", [2, 3, 5])
@pytest.mark.parametrize("kind", list(SCALES))
def test_lists(kind, dim, mode, backend):
    C.check_lists(BACKENDS[backend], problem(kind, dim, mode),
                  f"{kind} {dim}-D mode {mode} ({backend})", brute=True)
