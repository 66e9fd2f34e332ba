"""The radix sort's forms by the number of keys, on the CPU emulation (which
aborts on a block slot taken twice, a slot out of range or an unstable order):
one block, blocks that sum the others' counts themselves, scanned counts."""
import re

import numpy as np
import pytest

import emu_driver
import parity_cases as C
from paper_2510_18838_amd import synth


@pytest.mark.parametrize("n,form", [(1, "one block"), (63, "one block"), (64, "one block"),
                                    (4095, "one block"), (4096, "one block"), (4097, "direct"),
                                    (131072, "direct"), (131073, "scanned"), (140001, "scanned")])
@pytest.mark.parametrize("lbvh", [False, True], ids=["grid", "tree"])
def test_forms(n, form, lbvh):
    rng = np.random.default_rng(n)
    src = rng.uniform(0.0, 1.0, (n, 2))
    src[: n // 3] = np.round(src[: n // 3], 1)   # equal keys, to be kept in order
    p = C.custom(src, rng.uniform(0.0, 1.0, (1, n)), rng.uniform(0.0, 1.0, (3, 2)), 0, synth.KNN,
                 k=1, k_cap=4)
    emu_driver.run(p, 0, lbvh=lbvh)
    forms = re.findall(r"sort: (\d+) keys, (.*)", emu_driver.run.last_stderr)
    assert forms == [(str(n), form), ("3", "one block")]
