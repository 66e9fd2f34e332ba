"""The row tables and windowed selections of the search, at the sizes where
they can go wrong, on the CPU emulation (one lane per target and four) against
the oracle's lists, bit for bit: clouds that are flat or offset (bucket widths
above and below 1), rows of more sources than a table word holds, tables that
need filling more than once, more tied distances than are ranked in registers,
caps that bind in every dimension."""
import numpy as np
import pytest

import emu_driver
import parity_cases as C
from paper_2510_18838_amd import synth
from test_emulation import EmuBackend


@pytest.fixture(scope="module", autouse=True)
def _built():
    emu_driver.build()


BACKENDS = {"one": EmuBackend(1), "four": EmuBackend(4), "tree": EmuBackend(1, lbvh=True)}


def _problem(kind):
    rng = np.random.default_rng(sum(map(ord, kind)))
    u = lambda *s: rng.uniform(0.0, 1.0, s)   # noqa: E731
    if kind == "flat":           # wide buckets, targets off the plane of the sources
        src = u(3000, 3) * [900.0, 700.0, 0.0] + [0.0, 0.0, 5.0]
        tgt = u(300, 3) * [900.0, 700.0, 24.0] - [0.0, 0.0, 7.0]
        return C.custom(src, u(1, 3000), tgt, 1, synth.GROW, radius=20.0, n_min=8, k_cap=24)
    if kind == "outside":        # targets far from the box on every side
        return C.custom(u(2000, 3), u(1, 2000), u(200, 3) * 9.0 - 4.0, 1, synth.KNN, k=20, k_cap=40)
    if kind == "long rows":      # a dense clump: rows beyond 4095 sources
        src = np.concatenate([u(9000, 3) * [2e-3, 2e-4, 2e-4] + 0.5, u(500, 3)])
        tgt = np.concatenate([u(15, 3) * 2e-3 + 0.5, u(15, 3)])
        return C.custom(src, u(1, 9500), tgt, 1, synth.KNN, k=12, k_cap=32)
    if kind == "many rows":      # a growing radius of many small buckets
        return C.custom(u(4000, 3), u(1, 4000), u(60, 3), 1, synth.GROW, radius=0.02, n_min=60,
                        k_cap=20)
    if kind == "lattice ties":   # every distance shared by up to 48 sources
        g = np.stack(np.meshgrid(*[np.arange(9.0)] * 3, indexing="ij"), -1).reshape(-1, 3)
        return C.custom(g, u(1, len(g)), rng.integers(1, 8, (60, 3)) * 1.0, 1, synth.KNN, k=34,
                        k_cap=60)
    if kind == "lattice cap":
        g = np.stack(np.meshgrid(*[np.arange(9.0)] * 3, indexing="ij"), -1).reshape(-1, 3)
        return C.custom(g, u(1, len(g)), rng.integers(1, 8, (60, 3)) * 1.0, 1, synth.GROW,
                        radius=2.5, n_min=8, k_cap=30)
    d = int(kind[-1])            # "capped 1" .. "capped 5": most targets above the cap
    r = (30.0 / (3000 * synth.unit_ball_volume(d))) ** (1.0 / d) * (1.6 if d > 3 else 1.0)
    return C.custom(u(3000, d), u(1, 3000), u(150, d), 1, synth.GROW, radius=r, n_min=8, k_cap=16)


@pytest.mark.parametrize("backend", list(BACKENDS))
@pytest.mark.parametrize("kind", ["flat", "outside", "long rows", "many rows", "lattice ties",
                                  "lattice cap", "capped 1", "capped 2", "capped 3", "capped 4",
                                  "capped 5"])
def test_lists(kind, backend):
    ref = C.check_lists(BACKENDS[backend], _problem(kind), f"{kind} ({backend})")
    if kind.startswith("capped"):
        assert ((ref["status"] & C.CAPPED) != 0).mean() > 0.3


@pytest.mark.parametrize("precision", [C.FP64, C.MIXED_REFINE])
def test_four_lanes_give_the_same_bits(precision):
    """Four lanes per target sum every neighbour in list order, as one does."""
    for dim, degree, nf in ((2, 2, 1), (3, 1, 9), (3, 2, 3), (5, 1, 6)):
        p = synth.uniform_problem(71, 3000, 300, dim, degree, synth.KNN, n_fields=nf, k=30, k_cap=48)
        a = BACKENDS["one"].transfer(p, precision)
        b = BACKENDS["four"].transfer(p, precision)
        assert (a["status"] == b["status"]).all()
        assert np.array_equal(a["out"], b["out"], equal_nan=True), (dim, degree, nf)
