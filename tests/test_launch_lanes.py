"""Lanes per target of the launches, on the host against a stand-in for the HIP
runtime: the rule's lines, and the limit of a launch's threads."""
import os

import pytest

import fake_hip

pytestmark = pytest.mark.skipif(not os.path.exists(fake_hip.LIB),
                                reason="libpcms_mls.so not built (run __graft_entry__.build())")

CALL = """
class Opts(C.Structure):
    _fields_ = [("weight", i32), ("precision", i32), ("lam", C.c_double), ("flags", C.c_uint32),
                ("block", i32), ("summary", P)]

def threads(dim, degree, precision, n_tgt, mode=1, k=40, k_cap=64):
    # of every launch; the search is the last one up to 49,152 targets, whose
    # outputs it writes itself, and the last but one above
    g, rad, o = P(), Radius(mode, k, 8, 40, 0.1), Opts()
    o.precision = precision
    assert L.pcms_grid_build(PTR, i64(100000), dim, None, C.c_double(0), C.c_double(0), None,
                             C.byref(g)) == 0
    fake.fake_clear()
    code = L.pcms_mls_transfer_grid(g, PTR, 1, PTR, i64(n_tgt), degree, C.byref(rad), k_cap,
                                    C.byref(o), None, PTR, PTR)
    assert code == 0, L.pcms_last_error()
    launches = [c.split(" ") for c in log() if c.startswith("hipLaunchKernel")]
    return [int(c[1]) * int(c[2]) for c in launches]
"""


@pytest.fixture(scope="module")
def fake(tmp_path_factory):
    return fake_hip.build(tmp_path_factory.mktemp("fake_hip"))


@pytest.mark.parametrize("dim,degree,precision,line", [
    (3, 2, 0, 49152), (3, 2, 2, 49152), (5, 1, 0, 49152), (5, 1, 2, 49152), (4, 2, 0, 4096),
    (5, 2, 0, 4096), (4, 2, 1, 32768), (5, 2, 1, 32768), (4, 2, 2, 32768), (5, 2, 2, 32768)])
def test_few_targets(fake, dim, degree, precision, line):
    fake_hip.run(fake, CALL, f"""
    four = threads({dim}, {degree}, {precision}, {line})[-1]
    assert 4 * {line} <= four < 4 * {line} + 64 * 512, four
    many = threads({dim}, {degree}, {precision}, {line} + 1)[-1 if {line} < 49152 else -2]
    assert {line} < many < {line} + 64 * 513, many
    """)


def test_threads_of_a_launch(fake):
    """2^30 targets of long lists: four lanes each would be 2^32 threads."""
    fake_hip.run(fake, CALL, """
    most = max(threads(5, 1, 0, (1 << 30) - 1, mode=2, k_cap=128))
    assert most < 1 << 32, most
    assert max(threads(5, 1, 0, 1 << 29, mode=2, k_cap=128)) >= 1 << 31   # four lanes
    """)
