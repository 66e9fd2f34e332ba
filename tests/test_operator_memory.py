"""What an operator's build and release do with devices and memory, on the host
against a stand-in for the HIP runtime."""
import os

import pytest

import fake_hip

pytestmark = pytest.mark.skipif(not os.path.exists(fake_hip.LIB),
                                reason="libpcms_mls.so not built (run __graft_entry__.build())")

BUILD = """
def build(n=1000):
    op, rad = P(), Radius(1, 8, 0, 0, 0.0)
    code = L.pcms_operator_build(PTR, i64(n), 3, PTR, i64(n), 1, C.byref(rad), 16, None, None, None,
                                 PTR, C.byref(op))
    return op, code
"""


@pytest.fixture(scope="module")
def fake(tmp_path_factory):
    return fake_hip.build(tmp_path_factory.mktemp("fake_hip"))


def test_release_waits_for_the_operators_own_device(fake):
    """An apply may be running on the operator's device when another one is
    current: the block goes back only after that device is idle."""
    fake_hip.run(fake, BUILD, """
    fake.hipSetDevice(3)
    op, code = build()
    assert code == 0 and op.value, L.pcms_last_error()
    fake.hipSetDevice(1)
    fake.fake_clear()
    assert L.pcms_operator_free(op) == 0
    names = [c.split(" ")[0] for c in log()]
    assert names.index("hipDeviceSynchronize@3") < names.index("hipFreeAsync@3"), names
    assert names[-1] == "hipSetDevice@1", names
    """)


@pytest.mark.parametrize("call", ["hipDeviceSynchronize", "hipFreeAsync"])
def test_a_failed_release_is_reported_and_can_be_repeated(fake, call):
    fake_hip.run(fake, BUILD, f"""
    op, code = build()
    assert code == 0
    fake.fake_clear()
    fail("{call}", HIP_ERROR_CAPTURE, 1)
    assert L.pcms_operator_free(op) == 2, "PCMS_ERR_HIP"
    if "{call}" == "hipDeviceSynchronize":
        assert not any("hipFreeAsync" in c for c in log()), log()
    fake.fake_clear()
    assert L.pcms_operator_free(op) == 0
    assert sum("hipFreeAsync" in c for c in log()) == 1, log()
    """)


CALLS = {
    "operator": ("hipMallocFromPoolAsync", "build()[1]"),
    "grid": ("hipMalloc", """L.pcms_grid_build(PTR, i64(500), 2, None, C.c_double(0), C.c_double(0),
                                               None, C.byref(P()))"""),
    "transfer": ("hipMallocAsync", """L.pcms_mls_transfer(
        PTR, i64(500), 2, PTR, 1, PTR, i64(400), 1, C.byref(Radius(1, 8, 0, 0, 0.0)), 16, None, None,
        None, PTR, PTR)"""),
}


@pytest.mark.parametrize("call", list(CALLS))
def test_a_call_without_memory_takes_back_what_the_pool_holds(fake, call):
    """Memory kept for the next operator is given back to the device where an
    allocation of the library would fail without it."""
    name, code = CALLS[call]
    fake_hip.run(fake, BUILD, f"""
    op, code = build()
    assert code == 0 and L.pcms_operator_free(op) == 0
    fake.fake_clear()
    fail("{name}", HIP_ERROR_MEMORY, 1)
    assert {code} == 0, L.pcms_last_error()
    calls = log()
    asked = [i for i, c in enumerate(calls) if c.startswith("{name}@")]
    assert "hipMemPoolTrimTo@0 0" in calls[asked[0]:asked[1]], calls
    fake.fake_clear()
    fail("{name}", HIP_ERROR_MEMORY)
    assert {code} == 3, "PCMS_ERR_NOMEM"
    """)


def test_a_call_without_memory_and_without_a_pool_asks_once(fake):
    fake_hip.run(fake, BUILD, f"""
    fail("hipMalloc", HIP_ERROR_MEMORY)
    assert {CALLS["grid"][1]} == 3
    assert sum(c.startswith("hipMalloc@") for c in log()) == 1, log()
    """)
