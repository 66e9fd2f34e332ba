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
