"""Runs a piece of code in a child process in which the library's HIP calls go
to the stand-in of fake_hip.cpp."""
import os
import subprocess
import sys
import textwrap

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(os.path.dirname(HERE))
LIB = os.path.join(ROOT, "paper_2510_18838_amd", "libpcms_mls.so")

PRELUDE = """
import ctypes as C, sys
fake = C.CDLL(sys.argv[1], mode=C.RTLD_GLOBAL)   # before the library, which binds to it
L = C.CDLL(sys.argv[2])
fake.fake_log.restype = C.c_char_p
L.pcms_last_error.restype = C.c_char_p
P, i64, i32 = C.c_void_p, C.c_int64, C.c_int32

class Radius(C.Structure):
    _fields_ = [("mode", i32), ("k", i32), ("n_min", i32), ("max_iter", i32), ("r", C.c_double)]

def log():
    return fake.fake_log().decode().split("\\n")[:-1]

def fail(name, error, calls=1 << 30):
    fake.fake_fail(name.encode(), error, calls)

HIP_ERROR_MEMORY, HIP_ERROR_CAPTURE = 2, 900
PTR = P(0x1000)   # device memory, as far as the host code can tell
"""


def build(directory) -> str:
    out = os.path.join(str(directory), "libfake_hip.so")
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-o", out,
                           os.path.join(HERE, "fake_hip.cpp")])
    return out


def run(fake: str, *code: str):
    text = PRELUDE + "".join(textwrap.dedent(c) for c in code)
    res = subprocess.run([sys.executable, "-c", text, fake, LIB],
                         capture_output=True, text=True, timeout=120)
    assert res.returncode == 0, res.stdout[-3000:] + res.stderr[-3000:]
    return res.stdout
