"""Single host+device functions of the kernels, compiled for the host."""
import os
import subprocess

import emu_driver


def test_units(tmp_path):
    exe = str(tmp_path / "unit")
    subprocess.check_call(["g++", "-std=c++20", "-O1", "-g", "-fsanitize=address,undefined",
                           "-fno-sanitize-recover=undefined", "-DPCMS_HOST_EMULATION",
                           "-I", os.path.join(emu_driver.ROOT, "include"),
                           "-I", os.path.join(emu_driver.ROOT, "paper_2510_18838_amd", "csrc"),
                           "-I", emu_driver.EMU_DIR, os.path.join(emu_driver.EMU_DIR, "unit.cpp"),
                           "-o", exe])
    res = subprocess.run([exe], capture_output=True, text=True,
                         env=dict(os.environ, ASAN_OPTIONS="detect_leaks=0"))
    assert res.returncode == 0 and res.stdout.endswith("ok\n"), res.stdout + res.stderr[-2000:]
