"""What a kernel needs from the runtime once (more dynamic LDS than the default) is asked for on every device, not once in a
process: the class that keeps count, compiled alone, and that nothing goes past it."""
import glob
import os
import re
import subprocess

from paper_2207_04606_amd import build as sptir_build

HERE = os.path.dirname(os.path.abspath(__file__))


def test_once_per_device(tmp_path):
    exe = str(tmp_path / "per_device")
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-pthread", "-I", sptir_build.CSRC, "-o", exe,
                           os.path.join(HERE, "per_device_main.cpp")])
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert (r.returncode, r.stdout) == (0, "ok\n")


def test_large_lds_is_allowed_in_one_place():
    where = []
    for path in sorted(glob.glob(os.path.join(sptir_build.CSRC, "*"))):
        with open(path) as f:
            text = f.read()
        where += [os.path.basename(path)] * len(re.findall(r"\bhipFuncSetAttribute\b", text))
        assert "call_once" not in text, f"{path}: once in a process is not once per device"
    assert where == ["sptir_internal.h"]
