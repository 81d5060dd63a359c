"""Argument blocks of every form of a kernel whose operands the 32-bit fields could not hold as they are: chain.hip compiled into a small driver (no GPU)."""
import os
import subprocess

from paper_2503_19779_amd.build import FLAGS, LIB, build_library

HERE = os.path.dirname(os.path.abspath(__file__))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


def test_periods_longer_than_the_tensor(tmp_path):
    build_library(force=False)
    exe = str(tmp_path / "long_periods")
    flags = [f for f in FLAGS if f not in ("-shared", "-fPIC", "-O3")] + ["-O1"]
    res = subprocess.run([HIPCC] + flags + ["-x", "hip", os.path.join(HERE, "long_periods_driver.cpp"), "-x", "none", LIB, "-Wl,-rpath," + os.path.dirname(LIB), "-o", exe],
                         capture_output=True, text=True)
    assert res.returncode == 0, res.stdout + res.stderr
    res = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert res.returncode == 0 and "long periods: ok" in res.stdout, res.stdout + res.stderr
