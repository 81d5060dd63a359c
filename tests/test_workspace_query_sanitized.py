"""Workspace size queries over unvalidated sizes, with chain.hip built under UndefinedBehaviorSanitizer on the host side (no GPU)."""
import os
import subprocess

from paper_2503_19779_amd.build import FLAGS, LIB, build_library

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


def test_size_queries_do_not_overflow(tmp_path):
    build_library(force=False)
    flags = [f for f in FLAGS if f not in ("-shared", "-fPIC", "-O3")] + ["-O1", "-g", "-Xarch_host", "-fsanitize=undefined", "-Xarch_host", "-fno-sanitize-recover=all"]
    objs = [str(tmp_path / "chain.o"), str(tmp_path / "driver.o")]
    exe = str(tmp_path / "workspace_query")
    for cmd in ([HIPCC] + flags + ["-c", "-o", objs[0], os.path.join(ROOT, "paper_2503_19779_amd", "csrc", "chain.hip")],
                [HIPCC] + flags + ["-c", "-x", "hip", "-o", objs[1], os.path.join(HERE, "workspace_query_driver.cpp")],
                [HIPCC, "--offload-arch=gfx950", "--hip-link", "-fsanitize=undefined", "-fno-gpu-sanitize", "-o", exe] + objs + [LIB, "-Wl,-rpath," + os.path.dirname(LIB)],
                [exe]):
        res = subprocess.run(cmd, capture_output=True, text=True, timeout=240)
        assert res.returncode == 0, " ".join(cmd) + "\n" + res.stdout + res.stderr
    assert "workspace queries: ok" in res.stdout
