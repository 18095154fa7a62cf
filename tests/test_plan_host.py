"""Host code around the launches, checked on the CPU.

  * tests/plan_host.cpp: the RF image's segments and the root pass's grid stay within what one
    launch holds (fewer than 2^32 threads a dimension) for every size the entry points take;
  * tests/fetch_host.cpp: which way a server's results take into which kind of memory."""

import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")


def _run(tmp_path, name, *flags):
    """Build tests/<name>.cpp with the HIP headers and run it; its number of checks."""
    if not shutil.which("g++") or not os.path.exists(os.path.join(ROCM, "include", "hip", "hip_runtime.h")):
        pytest.skip("g++ or the HIP headers are not available")
    exe = str(tmp_path / name)
    subprocess.run(["g++", "-std=c++17", "-O1", "-g", "-Wall", *flags, "-fno-sanitize-recover=all",
                    "-D__HIP_PLATFORM_AMD__", "-I", os.path.join(ROOT, "include"), "-isystem",
                    os.path.join(ROCM, "include"), "-o", exe, os.path.join(HERE, name + ".cpp"), "-pthread"], check=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stderr
    assert r.stdout.startswith("ok "), r.stdout
    return int(r.stdout.split()[1])


def test_launch_sizes(tmp_path):
    assert _run(tmp_path, "plan_host", "-fsanitize=undefined") > 500


def test_fetch_routes(tmp_path):
    assert _run(tmp_path, "fetch_host", "-fsanitize=thread") > 50
