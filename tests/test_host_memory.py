"""Device memory kept between calls, on the host side: tests/host_memory.cpp runs the library against a HIP runtime of its
own, so that waits can fail, frees can take long and memory can run out without a GPU."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PKG = os.path.join(ROOT, "paper_2212_05009_amd")


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    if not os.path.exists(os.path.join(PKG, "libgcn.so")):
        import __graft_entry__
        __graft_entry__.build()
    out = str(tmp_path_factory.mktemp("host") / "host_memory")
    cmd = [os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), "-x", "hip", "--offload-host-only", "--offload-arch=gfx950", "-std=c++17", "-O1", "-I", os.path.join(PKG, "csrc"),
           os.path.join(ROOT, "tests", "host_memory.cpp"), "-o", out, "-L", PKG, "-lgcn", "-Wl,-rpath," + PKG, "-rdynamic", "-pthread"]
    res = subprocess.run(cmd, capture_output=True, text=True)
    assert res.returncode == 0, res.stdout + res.stderr
    return out


@pytest.mark.parametrize("check", ["plan", "lock", "exhausted", "workspace", "release", "host"])
def test_kept_memory(program, check):
    res = subprocess.run([program, check], capture_output=True, text=True, timeout=120)
    assert res.returncode == 0, res.stdout + res.stderr
