"""The ranges that end the requests of the streaming dense kernels, on the host: tests/rows_range.cpp over a grid of sizes."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_no_request_passes_the_end_of_a_matrix(tmp_path):
    out = str(tmp_path / "rows_range")
    cmd = [os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), "-x", "hip", "--offload-host-only", "--offload-arch=gfx950", "-std=c++17", "-O1",
           "-I", os.path.join(ROOT, "paper_2212_05009_amd", "csrc"), os.path.join(ROOT, "tests", "rows_range.cpp"), "-o", out]
    res = subprocess.run(cmd, capture_output=True, text=True)
    assert res.returncode == 0, res.stdout + res.stderr
    res = subprocess.run([out], capture_output=True, text=True, timeout=120)
    assert res.returncode == 0, res.stdout + res.stderr
