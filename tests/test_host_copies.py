"""Copies between a caller's memory and the device through pinned slots, on the
CPU (tests/host/host_copies.cpp, which stands in for the runtime calls; no GPU
call is made), also under the sanitizers."""

import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def on_host(*names):
    """Compiler flags of these sanitizers, for the host part only."""
    return [x for n in names for x in ("-Xarch_host", "-fsanitize=" + n)]


@pytest.mark.parametrize("flags", [[], on_host("address", "undefined"), on_host("thread")],
                         ids=["plain", "address-undefined", "thread"])
def test_host_copies(tmp_path, flags):
    hipcc = next((c for c in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", shutil.which("hipcc"))
                  if c and os.path.exists(c)), None)
    if hipcc is None:
        pytest.skip("hipcc not found")
    exe = str(tmp_path / "host_copies")
    b = subprocess.run([hipcc, "-O1", "-g", "-std=c++17", "--offload-arch=gfx950",
                        "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops", *flags,
                        "-I" + os.path.join(ROOT, "include"), "-I" + os.path.join(ROOT, "paper_2401_02756_amd", "csrc"),
                        "-o", exe, os.path.join(ROOT, "tests", "host", "host_copies.cpp"), "-pthread"],
                       capture_output=True, text=True, timeout=300)
    assert b.returncode == 0, b.stderr[-2000:]
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    out = r.stdout + r.stderr
    assert r.returncode == 0 and r.stdout.strip().endswith("ok"), out[-3000:]
    for marker in ("AddressSanitizer", "runtime error:", "ThreadSanitizer", "LeakSanitizer"):
        assert marker not in out, out[-3000:]
