"""The host side of the trigger scans on the CPU: libst.so under a program that takes the HIP runtime's place (tests/host/
scan_driver.cpp), so that what a launch is given and what a failing allocation leads to can be seen without a GPU."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PKG = os.path.join(ROOT, "paper_2504_12329_amd")


@pytest.mark.skipif(shutil.which("hipcc") is None, reason="hipcc not on PATH")
def test_scans_against_a_runtime_of_our_own(tmp_path):
    """Scans of up to one tile of positions are launched without LDS for bitmaps; the static variant where pinned memory cannot be
    allocated, or has no address on the device."""
    if not os.path.exists(os.path.join(PKG, "libst.so")):
        from paper_2504_12329_amd import build
        build.build()
    exe = str(tmp_path / "scan_driver")
    subprocess.run(["hipcc", "--offload-arch=gfx950", "-O1", "-std=c++17", "-Xclang", "-target-feature", "-Xclang",
                    "-packed-fp32-ops", os.path.join(ROOT, "tests", "host", "scan_driver.cpp"), "-o", exe, "-L" + PKG, "-lst",
                    "-Wl,-rpath," + PKG, "-rdynamic"], check=True, capture_output=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and "ok" in r.stdout, r.stdout + r.stderr
