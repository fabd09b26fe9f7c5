"""The LDS of the modified-equilibrium noise kernels fits a compute unit at
every extent, precision and batch that the model accepts (no GPU needed)."""

import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PKG = os.path.join(ROOT, "paper_1012_3632_amd")


def test_noise_lds_fits_every_extent(tmp_path):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("hipcc not found")
    exe = str(tmp_path / "noise_shape")
    r = subprocess.run([hipcc, "--offload-arch=gfx950", "--offload-host-only", "-O2", "-std=c++17",
                        os.path.join(ROOT, "tests", "noise_shape_check.cpp"), "-o", exe,
                        "-L" + PKG, "-l:libflb.so", "-Wl,-rpath," + PKG],
                       capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr[-3000:]
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and r.stdout.endswith(" 0 do not fit\n"), r.stdout + r.stderr
