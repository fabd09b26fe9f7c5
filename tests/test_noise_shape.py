"""Host-side checks of the modified-equilibrium model (no GPU needed): the LDS
of its noise kernels fits a compute unit, and the limit of every launch, at the
extents, precisions and batches that the model accepts; a run makes no copy of
the populations that its steps can do without; the division that the line
transforms index by is exact."""

import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PKG = os.path.join(ROOT, "paper_1012_3632_amd")


def _run(tmp_path, name):
    """The output of tests/<name>.cpp, built for the host against the library."""
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("hipcc not found")
    exe = str(tmp_path / name)
    r = subprocess.run([hipcc, "--offload-arch=gfx950", "--offload-host-only", "-O2", "-std=c++17",
                        os.path.join(ROOT, "tests", name + ".cpp"), "-o", exe,
                        "-L" + PKG, "-l:libflb.so", "-Wl,-rpath," + PKG, "-rdynamic"],
                       capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr[-3000:]
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout + r.stderr
    return r.stdout


def test_noise_lds_fits_every_extent(tmp_path):
    assert _run(tmp_path, "noise_shape_check").endswith(" 0 do not fit\n")


def test_noise_launches_raise_their_lds_limit(tmp_path):
    assert _run(tmp_path, "noise_launch_check").endswith(" 0 over their limit\n")


def test_even_runs_make_no_copy(tmp_path):
    assert _run(tmp_path, "modeq_run_check").endswith(" 0 with a copy too many\n")


def test_reciprocal_division(tmp_path):
    assert _run(tmp_path, "fft_div_check").endswith(" 0 wrong\n")
