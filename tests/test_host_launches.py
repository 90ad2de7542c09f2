"""CPU: what the library launches, seen from a fake HIP runtime.

The drivers in tests/hostsim export the runtime's functions (fake_hip.hpp) and load the built
libpsatd.so: its host code runs as it is, device memory is host memory, and every launch is
handed to the driver with the kernel's name and parameters instead of being run.  So a choice of kernels,
radices or tables is checked over whole ranges of sizes without a GPU.
"""

import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
PKG = os.path.join(ROOT, "paper_1812_07357_amd")
HIPCC = os.environ.get("HIPCC", shutil.which("hipcc") or "/opt/rocm/bin/hipcc")


def _build(tmp_path, name):
    if not os.path.exists(HIPCC):
        pytest.skip("needs hipcc")
    lib = os.environ.get("PSATD_HOSTSIM_LIB", PKG)
    exe = str(tmp_path / name)
    cmd = [HIPCC, "-std=c++17", "-O1", "--offload-arch=gfx950", "--offload-host-only", f"-I{ROOT}/include",
           f"-I{PKG}/csrc", "-x", "hip", os.path.join(HERE, "hostsim", name + ".cpp"), "-o", exe, "-rdynamic",
           f"-L{lib}", "-lpsatd", f"-Wl,-rpath,{lib}"]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-4000:]
    return exe


def _run(exe, *args):
    r = subprocess.run([exe, *args], capture_output=True, text=True, timeout=600)
    assert r.returncode == 0, r.stdout[-3000:] + r.stderr[-2000:]
    return r.stdout


def test_every_pml_z_pass_has_its_tables(tmp_path):
    """Twelve z lines per column may not fit the LDS where the step's eleven do (FP64)."""
    _run(_build(tmp_path, "pml_z_tables"))


def test_plans_and_batches_share_a_tune_cache(tmp_path):
    """Pair radices of a plan (25 * 24 for 600 points) never reach the Stockham kernels that a batch runs."""
    _run(_build(tmp_path, "tune_cache"))
