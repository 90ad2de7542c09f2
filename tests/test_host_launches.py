"""CPU: what the library launches, seen from a fake HIP runtime.

The drivers in tests/hostsim export the runtime's functions (fake_hip.hpp) and load the built
libpsatd.so: its host code runs as it is, device memory is host memory, and every launch is
handed to the driver with the kernel's name and parameters instead of being run.  So a choice of kernels,
radices or tables is checked over whole ranges of sizes without a GPU.
"""

import os
import re
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


_ROW_KERNELS = """
#include "row_run.hpp"
#define KERNEL(K, T, NAME) \\
  extern "C" __global__ void NAME(const T* p, T* out) { \\
    const auto r = psatd::load_run<K>(p + threadIdx.x); \\
    for (int c = 0; c <= K; ++c) out[(K + 1) * threadIdx.x + c] = r.v[c]; \\
  }
KERNEL(1, float, k1_float) KERNEL(2, float, k2_float) KERNEL(3, float, k3_float)
KERNEL(1, double, k1_double) KERNEL(2, double, k2_double) KERNEL(3, double, k3_double)
"""


def test_a_row_of_the_gather_is_read_and_no_value_more(tmp_path):
    """The words that the loads of a particle's row cover, from the assembly: K + 1 values, not a whole
    power of two of them (the fourth value after the last row of an array may not be mapped)."""
    if not os.path.exists(HIPCC):
        pytest.skip("needs hipcc")
    src, out = tmp_path / "rows.hip", tmp_path / "rows.s"
    src.write_text(_ROW_KERNELS)
    cmd = [HIPCC, "-std=c++17", "-O3", "--offload-arch=gfx950", "--offload-device-only", "-S", f"-I{PKG}/csrc", str(src),
           "-o", str(out)]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-4000:]
    text = out.read_text()
    for k in (1, 2, 3):
        for real, words in (("float", 1), ("double", 2)):
            body = re.search(rf"^k{k}_{real}:(.*?)s_endpgm", text, re.S | re.M).group(1)
            loads = re.findall(r"\b(?:global|flat|buffer)_load_dword(?:x(\d))?\b", body)
            assert loads and sum(int(n or 1) for n in loads) == (k + 1) * words, (k, real, loads)


def test_signed_zeros_are_given_up_in_the_chirp_z_units_only():
    """And alike in the kernels of a plan and of a batch (unit 8 and class 2 of unit 9)."""
    from paper_1812_07357_amd import build_lib

    assert "-fno-signed-zeros" not in build_lib.FLAGS
    for src, name, extra in build_lib.SOURCES:
        chirp = src == "passes.hip" and ("-DPSATD_UNIT=8" in extra or "-DPSATD_CLASS=2" in extra)
        assert ("-fno-signed-zeros" in extra) == chirp, name


def test_layers_hold_no_arrays_that_no_pass_uses(tmp_path):
    _run(_build(tmp_path, "pml_memory"))
