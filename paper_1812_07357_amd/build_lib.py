"""Build libpsatd.so (HIP, gfx950) in-tree with hipcc.

Usage: python -m paper_1812_07357_amd.build_lib [--incremental]  (or build() from Python).
Objects are compiled in parallel into _build/ and linked into
paper_1812_07357_amd/libpsatd.so.
"""

from __future__ import annotations

import concurrent.futures as cf
import os
import shutil
import subprocess
import sys

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
BUILD = os.path.join(ROOT, "_build")
LIB = os.path.join(PKG, "libpsatd.so")

ARCH = "gfx950"
HIPCC = os.environ.get("HIPCC", shutil.which("hipcc") or "/opt/rocm/bin/hipcc")

# Packed FP32 instructions are disabled: the compiler forms them from plain
# float code, and some of their forms are not trusted on this hardware.
FLAGS = [
    "-O3", "-std=c++17", "-fPIC", f"--offload-arch={ARCH}",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-function",
    f"-I{os.path.join(ROOT, 'include')}",
]

# Chirp-z lines: their zero padding folds out of the butterflies where -0 and +0 are the same value, which
# they are for a field.  The Stockham y pass spills more with the flag (FP32, chirp-z lines of 579 to 645 points
# 17 % slower), the direct pairs gain 2 % of one pass.  (A kernel and its form for batches are compiled alike:
# their results are the same bit for bit.)
_CHIRP_FLAGS = ["-fno-signed-zeros"]
# (source, object name, extra flags).  passes.hip is compiled once per unit and precision, the
# pair kernels (units 7..9) also once per pass, those of batches per class, so that the large pass
# kernels build in parallel; the slowest units come first.
_PAIR_UNITS = (("pair", ["-DPSATD_UNIT=7"]), ("pair_batch", ["-DPSATD_UNIT=9", "-DPSATD_CLASS=0"]),
               ("chirp", ["-DPSATD_UNIT=8", *_CHIRP_FLAGS]),
               ("chirp_batch", ["-DPSATD_UNIT=9", "-DPSATD_CLASS=2", *_CHIRP_FLAGS]))
_PASS_UNITS = [(f"{name}_{kind}", [*unit, f"-DPSATD_PART={part}"])
               for part, name in ((3, "zpush"), (2, "ypass"), (1, "xfwd"), (4, "xinv")) for kind, unit in _PAIR_UNITS]
_PASS_UNITS += [(name, [f"-DPSATD_UNIT={u}"])
                for u, name in ((1, "xfwd"), (2, "ypass"), (3, "zpush"), (4, "zpush_batch"), (5, "xinv"), (6, "zpush_pml"))]
SOURCES = [("passes.hip", f"passes_{name}_{prec}", [*extra, f"-DPSATD_REAL={prec}"])
           for name, extra in _PASS_UNITS for prec in ("float", "double")]
SOURCES += [(src, os.path.splitext(src)[0], []) for src in ("tables.hip", "guards.hip", "plan.hip", "mlp.hip", "pic.hip", "pml.hip")]


def _compile(unit) -> str:
    src, name, extra = unit
    obj = os.path.join(BUILD, name + ".o")
    cmd = [HIPCC, *FLAGS, *extra, "-c", os.path.join(CSRC, src), "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed on {src} ({name}):\n{r.stderr[-8000:]}")
    return obj


def _stale(unit) -> bool:
    """True if the unit's object is missing or older than its source or any header."""
    src, name, _ = unit
    obj = os.path.join(BUILD, name + ".o")
    if not os.path.exists(obj):
        return True
    deps = [os.path.join(CSRC, src)] + [os.path.join(CSRC, f) for f in os.listdir(CSRC) if f.endswith(".hpp")]
    deps.append(os.path.join(ROOT, "include", "psatd.h"))
    t = os.path.getmtime(obj)
    return any(os.path.getmtime(d) > t for d in deps)


def build(verbose: bool = True, incremental: bool = False) -> str:
    """Compile every unit (or, with ``incremental``, only the stale ones) and link the library."""
    os.makedirs(BUILD, exist_ok=True)
    units = [u for u in SOURCES if not incremental or _stale(u)]
    jobs = min(max(1, len(units)), max(1, (os.cpu_count() or 2)))
    with cf.ThreadPoolExecutor(jobs) as ex:
        list(ex.map(_compile, units))
    objs = [os.path.join(BUILD, name + ".o") for _, name, _ in SOURCES]
    tmp = LIB + ".tmp"
    cmd = [HIPCC, f"--offload-arch={ARCH}", "-shared", "-fPIC", "-o", tmp, *objs]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"link failed:\n{r.stderr[-8000:]}")
    os.replace(tmp, LIB)
    if verbose:
        print(f"built {LIB}", file=sys.stderr)
    return LIB


if __name__ == "__main__":
    build(incremental="--incremental" in sys.argv[1:])
