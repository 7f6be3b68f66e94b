"""Build the gfx950 shared library libmmx.so in place (hipcc; no GPU needed).

Usage: python -m paper_2406_16064_amd.build   (or call build()).
All HIP sources are compiled with packed-FP32 instructions disabled.
"""
import os
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
OUT = os.path.join(HERE, "libmmx.so")
SOURCES = ("hotpath.hip", "invx_f32_demag.hip", "invx_f32_local.hip", "invx_f64_demag.hip",
           "invx_f64_local.hip", "invx_f32_demag_cells.hip", "invx_f32_local_cells.hip",
           "invx_f64_demag_cells.hip", "invx_f64_local_cells.hip", "yzy_f32.hip", "yzy_f64.hip",
           "lengths_f32.hip", "lengths_f64.hip", "invx_f32_any_cells.hip", "invx_f64_any_cells.hip",
           "invx_f32_any1.hip", "invx_f32_any2.hip", "invx_f32_any4.hip", "invx_f64_any1.hip", "invx_f64_any2.hip",
           "invx_f64_any4.hip",
           "len_f32.hip", "long_f32.hip", "invx_f32_len1.hip", "invx_f32_len2.hip",
           "len_f64.hip", "long_f64.hip", "invx_f64_len1.hip", "invx_f64_len2.hip", "potential.hip", "setup.hip", "plan.hip")
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops"]


def _hipcc():
    for c in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", "hipcc"):
        if c and (os.path.isabs(c) and os.path.exists(c) or not os.path.isabs(c)):
            return c
    return "hipcc"


def _run(cmd):
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("build failed: %s\n%s%s" % (" ".join(cmd), r.stdout, r.stderr))


def build(verbose=False):
    """Compile every HIP source for gfx950 and link libmmx.so (always rebuilds)."""
    hipcc = _hipcc()
    objdir = os.path.join(HERE, "_build")
    os.makedirs(objdir, exist_ok=True)
    objs = []
    cmds = []
    for src in SOURCES:
        obj = os.path.join(objdir, src.replace(".hip", ".o"))
        objs.append(obj)
        cmds.append([hipcc] + FLAGS + ["-c", os.path.join(CSRC, src), "-o", obj])
    with ThreadPoolExecutor(max_workers=len(cmds)) as ex:
        list(ex.map(_run, cmds))
    tmp = OUT + ".tmp"
    _run([hipcc, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", tmp] + objs)
    os.replace(tmp, OUT)
    if verbose:
        print("built", OUT)
    return OUT


if __name__ == "__main__":
    build(verbose=True)
    sys.exit(0)
