"""Build the HIP library (gfx950) in-tree with hipcc.

    python -m paper_1802_10323_amd.build

produces ``paper_1802_10323_amd/libpoisson_hip.so`` from the translation units
in ``csrc/`` (objects in ``paper_1802_10323_amd/_build/``).
"""
import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
LIB = os.path.join(HERE, "libpoisson_hip.so")
LINE_PARTS = 8      # objects of r2r_line_part.hip, each with its share of the lengths
# (source, extra flags, object name)
UNITS = [(name, [], name + ".o")
         for name in ("poisson.hip", "r2r_async.hip", "r2r_async_wide.hip", "tri_async.hip",
                      "tri_line.hip")]
UNITS += [("r2r_line_part.hip", [f"-DPOISSON_LINE_PART_INDEX={i}"], f"r2r_line_part{i}.hip.o")
          for i in range(LINE_PARTS)]
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

FLAGS = [
    "-O3", "-std=c++17", "-fPIC", "-shared",
    "--offload-arch=gfx950",
    # no packed-FP32 instructions in device code
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-I" + os.path.join(ROOT, "include"),
    "-I" + os.path.join(HERE, "csrc"),
    "-Wall", "-Wno-unused-result",
]


def _run(cmd, verbose):
    if verbose:
        print(" ".join(cmd), flush=True)
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode != 0:
        sys.stderr.write(res.stdout + res.stderr)
        raise RuntimeError(f"hipcc failed with status {res.returncode}: {' '.join(cmd)}")


def build(verbose=False):
    """Compile every translation unit (in parallel) and link the library."""
    from concurrent.futures import ThreadPoolExecutor
    objdir = os.path.join(HERE, "_build")
    os.makedirs(objdir, exist_ok=True)
    objs = [os.path.join(objdir, obj) for _, _, obj in UNITS]
    compile_flags = [f for f in FLAGS if f != "-shared"]

    def compile_unit(unit):
        src, extra, obj = unit
        _run([HIPCC, *compile_flags, *extra, "-c", os.path.join(HERE, "csrc", src),
              "-o", os.path.join(objdir, obj)], verbose)

    with ThreadPoolExecutor(max_workers=min(len(UNITS), max(2, os.cpu_count() or 2))) as pool:
        list(pool.map(compile_unit, UNITS))
    tmp = LIB + ".tmp"
    _run([HIPCC, "-shared", "-fPIC", "--offload-arch=gfx950", *objs, "-o", tmp], verbose)
    os.replace(tmp, LIB)
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
