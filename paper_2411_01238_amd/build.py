"""Builds libsdrop.so (the C-ABI library) in-tree with hipcc for gfx950."""
import os
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
INCLUDE = os.path.join(os.path.dirname(HERE), "include")
LIB = os.path.join(HERE, "libsdrop.so")
# (source, object, defines): the GEMM kernels are one source, compiled per operand type and group of kernels.
# The longest units come first.
UNITS = [("sdrop_gemm_inst.hip", "sdrop_gemm_%s_%d.o" % (t.lower(), part), ["-DSDROP_T=" + t, "-DSDROP_PART=%d" % part])
         for part in (1, 0, 3, 2, 5, 4) for t in ("F16", "BF16")]
UNITS += [(src, os.path.splitext(src)[0] + ".o", []) for src in ("sdrop_gemm.hip", "sdrop_mask.hip", "sdrop_bias_grad.hip")]

HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-fno-gpu-rdc",
    # packed fp32 VALU forms are kept out of the generated code on purpose
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-variable", "-Wno-unused-but-set-variable",
    "-I", INCLUDE, "-I", CSRC,
]


def _hipcc():
    return os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


def _compile(unit):
    src, obj, defines = unit
    obj = os.path.join(CSRC, obj)
    cmd = [_hipcc()] + HIPCC_FLAGS + defines + ["-c", os.path.join(CSRC, src), "-o", obj]
    r = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    out = "\n".join(l for l in r.stdout.splitlines() if "packed-fp32-ops" not in l)
    if r.returncode != 0:
        raise RuntimeError("hipcc failed on %s:\n%s" % (src, out))
    if out.strip():
        sys.stderr.write(out + "\n")
    return obj


def build(verbose=True):
    """Compiles every HIP source and links libsdrop.so; always rebuilds."""
    with ThreadPoolExecutor(max_workers=min(8, len(UNITS))) as ex:
        objs = list(ex.map(_compile, UNITS))
    cmd = [_hipcc(), "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB] + objs
    subprocess.check_call(cmd)
    if verbose:
        print("built", LIB)
    return LIB


if __name__ == "__main__":
    build()
