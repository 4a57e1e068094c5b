"""Build libmesa.so in-tree with hipcc for gfx950 (cross-compiles without a GPU)."""
from __future__ import annotations

import os
import shutil
import subprocess
import sys
import sysconfig
from concurrent.futures import ThreadPoolExecutor
from pathlib import Path

PKG = Path(__file__).resolve().parent
CSRC = PKG / "csrc"
INCLUDE = PKG.parent / "include"
LIB = PKG / "libmesa.so"
FAST = PKG / ("_marshal" + sysconfig.get_config_var("EXT_SUFFIX"))
OBJ = PKG / "_build"
SOURCES = ["stream_kernels.hip", "softmax_fwd.hip", "softmax_bwd.hip", "layernorm_fwd.hip", "layernorm_bwd.hip", "linear_dw.hip", "attn_matmul_bwd.hip", "lowbit.hip", "conv_dw.hip", "mfma_probe.hip"]
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

# -ffp-contract=off: no implicit fused multiply-adds anywhere; kernels that may fuse call fmaf.
# Packed binary32 arithmetic is switched off: some of its forms have given wrong results now and then.
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-fvisibility=hidden", "-ffp-contract=off",
         "-fhip-fp32-correctly-rounded-divide-sqrt", "-fno-gpu-flush-denormals-to-zero",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-Wall", "-Wno-unused-function", "-Wno-unknown-warning-option",
         f"-I{INCLUDE}", f"-I{CSRC}"]


def _compile(src: str) -> Path:
    OBJ.mkdir(exist_ok=True)
    out = OBJ / (src + ".o")
    cmd = [HIPCC, *FLAGS, "-c", str(CSRC / src), "-o", str(out)]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        sys.stderr.write(r.stdout + r.stderr)
        raise RuntimeError(f"hipcc failed on {src}")
    errs = [l for l in r.stderr.splitlines() if "warning" in l and "packed-fp32-ops" not in l and "unused-value" not in l]
    if errs:
        sys.stderr.write("\n".join(errs[:20]) + "\n")
    return out


def build(verbose: bool = True) -> Path:
    with ThreadPoolExecutor(max_workers=4) as ex:
        objs = list(ex.map(_compile, SOURCES))
    tmp = LIB.with_suffix(f".tmp{os.getpid()}.so")
    cmd = [HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", str(tmp), *map(str, objs)]
    subprocess.run(cmd, check=True)
    os.replace(tmp, LIB)
    # the binding's native marshalling: plain C against the Python headers, bound to the library beside it.  The binding
    # does without it, at some 6 us a call, so it asks for nothing that the library does not: no headers, no extension
    headers, cc = sysconfig.get_path("include"), os.environ.get("CC", "gcc")
    if (Path(headers) / "Python.h").exists() and shutil.which(cc.split()[0]):
        tmp = PKG / f"_marshal.tmp{os.getpid()}.so"
        cmd = [*cc.split(), "-O2", "-std=c11", "-fPIC", "-shared", "-Wall", f"-I{INCLUDE}", f"-I{headers}", str(CSRC / "marshal.c"), "-o", str(tmp),
               f"-L{PKG}", "-l:libmesa.so", "-Wl,-rpath,$ORIGIN"]
        subprocess.run(cmd, check=True)
        os.replace(tmp, FAST)
    else:
        print(f"no Python headers in {headers}, or no C compiler {cc}: {FAST.name} not built, calls are marshalled by ctypes")
    if verbose:
        print(f"built {LIB}")
    return LIB


if __name__ == "__main__":
    build()
