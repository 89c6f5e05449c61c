"""Builds libmoe_gfx950.so in-tree with hipcc (cross-compiles for gfx950; no GPU needed)."""
from __future__ import annotations

import os
import subprocess
import sys
import tempfile
from concurrent.futures import ThreadPoolExecutor

PKG_DIR = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG_DIR)
CSRC = os.path.join(PKG_DIR, "csrc")
LIB_PATH = os.path.join(PKG_DIR, "libmoe_gfx950.so")
SOURCES = ["moe_api.hip", "index_build.hip", "grouped_gemm.hip", "decode_gemm.hip", "probes.hip"]


def build_library(verbose: bool = False, extra_flags=(), out_path: str = LIB_PATH) -> str:
    """Compiles the library, its sources side by side, to objects next to out_path.  extra_flags / out_path: builds with extra
    instrumentation go elsewhere than in-tree; the flags are those of every compilation and of the link."""
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    common = [hipcc, "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
              "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",   # no packed-fp32 code generation
              "-Wno-unused-command-line-argument",
              "-I", os.path.join(ROOT, "include"), "-I", CSRC] + list(extra_flags)

    def run(cmd):
        if verbose:
            print(" ".join(cmd), flush=True)
        res = subprocess.run(cmd, capture_output=True, text=True)
        # the host pass does not know the packed-fp32 feature and says so; that line is noise
        err = "\n".join(l for l in res.stderr.splitlines() if "packed-fp32-ops" not in l)
        if res.returncode != 0:
            raise RuntimeError(f"hipcc failed ({res.returncode}):\n{err}")
        if verbose and err.strip():
            print(err, file=sys.stderr)

    with tempfile.TemporaryDirectory(prefix="moe_build_", dir=os.path.dirname(os.path.abspath(out_path))) as tmp:
        objects = [os.path.join(tmp, s.replace(".hip", ".o")) for s in SOURCES]
        with ThreadPoolExecutor(len(SOURCES)) as pool:
            list(pool.map(run, [common + ["-c", os.path.join(CSRC, s), "-o", o] for s, o in zip(SOURCES, objects)]))
        run([hipcc, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", out_path] + list(extra_flags) + objects)
    return out_path


if __name__ == "__main__":
    print(build_library(verbose=True))
