"""Build libgsi.so (HIP kernels + C ABI) for gfx950 with hipcc, in-tree.

``python -m paper_2605_03109_amd.build`` compiles every ``csrc/*.hip`` and links
``paper_2605_03109_amd/libgsi.so``.  hipcc cross-compiles, so no GPU is needed to build.
"""
from __future__ import annotations

import concurrent.futures
import glob
import os
import shutil
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
OBJ = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "libgsi.so")

ARCH = "gfx950"
# Packed-FP32 instruction selection is switched off for every device compile (the host pass warns
# that it does not know the feature; that is harmless).
HIPCC_FLAGS = [
    "-O3",
    "-std=c++17",
    "-fPIC",
    f"--offload-arch={ARCH}",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall",
    "-Wno-unused-function",
    "-Wno-unknown-warning-option",
]


def hipcc() -> str:
    exe = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(exe):
        raise RuntimeError("hipcc not found: libgsi cannot be built")
    return exe


# Kernels that must not use scratch memory (register spills): a dispatch that needs scratch costs tens of
# microseconds here, more than the whole single-token step.
NO_SCRATCH = {"gsi_fused.hip": ("fused_token",), "gsi_wide.hip": ("wide_",), "gsi_basis.hip": ("basis_product",), "gsi_stage.hip": ("proj_stage", "table_partial", "table_cred", "table_gram", "table_rows")}


# Waves per SIMD that launches of these kernels count on: workgroups of a whole call resident at once.
MIN_WAVES = {
    "gsi_stage.hip": {"proj_stage": 5, "one_partial": 5, "table_partial": 5, "table_rows": 6},
    # two-term operand, tiles of 128 rows, no transposition: two workgroups of eight waves per compute unit
    "gsi_mfma.hip": {f"gemm_ntILi1ELi{epi}ELi128ELb0E": 4 for epi in (1, 5, 6)},
}


def check_resources(name: str, remarks: str) -> int:
    """Holds the compiler's resource remarks of one source against NO_SCRATCH and MIN_WAVES; the kernels it looked at."""
    scratch, waves = NO_SCRATCH.get(name, ()), MIN_WAVES.get(name, {})
    kernel, seen = None, set()
    for line in remarks.splitlines():
        if "Function Name:" in line:
            kernel = line.split("Function Name:")[1].split()[0]
        elif kernel and "ScratchSize [bytes/lane]:" in line and any(w in kernel for w in scratch):
            n = int(line.split("ScratchSize [bytes/lane]:")[1].split()[0])
            seen.add(kernel)
            if n != 0:
                raise RuntimeError(f"{name}: kernel {kernel} spills registers ({n} bytes of scratch per lane)")
        elif kernel and "Occupancy [waves/SIMD]:" in line:
            n = int(line.split("Occupancy [waves/SIMD]:")[1].split()[0])
            for w, want in waves.items():
                if w in kernel:
                    seen.add(kernel)
                    if n < want:
                        raise RuntimeError(f"{name}: kernel {kernel} runs {n} waves per SIMD instead of {want}")
    return len(seen)


def _compile(src: str, obj: str | None = None) -> str:
    name = os.path.basename(src)
    obj = obj or os.path.join(OBJ, name.replace(".hip", ".o"))
    cmd = [hipcc(), *HIPCC_FLAGS, "-Rpass-analysis=kernel-resource-usage", "-c", src, "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed for {src}:\n{r.stdout}\n{r.stderr}")
    if check_resources(name, r.stderr) == 0 and (name in NO_SCRATCH or name in MIN_WAVES):
        raise RuntimeError(f"{src}: no resource remark of the kernels that are to be checked")
    return obj


def build(verbose: bool = True) -> str:
    os.makedirs(OBJ, exist_ok=True)
    srcs = sorted(glob.glob(os.path.join(CSRC, "*.hip")))
    if not srcs:
        raise RuntimeError("no HIP sources found")
    with concurrent.futures.ThreadPoolExecutor(max_workers=min(8, len(srcs))) as ex:
        objs = list(ex.map(_compile, srcs))
    cmd = [hipcc(), "-shared", "-fPIC", f"--offload-arch={ARCH}", *objs, "-o", LIB]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"link failed:\n{r.stdout}\n{r.stderr}")
    if verbose:
        print(f"built {LIB} from {len(srcs)} sources")
    return LIB


if __name__ == "__main__":
    build()
    sys.exit(0)
