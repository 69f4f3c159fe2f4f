"""Compile the HIP sources under csrc/ into paper_2602_11235_amd/libmtfm_hta.so for gfx950."""
from __future__ import annotations

import concurrent.futures
import glob
import os
import shutil
import subprocess
import tempfile

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libmtfm_hta.so")

HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared", "-fvisibility=hidden",
    "-Wall", "-Wextra", "-Wno-unused-parameter", "-munsafe-fp-atomics",
    # the global->LDS copies name M0 in their clobber lists on purpose (the compiler reserves M0 and says so each time)
    "-Wno-inline-asm",
    # packed fp32 VALU forms are kept off for every device function in this library
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
]

# Instruction scheduling strategy of single translation units.  The compiler's default strategy schedules for occupancy
# first; "max-ilp" orders for instruction-level parallelism, which in the dQ kernels puts the dQ products of one row block
# between the weight arithmetic of the other and in the 128-wide dK/dV kernel (one wave per SIMD) spreads the matrix
# instructions through the vector work.  Measured on MI355X: dQ 2-5 % faster, dK/dV at head_dim 128 3.7 %; the forward and
# the other dK/dV kernels are slower with it (lower occupancy, spills) and keep the default.
MAX_ILP = ["-mllvm", "-amdgpu-sched-strategy=max-ilp"]
# A kernel that owns more than 256 registers per wave has its matrix results placed in accumulation registers, from where every score
# had to be copied before vector instructions could use it (64 copies per 64 matrix instructions at head_dim 128).  This leaves the
# choice to the register allocator, which then keeps operands there instead.  dK/dV of 128 users of 750..8192 keys 23.15 -> 22.7 ms;
# whole steps at head_dim 128: 32 users of 60..120 keys 72.0 -> 69.5 us, 200 target layers of 250..1000 keys 422 -> 416.  (The
# pointwise dK/dV kernel loses by it, 1243 -> 1259 us per step: its unit keeps the default.)
VGPR_FORM = ["-mllvm", "-amdgpu-mfma-vgpr-form=1"]
# Kernel arguments in scalar registers when a kernel starts, up to the first one that is a struct: the command processor fetches them with the
# launch, where a load of the kernel's own takes 1100 cycles (0.45 us) before the first address is known.  For the kernels of a few
# requests, which live for 3 to 30 us and start with those.
KERNARG_PRELOAD = ["-mllvm", "-amdgpu-kernarg-preload-count=14"]
FILE_FLAGS = {
    "hta_bwd_dq_bf16.hip": MAX_ILP,
    "hta_bwd_dkdv128_bf16.hip": MAX_ILP + VGPR_FORM,
    "hta_bwd_brief_bf16.hip": VGPR_FORM,
    "hta_serve_bf16.hip": KERNARG_PRELOAD,
}


def sources():
    return sorted(glob.glob(os.path.join(CSRC, "*.hip")))


def _run(cmd, verbose):
    if verbose:
        print(" ".join(cmd))
    proc = subprocess.run(cmd, capture_output=True, text=True)
    noise = "'-packed-fp32-ops' is not a recognized feature"
    err = "\n".join(line for line in proc.stderr.splitlines() if noise not in line)
    if proc.returncode != 0:
        raise RuntimeError(f"hipcc failed:\n{err}")
    if verbose and err.strip():
        print(err)


def build(verbose: bool = False, extra_flags=()) -> str:
    """Compile every source to an object file (in parallel, one hipcc per file), link, and move the library into place
    only when all of it succeeded."""
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    compile_flags = [f for f in HIPCC_FLAGS if f != "-shared"]
    srcs = sources()
    with tempfile.TemporaryDirectory(prefix="mtfm_hta_build_") as tmp:
        objs = [os.path.join(tmp, os.path.basename(src) + ".o") for src in srcs]
        jobs = [[hipcc, *compile_flags, *FILE_FLAGS.get(os.path.basename(src), []), *extra_flags, "-c", "-o", obj, src]
                for src, obj in zip(srcs, objs)]
        workers = max(1, min(len(jobs), int(os.environ.get("MAX_JOBS", os.cpu_count() or 1))))
        with concurrent.futures.ThreadPoolExecutor(workers) as pool:
            list(pool.map(lambda cmd: _run(cmd, verbose), jobs))
        out = os.path.join(tmp, "libmtfm_hta.so")
        _run([hipcc, "--offload-arch=gfx950", "-shared", "-fPIC", "-fvisibility=hidden", "-o", out, *objs], verbose)
        staged = LIB + f".tmp{os.getpid()}"
        shutil.copyfile(out, staged)
    os.chmod(staged, 0o755)
    os.replace(staged, LIB)
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
