"""Compile the HIP sources into paper_2402_00025_amd/libw4a16.so for gfx950 (cross-compiles
without a GPU) and the Python calls of its GEMM entry points into paper_2402_00025_amd/_call.so.
Both are built in-tree so they travel with the source tree."""
from __future__ import annotations

import pathlib
import subprocess
import sysconfig
import tempfile

HERE = pathlib.Path(__file__).resolve().parent
SOURCES = [HERE / "csrc" / "w4a16.hip", HERE / "csrc" / "w4a16_rows.hip", HERE / "csrc" / "w4a16_batch.hip",
           HERE / "csrc" / "w4a16_fine.hip"]
LIB = HERE / "libw4a16.so"
CALL_SRC = HERE / "csrc" / "py_call.cpp"
CALL_LIB = HERE / "_call.so"

HIPCC_FLAGS = [
    "-O3", "--offload-arch=gfx950", "-std=c++17", "-fPIC",
    "-munsafe-fp-atomics",                                     # hardware fp32 / packed-fp16 atomic adds
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",  # no v_pk_*_f32
    "-mllvm", "-amdgpu-kernarg-preload-count=14",                # leading kernel arguments arrive in SGPRs
    "-Wall", "-Wno-unused-function",
]


def build_call(verbose: bool = False) -> pathlib.Path:
    """_call.so: host code only, against torch's headers and libw4a16.so (which is found beside it)."""
    from torch.utils import cpp_extension

    rocm = pathlib.Path(cpp_extension.ROCM_HOME or "/opt/rocm")
    include = [sysconfig.get_path("include"), *cpp_extension.include_paths(), str(rocm / "include")]
    cmd = ["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-D__HIP_PLATFORM_AMD__", "-DUSE_ROCM",
           *(f for i in include for f in ("-isystem", i)), str(CALL_SRC), "-o", str(CALL_LIB),
           f"-L{HERE}", "-l:libw4a16.so", "-Wl,-rpath,$ORIGIN",
           *(f"-L{p}" for p in cpp_extension.library_paths()), "-ltorch_python", "-ltorch", "-ltorch_cpu", "-lc10", "-lc10_hip",
           "-Wall"]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.run(cmd, check=True)
    return CALL_LIB


def build(verbose: bool = False, extra=()) -> pathlib.Path:
    with tempfile.TemporaryDirectory() as tmp:
        objects, running = [], []
        for src in SOURCES:  # side by side
            objects.append(str(pathlib.Path(tmp) / (src.stem + ".o")))
            cmd = ["hipcc", *HIPCC_FLAGS, *extra, "-c", "-o", objects[-1], str(src)]
            if verbose:
                print(" ".join(cmd), flush=True)
            running.append((cmd, subprocess.Popen(cmd)))
        for cmd, p in running:
            if p.wait() != 0:
                for _, other in running:
                    other.kill()
                raise subprocess.CalledProcessError(p.returncode, cmd)
        cmd = ["hipcc", "-shared", "--offload-arch=gfx950", "-o", str(LIB), *objects]
        if verbose:
            print(" ".join(cmd), flush=True)
        subprocess.run(cmd, check=True)
    build_call(verbose)
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
