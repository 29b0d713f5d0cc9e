"""Compile the HIP sources under csrc/ for gfx950 into paper_2408_08554_amd/libabq.so, and csrc/python/ (host code) into
the extension module abq_native beside it.

Run here on the CPU container (hipcc cross-compiles); the built library travels with the
tree.  `python -m paper_2408_08554_amd.build` rebuilds everything
(`--incremental`: only what changed).
"""
import concurrent.futures
import glob
import os
import subprocess
import sysconfig

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
OBJ = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "libabq.so")
NATIVE = os.path.join(HERE, "abq_native.so")           # the online entry points as a Python extension module
PROBE_LIB = os.path.join(HERE, "libabq_probe.so")   # measurement aids of the benchmark, not part of libabq.so

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-ffp-contract=off",
    # packed-FP32 instructions are kept out of all device code
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-function", "-Wno-unknown-warning-option",
]
if os.environ.get("ABQ_BUILD_TUNING") == "1":   # the tuner's A/B builds only: lets ABQ_* environment variables override launch plans
    FLAGS.append("-DABQ_TUNING_ENV")


def _compile(src: str, newest_header: float = 0.0) -> str:
    obj = os.path.join(OBJ, os.path.relpath(src, CSRC).replace(os.sep, "_") + ".o")
    if newest_header and os.path.exists(obj) and os.path.getmtime(obj) >= max(newest_header, os.path.getmtime(src)):
        return obj   # --incremental: neither the source nor any header is newer than the object
    extra = ["-Rpass-analysis=kernel-resource-usage"] if os.path.basename(src) in NO_SCRATCH else []
    if os.path.basename(src).startswith(("abq_block_p", "abq_f4")):
        # accumulators in ordinary registers also where one workgroup of four waves has a unit to itself; left alone, the compiler
        # puts them into the other register file and copies them to and fro inside the K loop
        extra += ["-mllvm", "-amdgpu-mfma-vgpr-form=1"]
    done = subprocess.run([HIPCC, *FLAGS, *extra, "-c", src, "-o", obj], check=True, stderr=subprocess.PIPE, text=True)
    if os.path.basename(src) in NO_SCRATCH:
        _check_no_scratch(src, done.stderr, NO_SCRATCH[os.path.basename(src)])
    return obj


# Kernels that may not use scratch memory; the build fails if one does.  Their K loops count on loads staying in flight: a reload from
# scratch inside one waits for all of them.  direct_kernel has all loads of a wave in flight at once, and spills them ahead of the weights it waits for.
NO_SCRATCH = {"abq_f4.hip": "f4_gemm_kernel", "abq_gemm_tiled.hip": "tiled_kernel", **{f"abq_ksplit_p{p}.hip": "ksplit_kernel" for p in range(1, 9)},
              **{f"abq_block_p{p}.hip": "block_" for p in range(1, 9)},
              **{f"abq_direct_p{p}.hip": "direct_kernel" for p in (12, 34, 56, 78)}}
# (64 x 256 tiles at p = 7, three plane groups of four tiles per wave: two registers over the 256 of two workgroups per CU)
SCRATCH_ALLOWED = ("tiled_kernelILi7ELi4ELi4ELi2E",)


def _check_no_scratch(src: str, remarks: str, kernel: str) -> None:
    name, seen = None, 0
    for line in remarks.splitlines():
        if "Function Name:" in line:
            name = line.split("Function Name:")[1].strip()
        elif "ScratchSize [bytes/lane]:" in line and name and kernel in name and not any(k in name for k in SCRATCH_ALLOWED):
            seen += 1
            if int(line.split(":")[-1].split()[0]) != 0:
                os.remove(os.path.join(OBJ, os.path.relpath(src, CSRC).replace(os.sep, "_") + ".o"))
                raise RuntimeError(f"{src}: kernel {name} uses scratch memory (see NO_SCRATCH)")
    if not seen:
        raise RuntimeError(f"{src}: no resource-usage remark for {kernel}; the scratch check did not run")


def _build_native(newest_header: float = 0.0) -> None:
    """abq_native (csrc/python/): host code against the installed torch's headers and libraries, and libabq.so beside it."""
    import torch
    src = os.path.join(CSRC, "python", "abq_native.cpp")
    if newest_header and os.path.exists(NATIVE) and os.path.getmtime(NATIVE) >= max(newest_header, os.path.getmtime(src)):
        return
    root = os.path.dirname(torch.__file__)
    cmd = ["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-fvisibility=hidden", "-Wall", "-Wno-missing-field-initializers",
           "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1", f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}",
           "-isystem", sysconfig.get_paths()["include"], "-isystem", os.path.join(root, "include"),
           "-isystem", os.path.join(root, "include", "torch", "csrc", "api", "include"), "-isystem", os.path.join(os.path.dirname(os.path.dirname(HIPCC)), "include"),
           src, "-o", NATIVE, "-L" + HERE, "-labq", "-L" + os.path.join(root, "lib"), "-lc10", "-lc10_hip", "-ltorch_cpu", "-ltorch_python",
           "-Wl,-rpath,$ORIGIN"]
    done = subprocess.run(cmd, stderr=subprocess.PIPE, text=True)
    if done.returncode:
        raise RuntimeError(f"g++ failed on {src}:\n{done.stderr}")


def build(verbose: bool = False, incremental: bool = False) -> str:
    """Compiles every source (always, unless `incremental`: then only what is older than its source or a header)."""
    os.makedirs(OBJ, exist_ok=True)
    srcs = sorted(glob.glob(os.path.join(CSRC, "*.hip")))
    probe_srcs = sorted(glob.glob(os.path.join(CSRC, "probe", "*.hip")))
    headers = glob.glob(os.path.join(CSRC, "*.h")) + glob.glob(os.path.join(HERE, "..", "include", "*.h")) + [__file__]
    newest = max(os.path.getmtime(h) for h in headers) if incremental else 0.0
    with concurrent.futures.ThreadPoolExecutor(max_workers=min(8, len(srcs))) as ex:
        futs = {ex.submit(_compile, s, newest): s for s in srcs + probe_srcs}
        objs, probe_objs = [], []
        for f, s in futs.items():
            try:
                (probe_objs if s in probe_srcs else objs).append(f.result())
            except subprocess.CalledProcessError as e:
                raise RuntimeError(f"hipcc failed on {s}:\n{e.stderr}") from None
            if verbose:
                print("compiled", os.path.basename(s), flush=True)
    subprocess.run([HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", *sorted(objs), "-o", LIB], check=True)
    subprocess.run([HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", *sorted(probe_objs), "-o", PROBE_LIB], check=True)
    _build_native(newest)
    return LIB


if __name__ == "__main__":
    import sys
    print(build(verbose=True, incremental="--incremental" in sys.argv))
