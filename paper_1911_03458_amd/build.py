"""Build libmerit.so (HIP kernels + C ABI; needs hipcc only) in-tree for gfx950, and _torch_calls.so beside it (a Python
module over the library; needs g++ and PyTorch's headers)."""
from __future__ import annotations

import os
import shutil
import subprocess
from concurrent.futures import ThreadPoolExecutor

_HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(_HERE)
CSRC = os.path.join(_HERE, "csrc")
LIB_PATH = os.path.join(_HERE, "libmerit.so")
CALLS_SRC = os.path.join(CSRC, "torch_calls.cpp")
CALLS_PATH = os.path.join(_HERE, "_torch_calls.so")      # a Python module over libmerit.so and PyTorch

SOURCES = ["merit_plan.cpp", "pool2d.hip", "sad_search.hip", "conv2d.hip", "conv2d_chws.hip", "conv2d_px.hip", "conv2d_split.hip", "maxpool_f16.hip", "generic.hip", "corr.hip", "dwconv.hip", "sepfilter.hip", "bilateral.hip", "probe.hip"]
HEADERS = [os.path.join(CSRC, "merit_internal.h"), os.path.join(ROOT, "include", "merit.h"),
           os.path.join(ROOT, "include", "merit_probe.h")]
CALLS_DEPS = [CALLS_SRC, os.path.join(ROOT, "include", "merit.h")]


def hipcc_path() -> str:
    for cand in (shutil.which("hipcc"), "/opt/rocm/bin/hipcc"):
        if cand and os.path.exists(cand):
            return cand
    raise RuntimeError("hipcc not found: the MERIT HIP library cannot be built")


def is_stale() -> bool:
    if not os.path.exists(LIB_PATH):
        return True
    t = os.path.getmtime(LIB_PATH)
    deps = [os.path.join(CSRC, s) for s in SOURCES] + HEADERS
    return any(os.path.getmtime(d) > t for d in deps)


def build_library(force: bool = True, extra_flags=()) -> str:
    """Compile every HIP source for gfx950 into one shared library."""
    if not force and not is_stale():
        return LIB_PATH
    common = [hipcc_path(), "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
              # keep hipcc from forming packed-fp32 VALU ops
              "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
              "-Wall", "-Wno-unused-command-line-argument",
              "-I", os.path.join(ROOT, "include"), "-I", CSRC, *extra_flags]
    # one object per source, compiled side by side (the convolution file dominates), then one link
    objdir = os.path.join(_HERE, "_build")
    os.makedirs(objdir, exist_ok=True)
    objs = [os.path.join(objdir, os.path.splitext(s)[0] + ".o") for s in SOURCES]

    def compile_one(job):
        src, obj = job
        return subprocess.run(common + ["-c", os.path.join(CSRC, src), "-o", obj], capture_output=True, text=True)

    with ThreadPoolExecutor(max_workers=min(len(SOURCES), os.cpu_count() or 1)) as pool:
        for proc in pool.map(compile_one, zip(SOURCES, objs)):
            if proc.returncode != 0:
                raise RuntimeError("hipcc failed:\n" + proc.stdout + proc.stderr)
    proc = subprocess.run(common + ["-shared", "-o", LIB_PATH] + objs, capture_output=True, text=True)
    if proc.returncode != 0:
        raise RuntimeError("hipcc (link) failed:\n" + proc.stdout + proc.stderr)
    return LIB_PATH


def calls_are_stale() -> bool:
    if not os.path.exists(CALLS_PATH):
        return True
    t = os.path.getmtime(CALLS_PATH)
    return any(os.path.getmtime(d) > t for d in CALLS_DEPS)


def build_torch_calls(force: bool = True) -> str:
    """Compile csrc/torch_calls.cpp (host code, no kernels) against PyTorch and the built library."""
    if not force and not calls_are_stale():
        return CALLS_PATH
    import sysconfig

    import torch
    from torch.utils import cpp_extension as ext

    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    libs = ext.library_paths()
    tmp = CALLS_PATH + ".%d.tmp" % os.getpid()      # (never a half-written module in the way of another process)
    cmd = ["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1",
           "-D_GLIBCXX_USE_CXX11_ABI=%d" % int(torch._C._GLIBCXX_USE_CXX11_ABI),
           '-DMERIT_TORCH="%s"' % torch.__version__, CALLS_SRC, "-o", tmp,
           "-I", os.path.join(ROOT, "include"), "-I", sysconfig.get_paths()["include"]]
    cmd += ["-isystem" + d for d in ext.include_paths() + [os.path.join(rocm, "include")]]
    cmd += ["-L" + _HERE, "-l:" + os.path.basename(LIB_PATH), "-Wl,-rpath,$ORIGIN"] + ["-L" + d for d in libs]
    cmd += ["-ltorch_python", "-ltorch_cpu", "-ltorch_hip", "-lc10_hip", "-lc10"]
    proc = subprocess.run(cmd, capture_output=True, text=True)
    if proc.returncode != 0:
        raise RuntimeError("g++ (torch_calls) failed:\n" + proc.stdout + proc.stderr)
    os.replace(tmp, CALLS_PATH)
    return CALLS_PATH


def build_all(force: bool = True) -> None:
    """The library and the Python module over it."""
    build_library(force=force)
    build_torch_calls(force=force)


def build_host_check(sanitizer: str = "address,undefined") -> str:
    """CPU-only build for host robustness checks: the host side of every source (no device code,
    so it takes seconds) with -fsanitize=<sanitizer>, linked with csrc/host_check.cpp into an
    executable that exercises the plan code through the C ABI without touching a GPU.
    `sanitizer` = "address,undefined" or "thread".  Returns the executable's path."""
    tag = sanitizer.replace(",", "_")
    objdir = os.path.join(_HERE, "_build", "host_" + tag)
    os.makedirs(objdir, exist_ok=True)
    exe = os.path.join(objdir, "host_check")
    srcs = [os.path.join(CSRC, s) for s in SOURCES] + [os.path.join(CSRC, "host_check.cpp")]
    if os.path.exists(exe) and all(os.path.getmtime(d) <= os.path.getmtime(exe) for d in srcs + HEADERS):
        return exe
    common = [hipcc_path(), "--offload-arch=gfx950", "--cuda-host-only", "-O1", "-g", "-std=c++17",
              "-fsanitize=" + sanitizer, "-fno-sanitize-recover=all", "-Wno-unused-command-line-argument",
              "-I", os.path.join(ROOT, "include"), "-I", CSRC]
    objs = [os.path.join(objdir, os.path.splitext(os.path.basename(s))[0] + ".o") for s in srcs]

    def compile_one(job):
        src, obj = job
        return subprocess.run(common + ["-c", src, "-o", obj], capture_output=True, text=True)

    with ThreadPoolExecutor(max_workers=min(len(srcs), os.cpu_count() or 1)) as pool:
        for proc in pool.map(compile_one, zip(srcs, objs)):
            if proc.returncode != 0:
                raise RuntimeError("hipcc (host check) failed:\n" + proc.stdout + proc.stderr)
    # Host-only objects still refer to the device code object they would register at load time
    # (one symbol per source, named after a hash); there is none in this build: define each as
    # a few zero bytes, which the HIP runtime declines to load -- nothing here launches a kernel.
    undef = set()
    for obj in objs:
        nm = subprocess.run(["nm", "-u", obj], capture_output=True, text=True)
        undef |= {ln.split()[-1] for ln in nm.stdout.splitlines() if "__hip_fatbin_" in ln}
    stub = os.path.join(objdir, "no_device_code.c")
    with open(stub, "w") as f:
        for name in sorted(undef):
            f.write(f"const unsigned long long {name}[8] = {{0}};\n")
    stub_o = os.path.join(objdir, "no_device_code.o")
    proc = subprocess.run(["gcc", "-c", stub, "-o", stub_o], capture_output=True, text=True)
    if proc.returncode != 0:
        raise RuntimeError("gcc (host check stub) failed:\n" + proc.stdout + proc.stderr)
    proc = subprocess.run([hipcc_path(), "--offload-arch=gfx950", "-fsanitize=" + sanitizer, "-o", exe] + objs
                          + [stub_o, "-lpthread"], capture_output=True, text=True)
    if proc.returncode != 0:
        raise RuntimeError("hipcc (host check link) failed:\n" + proc.stdout + proc.stderr)
    return exe


if __name__ == "__main__":
    build_all()
    print(LIB_PATH, CALLS_PATH)
