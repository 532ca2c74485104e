"""Builds the HIP library (libradar.so) in-tree with hipcc for gfx950."""
import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libradar.so")
SOURCES = ["radar_common.hip", "radar_expand.hip", "radar_accept.hip", "radar_attention.hip", "radar_policy.hip", "radar_accept_q.hip"]
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
         # packed fp32 arithmetic is kept off for device code
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         # a kernel's leading scalar arguments are in registers when it starts (as many as fit into the 16 that the
         # hardware fills), so that its first loads do not wait for the argument segment
         "-mllvm", "-amdgpu-kernarg-preload-count=14",
         # the loads that write LDS directly are issued as assembly and name m0, a reserved register, as clobbered
         "-Wno-inline-asm"]


NATIVE = os.path.join(HERE, "_native.so")
CXX = os.environ.get("CXX", "g++")


def _stale(target, deps):
    if not os.path.exists(target):
        return True
    t = os.path.getmtime(target)
    return any(os.path.getmtime(d) > t for d in deps)


SAN_LIB = os.path.join(HERE, "libradar_san.so")
SAN_NATIVE = os.path.join(HERE, "_native_san.so")
# host code only (the GPU side has no sanitizer here): each option directly after -Xarch_host
SAN_FLAGS = ["-Xarch_host", "-fsanitize=address", "-Xarch_host", "-fsanitize=undefined",
             "-Xarch_host", "-fno-sanitize-recover=undefined", "-Xarch_host", "-fno-omit-frame-pointer", "-g"]


def sanitizer_runtime():
    """Path of the address-sanitizer runtime the sanitized library needs preloaded."""
    r = subprocess.run([os.path.join(os.path.dirname(HIPCC), "..", "lib", "llvm", "bin", "clang"),
                        "--print-file-name=libclang_rt.asan-x86_64.so"], capture_output=True, text=True)
    return r.stdout.strip()


def build_library(force=True, verbose=False, sanitize=False):
    """Compile every kernel source and link paper_2512_14069_amd/libradar.so, and the binding's native half.  sanitize=True builds
    libradar_san.so and _native_san.so instead: the same sources with the HOST code (argument checks, planning,
    launch paths, argument marshalling) under AddressSanitizer and UndefinedBehaviorSanitizer; used by the CPU tests only."""
    headers = [os.path.join(CSRC, f) for f in os.listdir(CSRC) if f.endswith(".h")]
    headers.append(os.path.join(os.path.dirname(HERE), "include", "radar.h"))
    if sanitize:
        build_native(force, sanitize=True)
        return _build(os.path.join(HERE, "_build", "san"), SAN_LIB, [f for f in FLAGS if f != "-O3"] + ["-O1"] + SAN_FLAGS,
                      ["-fsanitize=address", "-fsanitize=undefined", "-shared-libsan"], headers, force, verbose)
    build_native(force)
    return _build(os.path.join(HERE, "_build"), LIB, FLAGS, [], headers, force, verbose)


def build_native(force=True, sanitize=False):
    """Compile the binding's argument marshaller (host code only) against the installed torch."""
    import sysconfig

    import torch
    src, root = os.path.join(CSRC, "radar_native.cpp"), os.path.dirname(torch.__file__)
    target = SAN_NATIVE if sanitize else NATIVE
    if not (force or _stale(target, [src, os.path.join(os.path.dirname(HERE), "include", "radar.h")])):
        return target
    # the sanitized one is built by clang, whose runtime the sanitized library brings along; torch has no type
    # information that the vptr check could use
    front = [CXX, "-O2"]
    if sanitize:
        front = [os.path.join(os.path.dirname(HIPCC), "..", "lib", "llvm", "bin", "clang++"), "-O1", "-g", "-fno-omit-frame-pointer",
                 "-fsanitize=address", "-fsanitize=undefined", "-fno-sanitize=vptr", "-fno-sanitize=function",
                 "-fno-sanitize-recover=undefined", "-shared-libsan"]
    cmd = front + ["-std=c++17", "-fPIC", "-shared", "-DUSE_ROCM=1", "-D__HIP_PLATFORM_AMD__=1",
           "-D_GLIBCXX_USE_CXX11_ABI=%d" % torch._C._GLIBCXX_USE_CXX11_ABI]
    for inc in (os.path.join(root, "include"), os.path.join(root, "include", "torch", "csrc", "api", "include"),
                os.path.join(os.path.dirname(HIPCC), "..", "include"), sysconfig.get_paths()["include"]):
        cmd += ["-isystem", inc]
    lib = os.path.join(root, "lib")
    cmd += [src, "-o", target, "-L" + lib, "-Wl,-rpath," + lib, "-lc10", "-lc10_hip", "-ltorch_cpu", "-ltorch_python", "-ldl"]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"{front[0]} failed for radar_native.cpp:\n{r.stderr}")
    return target


def _build(objdir, lib, flags, link_flags, headers, force, verbose):
    os.makedirs(objdir, exist_ok=True)
    objs = []
    for src in SOURCES:
        sp = os.path.join(CSRC, src)
        if not os.path.exists(sp):
            raise RuntimeError(f"kernel source {sp} is missing")
        obj = os.path.join(objdir, src.replace(".hip", ".o"))
        if force or _stale(obj, [sp] + headers):
            cmd = [HIPCC] + flags + ["-c", sp, "-o", obj]
            r = subprocess.run(cmd, capture_output=True, text=True)
            err = "\n".join(l for l in r.stderr.splitlines() if "not a recognized feature" not in l)
            if r.returncode != 0:
                raise RuntimeError(f"hipcc failed for {src}:\n{err}")
            if verbose and err.strip():
                print(err, file=sys.stderr)
        objs.append(obj)
    if force or _stale(lib, objs):
        r = subprocess.run([HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC"] + link_flags + ["-o", lib] + objs,
                           capture_output=True, text=True)
        if r.returncode != 0:
            raise RuntimeError(f"link failed:\n{r.stderr}")
    return lib


if __name__ == "__main__":
    print(build_library(force="--force" in sys.argv, verbose=True))
