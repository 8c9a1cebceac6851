"""Builds libpdd.so (HIP kernels + C ABI) for gfx950 with hipcc.

Sources compile in parallel into objects under _build/ and link into
paper_1705_03666_amd/libpdd.so.  Usage: python -m paper_1705_03666_amd.build
"""
from __future__ import annotations

import concurrent.futures as cf
import os
import shutil
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
BUILD = os.path.join(ROOT, "_build")
LIB = os.path.join(HERE, "libpdd.so")
ARCH = os.environ.get("PDD_OFFLOAD_ARCH", "gfx950")

SOURCES = ["walk_fwd.hip", "walk_adj_f32.hip", "walk_adj_f64.hip", "walk_common.hip", "branching.hip",
           "walk_batch.hip", "noalloc.hip", "capi.cpp", "schedule.cpp", "specialize.cpp"]
# device headers embedded into the library for runtime compilation of
# problem-specialised kernels (see csrc/pdd_spec.hpp)
RTC_HEADERS = ["pdd_internal.hpp", "pdd_device.hpp", "walk_kernels.hpp", "walk_stream.hpp", "branch_kernels.hpp"]
RTC_SOURCE = "rtc_sources.cpp"

FLAGS = ["-O3", "-std=c++17", "-fPIC", f"--offload-arch={ARCH}", "-I", os.path.join(ROOT, "include"), "-I", CSRC,
         # no packed FP32 instructions in device code
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-Wall", "-Wno-unused-function", "-Wno-unused-variable", "-Wno-unused-but-set-variable"]


def _hipcc() -> str:
    p = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(p):
        raise RuntimeError("hipcc not found")
    return p


def _write_rtc_source() -> str:
    """C++ file holding the text of RTC_HEADERS as raw string literals."""
    delim = "PDDRTC"
    names, bodies = [], []
    for h in RTC_HEADERS:
        with open(os.path.join(CSRC, h)) as fh:
            text = fh.read()
        if f'){delim}"' in text:
            raise RuntimeError(f"{h} contains the raw-string delimiter")
        names.append(f'"{h}"')
        bodies.append(f'R"{delim}({text}){delim}"')
    out = os.path.join(BUILD, RTC_SOURCE)
    body = ("// Generated by build.py: device headers for runtime compilation.\n"
            "namespace pdd {\n"
            f"extern const int kRtcHeaderCount = {len(names)};\n"
            f"extern const char* const kRtcHeaderNames[] = {{{', '.join(names)}}};\n"
            f"extern const char* const kRtcHeaderBodies[] = {{\n" + ",\n".join(bodies) + "};\n"
            "}  // namespace pdd\n")
    tmp = out + ".tmp"
    with open(tmp, "w") as fh:
        fh.write(body)
    os.replace(tmp, out)
    return out


def _compile(src: str) -> str:
    obj = os.path.join(BUILD, os.path.splitext(src)[0] + ".o")
    path = os.path.join(BUILD, src) if src == RTC_SOURCE else os.path.join(CSRC, src)
    cmd = [_hipcc()] + FLAGS + ["-c", path, "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"compiling {src} failed:\n{r.stderr}")
    return obj


def build(jobs: int = 0, verbose: bool = True) -> str:
    os.makedirs(BUILD, exist_ok=True)
    _write_rtc_source()
    srcs = SOURCES + [RTC_SOURCE]
    jobs = jobs or min(len(srcs), max(1, (os.cpu_count() or 4)))
    with cf.ThreadPoolExecutor(jobs) as ex:
        objs = list(ex.map(_compile, srcs))
    tmp = LIB + ".tmp"
    cmd = [_hipcc(), "-shared", "-fPIC", f"--offload-arch={ARCH}", "-o", tmp] + objs + ["-lhiprtc"]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"linking libpdd.so failed:\n{r.stderr}")
    os.replace(tmp, LIB)
    if verbose:
        print(f"built {LIB}")
    return LIB


# Host code with argument checking, built again under AddressSanitizer and
# UndefinedBehaviorSanitizer by build_host_sanitized (device code unchanged:
# every -fsanitize applies to the host pass only).
SANITIZED_HOST_SOURCES = ["capi.cpp", "schedule.cpp", "specialize.cpp", "noalloc.hip"]
HOST_SANITIZER_FLAGS = ["-Xarch_host", "-fsanitize=address", "-Xarch_host", "-fsanitize=undefined",
                        "-Xarch_host", "-fno-sanitize-recover=undefined", "-Xarch_host", "-fno-omit-frame-pointer"]


def sanitizer_runtime() -> str:
    """Path of the AddressSanitizer runtime the sanitized library needs
    (LD_PRELOAD it into a process that is not itself instrumented)."""
    clang = os.path.join(os.path.dirname(os.path.realpath(_hipcc())), "..", "lib", "llvm", "bin", "clang")
    if not os.path.exists(clang):
        clang = shutil.which("clang") or "/opt/rocm/llvm/bin/clang"
    r = subprocess.run([clang, "-print-file-name=libclang_rt.asan-x86_64.so"], capture_output=True, text=True)
    path = r.stdout.strip()
    if r.returncode != 0 or not os.path.isabs(path) or not os.path.exists(path):
        raise RuntimeError("AddressSanitizer runtime not found")
    return path


def build_host_sanitized(out_dir: str) -> str:
    """libpdd_san.so in out_dir: the host sources that check arguments
    (SANITIZED_HOST_SOURCES) compiled with the host sanitizers, linked with
    the kernel objects of the regular build (built first if missing)."""
    os.makedirs(out_dir, exist_ok=True)
    plain = [s for s in SOURCES + [RTC_SOURCE] if s not in SANITIZED_HOST_SOURCES]
    objs = [os.path.join(BUILD, os.path.splitext(s)[0] + ".o") for s in plain]
    if not all(os.path.exists(o) for o in objs):
        build(verbose=False)

    def compile_san(src: str) -> str:
        obj = os.path.join(out_dir, os.path.splitext(src)[0] + ".o")
        cmd = [_hipcc()] + [f for f in FLAGS if f != "-O3"] + ["-O1", "-g"] + HOST_SANITIZER_FLAGS + \
            ["-c", os.path.join(CSRC, src), "-o", obj]
        r = subprocess.run(cmd, capture_output=True, text=True)
        if r.returncode != 0:
            raise RuntimeError(f"compiling {src} with sanitizers failed:\n{r.stderr}")
        return obj

    with cf.ThreadPoolExecutor(len(SANITIZED_HOST_SOURCES)) as ex:
        san = list(ex.map(compile_san, SANITIZED_HOST_SOURCES))
    lib = os.path.join(out_dir, "libpdd_san.so")
    cmd = [_hipcc(), "-shared", "-fPIC", f"--offload-arch={ARCH}", "-o", lib] + objs + san + ["-lhiprtc"] + \
        ["-Xarch_host", "-fsanitize=address", "-Xarch_host", "-fsanitize=undefined", "-shared-libsan"]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"linking libpdd_san.so failed:\n{r.stderr}")
    return lib


if __name__ == "__main__":
    build(int(sys.argv[1]) if len(sys.argv) > 1 else 0)
