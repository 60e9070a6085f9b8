"""Builds libcoexec.so in-tree: HIP kernels with hipcc for gfx950, host code
with g++, linked with hipcc."""
from __future__ import annotations

import os
import subprocess
import sys

PKG = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(PKG, "csrc")
BUILD = os.path.join(PKG, "_build")
LIB = os.path.join(PKG, "libcoexec.so")
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")
HIPCC = os.path.join(ROCM, "bin", "hipcc")

# No FP contraction anywhere: every payload operation is written explicitly.
# Packed FP32 instructions are disabled for all device code.
HIP_FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-ffp-contract=off", "-fno-fast-math",
             "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops", "-Wall"]
# functions on cache lines: the host's binomial loop takes half as long again where
# the linker happens to put it at 48 past one
CXX_FLAGS = ["-O3", "-std=c++17", "-fPIC", "-ffp-contract=off", "-fno-fast-math", "-fno-math-errno", "-Wall",
             "-falign-functions=64", "-D__HIP_PLATFORM_AMD__", "-I" + os.path.join(ROCM, "include"), "-pthread"]


def _run(cmd, verbose):
    if verbose:
        print(" ".join(cmd), flush=True)
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        sys.stderr.write(r.stdout + r.stderr)
        raise RuntimeError("build step failed: " + " ".join(cmd[:3]))
    # hipcc's host pass does not know the packed-fp32 target feature; that warning is harmless
    noise = [ln for ln in (r.stdout + r.stderr).splitlines() if "packed-fp32-ops" not in ln and ln.strip()]
    if verbose and noise:
        print("\n".join(noise))


# Device headers compiled again, with the caller's work-item function, when a
# payload is supplied as source at run time (hipRTC has no HIP runtime header
# and no <stddef.h>: those includes are dropped, and the public header is
# found by its bare name).
RT_HEADERS = [("common.hpp", os.path.join(CSRC, "common.hpp")),
              ("device_atomics.hpp", os.path.join(CSRC, "device_atomics.hpp")),
              ("device_divide.hpp", os.path.join(CSRC, "device_divide.hpp")),
              ("sched_device.hpp", os.path.join(CSRC, "sched_device.hpp")),
              ("rt_tile.hpp", os.path.join(CSRC, "rt_tile.hpp")),
              ("coexec.h", os.path.join(PKG, "..", "include", "coexec.h"))]
_DROP = ("#include <hip/hip_runtime.h>", "#include <hip/hip_runtime_api.h>", "#include <stddef.h>")


def _embed_headers() -> str:
    out = os.path.join(BUILD, "rt_embed.cpp")
    names, texts = [], []
    for name, path in RT_HEADERS:
        with open(path) as f:
            t = f.read().replace('#include "../../include/coexec.h"', '#include "coexec.h"')
        t = "\n".join(ln for ln in t.split("\n") if ln.strip() not in _DROP)
        if ")CE_RT_EMBED" in t:
            raise RuntimeError(f"{path} holds the embedding delimiter")
        names.append(f'"{name}"')
        texts.append('R"CE_RT_EMBED(' + t + ')CE_RT_EMBED"')
    src = ("// Generated by _build.py: device headers for runtime-compiled payloads.\n"
           "namespace ce {\n"
           f"extern const int kRtHeaderCount = {len(names)};\n"
           f"extern const char* const kRtHeaderNames[] = {{{', '.join(names)}}};\n"
           f"extern const char* const kRtHeaderTexts[] = {{\n{(',' + chr(10)).join(texts)}}};\n"
           "}  // namespace ce\n")
    with open(out, "w") as f:
        f.write(src)
    return out


def build(verbose: bool = False) -> str:
    os.makedirs(BUILD, exist_ok=True)
    objs = []
    for src in ("kernels.hip", "binomial_call.hip", "batch_kernels.hip", "serve_kernels.hip", "noalloc.hip"):
        o = os.path.join(BUILD, src + ".o")
        _run([HIPCC, *HIP_FLAGS, "-c", os.path.join(CSRC, src), "-o", o], verbose)
        objs.append(o)
    for src in ("host_payloads.cpp", "dma.cpp", "engine.cpp", "batch.cpp", "serve.cpp", "rt_module.cpp",
                _embed_headers()):
        o = os.path.join(BUILD, os.path.basename(src) + ".o")
        _run(["g++", *CXX_FLAGS, "-c", os.path.join(CSRC, src), "-o", o], verbose)
        objs.append(o)
    tmp = LIB + ".tmp"
    _run([HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", tmp, *objs, "-pthread", "-L" + os.path.join(ROCM, "lib"), "-lhsa-runtime64", "-lhiprtc",
          "-Wl,-soname,libcoexec.so", "-Wl,--no-undefined"], verbose)
    os.replace(tmp, LIB)
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
