"""Build the HIP library in-tree: ``paper_2209_09711_amd/libbat_hip.so``.

Steps: embed the headers with device code (``bat_device.hpp``,
``bat_cube.hpp``, ``bat_ms_cube.hpp``) as string literals (the source the
library hands to hiprtc for graph-specialised kernels) with a digest of the
ahead-of-time kernel sources, then compile the ahead-of-time kernels and the C ABI with hipcc for gfx950, and the compile
helper ``bat_jitc`` (a host program the library runs to compile several
graph-specialised kernels side by side) with the host compiler.
"""
from __future__ import annotations

import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
INCLUDE = os.path.join(ROOT, "include")
LIB = os.path.join(HERE, "libbat_hip.so")
JITC = os.path.join(HERE, "bat_jitc")
ARCH = os.environ.get("BAT_OFFLOAD_ARCH", "gfx950")

HIP_FLAGS = ["-O3", "-std=c++17", "-fPIC", f"--offload-arch={ARCH}",
             "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
             "-Wall", "-Wno-unused-function", "-Wno-unknown-pragmas"]


def embed_device_source() -> str:
    import hashlib
    delim = "BATDEV"
    srcs = {}
    for f in ("bat_device.hpp", "bat_cube.hpp", "bat_ms_cube.hpp"):
        srcs[f] = open(os.path.join(CSRC, f)).read()
        assert f"){delim}\"" not in srcs[f]
    # digest of everything the ahead-of-time kernels are compiled from,
    # reported in each launch's kernel identity
    h = hashlib.sha256()
    for f in ("bat_device.hpp", "bat_cube.hpp", "bat_kernels.hip", "bat_cube.hip", "bat_cube_batch.hip",
              "bat_ms_cube.hpp", "bat_launch.hpp", "bat_ms.hip"):
        with open(os.path.join(CSRC, f), "rb") as fh:
            h.update(fh.read())
    out = os.path.join(CSRC, "bat_device_embed.inc")
    text = ("// Generated by build.py from bat_device.hpp, bat_cube.hpp and\n"
            "// bat_ms_cube.hpp: the device templates as text, compiled at run time by\n"
            "// hiprtc for graph-specialised kernels.\n"
            f"static const char kDeviceSource[] = R\"{delim}(\n{srcs['bat_device.hpp']}\n){delim}\";\n"
            f"static const char kCubeSource[] = R\"{delim}(\n{srcs['bat_cube.hpp']}\n){delim}\";\n"
            f"static const char kMsCubeSource[] = R\"{delim}(\n{srcs['bat_ms_cube.hpp']}\n){delim}\";\n"
            f"static const char kAotKernelDigest[] = \"{h.hexdigest()[:32]}\";\n")
    if not os.path.exists(out) or open(out).read() != text:
        with open(out, "w") as f:
            f.write(text)
    return out


def build(verbose: bool = False) -> str:
    embed_device_source()
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    tmp = LIB + f".tmp{os.getpid()}"
    cmd = [hipcc, *HIP_FLAGS, "-shared", f"-I{INCLUDE}", f"-I{CSRC}",
           *(os.path.join(CSRC, f) for f in ("bat_kernels.hip", "bat_cube.hip", "bat_cube_batch.hip", "bat_ms.hip",
                                             "bat_host.cpp")),
           "-o", tmp, "-lhiprtc"]
    if verbose:
        print(" ".join(cmd), flush=True)
    r = subprocess.run(cmd, capture_output=True, text=True)
    msgs = [ln for ln in (r.stdout + r.stderr).splitlines()
            if "unknown target feature" not in ln and "packed-fp32-ops" not in ln
            and "argument unused during compilation" not in ln]
    if r.returncode != 0:
        sys.stderr.write("\n".join(msgs) + "\n")
        raise RuntimeError(f"hipcc failed ({r.returncode})")
    if verbose and msgs:
        print("\n".join(msgs))
    os.replace(tmp, LIB)
    build_jitc(verbose)
    return LIB


def build_jitc(verbose: bool = False) -> str:
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    tmp = JITC + f".tmp{os.getpid()}"
    cmd = [os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-D__HIP_PLATFORM_AMD__", f"-I{rocm}/include",
           os.path.join(CSRC, "bat_jitc.cpp"), "-o", tmp, "-ldl"]
    if verbose:
        print(" ".join(cmd), flush=True)
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        sys.stderr.write(r.stdout + r.stderr)
        raise RuntimeError(f"building bat_jitc failed ({r.returncode})")
    os.replace(tmp, JITC)
    return JITC


if __name__ == "__main__":
    print(build(verbose=True))
