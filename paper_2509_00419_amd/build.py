"""Builds liblvlm.so (the C-ABI library) in-tree with hipcc for gfx950, and the native side of the torch binding."""
from __future__ import annotations

import importlib.util
import os
import subprocess
import sys
import sysconfig

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB_PATH = os.path.join(HERE, "liblvlm.so")
BINDING_PATH = os.path.join(HERE, "_torch_binding.so")
SOURCES = ["api.hip", "score.hip", "merge.hip", "sim.hip", "kv.hip", "attn.hip", "prefill.hip", "scratch.hip", "probe.hip"]

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-fvisibility=hidden",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",   # no packed fp32 ALU forms
    "-Wno-unused-command-line-argument",
]


def binding_command(out: str = BINDING_PATH, flags: tuple = ("-O2",)) -> list:
    """The command that builds the native side of binding.py (host code only: torch tensors to the C ABI)."""
    torch_dir = os.path.dirname(importlib.util.find_spec("torch").origin)
    rocm = os.path.dirname(os.path.dirname(HIPCC))
    return [os.environ.get("CXX", "g++"), *flags, "-std=c++17", "-fPIC", "-shared", "-fvisibility=hidden",
            "-D__HIP_PLATFORM_AMD__", "-DUSE_ROCM",          # what the HIP and torch headers ask of a host compiler
            "-I" + os.path.join(torch_dir, "include"), "-I" + os.path.join(torch_dir, "include/torch/csrc/api/include"),
            "-I" + os.path.join(rocm, "include"), "-I" + sysconfig.get_paths()["include"],
            os.path.join(CSRC, "torch_binding.cpp"), "-o", out, "-L" + os.path.join(torch_dir, "lib"),
            "-lc10", "-lc10_hip", "-ltorch_cpu", "-ltorch_python"]


def build_library(verbose: bool = True) -> str:
    """Compiles every source, links the shared library and the torch binding; returns the library's path."""
    objs = []
    build_dir = os.path.join(HERE, "_build")
    os.makedirs(build_dir, exist_ok=True)
    procs = []
    for src in SOURCES:
        obj = os.path.join(build_dir, src.replace(".hip", ".o"))
        cmd = [HIPCC, *FLAGS, "-c", os.path.join(CSRC, src), "-o", obj]
        if verbose:
            print(" ".join(cmd), flush=True)
        procs.append((src, subprocess.Popen(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)))
        objs.append(obj)
    cmd = binding_command()
    if verbose:
        print(" ".join(cmd), flush=True)
    procs.append(("torch_binding.cpp", subprocess.Popen(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)))
    failed = False
    for src, p in procs:
        out, _ = p.communicate()
        out = "\n".join(l for l in out.splitlines() if "packed-fp32-ops" not in l and l.strip())
        if p.returncode != 0:
            failed = True
            print(f"[build] {src} FAILED\n{out}", file=sys.stderr)
        elif verbose and out:
            print(out)
    if failed:
        raise RuntimeError("the compiler failed")
    cmd = [HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB_PATH, *objs]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.run(cmd, check=True)
    return LIB_PATH


def build_host_sanitized(out_dir: str) -> tuple:
    """The same sources with the HOST side under the undefined-behaviour sanitizer in trap mode (no runtime library:
    undefined behaviour in the library's host code ends the process with an illegal-instruction signal).  The device
    code is compiled as always, at -O1.  Returns the paths of the library and of the torch binding written into out_dir."""
    os.makedirs(out_dir, exist_ok=True)
    flags = [f for f in FLAGS if f != "-O3"] + ["-O1", "-Xarch_host", "-fsanitize=undefined", "-Xarch_host",
                                                "-fsanitize-trap=undefined"]
    procs, objs = [], []
    for src in SOURCES:
        obj = os.path.join(out_dir, src.replace(".hip", ".o"))
        procs.append((src, subprocess.Popen([HIPCC, *flags, "-c", os.path.join(CSRC, src), "-o", obj],
                                            stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)))
        objs.append(obj)
    binding = os.path.join(out_dir, "_torch_binding.so")
    cmd = binding_command(binding, ("-O1", "-fsanitize=undefined", "-fno-sanitize=vptr", "-fsanitize-undefined-trap-on-error"))
    procs.append(("torch_binding.cpp", subprocess.Popen(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)))
    for src, p in procs:
        out, _ = p.communicate()
        if p.returncode != 0:
            raise RuntimeError(f"the compiler failed on {src}:\n{out}")
    lib = os.path.join(out_dir, "liblvlm_ubsan.so")
    subprocess.run([HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", lib, *objs], check=True)
    return lib, binding


if __name__ == "__main__":
    print(build_library())
