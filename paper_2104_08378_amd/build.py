"""Build libsp24.so (hand-written HIP, gfx950 only) in-tree with hipcc, and the native half of the Python binding
(_sp24_host.so, host code only) with g++ against the installed torch.  Where torch or its headers are not installed that
half is left out: the library does not need it, and the binding's Python code does without.

    python -m paper_2104_08378_amd.build

The shared library lands next to this file so that it travels with the source
tree; nothing is installed.  There is one code path and one target: no CUDA
shims, no fallback.
"""
import os
import subprocess
import sys
import sysconfig

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libsp24.so")
HOST = os.path.join(HERE, "_sp24_host.so")      # native marshalling of the binding's calls (csrc/host_calls.cpp)
PROBE = os.path.join(HERE, "sp24_probe")        # stand-alone measurement of the chip's ceilings (csrc/probe.hip)
SOURCES = ["api.hip", "prune_compress.hip", "permute.hip", "permute_search.hip", "permute_search_columns.hip", "splitk.hip", "mm_simple.hip", "mm_ksplit.hip", "conv_narrow.hip", "mm_skinny.hip", "mm_stream.hip", "mm_tiled.hip", "mm_staged.hip",
           "mm_staged_f16.hip", "mm_staged_bf16.hip", "mm_staged_i8.hip", "mm_staged_f8.hip"] + [
    "mm_tiled_%s_%s.hip" % (i, o) for i, o in
    [("f16", "f32"), ("f16", "f16"), ("f16", "bf16"), ("bf16", "f32"), ("bf16", "f16"), ("bf16", "bf16"),
     ("i8", "i32"), ("i8", "i8"), ("i8", "f32"), ("i8", "f16"), ("i8", "bf16"), ("f8", "f32"), ("f8", "f16"), ("f8", "bf16")]]
FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-fno-gpu-rdc",
    # hipcc must not form packed-fp32 instructions by itself on this target
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    # -Winline-asm: a note for every transfer that sets m0, megabytes of them, which stall the compilers on their pipes
    "-Wall", "-Wno-unused-command-line-argument", "-Wno-inline-asm",
]


def host_flags():
    """(compile flags, link flags), or None without torch and its headers."""
    try:
        import torch
    except ImportError:
        return None
    root = os.path.dirname(torch.__file__)
    if not os.path.exists(os.path.join(root, "include", "torch", "csrc", "autograd", "python_variable.h")):
        return None
    compile_flags = ["-O2", "-std=c++17", "-fPIC", "-fvisibility=hidden", "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1",
                     f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}", f"-I{root}/include", f"-I{root}/include/torch/csrc/api/include",
                     "-I/opt/rocm/include", f"-I{sysconfig.get_paths()['include']}"]
    link_flags = [f"-L{HERE}", "-l:libsp24.so", f"-L{root}/lib", "-ltorch_python", "-ltorch", "-ltorch_cpu", "-lc10", "-lc10_hip", "-Wl,-rpath,$ORIGIN"]
    return compile_flags, link_flags


def build(verbose=False):
    objs = []
    procs = []
    for src in SOURCES:
        obj = os.path.join(CSRC, src.replace(".hip", ".o"))
        cmd = ["hipcc", *FLAGS, "-c", os.path.join(CSRC, src), "-o", obj]
        if verbose:
            print(" ".join(cmd))
        procs.append((src, subprocess.Popen(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)))
        objs.append(obj)
    probe_cmd = ["hipcc", *[f for f in FLAGS if f != "-fPIC"], os.path.join(CSRC, "probe.hip"), "-o", PROBE]
    procs.append(("probe.hip", subprocess.Popen(probe_cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)))
    host, host_obj = host_flags(), os.path.join(CSRC, "host_calls.o")
    if host:
        procs.append(("host_calls.cpp", subprocess.Popen(["g++", *host[0], "-c", os.path.join(CSRC, "host_calls.cpp"), "-o", host_obj],
                                                         stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)))
    failed = False
    for src, p in procs:
        out, _ = p.communicate()
        out = "\n".join(l for l in out.splitlines() if "is not a recognized feature for this target" not in l)
        if p.returncode != 0:
            failed = True
            print(f"compilation failed for {src}:\n{out}", file=sys.stderr)
        elif verbose and out.strip():
            print(out)
    if failed:
        raise RuntimeError("libsp24 build failed")
    subprocess.check_call(["hipcc", "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB, *objs])
    if host:
        subprocess.check_call(["g++", "-shared", "-o", HOST, host_obj, *host[1]])
    else:
        print("torch or its headers are missing: _sp24_host.so is not built", file=sys.stderr)
        if os.path.exists(HOST):
            os.remove(HOST)                       # of another torch
    return LIB


if __name__ == "__main__":
    print(build(verbose="-v" in sys.argv))
