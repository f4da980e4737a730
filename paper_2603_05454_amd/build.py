"""Build liblsp.so (the C-ABI HIP library) for gfx950 and the native part of its Python binding, in-tree."""
import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "liblsp.so")
BINDING = os.path.join(HERE, "_binding.so")
SOURCES = ["lsp_common.hip", "lsp_confidence.hip", "lsp_commit.hip", "lsp_attn.hip",
           "lsp_attn_f32.hip", "lsp_attn_bf16.hip", "lsp_scattered.hip", "lsp_lm_head.hip"]
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-fno-gpu-rdc",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-I", os.path.join(ROOT, "include"), "-I", CSRC, "-Wall", "-Wno-unused-result"]


def binding_command():
    """The marshalling module is host code against torch's own headers (tensor layout, current stream)."""
    import sysconfig
    import torch
    from torch.utils.cpp_extension import include_paths
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    incs = [os.path.join(ROOT, "include"), *include_paths(), os.path.join(rocm, "include"), sysconfig.get_paths()["include"]]
    libs = os.path.join(os.path.dirname(torch.__file__), "lib")
    return [os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall", "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1",
            f"-D_GLIBCXX_USE_CXX11_ABI={int(torch.compiled_with_cxx11_abi())}", *[x for i in incs for x in ("-isystem", i)],
            os.path.join(CSRC, "binding.cpp"), "-o", BINDING, "-L", libs, "-lc10", "-lc10_hip", "-ltorch_cpu", "-ltorch_python"]


def build(verbose: bool = False, jobs: int = 6) -> str:
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    # the hand-scheduled loops are generated (csrc/gen_attn_pipe.py -> csrc/lsp_attn_{pipe,pipe_idle,half,half_either,half_idle}_loop.inc;
    # csrc/gen_lm_head.py -> csrc/lsp_lm_head_loop_{256,128,64}.inc)
    for gen in ("gen_attn_pipe.py", "gen_lm_head.py"):
        subprocess.run([sys.executable, os.path.join(CSRC, gen)], check=True, stdout=subprocess.DEVNULL)
    objdir = os.path.join(HERE, "_build")
    os.makedirs(objdir, exist_ok=True)
    procs = []
    objs = []
    for src in SOURCES:
        obj = os.path.join(objdir, src.replace(".hip", ".o"))
        objs.append(obj)
        cmd = [hipcc, *FLAGS, "-c", os.path.join(CSRC, src), "-o", obj]
        if verbose:
            print(" ".join(cmd), flush=True)
        procs.append((src, subprocess.Popen(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)))
        while sum(p.poll() is None for _, p in procs) >= jobs:
            for _, p in procs:
                if p.poll() is None:
                    p.wait()
                    break
    procs.append(("binding.cpp", subprocess.Popen(binding_command(), stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)))
    for src, p in procs:
        out, _ = p.communicate()
        lines = [l for l in out.splitlines() if "packed-fp32-ops" not in l]
        if p.returncode != 0:
            raise RuntimeError(f"the compiler failed on {src}:\n" + "\n".join(lines))
        if verbose and lines:
            print("\n".join(lines))
    subprocess.run([hipcc, "--offload-arch=gfx950", "-shared", "-fPIC", *objs, "-o", LIB], check=True)
    return LIB


if __name__ == "__main__":
    print(build(verbose="-v" in sys.argv))
