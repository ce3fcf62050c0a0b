"""Builds liboomb.so (the C-ABI library, for gfx950 with hipcc) and _binding.so (the native half of the Python binding), in-tree."""
from __future__ import annotations

import os
import subprocess
import sys
import sysconfig

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
OUT = os.path.join(HERE, "liboomb.so")
BINDING = os.path.join(HERE, "_binding.so")
SOURCES = ["api.hip", "score_topk.hip", "vote_topk.hip", "kv_manager.hip", "page_pool.hip", "offload.hip", "check.hip", "attn_generic.hip", "kv_layout.hip", "qp_lists.hip", "attn_fwd_mfma.hip", "attn_bwd_mfma.hip", "attn_bwd_dkv_mfma.hip", "profile.hip", "calibrate.hip"]
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-ffp-contract=off",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-Wno-unused-command-line-argument", "-Wno-unknown-warning-option"]


def _binding_command(obj: str) -> list:
    """The binding holds no device code: plain C++ against Python and torch."""
    import torch
    from torch.utils.cpp_extension import include_paths
    inc = [f"-I{p}" for p in include_paths() + [sysconfig.get_paths()["include"]]]
    return ["g++", "-O2", "-std=c++17", "-fPIC", "-w", f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}", *inc,
            "-c", os.path.join(CSRC, "binding.cpp"), "-o", obj]


def _link_binding(obj: str) -> None:
    import torch
    lib = os.path.join(os.path.dirname(torch.__file__), "lib")
    subprocess.check_call(["g++", "-shared", "-o", BINDING, obj, f"-L{HERE}", "-l:liboomb.so", "-Wl,-rpath,$ORIGIN", f"-L{lib}", "-ltorch_python", "-ltorch_cpu",
                           "-lc10"])


def build(verbose: bool = False) -> str:
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    objs = []
    procs = []
    bdir = os.path.join(HERE, "_build")
    os.makedirs(bdir, exist_ok=True)
    binding = os.path.join(bdir, "binding.o")
    native = subprocess.Popen(_binding_command(binding), stdout=subprocess.PIPE, stderr=subprocess.STDOUT)
    for src in SOURCES:
        obj = os.path.join(bdir, src.replace(".hip", ".o"))
        cmd = [hipcc, *FLAGS, "-c", os.path.join(CSRC, src), "-o", obj]
        if verbose:
            print(" ".join(cmd), flush=True)
        procs.append((src, subprocess.Popen(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT)))
        objs.append(obj)
    for src, pr in procs:
        out, _ = pr.communicate()
        text = out.decode(errors="replace")
        # the host pass does not know the packed-fp32 feature name; that warning is harmless
        text = "\n".join(l for l in text.splitlines() if "packed-fp32-ops" not in l and l.strip())
        if pr.returncode != 0:
            raise RuntimeError(f"hipcc failed on {src}:\n{text}")
        if verbose and text:
            print(text, flush=True)
    subprocess.check_call([hipcc, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", OUT, *objs])
    out, _ = native.communicate()
    if native.returncode != 0:
        raise RuntimeError("g++ failed on binding.cpp:\n" + out.decode(errors="replace"))
    _link_binding(binding)
    return OUT


if __name__ == "__main__":
    print(build(verbose="-v" in sys.argv))
