"""Compile the HIP sources under csrc/ into paper_2305_11624_amd/libconvbn.so for gfx950, and the host code that hands
tensors to it into the CPython extension _call.so."""
import os
import subprocess
import sysconfig

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libconvbn.so")
CALL = os.path.join(HERE, "_call.so")
OBJDIR = os.path.join(HERE, "_build")   # objects and compiler temporaries stay out of the source folder
SOURCES = ["api.hip", "fold.hip", "fold_t.hip", "depthwise.hip", "conv_grouped.hip", "conv_grouped3.hip", "conv_direct.hip", "conv_igemm.hip", "conv_tile.hip", "conv_st.hip", "conv_rw.hip", "conv_pw.hip", "conv_gm.hip", "conv_stem.hip", "conv_wave.hip", "conv_win.hip", "wgrad_win.hip", "win_pair.hip", "wgrad_sq.hip", "aux_ops.hip"]
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-Wall", "-Wno-unused-function"]


def _call_command():
    from torch.utils import cpp_extension   # (paths only: nothing is compiled by it)
    inc = cpp_extension.include_paths() + [sysconfig.get_paths()["include"], "/opt/rocm/include"]
    libdirs = [os.path.join(os.path.dirname(p), "lib") for p in cpp_extension.include_paths() if os.path.basename(p) == "include"]
    import torch
    return (["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM",
             "-D_GLIBCXX_USE_CXX11_ABI=%d" % int(torch._C._GLIBCXX_USE_CXX11_ABI)]
            + ["-isystem" + i for i in inc] + [os.path.join(CSRC, "py_call.cpp"), "-o", CALL]
            + ["-L" + d for d in libdirs if os.path.isdir(d)] + ["-ltorch_python", "-ltorch_cpu", "-lc10", "-lc10_hip"])


def build(verbose: bool = False) -> str:
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    os.makedirs(OBJDIR, exist_ok=True)
    objs = []
    procs = []
    for src in SOURCES:
        obj = os.path.join(OBJDIR, src.replace(".hip", ".o"))
        objs.append(obj)
        cmd = [hipcc] + [f for f in FLAGS if f != "-shared"] + ["-c", os.path.join(CSRC, src), "-o", obj]
        procs.append((cmd, subprocess.Popen(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)))
    cmd = _call_command()
    procs.append((cmd, subprocess.Popen(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)))
    for cmd, p in procs:
        out, _ = p.communicate()
        # the host pass does not know the packed-fp32 target feature: that warning is harmless
        out = "\n".join(l for l in out.splitlines() if "packed-fp32-ops" not in l)
        if p.returncode != 0:
            raise RuntimeError("compiler failed: %s\n%s" % (" ".join(cmd), out))
        if verbose and out.strip():
            print(out)
    link = [hipcc, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB] + objs
    subprocess.run(link, check=True)
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
