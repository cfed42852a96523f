"""Builds libspecpv.so (HIP, gfx950) in-tree with hipcc, and the extension module of the binding with g++."""
import os
import subprocess
import sys
import sysconfig

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libspecpv.so")
NATIVE = os.path.join(HERE, "_native.so")
# the same library with time stamps inside the partial-verify attention kernel (timeline.py uses it)
LIB_TIMELINE = os.path.join(HERE, "libspecpv_timeline.so")
SOURCES = ["api.hip", "summarize.hip", "select.hip", "score_mfma.hip", "attn_generic.hip", "attn_f32.hip",
           "attn_mfma.hip", "attn_tile.hip", "combine.hip", "refresh_tail.hip", "commit.hip"]
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         # leading scalar kernel arguments arrive in registers instead of through a load
         "-mllvm", "-amdgpu-kernarg-preload-count=12",
         "-I" + os.path.join(ROOT, "include"), "-I" + CSRC]


def build(verbose=False, jobs=8, lib=LIB, defines=()):
    """Compile every HIP source to an object (in parallel) and link the shared library `lib`."""
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    extra = os.environ.get("SPECPV_EXTRA_HIPCC_FLAGS", "").split() + ["-D" + d for d in defines]
    objdir = os.path.join(HERE, "_build", os.path.basename(lib).replace(".so", ""))
    os.makedirs(objdir, exist_ok=True)
    procs = []
    objs = []
    for src in SOURCES:
        obj = os.path.join(objdir, src.replace(".hip", ".o"))
        objs.append(obj)
        cmd = [hipcc] + FLAGS + extra + ["-c", os.path.join(CSRC, src), "-o", obj]
        procs.append((src, subprocess.Popen(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)))
        while sum(p.poll() is None for _, p in procs) >= jobs:
            procs[0][1].wait() if procs[0][1].poll() is None else None
            for _, p in procs:
                if p.poll() is None:
                    p.wait()
                    break
    for src, p in procs:
        out, _ = p.communicate()
        # the host pass does not know the packed-fp32 target feature and says so: harmless
        out = "\n".join(l for l in out.splitlines() if "packed-fp32-ops" not in l)
        if p.returncode != 0:
            raise RuntimeError("hipcc failed on %s:\n%s" % (src, out))
        if verbose and out.strip():
            print(out)
    tmp = lib + ".tmp%d" % os.getpid()
    subprocess.run([hipcc, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", tmp] + objs, check=True)
    os.replace(tmp, lib)
    return lib


def build_native():
    """The extension module: host code against the C ABI's header, Python and torch."""
    import torch
    from torch.utils import cpp_extension
    root = os.path.dirname(torch.__file__)
    tmp = NATIVE + ".tmp%d" % os.getpid()
    cmd = ["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-D__HIP_PLATFORM_AMD__", "-DUSE_ROCM",
           "-D_GLIBCXX_USE_CXX11_ABI=%d" % int(torch._C._GLIBCXX_USE_CXX11_ABI), "-I" + os.path.join(ROOT, "include"),
           "-I" + sysconfig.get_paths()["include"]]
    cmd += ["-isystem" + p for p in cpp_extension.include_paths("cuda")]
    cmd += [os.path.join(CSRC, "binding_native.cpp"), "-o", tmp, "-L" + os.path.join(root, "lib"), "-ltorch_python", "-ltorch_cpu", "-lc10", "-lc10_hip"]
    p = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    if p.returncode != 0:
        raise RuntimeError("g++ failed on binding_native.cpp:\n" + p.stdout)
    os.replace(tmp, NATIVE)
    return NATIVE


def build_timeline(verbose=False):
    """The instrumented variant: same sources, -DSPECPV_TIMELINE, its own file name."""
    return build(verbose=verbose, lib=LIB_TIMELINE, defines=("SPECPV_TIMELINE",))


if __name__ == "__main__":
    if "--timeline" in sys.argv[1:]:
        print(build_timeline(verbose=True))
    else:
        print(build(verbose=True))
        print(build_native())
