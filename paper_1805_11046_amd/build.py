"""Builds libq8t.so (all HIP kernels + the C ABI) for gfx950 with hipcc, and _q8t_calls.so (its calls as functions of a Python
module over torch tensors) with g++, in-tree."""
import glob
import os
import subprocess
import sys
import sysconfig

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libq8t.so")
CALLS = os.path.join(HERE, "_q8t_calls.so")

# -ffp-contract=off: rounding decisions need one fp32 rounding per written operation.
# packed-fp32 ops are switched off for the device pass (the host pass does not know the feature).
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-ffp-contract=off", "-fno-fast-math",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-fPIC", "-I" + os.path.join(ROOT, "include"), "-I" + CSRC]


def sources():
    return sorted(glob.glob(os.path.join(CSRC, "*.hip")))


def _calls_commands():
    import torch
    root = os.path.dirname(torch.__file__)
    obj = os.path.join(HERE, "_build", "python_calls.o")
    inc = [os.path.join(ROOT, "include"), sysconfig.get_paths()["include"], os.path.join(root, "include"),
           os.path.join(root, "include", "torch", "csrc", "api", "include"), "/opt/rocm/include"]
    compile_ = ["g++", "-O2", "-std=c++17", "-fPIC", "-fvisibility=hidden", "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1",
                "-D_GLIBCXX_USE_CXX11_ABI=%d" % int(torch._C._GLIBCXX_USE_CXX11_ABI)] + ["-I" + i for i in inc]
    link = ["g++", "-shared", "-o", CALLS, obj, "-L" + os.path.join(root, "lib"), "-ltorch_python", "-ltorch", "-lc10", "-lc10_hip",
            "-L" + HERE, "-l:libq8t.so", "-Wl,-rpath,$ORIGIN"]
    return compile_ + ["-c", os.path.join(CSRC, "python_calls.cpp"), "-o", obj], link


def build(verbose=False):
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    objs = []
    procs = []
    os.makedirs(os.path.join(HERE, "_build"), exist_ok=True)
    for src in sources():
        obj = os.path.join(HERE, "_build", os.path.basename(src) + ".o")
        objs.append(obj)
        procs.append((src, subprocess.Popen([hipcc] + FLAGS + ["-c", src, "-o", obj],
                                            stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)))
    compile_, link = _calls_commands()
    procs.append((compile_[-3], subprocess.Popen(compile_, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)))
    for src, p in procs:
        out, _ = p.communicate()
        out = "\n".join(l for l in out.splitlines() if "packed-fp32-ops" not in l)
        if p.returncode != 0:
            raise RuntimeError("compiling %s failed:\n%s" % (src, out))
        if verbose and out.strip():
            print(out)
    r = subprocess.run([hipcc, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB] + objs,
                       stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    if r.returncode != 0:
        raise RuntimeError("link failed:\n" + r.stdout)
    r = subprocess.run(link, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    if r.returncode != 0:
        raise RuntimeError("link failed:\n" + r.stdout)
    return LIB


if __name__ == "__main__":
    print(build(verbose="-v" in sys.argv))
