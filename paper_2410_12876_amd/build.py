"""Compile the HIP sources under csrc/ into paper_2410_12876_amd/libag.so for gfx950, and the Python binding into _binding.so."""
import glob
import os
import subprocess
import sys
import sysconfig

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
LIB = os.path.join(HERE, "libag.so")
BINDING = os.path.join(HERE, "_binding.so")
BINDING_SOURCE = os.path.join(HERE, "csrc", "ag_binding.cpp")
SOURCES = sorted(glob.glob(os.path.join(HERE, "csrc", "*.hip")))
HEADERS = sorted(glob.glob(os.path.join(HERE, "csrc", "*.h"))) + sorted(glob.glob(os.path.join(ROOT, "include", "*.h")))

FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-fno-gpu-rdc",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-Wall", "-Wno-unused-command-line-argument",
         "-I" + os.path.join(ROOT, "include"), "-I" + os.path.join(HERE, "csrc")]
# Flags of single sources (none at present): {"file.hip": ["-mllvm", "-some-option"]}
FILE_FLAGS = {}
OBJ_DIR = os.path.join(HERE, "_build")


def stale() -> bool:
    if not os.path.exists(LIB) or not os.path.exists(BINDING):
        return True
    t = min(os.path.getmtime(LIB), os.path.getmtime(BINDING))
    return any(os.path.getmtime(f) > t for f in SOURCES + HEADERS + [BINDING_SOURCE])


def compile_binding(obj: str) -> str:
    """The host-only binding module: compiled against torch's headers, linked by build() against libag.so beside it."""
    import torch
    base = os.path.join(os.path.dirname(torch.__file__), "include")
    cmd = ["g++", "-O2", "-std=c++17", "-fPIC", "-Wall", "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1",
           "-D_GLIBCXX_USE_CXX11_ABI=%d" % int(torch._C._GLIBCXX_USE_CXX11_ABI),
           "-isystem", base, "-isystem", os.path.join(base, "torch", "csrc", "api", "include"), "-isystem", "/opt/rocm/include",
           "-isystem", sysconfig.get_paths()["include"], "-I" + os.path.join(ROOT, "include"), "-c", BINDING_SOURCE, "-o", obj]
    r = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    if r.returncode != 0:
        raise RuntimeError("g++ failed on ag_binding.cpp:\n" + r.stdout)
    return os.path.join(os.path.dirname(torch.__file__), "lib")


def link_binding(obj: str, torch_lib: str) -> None:
    cmd = ["g++", "-shared", obj, "-o", BINDING + ".tmp", "-L" + HERE, "-l:libag.so", "-L" + torch_lib, "-lc10", "-lc10_hip",
           "-ltorch_cpu", "-ltorch_python", "-Wl,-rpath,$ORIGIN", "-Wl,-rpath," + torch_lib]
    r = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    if r.returncode != 0:
        raise RuntimeError("link of _binding.so failed:\n" + r.stdout)
    os.replace(BINDING + ".tmp", BINDING)


def build(force: bool = True, verbose: bool = False) -> str:
    if not force and not stale():
        return LIB
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    extra = os.environ.get("AG_EXTRA_FLAGS", "").split()
    os.makedirs(OBJ_DIR, exist_ok=True)

    def compile_one(src):
        obj = os.path.join(OBJ_DIR, os.path.basename(src) + ".o")
        cmd = [hipcc] + FLAGS + extra + FILE_FLAGS.get(os.path.basename(src), []) + ["-c", src, "-o", obj]
        if verbose:
            print(" ".join(cmd), flush=True)
        r = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
        out = "\n".join(l for l in r.stdout.splitlines() if "not a recognized feature" not in l)
        if r.returncode != 0:
            raise RuntimeError("hipcc failed on %s:\n%s" % (os.path.basename(src), out))
        return obj, out

    from concurrent.futures import ThreadPoolExecutor
    with ThreadPoolExecutor(max_workers=8) as pool:   # one compiler process per source
        binding_obj = os.path.join(OBJ_DIR, "ag_binding.o")
        torch_lib = pool.submit(compile_binding, binding_obj)
        results = list(pool.map(compile_one, SOURCES))
        torch_lib = torch_lib.result()
    out = "\n".join(o for _, o in results if o.strip())
    cmd = [hipcc, "--offload-arch=gfx950", "-shared", "-fPIC", "-fno-gpu-rdc"] + [o for o, _ in results] + ["-o", LIB + ".tmp"]
    if verbose:
        print(" ".join(cmd), flush=True)
    r = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    if r.returncode != 0:
        raise RuntimeError("link failed:\n" + r.stdout)
    if verbose and out.strip():
        print(out)
    os.replace(LIB + ".tmp", LIB)
    link_binding(binding_obj, torch_lib)
    return LIB


if __name__ == "__main__":
    print(build(force="--if-stale" not in sys.argv, verbose=True))
