"""Builds in-tree: the HIP library (hipcc --offload-arch=gfx950 -> csrc/../lib/libwinograd_mi355x.so) and the CPython
extension that hands torch tensors to it (g++ -> lib/_winograd_torch.so)."""
import concurrent.futures
import glob
import os
import subprocess
import sysconfig

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
LIB_DIR = os.path.join(HERE, "lib")
OBJ_DIR = os.path.join(LIB_DIR, "obj")
LIB_PATH = os.path.join(LIB_DIR, "libwinograd_mi355x.so")
EXT_SOURCE = os.path.join(CSRC, "torch_binding.cpp")
EXT_PATH = os.path.join(LIB_DIR, "_winograd_torch.so")

HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    # keep matrix-core results in ordinary vector registers where they fit: the vector ALU reads
    # them right away (limb joins, output transform) and would otherwise pay one copy per register
    "-mllvm", "-amdgpu-mfma-vgpr-form=1",
    # a kernel's leading scalar arguments are in registers when a wave starts (WG_GEOMETRY_PARAMS)
    "-mllvm", "-amdgpu-kernarg-preload-count=16",
    "-Wall", "-Wno-unused-function",
]


def sources():
    return sorted(glob.glob(os.path.join(CSRC, "*.hip")))


def _headers():
    return glob.glob(os.path.join(CSRC, "*.h")) + glob.glob(os.path.join(ROOT, "include", "*.h"))


def _extension_commands(obj):
    """(compile, link) of the extension: host code only, against torch's headers and libraries."""
    import torch
    root = os.path.dirname(torch.__file__)
    include, libs = os.path.join(root, "include"), os.path.join(root, "lib")
    compile_cmd = [os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-fPIC", "-Wall", "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1",
                   "-D_GLIBCXX_USE_CXX11_ABI=%d" % int(torch._C._GLIBCXX_USE_CXX11_ABI),
                   "-I", os.path.join(ROOT, "include"), "-I", CSRC, "-isystem", include,
                   "-isystem", os.path.join(include, "torch", "csrc", "api", "include"), "-isystem", "/opt/rocm/include",
                   "-isystem", sysconfig.get_paths()["include"], "-c", EXT_SOURCE, "-o", obj]
    link_cmd = [os.environ.get("CXX", "g++"), "-shared", "-o", EXT_PATH, obj, "-L", LIB_DIR, "-lwinograd_mi355x", "-L", libs,
                "-ltorch_python", "-ltorch_hip", "-ltorch_cpu", "-lc10_hip", "-lc10", "-Wl,-rpath,$ORIGIN"]
    return compile_cmd, link_cmd


def _run(cmd):
    proc = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    out = "\n".join(l for l in proc.stdout.splitlines() if "is not a recognized feature for this target" not in l)
    if proc.returncode != 0:
        raise RuntimeError("build step failed: %s\n%s" % (" ".join(cmd), out))
    return out


def build(verbose=False, incremental=False, jobs=None):
    """Compile every HIP source for gfx950 (one object per source, in parallel) and link them into one shared
    library, then the extension.  Everything is recompiled unless `incremental` is set, in which case a source is skipped when its
    object is newer than it and than every header."""
    os.makedirs(OBJ_DIR, exist_ok=True)
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    newest_header = max(os.path.getmtime(h) for h in _headers())
    todo, objects = [], []
    for src in sources():
        obj = os.path.join(OBJ_DIR, os.path.basename(src)[:-4] + ".o")
        objects.append(obj)
        fresh = (incremental and os.path.exists(obj) and
                 os.path.getmtime(obj) > max(os.path.getmtime(src), newest_header))
        if not fresh:
            todo.append([hipcc] + HIPCC_FLAGS + ["-I", os.path.join(ROOT, "include"), "-I", CSRC, "-c", src, "-o", obj])
    ext_obj = os.path.join(OBJ_DIR, "torch_binding.o")
    ext_compile, ext_link = _extension_commands(ext_obj)
    if not (incremental and os.path.exists(ext_obj) and os.path.getmtime(ext_obj) > max(os.path.getmtime(EXT_SOURCE), newest_header)):
        todo.append(ext_compile)
    jobs = jobs or min(8, int(os.environ.get("MAX_JOBS", "8")), max(1, len(todo)))
    with concurrent.futures.ThreadPoolExecutor(max_workers=jobs) as pool:
        for cmd, out in zip(todo, pool.map(_run, todo)):
            if verbose:
                print(" ".join(cmd))
                if out.strip():
                    print(out)
    out = _run([hipcc, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB_PATH] + objects)
    out += _run(ext_link)
    if verbose and out.strip():
        print(out)
    return LIB_PATH


if __name__ == "__main__":
    import sys
    print(build(verbose=True, incremental="--incremental" in sys.argv))
