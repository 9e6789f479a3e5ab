"""Builds libtaser.so (the C-ABI HIP library) for gfx950 with hipcc, and _binding.so (the native half of the Python
binding) against torch with g++, in-tree."""
import glob
import os
import subprocess
import sys
import sysconfig

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libtaser.so")
BINDING = os.path.join(HERE, "_binding.so")

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared", "-Wall", "-Wextra",
         "-Wno-unused-parameter", "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-I", os.path.join(ROOT, "include"), "-I", CSRC]


def sources():
    return sorted(glob.glob(os.path.join(CSRC, "*.hip")))


def binding_tag():
    """What a _binding.so has to be built for; it holds this text."""
    import torch
    return f"torch {torch.__version__}, Python {sys.version_info.major}.{sys.version_info.minor}"


def binding_fits():
    if not os.path.exists(BINDING):
        return False
    with open(BINDING, "rb") as f:
        return f"built for {binding_tag()}.".encode() in f.read()


def binding_command():
    from torch.utils import cpp_extension as torch_paths
    dirs = torch_paths.include_paths("cuda") + [sysconfig.get_paths()["include"]]
    libs = [p for p in torch_paths.library_paths("cuda") if os.path.isdir(p)]
    return (["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall", "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1",
             f'-DTASER_BINDING_TAG="{binding_tag()}"',
             "-I", os.path.join(ROOT, "include")] + [x for d in dirs for x in ("-isystem", d)] +
            ["-o", BINDING, os.path.join(CSRC, "binding.cpp")] + [x for d in libs for x in ("-L", d, "-Wl,-rpath," + d)] +
            ["-ltorch_python", "-ltorch", "-ltorch_cpu", "-lc10", "-lc10_hip"])


def build(verbose=False):
    commands = [[HIPCC] + FLAGS + ["-o", LIB] + sources(), binding_command()]
    running = []
    for cmd in commands:
        if verbose:
            print(" ".join(cmd), flush=True)
        running.append(subprocess.Popen(cmd))
    for cmd, p in zip(commands, running):
        if p.wait() != 0:
            for other in running:
                other.wait()
            raise subprocess.CalledProcessError(p.returncode, cmd)
    return LIB


def stale():
    if not (os.path.exists(LIB) and binding_fits()):
        return True
    t = min(os.path.getmtime(LIB), os.path.getmtime(BINDING))
    deps = sources() + [p for e in ("*.h", "*.cpp") for p in glob.glob(os.path.join(CSRC, e))] + glob.glob(os.path.join(ROOT, "include", "*.h"))
    return any(os.path.getmtime(d) > t for d in deps)


if __name__ == "__main__":
    build(verbose=True)
