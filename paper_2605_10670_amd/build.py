"""Compile the HIP sources under csrc/ into paper_2605_10670_amd/libeep.so for gfx950, and
native/marshal.cpp into the extension module that binding.py makes its per-step calls through."""
import glob
import os
import subprocess
import sysconfig

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
LIB = os.path.join(HERE, "libeep.so")
SOURCES = sorted(glob.glob(os.path.join(HERE, "csrc", "*.hip")) +
                 glob.glob(os.path.join(HERE, "csrc", "*.cpp")))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared",
    # packed fp32 instructions are kept out of the generated code
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    # The first 14 dwords of a kernel's arguments arrive in scalar registers instead of through
    # a load that every wavefront waits for; the kernels take what their first loads need first.
    # Measured on whole steps: 8 decode steps of 32 / 256 tokens 79.8 -> 78.9 / 165 -> 160.5 us.
    "-mllvm", "-amdgpu-kernarg-preload-count=14",
    "-Wall", "-Wno-unused-command-line-argument",
    "-I", os.path.join(ROOT, "include"), "-I", os.path.join(HERE, "csrc"),
]


# (with the interpreter's tag, so that no other one loads it)
MARSHAL = os.path.join(HERE, "_marshal" + sysconfig.get_config_var("EXT_SUFFIX"))


def _compile(cmd, out):
    """Run `cmd` with an output name of this process's own and move the result into place whole: another
    process may be about to load `out`, or be building it too."""
    own = f"{out}.{os.getpid()}.so"
    try:
        subprocess.run(cmd + ["-o", own], check=True)
        os.replace(own, out)
    finally:
        if os.path.exists(own):
            os.remove(own)
    return out


def build_marshal() -> str:
    return _compile([os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall", "-Wextra",
                     "-Wno-missing-field-initializers", "-I", sysconfig.get_path("include"),
                     os.path.join(HERE, "native", "marshal.cpp")], MARSHAL)


def build() -> str:
    _compile([HIPCC] + FLAGS + SOURCES, LIB)
    build_marshal()
    return LIB


if __name__ == "__main__":
    print(build())
