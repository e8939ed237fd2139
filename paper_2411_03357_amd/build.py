"""Builds libpgcm.so (HIP kernels + C ABI) for gfx950 with hipcc, and the Python binding's native
marshalling with the host compiler, in-tree."""
import os
import shutil
import subprocess
import sysconfig

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libpgcm.so")
MARSHAL = os.path.join(HERE, "_marshal.so")
SOURCES = ["pgcm_kernels.hip", "pgcm_bitsliced.hip", "pgcm_host.hip", "pgcm_bounce.hip", "pgcm_pipe.hip",
           "pgcm_seq.cpp"]
HEADERS = ["pgcm_kernels.h", "pgcm_types.h", "pgcm_arrive.h", "pgcm_contexts.h", "pgcm_one_launch.h",
           "pgcm_spans.h", "pgcm_routes.h", "pgcm_host_ivs.h", "pgcm_bitsliced_gen.h",
           os.path.join("..", "..", "include", "pgcm.h"),
           os.path.join("..", "..", "include", "pgcm_seq.h"),
           os.path.join("..", "..", "include", "pgcm_bounce.h"),
           os.path.join("..", "..", "include", "pgcm_pipe.h")]

FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared", "-fvisibility=hidden",
    "-Wall", "-Wno-unused-command-line-argument",
    # keep the compiler from forming packed-FP32 instructions
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    # the leading kernel arguments come in registers instead of being loaded from host memory
    "-mllvm", "-amdgpu-kernarg-preload-count=14",
    # one lane's atomic stays one instruction, whose result is waited for where it is used
    "-mllvm", "-amdgpu-atomic-optimizer-strategy=None",
]


def hipcc() -> str:
    exe = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(exe):
        raise RuntimeError("hipcc not found")
    return exe


def is_stale() -> bool:
    if not os.path.exists(LIB) or not os.path.exists(MARSHAL):
        return True
    t = min(os.path.getmtime(LIB), os.path.getmtime(MARSHAL))
    deps = [os.path.join(CSRC, s) for s in SOURCES + HEADERS + ["marshal.cpp"]] + \
        [os.path.abspath(__file__)]
    return any(os.path.getmtime(d) > t for d in deps)


def build_marshal() -> None:
    cxx = shutil.which("g++") or shutil.which("c++")
    if cxx is None:
        raise RuntimeError("no host C++ compiler")
    tmp = MARSHAL + ".tmp%d" % os.getpid()
    proc = subprocess.run([cxx, "-O2", "-std=c++17", "-fPIC", "-shared", "-fvisibility=hidden",
                           "-Wall", "-I" + sysconfig.get_paths()["include"],
                           os.path.join(CSRC, "marshal.cpp"), "-o", tmp],
                          stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    if proc.returncode != 0:
        raise RuntimeError("compiling marshal.cpp failed:\n" + proc.stdout)
    os.replace(tmp, MARSHAL)


def build(force: bool = True, verbose: bool = False) -> str:
    if not force and not is_stale():
        return LIB
    tmp = LIB + ".tmp%d" % os.getpid()
    cmd = [hipcc()] + FLAGS + [os.path.join(CSRC, s) for s in SOURCES] + ["-o", tmp]
    if verbose:
        print(" ".join(cmd))
    proc = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    out = "\n".join(l for l in proc.stdout.splitlines() if "packed-fp32-ops" not in l)
    if proc.returncode != 0:
        raise RuntimeError("hipcc failed:\n" + out)
    if verbose and out.strip():
        print(out)
    os.replace(tmp, LIB)
    build_marshal()
    return LIB


if __name__ == "__main__":
    print(build(force=True, verbose=True))
