"""Build step for the HIP library: compiles csrc/ for gfx950 into libfastseq_hip.so.

Every source is compiled with hipcc for gfx950 only.  Packed-fp32 VALU
instructions are disabled for device code (``-packed-fp32-ops``); the host
pass warns that it does not know that feature, which is harmless.

The CPython marshalling module (csrc/pyext.c, plain C) is then compiled with
gcc and linked against the library, and so is the tensor front end's native
half (csrc/torch_ext.cpp, C++ against the installed torch's headers).

``build(trace=True)`` (``--trace``) compiles every source with FS_TRACE=1: the
attention and selection kernels then write per-workgroup timelines to a
buffer set with fs_trace_set (for measurements of where a launch spends its
time; a plain ``build()`` restores the normal kernels).

``build(sanitize=True)`` (``python -m paper_2106_04718_amd.build --sanitize``)
instruments the host code of every source with AddressSanitizer and
UndefinedBehaviorSanitizer (``-Xarch_host``: device code is built as usual),
links the library against clang's shared sanitizer runtime and builds the
marshalling module with clang and the same sanitizers.  Such a build is for
CPU test runs only (tests/run_sanitized.sh); a plain ``build()`` restores the
normal library.
"""
import concurrent.futures
import os
import pathlib
import subprocess
import sysconfig

PKG = pathlib.Path(__file__).resolve().parent
ROOT = PKG.parent
CSRC = PKG / "csrc"
BUILD = PKG / "_build"
LIB = PKG / "libfastseq_hip.so"
EXT = PKG / ("_fastseq_ext" + sysconfig.get_config_var("EXT_SUFFIX"))
SOURCES = ["capi.cpp", "cross_attn.hip", "ngram_block.hip", "beam_select.hip", "cache_reorder.hip", "postproc.cpp"]  # pyext.c is built by build_ext
TORCH_EXT = PKG / ("_fastseq_torch" + sysconfig.get_config_var("EXT_SUFFIX"))
ARCH = "gfx950"

COMMON = ["-O3", "-std=c++17", "-fPIC", f"--offload-arch={ARCH}",
          "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
          # kernel arguments arrive preloaded in SGPRs: the first wave of a
          # workgroup skips one dependent scalar load before its first
          # address computation
          "-mllvm", "-amdgpu-kernarg-preload-count=16",
          "-Wall", "-Wno-unused-command-line-argument",
          f"-I{ROOT / 'include'}", f"-I{CSRC}"]


def hipcc() -> str:
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    return os.path.join(rocm, "bin", "hipcc")


# host-side sanitizer flags: every one behind -Xarch_host, so no device code
# is built with a sanitizer
SANITIZE_HOST = ["-Xarch_host", "-fsanitize=address", "-Xarch_host", "-fsanitize=undefined",
                 "-Xarch_host", "-fno-sanitize-recover=undefined", "-Xarch_host", "-fno-omit-frame-pointer"]
SANITIZE_LINK = ["-Xarch_host", "-fsanitize=address", "-Xarch_host", "-fsanitize=undefined",
                 "-Xarch_host", "-shared-libasan"]


def clang() -> str:
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    return os.path.join(rocm, "llvm", "bin", "clang")


def sanitizer_runtime() -> str:
    """Path of clang's shared AddressSanitizer runtime (to preload into python)."""
    return subprocess.run([clang(), "-print-file-name=libclang_rt.asan-x86_64.so"], check=True,
                          capture_output=True, text=True).stdout.strip()


# (source, defines) of every object: the attention kernels' instances, by far
# the longest to compile, are built in four parts side by side
OBJECTS = [(s, ()) for s in SOURCES] + [("cross_attn.hip", (f"-DFS_ATTN_PART={part}",)) for part in (1, 2, 3)]


def _compile(src: str, defines: tuple, verbose: bool, sanitize: bool = False, trace: bool = False) -> pathlib.Path:
    obj = BUILD / (src + "".join(d.replace("-D", ".").replace("=", "") for d in defines) + ".o")
    cmd = [hipcc(), *COMMON, *defines, *(SANITIZE_HOST if sanitize else []), *(["-DFS_TRACE=1"] if trace else []),
           "-x", "hip", "-c", str(CSRC / src), "-o", str(obj)]
    if verbose:
        print(" ".join(cmd), flush=True)
    r = subprocess.run(cmd, capture_output=True, text=True)
    noise = "'-packed-fp32-ops' is not a recognized feature"
    err = "\n".join(l for l in r.stderr.splitlines() if noise not in l)
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed for {src}:\n{err}")
    if err.strip() and verbose:
        print(err, flush=True)
    return obj


def build(verbose: bool = False, sanitize: bool = False, trace: bool = False) -> pathlib.Path:
    BUILD.mkdir(exist_ok=True)
    with concurrent.futures.ThreadPoolExecutor(max_workers=len(OBJECTS) + 1) as ex:
        front = ex.submit(compile_torch_ext, verbose)
        objs = list(ex.map(lambda o: _compile(*o, verbose, sanitize, trace), OBJECTS))
    tmp = str(LIB) + ".tmp"
    cmd = [hipcc(), "-shared", "-fPIC", f"--offload-arch={ARCH}", "-Wl,-soname,libfastseq_hip.so",
           *(SANITIZE_LINK if sanitize else []), *map(str, objs), "-o", tmp]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.run(cmd, check=True)
    os.replace(tmp, LIB)
    build_ext(verbose, sanitize)
    link_torch_ext(front.result(), verbose)
    return LIB


def build_ext(verbose: bool = False, sanitize: bool = False) -> pathlib.Path:
    """The CPython module that marshals arguments into the C ABI."""
    tmp = str(EXT) + ".tmp"
    cc = [clang(), "-fsanitize=address,undefined", "-fno-sanitize-recover=undefined", "-shared-libasan",
          "-fno-omit-frame-pointer"] if sanitize else ["gcc"]
    cmd = [*cc, "-std=c11", "-O2", "-fPIC", "-shared", "-Wall", "-Wextra", "-Werror",
           f"-I{sysconfig.get_paths()['include']}", f"-I{ROOT / 'include'}", str(CSRC / "pyext.c"),
           f"-L{PKG}", "-lfastseq_hip", "-Wl,-rpath,$ORIGIN", "-o", tmp]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.run(cmd, check=True)
    os.replace(tmp, EXT)
    return EXT


def compile_torch_ext(verbose: bool = False) -> pathlib.Path:
    """Object file of the tensor front end's native half (never sanitized: torch is not)."""
    import torch
    from torch.utils.cpp_extension import include_paths
    obj = BUILD / "torch_ext.o"
    cmd = ["g++", "-std=c++17", "-O2", "-fPIC", "-Wall", "-fvisibility=hidden",
           f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}",
           *(f"-isystem{p}" for p in include_paths()), f"-I{sysconfig.get_paths()['include']}",
           f"-I{ROOT / 'include'}", "-c", str(CSRC / "torch_ext.cpp"), "-o", str(obj)]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.run(cmd, check=True)
    return obj


def link_torch_ext(obj: pathlib.Path, verbose: bool = False) -> pathlib.Path:
    from torch.utils.cpp_extension import library_paths
    tmp = str(TORCH_EXT) + ".tmp"
    cmd = ["g++", "-shared", str(obj), f"-L{PKG}", "-lfastseq_hip", *(f"-L{p}" for p in library_paths()),
           "-ltorch_python", "-ltorch_cpu", "-lc10", "-Wl,-rpath,$ORIGIN", "-o", tmp]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.run(cmd, check=True)
    os.replace(tmp, TORCH_EXT)
    return TORCH_EXT


if __name__ == "__main__":
    import sys
    print(build(verbose=True, sanitize="--sanitize" in sys.argv[1:], trace="--trace" in sys.argv[1:]))
