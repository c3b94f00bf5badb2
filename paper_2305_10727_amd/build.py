"""Builds libgpusq.so (hand-written HIP for gfx950) in-tree with hipcc.  `python -m paper_2305_10727_amd.build`."""
import os
import subprocess
import sys
import sysconfig

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libgpusq.so")
SOURCES = ["api.hip", "prep.hip", "int4.hip", "spgemm.hip", "fewrows.hip", "wide.hip", "mlp.hip", "patches.hip", "tile1_i8.hip", "tile1_f16.hip",
           "tile1_i8_ragged.hip", "tile1_f16_ragged.hip", "tile2.hip", "dense.hip"]
# Python's side of the binding: a host-only extension module beside the library (no GPU code, so the host compiler)
FASTCALL = os.path.join(HERE, "_fastcall" + sysconfig.get_config_var("EXT_SUFFIX"))
FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared", "-ffp-contract=off",
    # packed-fp32 instructions are kept out of the generated code: some of their forms give wrong results
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-value", "-Wno-inline-asm",
]


def _run(cmd, verbose):
    if verbose:
        print(" ".join(cmd), flush=True)
    res = subprocess.run(cmd, capture_output=True, text=True)
    # the host pass does not know the packed-fp32 target feature and says so; that line is noise
    err = "\n".join(l for l in res.stderr.splitlines() if "packed-fp32-ops" not in l)
    if res.returncode != 0:
        raise RuntimeError("hipcc failed:\n" + err)
    if verbose and err.strip():
        print(err, file=sys.stderr)


def _fastcall_command():
    """The extension module uses torch's C++ interface: its headers (as system headers), its ABI, its libraries by their own path."""
    import torch
    root = os.path.dirname(torch.__file__)
    libs = os.path.join(root, "lib")
    return ["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall", "-D_GLIBCXX_USE_CXX11_ABI=%d" % torch._C._GLIBCXX_USE_CXX11_ABI,
            "-I" + sysconfig.get_paths()["include"], "-isystem", os.path.join(root, "include"), "-isystem",
            os.path.join(root, "include", "torch", "csrc", "api", "include"), os.path.join(CSRC, "fastcall.cpp"), "-o", FASTCALL,
            "-L" + libs, "-Wl,-rpath," + libs, "-ltorch_python", "-ltorch_cpu", "-lc10"]


def build(verbose=False):
    """Compile every HIP source (one hipcc process each, side by side) and link paper_2305_10727_amd/libgpusq.so, and the
    extension module that calls it; always recompiles; raises on failure.  The objects live in a temporary directory, not in the tree."""
    import concurrent.futures
    import tempfile
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    compile_flags = [f for f in FLAGS if f != "-shared"]
    with tempfile.TemporaryDirectory(prefix="gpusq_build_") as tmp:
        objs = [os.path.join(tmp, s.replace(".hip", ".o")) for s in SOURCES]
        cmds = [[hipcc, *compile_flags, "-c", os.path.join(CSRC, s), "-o", o] for s, o in zip(SOURCES, objs)]
        cmds.append(_fastcall_command())
        with concurrent.futures.ThreadPoolExecutor(max_workers=min(len(cmds), os.cpu_count() or 1)) as pool:
            for f in [pool.submit(_run, c, verbose) for c in cmds]:
                f.result()
        _run([hipcc, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB, *objs], verbose)
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
