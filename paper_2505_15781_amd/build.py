"""Compile the HIP library for gfx950 (cross-compiles without a GPU)."""
from concurrent.futures import ThreadPoolExecutor
import glob
import os
import subprocess
import sys
import sysconfig

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
OBJ_DIR = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "libdkv.so")
MARSHAL = os.path.join(HERE, "_marshal.so")      # CPython module of the binding (csrc/marshal.c)
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-Wno-unused-command-line-argument", "-Wno-inline-asm"]
NOISE = "packed-fp32-ops"      # the host pass does not know the device feature and says so


def sources():
    return sorted(glob.glob(os.path.join(CSRC, "*.hip")))


def _run(cmd, verbose):
    if verbose:
        print(" ".join(cmd), flush=True)
    res = subprocess.run(cmd, capture_output=True, text=True)
    err = "\n".join(l for l in res.stderr.splitlines() if NOISE not in l)
    if res.returncode != 0:
        raise RuntimeError("hipcc failed:\n" + err)
    if verbose and err.strip():
        print(err, file=sys.stderr)


def build(verbose=False, incremental=False):
    """Compiles every source (one hipcc process each, in parallel) and links the shared library.
    `incremental` skips sources older than their object file (for edit-compile loops; headers are not tracked)."""
    os.makedirs(OBJ_DIR, exist_ok=True)
    headers = glob.glob(os.path.join(CSRC, "*.h")) + glob.glob(os.path.join(HERE, "..", "include", "*.h"))
    newest_header = max(os.path.getmtime(h) for h in headers)
    jobs, objs = [], []
    for src in sources():
        obj = os.path.join(OBJ_DIR, os.path.basename(src)[:-4] + ".o")
        objs.append(obj)
        if incremental and os.path.exists(obj) and os.path.getmtime(obj) > max(os.path.getmtime(src), newest_header):
            continue
        jobs.append([HIPCC] + FLAGS + ["-c", src, "-o", obj])
    with ThreadPoolExecutor(max(1, min(8, len(jobs)))) as ex:
        list(ex.map(lambda c: _run(c, verbose), jobs))
    _run([HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC"] + objs + ["-o", LIB], verbose)
    # plain C by the same compiler; needs the Python headers, not the HIP runtime
    _run([HIPCC, "-no-hip-rt", "-x", "c", "-O2", "-shared", "-fPIC", "-Wall", "-I", sysconfig.get_paths()["include"],
          os.path.join(CSRC, "marshal.c"), "-o", MARSHAL], verbose)
    return LIB


if __name__ == "__main__":
    print(build(verbose="-q" not in sys.argv, incremental="--incremental" in sys.argv))
