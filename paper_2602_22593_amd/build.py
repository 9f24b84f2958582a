"""Build libflyingkv.so (HIP, gfx950 only) in-tree with hipcc, and the binding's _calls module with the C compiler.

``python -m paper_2602_22593_amd.build`` compiles every ``csrc/*.hip`` into an object under
``_build/`` and links them into ``paper_2602_22593_amd/libflyingkv.so``.  hipcc cross-compiles
without a GPU, so this runs on a CPU-only machine too.  The _calls module belongs to the interpreter that runs the build (its
headers and file suffix); where it cannot be compiled the library still is, and the binding does without it.
"""
from __future__ import annotations

import concurrent.futures as cf
import glob
import os
import subprocess
import sys
import sysconfig

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
OBJ_DIR = os.path.join(ROOT, "_build")
LIB = os.path.join(PKG, "libflyingkv.so")
CALLS = os.path.join(PKG, "_calls" + sysconfig.get_config_var("EXT_SUFFIX"))

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-Wall", "-Wno-unused-function",
    # packed fp32 VALU forms are kept off for all device code of this library
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-I", os.path.join(ROOT, "include"), "-I", CSRC,
]


def sources():
    return sorted(glob.glob(os.path.join(CSRC, "*.hip")))


def _compile(src: str, force: bool) -> str:
    obj = os.path.join(OBJ_DIR, os.path.basename(src).replace(".hip", ".o"))
    deps = [src] + glob.glob(os.path.join(CSRC, "*.h")) + glob.glob(os.path.join(ROOT, "include", "*.h"))
    if not force and os.path.exists(obj) and all(os.path.getmtime(obj) >= os.path.getmtime(d) for d in deps):
        return obj
    cmd = [HIPCC] + FLAGS + ["-c", src, "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    noise = "is not a recognized feature for this target"
    err = "\n".join(x for x in r.stderr.splitlines() if noise not in x and x.strip())
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed for {src}:\n{err}")
    if err:
        sys.stderr.write(err + "\n")
    return obj


def _build_calls(force: bool) -> None:
    untagged = os.path.join(PKG, "_calls.so")   # of an earlier build: any interpreter would load it
    if os.path.exists(untagged):
        os.remove(untagged)
    src, header = os.path.join(CSRC, "binding_calls.c"), os.path.join(ROOT, "include", "flying_kv.h")
    if not force and os.path.exists(CALLS) and all(os.path.getmtime(CALLS) >= os.path.getmtime(d) for d in (src, header)):
        return
    cmd = [os.environ.get("CC", "gcc"), "-O2", "-Wall", "-shared", "-fPIC", "-I", sysconfig.get_paths()["include"],
           "-I", os.path.join(ROOT, "include"), src, "-o", CALLS]
    try:
        r = subprocess.run(cmd, capture_output=True, text=True)
        failed, said = r.returncode != 0, r.stderr.strip()
    except OSError as e:
        failed, said = True, str(e)
    if failed:
        if os.path.exists(CALLS):
            os.remove(CALLS)   # of older sources
        said = f"{src} not compiled, calls are marshalled in Python:\n{said}"
    if said:
        sys.stderr.write(said + "\n")


def ensure_built() -> None:
    """Build what is missing: everything without the library, the _calls module alone without that."""
    if not os.path.exists(LIB):
        build()
    elif not os.path.exists(CALLS):
        _build_calls(force=True)


def build(force: bool = True, verbose: bool = False) -> str:
    os.makedirs(OBJ_DIR, exist_ok=True)
    srcs = sources()
    with cf.ThreadPoolExecutor(max_workers=min(8, len(srcs))) as ex:
        objs = list(ex.map(lambda s: _compile(s, force), srcs))
    cmd = [HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB] + objs
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"link failed:\n{r.stderr}")
    _build_calls(force)
    if verbose:
        print(f"built {LIB} from {len(objs)} objects")
    return LIB


if __name__ == "__main__":
    build(force="--incremental" not in sys.argv, verbose=True)
