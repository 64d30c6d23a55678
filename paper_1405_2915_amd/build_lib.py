"""Build libskel.so (HIP, gfx950) in-tree, and the CPU-only host-logic test
library used by the container-protocol tests.

    python -m paper_1405_2915_amd.build_lib [-v]

Every HIP source is compiled by hipcc for gfx950 only, with packed-FP32
instruction generation disabled.  The container protocol, the execution plan
and error reporting are plain C++ and are also compiled by g++, together with
a host-memory fake of the copy backend, into libskel_hosttest.so.
"""
from __future__ import annotations

import concurrent.futures as cf
import os
import subprocess
import sys
import sysconfig

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
INC = os.path.join(ROOT, "include")
BUILD = os.path.join(PKG, "_build")
LIB = os.path.join(PKG, "libskel.so")
HOSTTEST_LIB = os.path.join(PKG, "libskel_hosttest.so")

HIP_SOURCES = ["common.cpp", "container.cpp", "dispatch.cpp", "runtime.cpp", "chain_table.cpp",
               "skeletons.cpp", "k_map.hip", "k_reduce.hip", "k_scan.hip", "k_scan_rows.hip",
               "k_overlap.hip", "k_segments.hip", "k_grad.hip", "k_chain.hip"]
HOST_SOURCES = ["common.cpp", "container.cpp", "dispatch.cpp", "chain_table.cpp"]

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
HIP_FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
             "-Wall", "-Wno-unused-function",
             "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
             f"-I{INC}", f"-I{CSRC}"]


def _run(cmd, verbose):
    if verbose:
        print(" ".join(cmd), flush=True)
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"command failed ({r.returncode}): {' '.join(cmd)}\n"
                           f"{r.stdout}\n{r.stderr}")
    if verbose and r.stderr.strip():
        print(r.stderr, flush=True)


def _compile(jobs_of, verbose, jobs: int = 8) -> None:
    """Compile (source, object, extra flags) triples side by side."""
    os.makedirs(BUILD, exist_ok=True)
    cmds = [[HIPCC] + HIP_FLAGS + flags + (["-x", "hip"] if src.endswith(".hip") else []) +
            ["-c", os.path.join(CSRC, src), "-o", obj] for src, obj, flags in jobs_of]
    with cf.ThreadPoolExecutor(max_workers=jobs) as ex:
        list(ex.map(lambda c: _run(c, verbose), cmds))


def _link(lib, objs, verbose) -> str:
    _run([HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", lib + ".tmp"] + objs, verbose)
    os.replace(lib + ".tmp", lib)
    return lib


def _objects():
    return {s: os.path.join(BUILD, s + ".o") for s in HIP_SOURCES}


def build_hip(verbose: bool = False, jobs: int = 8) -> str:
    _compile([(s, o, []) for s, o in _objects().items()], verbose, jobs)
    return _link(LIB, list(_objects().values()), verbose)


# named for this interpreter, so that one of another version does not load it
CALL_LIB = os.path.join(PKG, "_skelcall" + sysconfig.get_config_var("EXT_SUFFIX"))


def build_call(verbose: bool = False) -> str:
    """_skelcall: the Python binding's skeleton calls without ctypes."""
    tmp = CALL_LIB + ".tmp"
    _run(["g++", "-std=c++17", "-O2", "-fPIC", "-shared", "-Wall", f"-I{INC}",
          "-I" + sysconfig.get_paths()["include"], "-o", tmp,
          os.path.join(CSRC, "pycall.cpp")], verbose)
    os.replace(tmp, CALL_LIB)
    untagged = os.path.join(PKG, "_skelcall.so")
    if os.path.exists(untagged):  # of an older build; any interpreter would load it
        os.remove(untagged)
    return CALL_LIB


HOSTTEST_SAN_LIB = os.path.join(PKG, "libskel_hosttest_san.so")
# AddressSanitizer and UndefinedBehaviorSanitizer for the host-only builds
SANITIZE = ["-fsanitize=address,undefined", "-fno-omit-frame-pointer",
            "-fno-sanitize-recover=undefined"]


def build_hosttest(verbose: bool = False, sanitize: bool = False) -> str:
    srcs = [os.path.join(CSRC, s) for s in HOST_SOURCES]
    srcs.append(os.path.join(ROOT, "tests", "host", "fake_backend.cpp"))
    out = HOSTTEST_SAN_LIB if sanitize else HOSTTEST_LIB
    tmp = out + ".tmp"
    _run(["g++", "-std=c++17", "-O1", "-g", "-fPIC", "-shared", "-Wall"] +
         (SANITIZE if sanitize else []) + [f"-I{INC}", f"-I{CSRC}", "-o", tmp] + srcs, verbose)
    os.replace(tmp, out)
    return out


SCAN_STRESS_LIB = os.path.join(PKG, "libskel_scan_w2.so")


SCAN_STRESS_FLAGS = ["-DSKEL_SCAN_WAVES=2", "-DSKEL_FLAT_PATIENCE=1"]
SCAN_STRESS_OBJS = {s: os.path.join(BUILD, s + ".w2.o") for s in ("k_scan.hip", "k_scan_rows.hip")}


def build_scan_stress(verbose: bool = False) -> str:
    """libskel_scan_w2.so: the library with the scan tiles shrunk to two
    wavefronts (4096 elements for 4-byte inputs instead of 32768), eight times
    as many tiles and a deeper decoupled look-back, and with flat tiles that
    wait for one poll only before they compute the totals they miss, for the
    stress tests of both.  The other objects are those of the product build."""
    _compile([(s, o, SCAN_STRESS_FLAGS) for s, o in SCAN_STRESS_OBJS.items()], verbose)
    return _link(SCAN_STRESS_LIB, list({**_objects(), **SCAN_STRESS_OBJS}.values()), verbose)


def build(verbose: bool = False) -> None:
    # (the longest sources first; the stress build's beside the product's)
    todo = [(s, o, SCAN_STRESS_FLAGS) for s, o in SCAN_STRESS_OBJS.items()]
    todo += [(s, o, []) for s, o in _objects().items()]
    slow = ("k_scan.hip", "k_overlap.hip", "k_scan_rows.hip")
    todo.sort(key=lambda t: slow.index(t[0]) if t[0] in slow else len(slow))
    _compile(todo, verbose)
    _link(LIB, list(_objects().values()), verbose)
    _link(SCAN_STRESS_LIB, list({**_objects(), **SCAN_STRESS_OBJS}.values()), verbose)
    build_call(verbose)
    build_hosttest(verbose)


if __name__ == "__main__":
    if "--sanitize" in sys.argv:
        # the container protocol, plan and chain table (and the oracle) built
        # with the sanitizers; see sanitize_env() for running the CPU tests
        print(build_hosttest("-v" in sys.argv, sanitize=True))
        sys.path.insert(0, ROOT)
        from oracle import build as oracle_build
        print(oracle_build.build("-v" in sys.argv, sanitize=True))
    else:
        build(verbose="-v" in sys.argv)
        print(LIB)
