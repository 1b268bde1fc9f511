"""Compile the HIP library for gfx950 into paper_2305_13525_amd/libaxo.so, and beside it the extension module _calls where that can be built (in-tree)."""
import glob
import os
import subprocess
import sys
import sysconfig
import warnings

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libaxo.so")
# named for the interpreter whose headers it is built with, so that no other one loads it
CALLS = os.path.join(HERE, "_calls" + (sysconfig.get_config_var("EXT_SUFFIX") or ".so"))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-function",
]


def sources():
    # *.hip: device code and the launch API; *.cpp: host-only parts of the C ABI
    return sorted(glob.glob(os.path.join(CSRC, "*.hip"))) + sorted(glob.glob(os.path.join(CSRC, "*.cpp")))


def _run(cmd, verbose):
    if verbose:
        print(" ".join(cmd))
    r = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    out = "\n".join(l for l in r.stdout.splitlines() if "packed-fp32-ops" not in l)
    if r.returncode != 0:
        raise RuntimeError(f"{os.path.basename(cmd[0])} failed:\n" + out)
    if verbose and out.strip():
        print(out)


def build_calls(verbose: bool = False) -> bool:
    """The extension module.  Without a C compiler or Python's headers the package does without it: its functions are then the ctypes
    wrappers, which do the same and take 0.7-2 us longer per call."""
    new = CALLS + ".new"  # moved into place: a running process may have the old one mapped
    untagged = os.path.join(os.path.dirname(CALLS), "_calls.so")  # of older builds; any interpreter would load it
    if untagged != CALLS and os.path.exists(untagged):
        os.remove(untagged)
    try:
        _run([os.environ.get("CC", "gcc"), "-O2", "-std=c11", "-fPIC", "-shared", "-Wall", "-I" + sysconfig.get_paths()["include"],
              os.path.join(CSRC, "calls.c"), "-o", new], verbose)
    except (OSError, RuntimeError) as e:
        for path in (CALLS, new):  # an older one need not fit the library
            if os.path.exists(path):
                os.remove(path)
        warnings.warn(f"the extension module _calls was not built, calls go through ctypes: {e}")
        return False
    os.replace(new, CALLS)
    return True


def build(verbose: bool = False, extra=()) -> str:
    _run([HIPCC] + FLAGS + list(extra) + sources() + ["-o", LIB], verbose)
    build_calls(verbose)
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
    sys.exit(0)
