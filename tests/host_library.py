"""The library built for the CPU: its own sources, compiled as plain C++ against
the HIP stand-in under tests/host, which runs the kernels lane by lane and stops
at an access outside an allocation or a resource.  Tests run it in a process of
their own (a stop ends the process)."""
import concurrent.futures as cf
import glob
import os
import subprocess
import sys

import pytest

TESTS = os.path.dirname(os.path.abspath(__file__))
HOST = os.path.join(TESTS, "host")
CSRC = os.path.join(os.path.dirname(TESTS), "paper_2407_18947_amd", "csrc")
CLANG = "/opt/rocm/llvm/bin/clang++"


def _cc(args):
    r = subprocess.run([CLANG] + args, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(r.stderr[-4000:])


@pytest.fixture(scope="session")
def host_library(tmp_path_factory):
    """Path of the shared library."""
    out = str(tmp_path_factory.mktemp("host_library"))
    srcs = sorted(glob.glob(os.path.join(CSRC, "*.cpp")) + glob.glob(os.path.join(CSRC, "*.hip"))
                  + glob.glob(os.path.join(HOST, "*.cpp")))
    objs = [os.path.join(out, os.path.basename(s) + ".o") for s in srcs]
    flags = ["-x", "c++", "-std=c++17", "-O2", "-fPIC", "-w", f"-I{HOST}", f"-I{CSRC}", "-c"]
    with cf.ThreadPoolExecutor(max_workers=min(8, len(srcs))) as ex:
        list(ex.map(lambda p: _cc(flags + [p[0], "-o", p[1]]), zip(srcs, objs)))
    lib = os.path.join(out, "librtcc3_host.so")
    _cc(["-shared", "-o", lib] + objs)
    return lib


def host_run(lib, name, *args, timeout=300):
    """Runs function `name` of host_runs.py on the library; its output, or a failure with it."""
    r = subprocess.run([sys.executable, os.path.join(TESTS, "host_runs.py"), lib, name] + [str(a) for a in args],
                       capture_output=True, text=True, timeout=timeout)
    assert r.returncode == 0, f"{name} {args}: exit {r.returncode}\n{r.stdout[-2000:]}{r.stderr[-2000:]}"
    return r.stdout
