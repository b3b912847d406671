"""CPU-side checks of the C-ABI library: it is built, loads, and exports every
function that include/vie.h declares (no compute calls here)."""

import ctypes
import os
import re

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HEADER = os.path.join(ROOT, "include", "vie.h")
LIB = os.path.join(ROOT, "paper_2508_16471_amd", "libvie.so")


def _declared():
    src = open(HEADER).read()
    src = re.sub(r"/\*.*?\*/", "", src, flags=re.S)
    names = re.findall(r"^\s*(?:int64_t|int|void|const char)\s+\**\s*(\w+)\s*\(", src, flags=re.M)
    return sorted(set(names))


def test_header_declares_the_boundary_calls():
    names = _declared()
    for n in ("vie_setup", "vie_solve", "vie_farfield", "hom_g2", "vie_get_current",
              "vie_set_stream", "vie_destroy", "vie_strerror", "vie_matvec"):
        assert n in names


def test_library_exports_every_declared_symbol():
    assert os.path.exists(LIB), "run __graft_entry__.build() first"
    lib = ctypes.CDLL(LIB)
    missing = [n for n in _declared() if not hasattr(lib, n)]
    assert not missing, missing


def test_binding_names_match_header():
    from paper_2508_16471_amd import vie

    for n in _declared():
        assert hasattr(vie, n), n


CHILD = """
import ctypes, resource, sys
import numpy as np
from paper_2508_16471_amd import vie as V
eps = np.full((128, 128, 128), 2.0)
V.lib()
vm = int([l for l in open("/proc/self/status") if l.startswith("VmSize")][0].split()[1]) << 10
resource.setrlimit(resource.RLIMIT_AS, (vm + (24 << 20), resource.RLIM_INFINITY))
try:
    V.vie_rt_setup(eps, 0.05, (0, 0, 0), 6.28)
except V.VieError as e:
    print("code", e.code)
"""


def test_host_memory_that_runs_out_is_an_error_code():
    """The face data of 128^3 cells take 120 MB of host memory before any device
    call: with 24 MB left the entry point returns VIE_ENOMEM, nothing is thrown
    across the ABI (which would end the process)."""
    import subprocess
    import sys

    p = subprocess.run([sys.executable, "-c", CHILD], cwd=ROOT, capture_output=True, text=True,
                       timeout=300)
    assert p.returncode == 0 and p.stdout.split() == ["code", "-2"], (p.returncode, p.stdout,
                                                                      p.stderr[-500:])
