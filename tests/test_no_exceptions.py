"""No C++ exception leaves a C entry: a host allocation that fails is a status."""
import os
import subprocess
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

# a lattice of 2^24 - 4096 tiles, whose counts take 64 MiB of host memory, in a
# process that may have 16 MiB more than it has
PROGRAM = """
import ctypes, resource
import paper_2006_12838_amd._lib as L
status = L._lib.plic_curvature_status
cells, need = ctypes.c_int64(0), ctypes.c_size_t(0)
with open("/proc/self/statm") as f:
    size = int(f.read().split()[0]) * resource.getpagesize()
resource.setrlimit(resource.RLIMIT_AS, (size + (16 << 20), resource.RLIM_INFINITY))
rc = status(4096, 1 << 46, 64, 4 * 4095, 4 * 4096, 0, ctypes.byref(cells), ctypes.byref(need), None)
print("status", rc, L.plic_last_hip_error(), flush=True)
"""


def test_status_without_host_memory():
    r = subprocess.run([sys.executable, "-c", PROGRAM], cwd=ROOT, capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and r.stdout.split() == ["status", "-2", "2"], (r.returncode, r.stdout, r.stderr)
