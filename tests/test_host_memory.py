"""Host memory that runs out inside an entry point comes back as OIM_E_NOMEM; no
C++ exception leaves the library (no GPU needed)."""
import os
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

CHILD = """
import ctypes, resource, sys
sys.path.insert(0, {root!r})
import numpy as np
from paper_2505_22631_amd import _lib
L = _lib.lib()
n = {n}
i = np.arange(n)
off = np.concatenate([np.arange(1, 33), -np.arange(1, 33)])
col = np.sort((i[:, None] + off) % n, axis=1).astype(np.int32).ravel()
rp = (64 * np.arange(n + 1)).astype(np.int64)
J = np.full(col.size, -1.5, np.float32)
ptr = lambda a: a.ctypes.data_as(ctypes.c_void_p)
h = ctypes.c_void_p()
for line in open("/proc/self/status"):
    if line.startswith("VmSize"):
        now = int(line.split()[1]) << 10
resource.setrlimit(resource.RLIMIT_AS, (now + ({room} << 20), resource.RLIM_INFINITY))
st = L.oim_problem_from_csr(n, col.size, ptr(rp), ptr(col), ptr(J), 0, ctypes.byref(h))
resource.setrlimit(resource.RLIMIT_AS, (resource.RLIM_INFINITY, resource.RLIM_INFINITY))
assert h.value is None
print(L.oim_status_str(st).decode(), L.oim_last_error().decode())
"""


# rooms (MiB) below the 98 MiB of the 8-byte entries (1.28e7 of them)
@pytest.mark.parametrize("room", [8, 64])
def test_creation_without_host_memory(room):
    code = CHILD.format(root=ROOT, n=200000, room=room)
    env = dict(os.environ, HIP_VISIBLE_DEVICES="", OMP_NUM_THREADS="1")
    r = subprocess.run([sys.executable, "-c", code], capture_output=True, text=True, env=env,
                       timeout=300)
    assert r.returncode == 0, r.stderr[-2000:]
    assert r.stdout.startswith("OIM_E_NOMEM host allocation failed"), r.stdout
