"""Host tier: aim_setup under a limit on the address space that its host tables
do not fit returns AIM_E_OOM; no C++ exception leaves the C entry.  In a process
of its own (the limit stays with it); no device is reached."""
import os
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

CODE = """
import ctypes, resource
from paper_2606_10784_amd import aim
from paper_2606_10784_amd import workloads as wl
lib = aim._lib()
p, keep = aim.make_params(wl.circle(90.0, 3000000), wl.K0, wl.ETA0, 0, 2048, 0.1, near_radius=3)
size = int([l for l in open('/proc/self/status') if l.startswith('VmSize')][0].split()[1]) * 1024
resource.setrlimit(resource.RLIMIT_AS, (size + %d * 2**20, resource.RLIM_INFINITY))
h = ctypes.c_void_p()
print(lib.aim_setup(ctypes.byref(p), ctypes.byref(h)), h.value)
"""


@pytest.mark.parametrize("megabytes", [64, 400, 1200])   # geometry, map weights, map points
def test_host_tables_that_do_not_fit(megabytes):
    r = subprocess.run([sys.executable, "-c", CODE % megabytes], capture_output=True, text=True, cwd=ROOT, timeout=300)
    assert r.returncode == 0, (r.returncode, r.stderr[-2000:])
    assert r.stdout.split() == ["3", "None"], r.stdout
