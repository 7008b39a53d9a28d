"""Host tier: set-up calls whose host tables cannot be made, through the C entry
and before any device is reached: a limit on the address space that the tables do
not fit gives AIM_E_OOM, more near pairs than the row pointers count AIM_E_ARG; no
C++ exception leaves aim_setup.  Each in a process of its own."""
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
p, keep = aim.make_params(wl.circle({radius}, {n}), wl.K0, wl.ETA0, 0, {m}, 0.1, near_radius={near})
size = int([l for l in open('/proc/self/status') if l.startswith('VmSize')][0].split()[1]) * 1024
resource.setrlimit(resource.RLIMIT_AS, (size + {megabytes} * 2**20, resource.RLIM_INFINITY))
h = ctypes.c_void_p()
print(lib.aim_setup(ctypes.byref(p), ctypes.byref(h)), h.value)
"""


def _setup(**kw):
    r = subprocess.run([sys.executable, "-c", CODE.format(**kw)], capture_output=True, text=True, cwd=ROOT, timeout=300)
    assert r.returncode == 0, (r.returncode, r.stderr[-2000:])
    return r.stdout.split()


@pytest.mark.parametrize("megabytes", [64, 400, 1200])   # geometry, map weights, map points
def test_host_tables_that_do_not_fit(megabytes):
    assert _setup(radius=90.0, n=3000000, m=2048, near=3, megabytes=megabytes) == ["3", "None"]


def test_near_pairs_past_the_row_pointers():
    """46 341 bases inside one near zone: more than 2^31 - 1 pairs, refused before any list of them is made."""
    assert _setup(radius=0.45, n=46341, m=16, near=12, megabytes=4096) == ["1", "None"]
