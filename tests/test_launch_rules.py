"""Host tier: launch arithmetic of the library (csrc/aim_internal.h, built with
g++), checked on the CPU at the limits HIP sets."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("host") / "launch_rules")
    cmd = ["g++", "-std=c++17", "-O1", "-fsanitize=undefined", "-fno-sanitize-recover=all", "-D__HIP_PLATFORM_AMD__",
           "-I/opt/rocm/include", "-I" + os.path.join(ROOT, "include"),
           os.path.join(ROOT, "tests", "host", "launch_rules.cpp"), "-o", exe]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]

    def run(*args):
        out = subprocess.run([exe, *map(str, args)], capture_output=True, text=True, check=True).stdout
        return [[int(v) for v in line.split()] for line in out.splitlines()]
    return run


@pytest.mark.parametrize("nnz", [1, 8, 9, 2**26 - 1, 2**26, 2**26 + 1, 2**28 - 8, 2**28 - 1, 2**28, 2**28 + 1,
                                 16385**2, 2**31 - 1])
def test_near_build_launches(rules, nnz):
    """The launches take every near entry once (up to the 2^31 - 1 a CSR row
    pointer can count) and stay below the 2^32 work-items of a launch."""
    (lanes, block), *launches = rules("near", nnz)
    per = block // lanes
    end = 0
    for q0, blocks in launches:
        assert q0 == end
        assert 0 < blocks * block < 2**32
        end = q0 + blocks * per
    assert nnz <= end < nnz + per
