"""Host tier: launch arithmetic and dispatch rules of the library
(csrc/aim_internal.h, built with g++), checked on the CPU at their limits."""
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


@pytest.mark.parametrize("f32,limit", [(0, 768), (1, 1536)])
def test_timed_kernels_run_apart(rules, f32, limit):
    """The forward row pass takes the anterpolation along up to its limit of rows, except where one of the two is timed."""
    for n, rows, fused in ((128, limit, 1), (512, limit, 1), (512, limit + 1, 0), (1024, 8, 0)):
        assert rules("fused", n, f32, rows, 1, 0) == [[fused]]
        assert rules("fused", n, f32, rows, 1, 1) == [[0]]


def test_few_columns_rule(rules):
    """Sums over the kept columns only from n = 1024, up to n / 16 pairs and 3/5 of the FFTs' steps."""
    for n in (32, 256, 512):
        assert rules("few", n, 1, 10 * n, n) == [[0]]
    for n in (1024, 2048, 4096):
        assert rules("few", n, n // 16, 9 * n // 4, n // 4) == [[1]]        # 9 points a row: n / 16 binds
        assert rules("few", n, n // 16 + 1, 9 * n // 4, n // 4) == [[0]]
        assert rules("few", n, n // 25, 15 * n // 4, n // 4) == [[1]]       # 15 points a row: pk <= n / 25
        assert rules("few", n, n // 25 + 1, 15 * n // 4, n // 4) == [[0]]
    assert rules("few", 4096, 256, 2**20, 2048) == [[0]]                    # products past 32 bits
