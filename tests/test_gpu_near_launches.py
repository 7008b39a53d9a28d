"""A near field of more than 2^28 entries (16 400 pulses inside one near zone):
the build's sixteen lanes per entry take more than the 2^32 work-items of one
launch.  The matrix is symmetric and entries (i, j), (j, i) come from different
launches: rows at the first and last entries and around entries 2^26 and 2^28
agree with each other to rounding (1e-12 of the largest entry, the tolerance of
the quadrature tests; the entry of two neighbours is far above it)."""
import numpy as np
import pytest

from paper_2606_10784_amd import workloads as wl

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no HIP device", allow_module_level=True)

from paper_2606_10784_amd import aim  # noqa: E402


def test_more_than_2_to_28_entries():
    N = 16400
    ctx = aim.Context(wl.circle(0.45, N), wl.K0, wl.ETA0, 0, 16, 0.1, near_radius=12, max_restart=0)
    assert ctx.info()["near_nnz_s"] == N * N > 2**28
    rows = [0, 1, 2, 2**26 // N - 1, 2**26 // N, 2**26 // N + 1, 2**28 // N - 1, 2**28 // N, 2**28 // N + 1, N - 2,
            N - 1]
    C = np.empty((len(rows), len(rows)), complex)
    for i, row in enumerate(rows):
        cols, vals = ctx.near_row("S", row)
        assert np.array_equal(cols, np.arange(N))
        C[i] = vals[rows]
    top = np.abs(C).max()
    print(f"largest {top:.3e} neighbours {abs(C[0, -1]):.3e} asymmetry {np.abs(C - C.T).max() / top:.2e}", flush=True)
    assert abs(C[0, -1]) > 0.1 * top
    assert np.abs(C - C.T).max() < 1e-12 * top
    ctx.close()
