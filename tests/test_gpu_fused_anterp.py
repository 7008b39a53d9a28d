"""The row pass that sums the anterpolation itself (few rows) gives the bits of
the separate kernels (many rows): a product alone against the same column of a
batch that is past the rule's limit, for FFT lengths 32 .. 512 (1024: never fused), pulses and
hats (one and three channels), FP64 and FP32 grids, filtered and not; contours
with few and with many (over 32) contributions per point, and with rows of
more points than one sweep of a block takes.  The column pass of
the single product takes one-wave blocks for FFT length 512, that of the batch
wide ones.  Equality is exact: the same terms in the same order."""
import math

import pytest

from paper_2606_10784_amd import workloads as wl

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no HIP device", allow_module_level=True)

from paper_2606_10784_amd import aim  # noqa: E402

EPS = 0.1


@pytest.mark.parametrize("m,n", [(16, 40), (32, 300), (50, 61), (100, 2500), (251, 1999), (300, 900), (512, 6001)])
@pytest.mark.parametrize("basis", [0, 1])
def test_single_equals_batch_column(m, n, basis):
    nrhs = max(2, min(128, 6000 // m))
    ctx = aim.Context(wl.circle(0.42 * (m - 1) * EPS, n), wl.K0, wl.ETA0, basis, m, EPS, max_rhs=nrhs,
                      precision=aim.AIM_MIXED, max_restart=0)
    ctx.filter(wl.alpha_half_bins(EPS))
    rows = ctx.info()["active_rows"]
    g = torch.Generator(device="cuda")
    g.manual_seed(m)
    x = torch.randn(nrhs, n, dtype=torch.complex128, device="cuda", generator=g)
    print(f"m={m} n={n} rows={rows} nrhs={nrhs}", flush=True)
    for op in (("S", "S_ALPHA") if basis == 0 else ("N", "S_ALPHA")):
        for q in (aim.OPS[op], aim.OPS[op] | aim.AIM_OP_GRID_FP32):
            y = ctx.matvec(q, x)
            for r in (0, nrhs - 1):
                assert torch.equal(ctx.matvec(q, x[r:r + 1].contiguous()).reshape(-1), y[r]), (op, q, r)
    ctx.close()
