"""Interpolation of batches split over blocks: every column of a batch equals the
product alone, bit for bit, for shares that divide the batch and that do not,
on the banded near field, the row-wise one (a hairpin, whose far arm is near)
and the per-node map (64 lanes per row), with and without near field."""
import math

import numpy as np
import pytest

from paper_2606_10784_amd import workloads as wl

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no HIP device", allow_module_level=True)

from paper_2606_10784_amd import aim  # noqa: E402

EPS = 0.1


def _hairpin(n):
    s = 2 * math.pi * np.arange(n) / n
    return np.stack([2.0 * np.cos(s), 0.1 * np.sin(s) + 0.037], axis=1)


CASES = {
    "band": (wl.circle(2.5, 3000), 64, 0),        # 192 blocks: shares of 1, 2, 5
    "rows": (_hairpin(1501), 64, 0),
    "nodes": (wl.circle(2.0, 801), 64, 6),
}


@pytest.mark.parametrize("nrhs", [2, 7, 37])
@pytest.mark.parametrize("basis", [0, 1])
@pytest.mark.parametrize("name", sorted(CASES))
def test_batch_columns_equal_single_products(name, basis, nrhs):
    xy, m, order = CASES[name]
    N = xy.shape[0]
    ctx = aim.Context(xy, wl.K0, wl.ETA0, basis, m, EPS, max_rhs=nrhs, node_order=order, max_restart=0)
    ctx.filter(wl.alpha_half_bins(EPS))
    g = torch.Generator(device="cuda")
    g.manual_seed(nrhs)
    x = torch.randn(nrhs, N, dtype=torch.complex128, device="cuda", generator=g)
    for op in (("S_ALPHA",) if order else ("S", "S_ALPHA")):
        y = ctx.matvec(op, x)
        for r in sorted({0, 1, nrhs // 2, nrhs - 1}):
            assert torch.equal(ctx.matvec(op, x[r:r + 1].contiguous()).reshape(-1), y[r]), (op, r)
    ctx.close()
