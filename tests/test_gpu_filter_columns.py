"""Filtered products leave out the tiles past the largest kept |kx|, and where
few columns are left their row transforms are sums over the active points:
cutoffs at the edges of these rules (only kx = 0; the first tiles; around one
wave's 32 columns, n/32, n/16, n/8 and n/4; all but the last bin; every bin)
for n = 128, 1024 (pulses, hats) and 2048, after a product that filled the
whole tile set.  Columns of a batch equal the single product bit for bit.
Against the oracle with the same embedding: FP64 to 1e-12 and the FP32 grid
to 1e-5 of max|y| (rounding of the kept bins, white for the seeded probe)."""
import math

import numpy as np
import pytest

from oracle import aim as oaim
from paper_2606_10784_amd import workloads as wl

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no HIP device", allow_module_level=True)

from paper_2606_10784_amd import aim  # noqa: E402

EPS = 0.1


@pytest.mark.parametrize("m,basis", [(64, 0), (512, 0), (300, 1), (600, 0)])
def test_cutoffs_match_oracle(m, basis):
    a = 0.3 * (m - 1) * EPS
    xy = wl.circle(a, max(9, int(2 * math.pi * a / (2.0 * EPS)) | 1))
    N = xy.shape[0]
    ctx = aim.Context(xy, wl.K0, wl.ETA0, basis, m, EPS, max_rhs=6, precision=aim.AIM_MIXED, max_restart=0)
    n = ctx.info()["n_pad"]
    rng = np.random.default_rng(m)
    x = rng.standard_normal((6, N)) + 1j * rng.standard_normal((6, N))
    xt = torch.from_numpy(x).cuda()
    op = "S_ALPHA" if basis == 0 else "N_ALPHA"
    for K in sorted({0, 1, 2, 3, 5, 31, 32, n // 32, n // 16, n // 16 + 2, n // 8, n // 4, n // 4 + 1, n // 2 - 1, n // 2}):
        alpha = (K + 0.5) * 2 * math.pi / (n * EPS)
        ctx.filter(math.inf)
        for q in (op, aim.OPS[op] | aim.AIM_OP_GRID_FP32):
            ctx.matvec(q, xt)
        ctx.filter(alpha)
        orc = oaim.AimOracle(xy, wl.K0, wl.ETA0, basis, m, EPS, alpha=alpha, near=False, n=n)
        ref = orc.apply(op, x[:1].T).T
        y = ctx.matvec(op, xt).cpu().numpy()
        yf = ctx.matvec(aim.OPS[op] | aim.AIM_OP_GRID_FP32, xt).cpu().numpy()
        e64 = np.max(np.abs(y[:1] - ref)) / np.max(np.abs(ref))
        e32 = np.max(np.abs(yf[:1] - ref)) / np.max(np.abs(ref))
        print(f"m={m} n={n} K={K}: {e64:.2e} {e32:.2e}", flush=True)
        assert e64 < 1e-12 and e32 < 1e-5
        one = ctx.matvec(op, xt[5:6].contiguous()).cpu().numpy()
        assert np.array_equal(one[0], y[5])
    ctx.close()
