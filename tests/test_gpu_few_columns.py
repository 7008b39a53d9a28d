"""Filtered products at FFT lengths 256, 512, 1024, 2048 and 4096 with cutoffs
on both sides of the rule that sums few kept columns (3/5 of the FFTs' steps;
n / 16 pairs, which binds at n = 2048 with 8 points a row) and small ones,
through the one-wave column blocks (256, 512) and the split tiles (512, 4096):
every column of a batch of six (a whole block of four right-hand sides and a
partial one) and of three (single ones) equals its product alone bit for bit,
and the FFT convolution of the oracle's tables: FP64 to 1e-12, the FP32 grid to
1e-5 of max|y|."""
import math

import numpy as np
import pytest
import scipy.fft

from oracle import aim as oaim
from paper_2606_10784_amd import workloads as wl

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no HIP device", allow_module_level=True)

from paper_2606_10784_amd import aim  # noqa: E402

EPS = 0.1


@pytest.mark.parametrize("m,cells", [(120, 2.0), (250, 2.0), (400, 2.0), (600, 6.0), (1401, 2.0)])
def test_every_column(m, cells):
    a = 0.3 * (m - 1) * EPS
    xy = wl.circle(a, int(2 * math.pi * a / (cells * EPS)) | 1)
    N = xy.shape[0]
    ctx = aim.Context(xy, wl.K0, wl.ETA0, 0, m, EPS, max_rhs=6, precision=aim.AIM_MIXED, max_restart=0)
    inf = ctx.info()
    n = inf["n_pad"]
    orc = oaim.AimOracle(xy, wl.K0, wl.ETA0, 0, m, EPS, near=False, n=n)
    F = scipy.fft.fft2(oaim.circulant_kernel(orc.grid, orc.T), workers=16)
    W, iy, ix = orc.W["phi"], orc.Gidx["phi"] // m, orc.Gidx["phi"] % m
    q = np.fft.fftfreq(n, 1.0 / n)
    rng = np.random.default_rng(m)
    x = rng.standard_normal((6, N)) + 1j * rng.standard_normal((6, N))
    xt = torch.from_numpy(x).cuda()
    G = []
    for r in range(6):
        g = np.zeros((n, n), complex)
        np.add.at(g, (iy, ix), W * x[r][:, None])
        G.append(F * scipy.fft.fft2(g, workers=16))
    lim = int(0.6 * n * inf["active_rows"] / inf["n_active"])
    for K in sorted({16, 33, lim - 17, lim - 1, lim, lim + 5, lim + 17, n // 16, n // 16 + 17} & set(range(10, n // 2))):
        ctx.filter((K + 0.5) * 2 * math.pi / (n * EPS))
        keep = q[:, None] ** 2 + q[None, :] ** 2 <= (K + 0.5) ** 2
        ref = [(W * scipy.fft.ifft2(np.where(keep, G[r], 0), workers=16)[iy, ix]).sum(1) for r in range(6)]
        for op, tol in ((aim.OPS["S_ALPHA"], 1e-12), (aim.OPS["S_ALPHA"] | aim.AIM_OP_GRID_FP32, 1e-5)):
            y = ctx.matvec(op, xt)
            y3 = ctx.matvec(op, xt[3:].contiguous())
            for r in range(6):
                one = ctx.matvec(op, xt[r].contiguous())
                assert torch.equal(one, y[r]), (K, op, r)
                assert r < 3 or torch.equal(one, y3[r - 3]), (K, op, r)
                e = np.max(np.abs(one.cpu().numpy() - ref[r])) / np.max(np.abs(ref[r]))
                assert e < tol, (K, op, r, e)
        print(f"m={m} n={n} K={K} limit={lim}: last column {e:.1e}", flush=True)
    ctx.close()
