"""The column pass of n = 1024 from the active grid points (n = 2048 beside
it: the pass over transformed rows), at the
shapes where its row tasks and staging can go wrong: the smallest and largest
grid side of the FFT length, the tallest and widest active sets, one very
long row next to short ones (a half disc: up to 64 lanes per row), rows dense
enough for the transformed-row form (a flat ellipse), odd sizes, several
right-hand sides and three channels.  Against the oracle with the same
embedding, FP64 to 1e-12 and the FP32 grid to 1e-5 of max|y| (O(1e5) terms
per output in either order; FP32 rounding over log2 n stages)."""
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

EPS = 0.05
K = 2 * math.pi / (40 * EPS)     # 40 cells per wavelength: long segments stay under one wavelength


def _ellipse(rx, ry, n):
    t = 2 * math.pi * (np.arange(n) + 0.3) / n
    return np.stack([rx * EPS * np.cos(t), ry * EPS * np.sin(t)], axis=1)


def _half_disc(r, n_flat, n_arc):
    """A flat bottom edge of 2 r cells (a few very long grid rows) under a half circle."""
    flat = np.stack([np.linspace(-r, r, n_flat, endpoint=False), np.full(n_flat, -0.4 * r)], axis=1)
    t = math.pi * np.arange(n_arc) / n_arc
    arc = np.stack([r * np.cos(t), -0.4 * r + 0.9 * r * np.sin(t)], axis=1)
    return EPS * np.concatenate([flat, arc])


CASES = [
    ("n1024_min_side", 257, _ellipse(122, 118, 151), 0),
    ("n1024_max_side", 512, _ellipse(250, 252, 211), 0),
    ("n1024_half_disc", 401, _half_disc(190, 300, 61), 1),
    ("n1024_tall", 500, _ellipse(9, 245, 103), 1),
    ("n1024_dense_rows", 512, _ellipse(250, 4, 301), 0),
    ("n2048_min_side", 513, _ellipse(249, 90, 173), 1),
    ("n2048_max_side", 1024, _ellipse(507, 508, 301), 0),
    ("n2048_tall", 1000, _ellipse(9, 490, 203), 1),
    ("n2048_half_disc", 1023, _half_disc(500, 500, 101), 0),
    ("n2048_dense_rows", 1024, _ellipse(500, 4, 601), 0),
]


@pytest.mark.parametrize("m,xy,basis", [c[1:] for c in CASES], ids=[c[0] for c in CASES])
def test_column_pass_matches_oracle(m, xy, basis):
    N = xy.shape[0]
    print(f"column pass m={m} basis={basis} N={N}", flush=True)
    ctx = aim.Context(xy, K, wl.ETA0, basis, m, EPS, max_rhs=5, precision=aim.AIM_MIXED, max_restart=0)
    n = ctx.info()["n_pad"]
    rng = np.random.default_rng(m)
    x = rng.standard_normal((5, N)) + 1j * rng.standard_normal((5, N))
    # the grid product alone (no near field), with the whole spectrum and with half of its bins
    op = "S_ALPHA" if basis == 0 else "N_ALPHA"
    for alpha in (math.inf, wl.alpha_half_bins(EPS)):
        ctx.filter(alpha)
        orc = oaim.AimOracle(xy, K, wl.ETA0, basis, m, EPS, alpha=alpha, near=False, n=n)
        ref = orc.apply(op, x[:3].T).T
        for nrhs in (1, 3):
            xt = torch.from_numpy(np.ascontiguousarray(x[:nrhs])).cuda()
            y = ctx.matvec(op, xt).cpu().numpy()
            yf = ctx.matvec(aim.OPS[op] | aim.AIM_OP_GRID_FP32, xt).cpu().numpy()
            e64 = np.max(np.abs(y - ref[:nrhs])) / np.max(np.abs(ref))
            e32 = np.max(np.abs(yf - ref[:nrhs])) / np.max(np.abs(ref))
            print(op, alpha, nrhs, e64, e32, flush=True)
            assert e64 < 1e-12 and e32 < 1e-5
    # a column's result does not depend on the batch it is in
    xt = torch.from_numpy(x).cuda()
    full = ctx.matvec(op, xt)
    for r in range(5):
        one = ctx.matvec(op, xt[r:r + 1].contiguous())
        assert (full[r] - one[0]).abs().max().item() <= 1e-14 * full.abs().max().item()
    ctx.close()
