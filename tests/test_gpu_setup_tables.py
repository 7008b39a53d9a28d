"""Set-up tables against the oracle's: the near pattern (every row's sorted
columns) and the active grid points (through a whole product), for contours
with many bases per cell, cells met again by a far part of the contour (a
hairpin whose arms lie two cells apart), bases spread wider than the near zone,
an odd grid side, the smallest near radius and a larger one.  Products to 1e-12
of max|y| (rounding only: the same formulas)."""
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


def _hairpin(n):
    # a thin ellipse: both arms run through the same cells
    s = 2 * math.pi * np.arange(n) / n
    return np.stack([2.0 * np.cos(s), 0.1 * np.sin(s) + 0.037], axis=1)


CASES = {
    "hairpin": (_hairpin(331), 57, 6),
    "dense": (wl.circle(0.9, 700), 33, 3),
    "sparse": (wl.circle(2.4, 60), 64, 3),
    "wide": (wl.circle(1.7, 150), 49, 9),
}


@pytest.mark.parametrize("basis", [0, 1])
@pytest.mark.parametrize("name", sorted(CASES))
def test_tables_match_oracle(name, basis):
    xy, m, radius = CASES[name]
    N = xy.shape[0]
    ctx = aim.Context(xy, wl.K0, wl.ETA0, basis, m, EPS, near_radius=radius, max_rhs=2)
    alpha = wl.alpha_half_bins(EPS)
    ctx.filter(alpha)
    n = ctx.info()["n_pad"]
    orc = oaim.AimOracle(xy, wl.K0, wl.ETA0, basis, m, EPS, near_radius=radius, alpha=alpha, n=n)
    for row in range(N):
        cols, _ = ctx.near_row("S", row)
        assert np.array_equal(cols, orc.near_sel_pairs[orc.near_sel_pairs[:, 0] == row, 1]), row
    x = wl.probe_vector(N, seed=3)
    for q in ("S", "S_ALPHA"):
        ref = orc.apply(q, x)
        y = ctx.matvec(q, torch.from_numpy(x).cuda()).cpu().numpy()
        err = np.max(np.abs(y - ref)) / np.max(np.abs(ref))
        print(f"{name} basis={basis} {q}: {err:.2e}", flush=True)
        assert err < 1e-12
    ctx.close()
