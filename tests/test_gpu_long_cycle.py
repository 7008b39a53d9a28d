"""GMRES cycles longer than one back-substitution block of 256 rows (blocks of
256, 512, 768 and 1024 threads) on a contour where every one of them still ends
far from convergence, so that each row of y counts: the step count is the one
asked for, and the residual is the least one over the same Krylov space (on an
orthonormal basis built here with two rounds of Gram-Schmidt) to 1e-9 |b| (both
are backward stable: rounding times |A||x| / |b|, below 1e-11).  What the bound
can see is checked on the reference itself: y with its rows from 256, 512 or
768 on left out (at 257, 513 and 769 steps a single row) misses it by more
than ten bounds."""
import numpy as np
import pytest

from paper_2606_10784_amd import workloads as wl

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no HIP device", allow_module_level=True)

from paper_2606_10784_amd import aim  # noqa: E402

BOUND = 1e-9


def _hessenberg(ctx, b, steps):
    Q = torch.zeros(steps + 1, ctx.N, dtype=b.dtype, device=b.device)
    H = torch.zeros(steps + 1, steps, dtype=b.dtype, device=b.device)
    Q[0] = b / torch.linalg.vector_norm(b)
    for j in range(steps):
        w = ctx.matvec("TM", Q[j])
        for _ in range(2):
            h = (Q[:j + 1].conj() * w).sum(1)
            w = w - (h[:, None] * Q[:j + 1]).sum(0)
            H[:j + 1, j] += h
        H[j + 1, j] = torch.linalg.vector_norm(w)
        Q[j + 1] = w / H[j + 1, j]
    return H.cpu().numpy()


def test_every_row_of_long_cycles_counts():
    eps, counts = 0.2, [255, 256, 257, 511, 512, 513, 768, 769, 1000]
    xy = wl.irregular_polygon(np.random.default_rng(1), 60.0, 6000)
    ctx = aim.Context(xy, wl.K0, wl.ETA0, 0, wl.grid_side_for(xy, eps), eps, max_restart=max(counts))
    b = ctx.rhs_planewave(0.4)
    H = _hessenberg(ctx, b, max(counts))
    for steps in counts:
        e = np.zeros(steps + 1, complex)
        e[0] = 1.0
        Q, R = np.linalg.qr(H[:steps + 1, :steps])
        y = np.linalg.solve(R, Q.conj().T @ e)
        least = np.linalg.norm(e - H[:steps + 1, :steps] @ y)
        for rows in (256, 512, 768):
            if rows < steps:
                cut = np.linalg.norm(e - H[:steps + 1, :steps] @ np.where(np.arange(steps) < rows, y, 0))
                assert abs(cut - least) > 10 * BOUND
        x, info = ctx.solve("TM", b, tol=1e-15, maxit=steps, restart=steps)
        rel = float(torch.linalg.vector_norm(b - ctx.matvec("TM", x)) / torch.linalg.vector_norm(b))
        print(f"steps={steps}: {rel:.3e} least {least:.3e} estimate {info[0]['resid_est']:.3e}", flush=True)
        assert info[0]["iterations"] == steps
        assert abs(rel - least) < BOUND
        assert abs(rel - info[0]["resid_est"]) < BOUND
    ctx.close()
