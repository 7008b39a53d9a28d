"""One GMRES cycle of r steps minimises the residual over the Krylov space: the
rotations of the Hessenberg columns (batches of up to eight, one lane each,
chains read four at a time) and the back substitution (columns read eight
steps ahead, blocks of 256, 512 and 768 threads) at the edges of those counts,
for one and three right-hand sides.  Reference: the least-squares problem on
an orthonormal basis of the same Krylov space, built here with two rounds of
Gram-Schmidt.  Residual norms to 1e-9 |b|: both are backward stable (rounding
times |A||x| / |b|, below 1e-11), a wrong rotation or row shows at once."""
import numpy as np
import pytest

from paper_2606_10784_amd import workloads as wl

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no HIP device", allow_module_level=True)

from paper_2606_10784_amd import aim  # noqa: E402


def _least_residuals(ctx, b, steps):
    V = [b / torch.linalg.vector_norm(b)]
    H = torch.zeros(steps + 1, steps, dtype=b.dtype, device=b.device)
    for j in range(steps):
        w = ctx.matvec("TM", V[j])
        Q = torch.stack(V)
        for _ in range(2):
            h = (Q.conj() * w).sum(1)
            w = w - (h[:, None] * Q).sum(0)
            H[:j + 1, j] += h
        H[j + 1, j] = torch.linalg.vector_norm(w)
        V.append(w / H[j + 1, j])
    H = H.cpu().numpy()
    beta = float(torch.linalg.vector_norm(b))
    out = {}
    for r in range(1, steps + 1):
        e = np.zeros(r + 1, complex)
        e[0] = 1.0
        Q, _ = np.linalg.qr(H[:r + 1, :r])
        out[r] = float(np.linalg.norm(e - Q @ (Q.conj().T @ e)))
    return out, beta


@pytest.mark.parametrize("nrhs,counts", [(1, [1, 2, 3, 4, 5, 7, 8, 9, 12, 16, 17, 25, 33]), (3, [1, 8, 13]),
                                         (1, [256, 257, 300, 513])])
def test_cycle_minimises_the_residual(nrhs, counts):
    rng = np.random.default_rng(12)
    eps, m = 0.1, 300
    xy = wl.random_star(rng, 6.0, 900)
    ctx = aim.Context(xy, wl.K0, wl.ETA0, 0, m, eps, max_rhs=nrhs, max_restart=max(counts))
    b = ctx.rhs_planewave([0.4 + 1.3 * r for r in range(nrhs)]).reshape(nrhs, -1)
    best = [_least_residuals(ctx, b[r], max(counts))[0] for r in range(nrhs)]
    for steps in counts:
        x, info = ctx.solve("TM", b, tol=1e-15, maxit=steps, restart=steps)
        res = b - ctx.matvec("TM", x.reshape(nrhs, -1)).reshape(nrhs, -1)
        for r in range(nrhs):
            rel = float(torch.linalg.vector_norm(res[r]) / torch.linalg.vector_norm(b[r]))
            print(f"steps={steps} rhs={r}: {rel:.3e} least {best[r][steps]:.3e} estimate {info[r]['resid_est']:.3e}", flush=True)
            assert abs(rel - best[r][steps]) < 1e-9
            assert abs(rel - info[r]["resid_est"]) < 1e-9
    ctx.close()
