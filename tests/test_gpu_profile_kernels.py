"""Event timing of the pipeline kernels where small grids take the
anterpolation inside the forward row pass: each of the five kernels can be
timed by itself (one launch per product; sampled ones and the others between
them count alike), and a product gives the same bits whichever kernel is timed."""
import pytest

from paper_2606_10784_amd import workloads as wl

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no HIP device", allow_module_level=True)

from paper_2606_10784_amd import aim  # noqa: E402


@pytest.mark.parametrize("m,n", [(64, 500), (200, 900), (300, 900)])
def test_each_kernel_is_timed(m, n):
    ctx = aim.Context(wl.circle(0.04 * m, n), wl.K0, wl.ETA0, 0, m, 0.1, precision=aim.AIM_MIXED, max_restart=0)
    g = torch.Generator(device="cuda")
    g.manual_seed(m)
    x = torch.randn(n, dtype=torch.complex128, device="cuda", generator=g)
    for op in (aim.OPS["TM"], aim.OPS["TM"] | aim.AIM_OP_GRID_FP32):
        y = ctx.matvec(op, x)
        for kernel, every in [(k, e) for k in range(5) for e in (1, 2)]:
            aim.aim_profile_start(ctx, kernel, every)
            got = [ctx.matvec(op, x) for _ in range(3)]
            ms, samples, launches = aim.aim_profile_stop(ctx)
            print(f"m={m} kernel={kernel}: {1e3 * ms:.1f} us", flush=True)
            assert launches == 3 and samples == 3 - (every - 1) and ms > 0
            assert all(torch.equal(v, y) for v in got)
    ctx.close()
