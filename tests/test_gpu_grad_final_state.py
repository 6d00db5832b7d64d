"""vp_grad leaves the state and the acceleration of vp_run: the same bits in FP64 on
every kind of grid (one-launch gravity, one-pass drifts over two and three axes,
plane passes, single sweeps), FP32 rounding in FP32."""
import numpy as np
import pytest

from helpers import small_workload
from paper_1206_6152_amd import VP_BC_ISOLATED, VP_BC_PERIODIC, VP_F32, VP_F64, Simulator, config_of

pytestmark = pytest.mark.gpu

STEPS = 3
GRIDS = [((4, 4, 4), (16, 16, 16), VP_BC_PERIODIC), ((4, 6, 8), (12, 8, 6), VP_BC_ISOLATED),
         ((16, 16, 16), (8, 8, 8), VP_BC_PERIODIC), ((6, 4, 48), (16, 16, 16), VP_BC_PERIODIC),
         ((24, 12, 48), (8, 12, 8), VP_BC_PERIODIC), ((48, 6, 4), (8, 32, 12), VP_BC_ISOLATED),
         ((2, 16, 16), (24, 24, 24), VP_BC_PERIODIC), ((128, 1, 1), (32, 1, 1), VP_BC_PERIODIC)]


@pytest.mark.parametrize("dtype", [VP_F64, VP_F32])
@pytest.mark.parametrize("n,nv,bc", GRIDS)
def test_gradient_leaves_the_state_of_a_run(n, nv, bc, dtype):
    print("case", n, nv, bc, dtype, flush=True)
    import torch
    w = small_workload(bc, n=n, nv=nv)
    g = torch.Generator("cuda:0").manual_seed(11)
    f0 = torch.rand(w.shape, dtype=torch.float64, device="cuda:0", generator=g) + 0.1
    f0 *= torch.rand(w.n, dtype=torch.float64, device="cuda:0", generator=g).reshape(w.n + (1, 1, 1)) + 0.5
    f0 = f0.to(torch.float32 if dtype == VP_F32 else torch.float64)
    dt = 0.4 * min(w.dx(l) / max(abs(w.vmin[l]), abs(w.vmax[l])) for l in range(3))
    fa, fb = f0.clone(), f0.clone()
    a, b = Simulator(config_of(w, dtype), fa), Simulator(config_of(w, dtype), fb)
    a.grad(STEPS, dt, 2)
    b.run(STEPS, dt)
    da, db = a.get_accel(), b.get_accel()
    a.close(), b.close()
    if dtype == VP_F64:
        assert torch.equal(fa, fb) and torch.equal(da, db)
        return
    # a coefficient that rounds the other way moves a sweep's result by two units of
    # 2^-23 of the line's largest value at most; nine sweeps a step
    tol = STEPS * 9 * 2.0 ** -22
    assert float((fa - fb).abs().max()) <= tol * float(fb.max())
    assert float((da - db).abs().max()) <= 10 * tol * float(db.abs().max())
