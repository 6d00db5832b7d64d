"""One step of vp_grad against its reverse sweeps called one by one, bit for bit: the
seed from the final potential, the closing half kick's three reverse sweeps at their
forward states, the density adjoint, the drift's three and the opening half kick's
three. Covers the one-pass reverse half kick at the sizes that vp_kick_adjoint does
not offer (FP64 16^3 and 24^3, FP32 32^3), accelerations of both signs with
whole-cell shifts, and blocks without that pass."""
import math

import numpy as np
import pytest

from helpers import small_workload
from paper_1206_6152_amd import VP_BC_ISOLATED, VP_BC_PERIODIC, VP_F32, VP_F64, Simulator, config_of

pytestmark = pytest.mark.gpu

# FP32 on grids beyond the one-launch gravity solve, which FP32 gradients leave out
CASES = [(VP_F64, (2, 3, 2), (16,) * 3, VP_BC_PERIODIC), (VP_F64, (2, 3, 2), (24,) * 3, VP_BC_ISOLATED),
         (VP_F64, (3, 2, 1), (8,) * 3, VP_BC_PERIODIC), (VP_F64, (4, 3, 2), (12, 8, 6), VP_BC_ISOLATED),
         (VP_F32, (8, 8, 12), (32,) * 3, VP_BC_ISOLATED), (VP_F32, (16, 16, 24), (8,) * 3, VP_BC_PERIODIC),
         (VP_F32, (8, 8, 12), (24,) * 3, VP_BC_ISOLATED), (VP_F32, (16, 16, 24), (12, 8, 6), VP_BC_PERIODIC)]


@pytest.mark.parametrize("dtype,n,nv,bc", CASES)
def test_one_step_of_the_gradient_equals_its_reverse_sweeps(dtype, n, nv, bc):
    print("case", dtype, n, nv, bc, flush=True)
    import torch
    w = small_workload(bc, n=n, nv=nv)
    t = torch.float32 if dtype == VP_F32 else torch.float64
    gen = torch.Generator("cuda:0").manual_seed(math.prod(nv))
    x0 = torch.rand(w.shape, dtype=torch.float64, device="cuda:0", generator=gen)
    x0 = torch.where(x0 < 0.2, torch.zeros_like(x0), x0).to(t)
    dt = 0.9 * min(w.dx(l) / max(abs(w.vmin[l]), abs(w.vmax[l])) for l in range(3))
    h = 0.5 * dt
    scale = np.array([w.dv(l) for l in range(3)]).reshape(3, 1, 1, 1) * 2.3 / h
    a0 = torch.from_numpy(np.random.default_rng(3).uniform(-1, 1, (3,) + w.n) * scale).to("cuda:0")

    f = x0.clone()
    sim = Simulator(config_of(w, dtype), f)
    sim.set_accel(a0)
    loss, grad = sim.grad(1, dt, 1)
    a1 = sim.get_accel()
    sim.close()

    g = x0.clone()                       # the forward states, one sweep at a time
    sim = Simulator(config_of(w, dtype), g)
    sim.set_accel(a0)
    states = {}
    for k, (axis, tau) in enumerate([(3, h), (4, h), (5, h), (2, dt), (1, dt), (0, dt), (3, h), (4, h), (5, h)]):
        if k == 6:
            sim.set_accel(a1)
        states[k] = g.clone()
        sim.sweep(axis, tau)
    assert torch.equal(g, f)
    dx3 = math.prod(w.dx(l) for l in range(3))
    dv3 = math.prod(w.dv(l) for l in range(3))
    phi = sim.potential()[1:-1, 1:-1, 1:-1]
    lam = ((-(dx3 * dv3) * phi).to(t).reshape(w.n + (1, 1, 1)).expand(w.shape)).contiguous()
    la = torch.zeros((3,) + w.n, dtype=torch.float64, device="cuda:0")
    for k, axis in ((8, 5), (7, 4), (6, 3)):
        sim.sweep_adjoint(axis, h, states[k], lam, la)
    sim.accel_adjoint(la, lam)
    for k, axis in ((5, 0), (4, 1), (3, 2)):
        sim.sweep_adjoint(axis, dt, states[k], lam)
    sim.set_accel(a0)
    la.zero_()
    for k, axis in ((2, 5), (1, 4), (0, 3)):
        sim.sweep_adjoint(axis, h, states[k], lam, la)
    sim.accel_adjoint(la, lam)
    sim.close()
    assert torch.equal(lam, grad), float((lam - grad).abs().max() / grad.abs().max())
