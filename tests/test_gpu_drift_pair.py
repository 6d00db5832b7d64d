"""Two position sweeps in one pass over tiles of the (y, x) or the (z, y) plane,
against the single sweeps, bit for bit: both planes, axes of unequal lengths,
lines that do not divide evenly among the lanes, 64- and 128-byte-row tiles, waves
whose velocity cells move both ways (12-cell vz rows), Courant numbers beyond one
cell, both directions and boundaries; and the density that the (y, x) pass's sums
give against the density pass (the same FP64 sums in another order)."""
import numpy as np
import pytest

from helpers import small_workload
from paper_1206_6152_amd import VP_BC_ISOLATED, VP_BC_PERIODIC, VP_F32, VP_F64, Simulator, config_of

pytestmark = pytest.mark.gpu

SHAPES = [((6, 4, 48), (16, 8, 16)), ((12, 16, 24), (16, 16, 12)), ((4, 64, 64), (8, 16, 12)),
          ((6, 64, 48), (8, 16, 12)), ((12, 48, 16), (16, 24, 12)),                            # y and x
          ((48, 6, 4), (8, 16, 12)), ((24, 24, 4), (16, 16, 12)), ((48, 8, 48), (8, 16, 12)),
          ((6, 6, 6), (32, 32, 12))]                                                           # z and y


@pytest.mark.parametrize("bc,mag", [(VP_BC_PERIODIC, 0.9), (VP_BC_PERIODIC, 2.3), (VP_BC_ISOLATED, 2.3)])
@pytest.mark.parametrize("dtype", [VP_F32, VP_F64])
@pytest.mark.parametrize("n,nv", SHAPES)
def test_pair_passes_equal_single_sweeps(n, nv, dtype, bc, mag):
    print("case", n, nv, dtype, bc, mag, flush=True)
    import torch
    w = small_workload(bc, n=n, nv=nv)
    t = torch.float32 if dtype == VP_F32 else torch.float64
    rng = torch.Generator("cuda:0").manual_seed(7)
    f = torch.rand(w.shape, dtype=t, device="cuda:0", generator=rng)
    f = torch.where(f < 0.3, torch.zeros_like(f), f ** 3)
    g = f.clone()
    one, split = Simulator(config_of(w, dtype), f), Simulator(config_of(w, dtype), g)
    tau = mag * min(w.dx(l) / max(abs(w.vmin[l]), abs(w.vmax[l])) for l in range(3))
    for tt in (tau, -tau):
        one.drift(tt)
        for axis in (2, 1, 0):
            split.sweep(axis, tt)
        assert torch.equal(f, g)
    # a step's density comes from the drift's sums: its acceleration against
    # that of the density pass over the same drifted state
    zero = torch.zeros((3,) + tuple(n), dtype=torch.float64, device="cuda:0")
    one.set_accel(zero)
    one.step(tau)
    for axis in (2, 1, 0):
        split.sweep(axis, tau)
    split.accel()
    want, got = split.get_accel(), one.get_accel()
    one.close(), split.close()
    assert float((got - want).abs().max()) <= 1e-12 * float(want.abs().max())
