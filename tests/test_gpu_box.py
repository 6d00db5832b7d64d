"""The run-time-shaped one-pass kick and drift (velocity blocks and spatial grids
of any accepted axis lengths that fit on chip) against the single sweeps, bit for
bit: unequal axes, every line length up to 128, lines of one cell, velocity rows
that are not whole 16-byte vectors, last chunks narrower than the others, boxes
with few lines (each split over several lanes), Courant numbers beyond one cell
and both directions; and the density that the drift's sums give against the
density pass (the same FP64 sums in another order)."""
import numpy as np
import pytest

from helpers import small_workload, structured_f
from paper_1206_6152_amd import VP_BC_ISOLATED, VP_BC_PERIODIC, VP_F32, VP_F64, Simulator, config_of

pytestmark = pytest.mark.gpu

SHAPES = [((8, 8, 8), (16, 16, 16)), ((4, 6, 8), (12, 8, 6)), ((3, 2, 4), (6, 6, 6)), ((2, 3, 1), (3, 4, 2)),
          ((1, 1, 24), (24, 3, 32)), ((12, 12, 12), (6, 6, 6)), ((16, 12, 2), (8, 48, 4)), ((2, 32, 8), (12, 12, 64)),
          ((6, 1, 2), (96, 2, 128)), ((48, 2, 4), (1, 64, 3)), ((4, 4, 4), (24, 32, 8)), ((64, 1, 2), (2, 96, 16))]


@pytest.mark.parametrize("mag", [0.9, 2.3])
@pytest.mark.parametrize("bc", [VP_BC_PERIODIC, VP_BC_ISOLATED])
@pytest.mark.parametrize("dtype", [VP_F32, VP_F64])
@pytest.mark.parametrize("n,nv", SHAPES)
def test_box_passes_equal_single_sweeps(n, nv, dtype, bc, mag):
    print("case", n, nv, dtype, bc, mag, flush=True)
    import torch
    w = small_workload(bc, n=n, nv=nv)
    x = structured_f(w.shape, 3).astype(np.float32 if dtype == VP_F32 else np.float64)
    f = torch.from_numpy(x).to("cuda:0")
    g = f.clone()
    one, split = Simulator(config_of(w, dtype), f), Simulator(config_of(w, dtype), g)
    tau = 0.23
    scale = np.array([w.dv(l) for l in range(3)]).reshape(3, 1, 1, 1) * mag / tau
    a = torch.from_numpy(np.random.default_rng(5).uniform(-1, 1, (3,) + tuple(n)) * scale).to("cuda:0")
    for s in (one, split):
        s.set_accel(a)
    one.kick(tau)
    for axis in (3, 4, 5):
        split.sweep(axis, tau)
    assert torch.equal(f, g)
    t = mag * min(w.dx(l) / max(abs(w.vmin[l]), abs(w.vmax[l])) for l in range(3))
    for tt in (t, -t):
        one.drift(tt)
        for axis in (2, 1, 0):
            split.sweep(axis, tt)
        assert torch.equal(f, g)
    # a step's density comes from the drift's sums: its acceleration against
    # that of the density pass over the drifted state
    h = f.clone()
    one.step(t)
    ref = Simulator(config_of(w, dtype), h)
    ref.set_accel(a)
    ref.kick(0.5 * t)
    ref.drift(t)
    ref.accel()
    want, got = ref.get_accel(), one.get_accel()
    one.close(), split.close(), ref.close()
    assert float((got - want).abs().max()) <= 1e-12 * float(want.abs().max()) + 1e-300 or \
        float(want.abs().max()) <= 1e-12
