"""Infinities and NaN go where the method sends them and no further: an adjoint
that is not finite in one cell, against the cells that the oracle's reverse
sweep reaches from it; and a state with infinite, NaN and nearly overflowing
cells through the one-pass kick and drift, against the single sweeps."""
import numpy as np
import pytest

import oracle
from helpers import oracle_grid, rel_l1, small_workload
from paper_1206_6152_amd import VP_BC_ISOLATED, VP_BC_PERIODIC, VP_F32, VP_F64, Simulator, config_of

pytestmark = pytest.mark.gpu

NP = {VP_F64: np.float64, VP_F32: np.float32}


def _dev(x):
    import torch
    return torch.from_numpy(np.ascontiguousarray(x)).to("cuda:0")


def _smooth(w, rng):
    """A bump along every axis: the line maxima are far from the first cells, and few corrector bounds act."""
    g = np.meshgrid(*[np.linspace(-1, 1, s) for s in w.shape], indexing="ij", sparse=True)
    return 0.2 + np.exp(-sum(x * x for x in g)) + 1e-3 * rng.uniform(0, 1, w.shape)


@pytest.mark.parametrize("bad", [np.inf, np.nan])
@pytest.mark.parametrize("dtype", [VP_F64, VP_F32])
@pytest.mark.parametrize("bc", [VP_BC_PERIODIC, VP_BC_ISOLATED])
@pytest.mark.parametrize("axis", range(6))
def test_reverse_sweep_of_a_non_finite_adjoint(axis, bc, dtype, bad):
    print("case", axis, bc, dtype, bad, flush=True)
    import torch
    w = small_workload(bc, n=(8, 12, 8), nv=(12, 8, 16))
    rng = np.random.default_rng(70 + axis)
    f_in = _smooth(w, rng).astype(NP[dtype]).astype(np.float64)
    lam = rng.standard_normal(w.shape).astype(NP[dtype]).astype(np.float64)
    lam[(1,) * 6] = bad
    tau = 0.31 if axis >= 3 else 0.4 * w.dx(axis) / max(abs(w.vmin[axis]), abs(w.vmax[axis]))
    a = rng.uniform(-1, 1, (3,) + w.n) * 0.8 * np.array([w.dv(l) for l in range(3)]).reshape(3, 1, 1, 1) / tau
    ref, _ = oracle.sweep_vjp(oracle_grid(w), f_in, axis, tau, lam, a)
    sim = Simulator(config_of(w, dtype), _dev(f_in.astype(NP[dtype])))
    sim.set_accel(_dev(a))
    out = _dev(lam.astype(NP[dtype]))
    sim.sweep_adjoint(axis, tau, sim.f, out)
    out = out.cpu().numpy().astype(np.float64)
    sim.close()
    fine = np.isfinite(ref)
    assert 1 <= (~fine).sum() <= 4      # the cell, and those that its face fluxes read
    assert np.array_equal(np.isfinite(out), fine)
    assert rel_l1(out[fine], ref[fine]) <= (1e-12 if dtype == VP_F64 else 2e-5)


@pytest.mark.parametrize("dtype,nv", [(VP_F32, 8), (VP_F32, 24), (VP_F64, 8)])
def test_one_pass_reverse_kick_of_a_non_finite_adjoint(dtype, nv):
    # the same cells, and the same bits elsewhere, as the three reverse sweeps
    print("case", dtype, nv, flush=True)
    import torch
    w = small_workload(VP_BC_PERIODIC, n=(2, 1, 2), nv=(nv,) * 3)
    rng = np.random.default_rng(nv)
    x = _smooth(w, rng).astype(NP[dtype])
    lam0 = rng.standard_normal(w.shape).astype(NP[dtype])
    lam0[0, 0, 1, 1, 2, 1] = np.inf
    tau = 0.27
    a = rng.uniform(-1, 1, (3,) + w.n) * 0.8 * np.array([w.dv(l) for l in range(3)]).reshape(3, 1, 1, 1) / tau
    g = _dev(x)
    sim = Simulator(config_of(w, dtype), g)
    sim.set_accel(_dev(a))
    sim.sweep(3, tau)
    in1 = g.clone()
    sim.sweep(4, tau)
    in2 = g.clone()
    lam_s, lam_f = _dev(lam0), _dev(lam0)
    for axis, at in ((5, in2), (4, in1), (3, _dev(x))):
        sim.sweep_adjoint(axis, tau, at, lam_s)
    sim.kick_adjoint(tau, _dev(x), lam_f)
    sim.close()
    fine = torch.isfinite(lam_s)
    assert 1 <= int((~fine).sum()) <= 64
    assert torch.equal(torch.isfinite(lam_f), fine)
    assert torch.equal(lam_f[fine], lam_s[fine])


@pytest.mark.parametrize("bad", [np.inf, -np.inf, np.nan, "max"])
@pytest.mark.parametrize("dtype", [VP_F64, VP_F32])
@pytest.mark.parametrize("bc", [VP_BC_PERIODIC, VP_BC_ISOLATED])
@pytest.mark.parametrize("n,nv", [((4, 1, 1), (6, 3, 4)), ((1, 4, 1), (4, 4, 4)), ((1, 1, 4), (3, 3, 3)),
                                  ((1, 1, 1), (12, 6, 8)), ((2, 3, 4), (8, 6, 4)), ((32, 1, 1), (64, 1, 1)),
                                  ((6, 24, 4), (8, 16, 12))])
def test_passes_of_a_non_finite_state(n, nv, bc, dtype, bad):
    print("case", n, nv, bc, dtype, bad, flush=True)
    import torch
    w = small_workload(bc, n=n, nv=nv)
    f0 = np.random.default_rng(8).uniform(0.5, 1.0, w.shape).astype(NP[dtype])
    mid = tuple(s // 2 for s in w.shape)
    f0[mid] = np.finfo(NP[dtype]).max if bad == "max" else bad
    tau = 0.23
    a = np.random.default_rng(5).uniform(-1, 1, (3,) + tuple(n)) * np.array([w.dv(l) for l in range(3)]).reshape(3, 1, 1, 1)
    t = 0.9 * min(w.dx(l) / max(abs(w.vmin[l]), abs(w.vmax[l])) for l in range(3))

    def bits(x):     # one pattern for every NaN
        x = torch.where(torch.isnan(x), torch.full_like(x, float("nan")), x)
        return x.view(torch.int64 if dtype == VP_F64 else torch.int32)
    for one_pass, axes, tt in (("kick", (3, 4, 5), tau), ("drift", (2, 1, 0), t)):
        f, g = _dev(f0), _dev(f0)
        one, split = Simulator(config_of(w, dtype), f), Simulator(config_of(w, dtype), g)
        for s in (one, split):
            s.set_accel(_dev(a / tau))
        getattr(one, one_pass)(tt)
        for axis in axes:
            split.sweep(axis, tt)
        one.close(), split.close()
        assert torch.equal(bits(f), bits(g)), one_pass
