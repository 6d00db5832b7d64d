"""The one-workgroup gravity solve (spatial grids whose transform grid fits the
LDS) against the oracle's direct-DFT solve: accelerations, potentials and the
transposed map, at the edges of its range: the largest grids of each of its two
sizes, rows of even and odd length, axes of one cell, lines in registers (up to
16 cells) and staged lines (longer). The bounds are those of the separate
transforms: the FP64 rounding of an O(log M) transform against a direct sum,
1e-12 of the largest potential, ten times that after the differences of the
gradient."""
import numpy as np
import pytest

import oracle
from helpers import oracle_grid, rel_l1, small_workload, structured_f
from paper_1206_6152_amd import VP_BC_ISOLATED, VP_BC_PERIODIC, VP_F64, Simulator, config_of

pytestmark = pytest.mark.gpu

CASES = [(VP_BC_PERIODIC, n) for n in
         [(1, 1, 1), (2, 1, 3), (8, 8, 8), (1, 1, 128), (128, 1, 4), (8, 8, 12), (16, 16, 16), (12, 24, 12),
          (3, 32, 48), (2, 16, 128), (1, 48, 96)]] + \
        [(VP_BC_ISOLATED, n) for n in [(1, 1, 1), (4, 4, 4), (1, 3, 2), (8, 8, 8), (2, 64, 1), (12, 6, 4), (4, 6, 24)]]


@pytest.mark.parametrize("bc,n", CASES)
def test_small_gravity_matches_oracle(bc, n):
    print("case", bc, n, flush=True)
    import torch
    w = small_workload(bc, n=n, nv=(2, 1, 2))
    f0 = structured_f(w.shape, 7) + 0.05
    rng = np.random.default_rng(9)
    f0 *= rng.uniform(0.5, 1.5, w.n).reshape(w.n + (1, 1, 1))
    g = oracle_grid(w)
    f = torch.from_numpy(f0).to("cuda:0")
    sim = Simulator(config_of(w, VP_F64), f)
    phi, acc = sim.potential().cpu().numpy(), sim.get_accel().cpu().numpy()
    la = rng.standard_normal((3,) + w.n)
    lam = torch.zeros(w.shape, dtype=torch.float64, device="cuda:0")
    sim.accel_adjoint(torch.from_numpy(la).to("cuda:0"), lam)
    sim.close()
    ref_phi, ref_a = oracle.potential(g, oracle.density(g, f0)), oracle.accel(g, f0)
    assert np.abs(phi - ref_phi).max() <= 1e-12 * max(np.abs(ref_phi).max(), 1e-300)
    assert np.abs(acc - ref_a).max() <= 1e-11 * max(np.abs(ref_phi).max() / min(w.dx(l) for l in range(3)), 1e-300)
    out = lam.cpu().numpy()
    if max(n) == 1:      # one cell: both ghosts of an axis hold the same value, and the map is zero
        assert not out.any()
        return
    ref_lam = oracle.accel_vjp(g, la)
    assert np.abs(out - ref_lam).max() <= 1e-11 * np.abs(ref_lam).max()
