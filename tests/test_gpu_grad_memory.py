"""vp_grad on a device with little memory left, in a process whose HIP
allocations have a budget (hip_memory_limit.c): one byte less than everything it
would like, exactly what it needs, and a byte less than that. In the first two it
does without its third work array, to the same bits; in the last it says so
before it touches f."""
import os
import shutil
import subprocess
import sys

import pytest

pytestmark = pytest.mark.gpu

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)

CHILD = r"""
import ctypes, re, sys
limit = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
import numpy as np, torch
runtime = set(re.findall(r"\S*/libamdhip64\S*", open("/proc/self/maps").read()))
assert len(runtime) == 1, runtime
assert limit.limit_open(runtime.pop().encode()) == 0      # before the first call that goes through it
limit.limit_asked.restype = ctypes.c_size_t
limit.limit_set.argtypes = [ctypes.c_size_t]
from helpers import small_workload, structured_f
from paper_1206_6152_amd import VP_BC_ISOLATED, VP_BC_PERIODIC, VP_F32, VP_F64, Simulator, VPError, _lib, config_of
CASES = [((4, 6, 8), (12, 8, 6), VP_F32, VP_BC_PERIODIC, 2), ((4, 6, 8), (12, 8, 6), VP_F64, VP_BC_ISOLATED, 2),
         ((4, 4, 4), (8, 8, 8), VP_F32, VP_BC_PERIODIC, 1), ((4, 4, 4), (16, 16, 16), VP_F64, VP_BC_PERIODIC, 3),
         ((2, 16, 16), (12, 24, 8), VP_F32, VP_BC_ISOLATED, 2), ((2, 2, 2), (48, 48, 48), VP_F32, VP_BC_PERIODIC, 4),
         ((16, 6, 24), (16, 8, 12), VP_F64, VP_BC_PERIODIC, 2)]
for n, nv, dtype, bc, ckpt in CASES:
    print("case", n, nv, dtype, bc, ckpt, flush=True)
    w = small_workload(bc, n=n, nv=nv)
    x = structured_f(w.shape, 9).astype(np.float32 if dtype == VP_F32 else np.float64) + 0.01
    fb = x.nbytes
    dt = 0.4 * min(w.dx(l) / max(abs(w.vmin[l]), abs(w.vmax[l])) for l in range(3))

    def grad(limit_bytes):
        f = torch.from_numpy(x).to("cuda:0")
        g = torch.full_like(f, float("nan"))
        sim = Simulator(config_of(w, dtype), f)
        torch.cuda.synchronize()
        limit.limit_off() if limit_bytes is None else limit.limit_set(limit_bytes)
        try:
            loss = _lib.vp_grad(sim.ctx, 3, dt, ckpt, g.data_ptr())
            asked, acc = limit.limit_asked(), sim.get_accel()
            return loss, g, f, acc, asked
        except VPError as e:
            assert e.code == _lib.VP_ENOMEM, e
            torch.cuda.synchronize()
            return None, None, f, None, None
        finally:
            limit.limit_off()
            sim.close()
    all_ = grad(None)
    assert torch.isfinite(all_[1]).all()
    for room in (all_[4] - 1, all_[4] - fb):
        lean = grad(room)
        assert lean[0] is not None, ("out of memory", all_[4] - room)
        assert lean[4] == all_[4] - fb              # without the third work array
        assert lean[0] == all_[0]
        for k in (1, 2, 3):
            assert torch.equal(lean[k], all_[k]), k
    none = grad(all_[4] - fb - 1)
    assert none[0] is None
    assert torch.equal(none[2].cpu(), torch.from_numpy(x))
print("done", flush=True)
"""


def test_gradient_with_little_memory(tmp_path):
    assert shutil.which("gcc"), "gcc is needed to build the allocation budget"
    so = str(tmp_path / "limit.so")
    r = subprocess.run(["gcc", "-shared", "-fPIC", "-O1", os.path.join(HERE, "hip_memory_limit.c"), "-o", so, "-ldl"],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    env = dict(os.environ, PYTHONPATH=os.pathsep.join([ROOT, HERE]))
    r = subprocess.run([sys.executable, "-u", "-c", CHILD, so], capture_output=True, text=True, env=env, cwd=ROOT,
                       timeout=100)
    print(r.stdout)
    assert r.returncode == 0, r.stderr
    assert r.stdout.endswith("done\n")
