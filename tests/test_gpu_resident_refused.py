"""A cooperative launch that the runtime refuses: the solve goes on with three
launches per iteration.  A child process loads, before the library, a stand-in
for hipLaunchCooperativeKernel that answers hipErrorCooperativeLaunchTooLarge
(720) and launches nothing."""
import os
import subprocess
import sys

import pytest

from gpu_helpers import require_gpu

pytestmark = pytest.mark.gpu

STAND_IN = "int refused_calls = 0;\nint hipLaunchCooperativeKernel(void) { ++refused_calls; return 720; }\n"

CHILD = """
import ctypes, sys
shim = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
sys.path[:0] = [sys.argv[2], sys.argv[2] + "/tests"]
calls = lambda: ctypes.c_int.in_dll(shim, "refused_calls").value
import torch
from gpu_helpers import random_velocity, sheet, to_dev
from paper_2008_00409_amd import binding as B, meshgen as mg
for dtype in ("f16", "f64"):
    for batch in (False, True):
        c = mg.config_batch(seed=91, sizes=[13, 40, 9, 27]) if batch else sheet(43, 31, seed=5)
        ctx = B.Context.from_cloth(c)
        if batch:
            ctx.set_instances([r[0] for r in c.sheet_ranges] + [c.nv])
        v = to_dev(torch, random_velocity(c, 0.05, seed=2))
        b = ctx.cloth_assemble(to_dev(torch, c.x0), v, dtype)
        before = calls()
        dv, info = ctx.cloth_pcg_solve(b, tol=1e-7, precond="block")
        assert calls() == before + 1, "the stand-in was not called"
        again, info2 = ctx.cloth_pcg_solve(b, tol=1e-7, precond="block")
        assert calls() == before + 1, "the next solve tried again"
        ctx.set_option(B.PC_OPT_LDS_WINDOW, 0)      # three launches, asked for
        want, winfo = ctx.cloth_pcg_solve(b, tol=1e-7, precond="block")
        assert torch.equal(dv, want) and torch.equal(again, want) and info == info2 == winfo, (info, winfo)
        ctx.close()
print("CHILD_OK", calls())
"""


def test_refused_launch(tmp_path):
    require_gpu()
    src, lib = tmp_path / "stand_in.c", tmp_path / "stand_in.so"
    src.write_text(STAND_IN)
    subprocess.run(["gcc", "-shared", "-fPIC", str(src), "-o", str(lib)], check=True, timeout=60)
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    out = subprocess.run([sys.executable, "-c", CHILD, str(lib), root], capture_output=True, text=True, timeout=100)
    assert out.returncode == 0 and "CHILD_OK 4" in out.stdout, out.stdout + out.stderr
