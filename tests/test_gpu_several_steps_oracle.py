"""Launches of several steps against the FP64 oracle, node by node on patches of
a lid-driven cavity, from the GPU's own state as the oracle's input: strips of
five steps (FP32 beyond the Infinity Cache) and four, tiles of four and three,
plain and with obstacles.  A call of n steps is one launch of n - 1 and one of
one (tests/test_launch_rules_cpu.py); with obstacles six are three, two and one."""
import numpy as np
import pytest
import torch

from helpers import oracle_for, rel_err
from paper_2108_08591_amd import cases as C
from paper_2108_08591_amd import mdf
from test_gpu_hbm_resident import TOL, _np

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("storage,N,n", [("f32", 1600, 6), ("f32", 1600, 5), ("f64", 1200, 5), ("f64", 1200, 4),
                                         ("f32", 1024, 5), ("f64", 200, 5), ("f32", 200, 4)])
@pytest.mark.parametrize("obstacles", [False, True])
def test_patches_of_a_cavity(storage, N, n, obstacles):
    spec = C.cavity_case(N=N, Re=1000.0)
    print(f"[gpu] several steps, oracle: {N}^2 {storage} n={n} obstacles={obstacles}", flush=True)
    P = 16
    patches = [(0, 0), (N - P, 0), (0, N - P), (N - P, N - P), (N // 2, N - P), (0, N // 3), (N - P, N // 2), (N // 4, 0),
               (N // 2, N // 2), (137 % (N - P), 151 % (N - P))]
    mask = None
    if obstacles:
        mask = np.zeros((N, N), np.uint8)
        for x0, y0 in patches:                 # a block and a single node in every patch
            mask[y0 + 5:y0 + 9, x0 + 4:x0 + 7] = 1
            mask[y0 + 12, x0 + 11] = 1
    s = mdf.Solver([spec], storage=storage, solid=[mask] if obstacles else None)
    s.set_launch(64, 4, 8, 2)
    s.step(200)
    f_t = s.populations()
    s.step(n)
    f_n = s.populations()
    for x0, y0 in patches:
        lo_x, hi_x, lo_y, hi_y = max(x0 - n, 0), min(x0 + P + n, N), max(y0 - n, 0), min(y0 + P + n, N)
        # sides inside the cavity get a wall too: what it does wrongly reaches n - 1 nodes in n steps
        sub = C.CaseSpec(C.D2Q5, (hi_x - lo_x, hi_y - lo_y), spec.s1, bc=(C.WALL,) * 4 + (C.PERIODIC,) * 2,
                         wall_u=spec.wall_velocity().copy())
        m = None if mask is None else np.ascontiguousarray(mask[lo_y:hi_y, lo_x:hi_x])
        o = oracle_for(sub, solid=m).set_populations(np.ascontiguousarray(_np(f_t[:, :, lo_y:hi_y, lo_x:hi_x])))
        o.run(n)
        iy, ix = slice(y0 - lo_y, y0 - lo_y + P), slice(x0 - lo_x, x0 - lo_x + P)
        ref, got = o.populations()[:, :, iy, ix], _np(f_n[:, :, y0:y0 + P, x0:x0 + P])
        fluid = np.ones((P, P), bool) if mask is None else mask[y0:y0 + P, x0:x0 + P] == 0
        assert rel_err(ref[..., fluid], got[..., fluid]) < TOL[storage], (x0, y0)
