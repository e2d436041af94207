"""The block-step loop of systems of at most 4096 bodies (active list built
and sources predicted by every workgroup itself) against the host-sized path.

Sizes at the edges of the sweep (256 next times per pass), of the source
tiles (256) and of the loop's range, and limits that hand larger blocks to
the host path and resume.  In FP64 the sums differ in their order only, so
the block steps, the N_act histogram and the interactions are the same; a
step's rounding (1e-16 of a coordinate of order 1) over at most a few hundred
steps of a softened system stays below 1e-12.  The other precisions round
jerk and snap to FP32 (6e-8): 1e-6.
"""
import numpy as np
import pytest

import ics
from gpu_helpers import cpu, log_case

pytestmark = pytest.mark.gpu

EPS = 0.01


def _run(n, prec, loop, span):
    from paper_1207_2367_amd import System
    m, x, v = ics.plummer(n, 300 + n)
    s = System(m, x, v, EPS, precision=prec)
    s.set_step_loop(loop)
    st = s.step(span)
    st2 = s.step(2 * span)
    return st, st2, {k: cpu(q) for k, q in s.get_state().items()}


@pytest.mark.parametrize("n", [2, 33, 255, 256, 257, 512, 513, 769, 1000, 2049, 3841, 4095, 4096,
                               4097])
@pytest.mark.parametrize("prec", [1, 0, 2], ids=["fp64", "mixed", "fp32pair"])
def test_small_loop_matches_host_path(n, prec):
    span = 1.0 / 32
    r1, r2, ref = _run(n, prec, 0, span)
    for lim in (n, 1, 33):
        log_case(test="small_loop", n=n, prec=prec, limit=lim)
        s1, s2, g = _run(n, prec, lim, span)
        assert np.all(g["t"] == 2 * span)
        if prec == 1:
            for a, b in ((s1, r1), (s2, r2)):
                for k in ("block_steps", "active_total", "interactions", "hist"):
                    assert a[k] == b[k], k
        tol = 1e-12 if prec == 1 else 1e-6
        assert np.abs(g["x"] - ref["x"]).max() < tol
        assert np.abs(g["v"] - ref["v"]).max() < 10 * tol
