"""The small systems' loop against the host-sized path in mixed precision.

Both form acceleration and jerk in FP64; they differ by the grouping of the
snap's FP32 partial sums (other lanes per particle), 1e-7 of the sum S of its
terms.  A step turns that into h^3 / 120 of it in velocity, so a time T into at
most T h^2 S / 120 x 1e-7; the step criterion keeps h^2 S of the order of the
acceleration, below 50 in these softened spheres: 3e-9 in velocity over 1/16,
a sixteenth of that in position, times ten for the growth of differences in
close encounters over that time.
"""
import numpy as np
import pytest

import ics
from gpu_helpers import cpu, log_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [33, 257, 1000, 2049, 4096])
def test_small_loop_mixed_rounding(n):
    from paper_1207_2367_amd import System
    m, x, v = ics.plummer(n, 300 + n)
    runs = []
    for loop in (0, n):
        log_case(test="small_loop_rounding", n=n, loop=loop)
        s = System(m, x, v, 0.01)
        s.set_step_loop(loop)
        s.step(1 / 16)
        runs.append({k: cpu(q) for k, q in s.get_state().items()})
        s.close()
    dx, dv = (np.abs(runs[0][k] - runs[1][k]).max() for k in ("x", "v"))
    print(f"n={n}: max difference of positions {dx:.1e}, velocities {dv:.1e}")
    assert dx <= 2e-9 and dv <= 3e-8
