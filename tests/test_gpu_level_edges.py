"""The schedule from per-level counts at the edges of its launches: systems
that leave the last workgroup of the compaction partly empty, and blocks on
both sides of the corrector size up to which the corrector's last workgroup
makes the next schedule (256 workgroups of 28 particles, or of 7 with 33 to
128 splits).  Against the sweep schedule on the same path: the same blocks and
the same bits, as no particle's evaluation or correction depends on its slot
in the active list."""
import numpy as np
import pytest

import ics
from gpu_helpers import cpu, log_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,t_end", [(2, 1 / 16), (255, 1 / 32), (257, 1 / 32), (5001, 1 / 64),
                                     (17000, 1 / 256)])
def test_level_schedule_edges(n, t_end):
    from paper_1207_2367_amd import System
    m, x, v = ics.plummer(n, 60 + n)
    log_case(test="level_edges", n=n)
    runs = []
    for mode in (0, 1):
        s = System(m, x, v, 1e-4)
        s.set_step_loop(0)
        s.set_schedule(mode)
        st = [s.step(t_end / 2), s.step(t_end)]
        runs.append((st, {k: cpu(q) for k, q in s.get_state().items()}))
        s.close()
    assert runs[0][0] == runs[1][0]
    for k in runs[0][1]:
        assert np.array_equal(runs[0][1][k], runs[1][1][k]), k
