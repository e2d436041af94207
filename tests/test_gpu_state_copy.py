"""State copies and the predictor's outputs at sizes around their workgroups of
256 particles: what goes in comes out bit for bit, arrays that are left out
stay as they are, and nothing is written past the last particle."""
import numpy as np
import pytest
import torch

import ics
import oracle
from gpu_helpers import cpu, log_case

pytestmark = pytest.mark.gpu
KEYS = ("x", "v", "a", "jk", "sn", "cr", "t", "dt")


@pytest.mark.parametrize("n", [1, 255, 256, 257, 1000])
def test_state_round_trip(n):
    from paper_1207_2367_amd import System
    m, x, v = ics.plummer(max(n, 2), 80)
    m, x, v = m[:n], x[:n], v[:n]
    log_case(test="state_round_trip", n=n)
    s = System(m, x, v, 1e-4, skip_startup=True)
    rng = np.random.default_rng(n)
    ref = {k: rng.standard_normal((n, 3)) for k in KEYS[:6]}
    ref["dt"] = 2.0 ** -rng.integers(4, 12, n).astype(float)
    ref["t"] = ref["dt"] * rng.integers(0, 6, n)
    s.set_state(**{k: ref[k] for k in ("x", "a", "cr", "t")})
    got = {k: cpu(q) for k, q in s.get_state().items()}
    for k in ("x", "a", "cr", "t"):
        assert np.array_equal(got[k], ref[k]), k
    assert np.array_equal(got["v"], v) and np.all(got["jk"] == 0) and np.all(got["sn"] == 0)
    s.set_state(**{k: ref[k] for k in ("v", "jk", "sn", "dt")})
    got = {k: cpu(q) for k, q in s.get_state().items()}
    for k in KEYS:
        assert np.array_equal(got[k], ref[k]), k
    p = [torch.full((n + 1, 3), 7.0, dtype=torch.float64, device="cuda") for _ in range(3)]
    from paper_1207_2367_amd import nbody
    s._check(nbody.load().nbody_predict(s.ctx, 0.4375, *[nbody._ptr(q) for q in p]))
    want = oracle.predict(*[ref[k] for k in KEYS[:6]], ref["t"], 0.4375)
    for g, r in zip(p, want):
        assert np.abs(cpu(g)[:n] - r).max() <= 4e-16 * 64 * np.abs(r).max()
        assert np.all(cpu(g)[n] == 7.0)
    s.close()
