"""Start-up passes at the edges of their launch shapes (lanes per particle,
particles per lane, source splits, ragged tiles) against the oracle's.

Tolerances: both sides form every pair term in FP64, so the error of a sum is
bounded by the sum S of its term magnitudes: 1e-12 S for a, da, d2a (some
thousand terms' rounding with room for the order of the sums), and 4e-12 of
the snap's condition number, relative, for the crackle, whose terms have one
more level of the same products.
"""
import math

import numpy as np
import pytest

import ics
import oracle
from gpu_helpers import abs_err_rows, cpu, log_case, norm_rows, term_sums

pytestmark = pytest.mark.gpu


def _check(sizes, eps, prec, n_sample=96):
    from paper_1207_2367_amd import System
    parts = [ics.plummer(k, 500 + q) if k > 1 else
             (np.ones(1), np.array([[0.3, -0.2, 0.1]]), np.array([[0.1, 0.2, -0.3]]))
             for q, k in enumerate(sizes)]
    m, x, v = (np.concatenate([p[q] for p in parts]) for q in range(3))
    off = np.concatenate([[0], np.cumsum(sizes)])
    log_case(test="startup", sizes=sizes, eps=eps, prec=prec)
    it = oracle.Integrator(m, x, v, eps, offsets=off)
    assert it.init(math.inf) == 0
    s = System(m, x, v, eps, precision=prec, offsets=list(off), device="cuda")
    g = {k: cpu(q) for k, q in s.get_state().items()}
    s.close()
    assert np.array_equal(g["x"], it.x) and np.array_equal(g["v"], it.v) and np.all(g["t"] == 0)
    for key in ("a", "jk", "sn", "cr", "dt"):
        assert np.isfinite(g[key]).all(), key
    rng = np.random.default_rng(9)
    for lo, hi in zip(off[:-1], off[1:]):
        if hi - lo == 1:
            for key in ("a", "jk", "sn", "cr"):
                assert np.all(g[key][lo] == 0.0), key
            continue
        ends = np.array([lo, hi - 1])
        idx = np.unique(np.concatenate([ends, rng.integers(lo, hi, n_sample)]))
        S = term_sums(m, x, v, it.a, eps, idx, (lo, hi))
        for key, q in (("a", 0), ("jk", 1), ("sn", 2)):
            e = abs_err_rows(g[key][idx], getattr(it, key)[idx])
            assert np.all(e <= 1e-12 * S[:, q]), (key, np.nanmax(e / S[:, q]))
        e = abs_err_rows(g["cr"][idx], it.cr[idx]) / norm_rows(it.cr[idx])
        assert np.all(e <= 4e-12 * S[:, 2] / norm_rows(it.sn[idx])), np.nanmax(e)


@pytest.mark.parametrize("eps", [1e-4, 0.0], ids=["soft", "eps0"])
@pytest.mark.parametrize("n", [2, 257, 1000, 4097, 16385, 33001])
def test_startup_sizes(n, eps):
    _check([n], eps, 0)


def test_startup_clusters():
    _check([1, 300, 5000, 2, 40, 9000], 1e-4, 1)
