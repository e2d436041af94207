"""The energy with a softening whose square is no normal FP32 number (accepted;
the state set without a start-up): a particle's own slot in its window of
sources has no finite 1/r there and must not enter the sum, with one, two and
four particles per lane and in clusters.  Against the oracle as in
test_gpu_energy_shapes.py: FP64 on both sides, the same pairs, 1e-12."""
import numpy as np
import pytest

import ics
import oracle
from gpu_helpers import log_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("eps", [1e-21, 1e-25, 1e-160])
@pytest.mark.parametrize("sizes", [[2], [300], [257, 1025], [32769], [66049]],
                         ids=lambda s: "-".join(map(str, s)))
def test_energy_tiny_softening(sizes, eps):
    from paper_1207_2367_amd import System
    parts = [ics.plummer(k, 800 + k) for k in sizes]
    m, x, v = (np.concatenate([p[q] for p in parts]) for q in range(3))
    off = np.concatenate([[0], np.cumsum(sizes)])
    log_case(test="energy_tiny_softening", sizes=sizes, eps=eps)
    s = System(m, x, v, eps, offsets=list(off), skip_startup=True)
    ek, ep, _ = s.energy()
    s.close()
    rk, rp, _ = oracle.energy(m, x, v, eps, off)
    assert abs(ek - rk) <= 1e-12 * abs(rk)
    assert abs(ep - rp) <= 1e-12 * abs(rp)


@pytest.mark.parametrize("sizes", [[33000] + [100] * 40, [40000, 33000, 129], [3000] + [1, 2, 255, 256, 257] * 5],
                         ids=["one-large", "two-per-lane", "one-of-3000"])
@pytest.mark.parametrize("eps", [1e-4, 0.0], ids=["soft", "eps0"])
def test_energy_mixed_clusters(sizes, eps):
    """Clusters of mixed sizes: splits counted for the large ones alone, which
    leave the small ones with more splits than they have tiles."""
    from paper_1207_2367_amd import System
    parts = [ics.plummer(max(k, 2), 810 + k) for k in sizes]
    m, x, v = (np.concatenate([p[q][:k] for p, k in zip(parts, sizes)]) for q in range(3))
    off = np.concatenate([[0], np.cumsum(sizes)])
    log_case(test="energy_mixed_clusters", sizes=sizes[:3], eps=eps)
    s = System(m, x, v, eps, offsets=list(off), skip_startup=True)
    ek, ep, _ = s.energy()
    s.close()
    rk, rp, _ = oracle.energy(m, x, v, eps, off)
    assert abs(ek - rk) <= 1e-12 * abs(rk)
    assert abs(ep - rp) <= 1e-12 * abs(rp)
