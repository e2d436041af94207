"""The energy's pair pass at the edges of its shapes: one, two and four
particles per lane (clusters below 32,768, from there, and from 65,536 bodies),
odd and even sizes, workgroups that are partly empty, one tile and several
splits.  Against the oracle's energy, both in FP64: the same pairs in another
order, so 1e-12 relative for the energies and for L against the sum of its
term magnitudes."""
import numpy as np
import pytest

import ics
import oracle
from gpu_helpers import log_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("sizes", [[1], [2], [3], [255, 257], [1025], [16384], [16901, 300], [32768], [33025, 300],
                                   [66049]],
                         ids=lambda s: "-".join(map(str, s)))
@pytest.mark.parametrize("eps", [1e-4, 0.0], ids=["soft", "eps0"])
def test_energy_shapes(sizes, eps):
    from paper_1207_2367_amd import System
    parts = [ics.plummer(max(k, 2), 700 + k) for k in sizes]
    m, x, v = (np.concatenate([p[q][:k] for p, k in zip(parts, sizes)]) for q in range(3))
    off = np.concatenate([[0], np.cumsum(sizes)])
    log_case(test="energy_shapes", sizes=sizes, eps=eps)
    s = System(m, x, v, eps, offsets=list(off), skip_startup=True)
    ek, ep, L = s.energy()
    s.close()
    rk, rp, rL = oracle.energy(m, x, v, eps, off)
    assert abs(ek - rk) <= 1e-12 * abs(rk)
    assert abs(ep - rp) <= 1e-12 * abs(rp)
    scale = (m[:, None] * np.abs(x)[:, [1, 2, 0]] * np.abs(v)[:, [2, 0, 1]]).sum(0) * 2
    assert np.all(np.abs(np.array(L) - rL) <= 1e-12 * scale)
