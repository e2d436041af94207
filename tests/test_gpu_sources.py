"""The evaluation's two source routes at sizes around its tiles and splits:
with the potential it reads the stored state (or the caller's arrays) as they
stand, without it records packed first.  Both against the oracle, with the
per-precision bounds of gpu_helpers.FORCE_TOL (pair rounding k of the sum of
the term magnitudes), and against each other: they take the same pairs in the
same order, so they may differ by the rounding of the FP64 sums only, 1e-13 of
that sum."""
import numpy as np
import pytest
import torch

import oracle
from gpu_helpers import FORCE_TOL, check_force, cpu, gpu_system, log_case, plummer_inputs, term_sums

pytestmark = pytest.mark.gpu
EPS = 1e-4


def _outs(na, pot):
    out = [torch.full((na, 3), float("nan"), dtype=torch.float64, device="cuda") for _ in range(3)]
    return out + [torch.full((na,), float("nan"), dtype=torch.float64, device="cuda") if pot else None]


@pytest.mark.parametrize("prec", [0, 1, 2], ids=["mixed", "fp64", "fp32pair"])
@pytest.mark.parametrize("n,na", [(2, 1), (63, 7), (257, 257), (4097, 130), (20011, 3), (16411, 2100)])
def test_routes_match_oracle(n, na, prec):
    from paper_1207_2367_amd.nbody import force_noalloc
    m, x, v, a = plummer_inputs(n, 900 + n)
    idx = np.sort(np.random.default_rng(n).choice(n, na, replace=False)).astype(np.int32)
    pos = np.unique(np.linspace(0, na - 1, min(na, 64)).astype(int))
    ref = oracle.force(m, x, v, a, EPS, idx[pos])
    S = term_sums(m, x, v, a, EPS, idx[pos])
    s = gpu_system(m, x, v, a, EPS, prec)
    log_case(test="routes", n=n, n_act=na, prec=prec, launch=s.get_launch(na))
    state = s.force(idx, out=_outs(na, True))
    packed = s.force(idx, out=_outs(na, False), pot=False)
    caller = force_noalloc(m, x, v, a, EPS, idx, precision=prec, out=_outs(na, True))
    caller_packed = force_noalloc(m, x, v, a, EPS, idx, precision=prec, out=_outs(na, False), pot=False)
    check_force(FORCE_TOL[prec], [cpu(g)[pos] for g in state], ref, S)
    for q in range(3):
        for other in (packed, caller, caller_packed):
            d = np.linalg.norm(cpu(other[q])[pos] - cpu(state[q])[pos], axis=1)
            assert np.all(d <= 1e-13 * S[:, q]), (q, (d / S[:, q]).max())
    d = np.abs(cpu(caller[3])[pos] - cpu(state[3])[pos])
    assert np.all(d <= 1e-13 * S[:, 3])
    s.close()
