"""``force_noalloc`` with outputs on top of its inputs gives the bits that it
gives in buffers apart from them: the inputs enter with their values from
before the call, in one split (no partial sums but for this) and in several,
with the potential (sources read where they are) and without (packed)."""
import pytest
import torch

from gpu_helpers import log_case, plummer_inputs

pytestmark = pytest.mark.gpu


def _dev(q):
    return torch.as_tensor(q, dtype=torch.float64, device="cuda").clone()


@pytest.mark.parametrize("prec", [0, 1, 2], ids=["mixed", "fp64", "fp32pair"])
@pytest.mark.parametrize("n", [64, 256, 511, 512, 1000, 300000])
def test_in_place(n, prec):
    from paper_1207_2367_amd.nbody import force_noalloc
    ins = plummer_inputs(n, 40 + n)
    every = torch.arange(n, dtype=torch.int32, device="cuda")
    few = every[:: max(2, n // 7)].contiguous()

    def go(idx, pot, place):
        m, x, v, a = (_dev(q) for q in ins)
        na = idx.shape[0]
        out = [torch.zeros((na, 3), dtype=torch.float64, device="cuda") for _ in range(3)]
        out.append(torch.zeros(na, dtype=torch.float64, device="cuda") if pot else None)
        for q, buf in place(m, x, v, a, na).items():
            out[q] = buf
        force_noalloc(m, x, v, a, 1e-4, idx, precision=prec, out=out, pot=pot)
        return [o for o in out if o is not None]

    def apart(m, x, v, a, na):
        return {}

    def update(m, x, v, a, na):          # the accelerations, in place
        return {0: a[:na]}

    def shifted(m, x, v, a, na):         # the last rows, and one output into each array
        return {0: a[a.shape[0] - na:], 1: v[:na], 2: x[x.shape[0] - na:]}

    def pots(m, x, v, a, na):
        return {3: m[:na]}

    for idx in (every, few):
        for pot in (True, False):
            log_case(test="in_place", n=n, n_act=idx.shape[0], prec=prec, pot=pot)
            ref = go(idx, pot, apart)
            assert all(torch.isfinite(q).all() for q in ref)
            for place in (update, shifted) + ((pots,) if pot else ()):
                for q, (g, r) in enumerate(zip(go(idx, pot, place), ref)):
                    assert torch.equal(g, r), (place.__name__, q)
