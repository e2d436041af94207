"""The sums over all particles of the energy pass keep their chains short.  2^20
particles of one kinetic energy c: a chain of equal terms rounds the same way in
every lane, so its error does not average out, while equal terms in a tree add
without rounding.  The orders' roundings that do not vanish: four waves of a
workgroup and four workgroups of a lane, at most two each (3c and 4c), 2^-53 of
the sum each.  (One chain of 64 workgroups per lane is 16 x 2^-53 off at this c.)"""
import numpy as np
import pytest

from gpu_helpers import log_case

pytestmark = pytest.mark.gpu


def test_kinetic_energy_of_equal_terms():
    from paper_1207_2367_amd import System
    n = 1 << 20
    c = 1.9419943792414571 / n
    log_case(test="energy_sums", n=n)
    v = np.zeros((n, 3))
    v[:, 0] = 1.0
    s = System(np.full(n, 2.0 * c), np.random.default_rng(4).standard_normal((n, 3)), v, 1e-4, skip_startup=True)
    ek, _, _ = s.energy()
    s.close()
    exact = np.longdouble(c) * n
    assert abs(float((np.longdouble(ek) - exact) / exact)) <= 4 * 2.0 ** -53
