"""Sphere quadrature of a field with one infinite or NaN value: it reaches the
outputs whose sphere touches that point and no others.  Which ones, the oracle's
integrals of the point's indicator say: exactly zero where the rule has no weight
there (rules of odd order have no mirror nodes along x)."""
import numpy as np
import pytest

from conftest import to_dev
from oracle.sphere_quad import shell_integrals
from paper_1407_0674_amd import FLAG_APERIODIC, FLAG_CUBIC, FP64, MIXED

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", [FP64, MIXED])
@pytest.mark.parametrize("k,reach,cubic", [(1, 2.6, False), (3, 1.4, False), (3, 3.3, True), (5, 2.0, False), (7, 4.4, False),
                                           (7, 2.7, True), (6, 3.5, False), (8, 2.2, True)])
def test_one_point(ev, precision, k, reach, cubic):
    h, shape, at = 0.05, (21, 19, 37), (10, 9, 17)
    f = 1.0 + np.random.default_rng(5400 + k).random((1,) + shape)
    one = np.zeros(shape)
    one[at] = 1.0
    for aperiodic in (False, True):
        I, Iv = shell_integrals(one, reach * h, h, k, aperiodic=aperiodic, cubic=cubic)
        weight = np.max(np.abs(np.stack([I, *Iv])), axis=0)
        flags = (FLAG_APERIODIC if aperiodic else 0) | (FLAG_CUBIC if cubic else 0)
        for bad in (np.inf, -np.inf, np.nan):
            f[0][at] = bad
            got = ev.sphere_quadrature(to_dev(f), [reach * h], h, k, precision=precision, flags=flags).cpu().numpy()[0]
            assert np.isfinite(got[:, weight == 0.0]).all()
            assert not np.isfinite(got[0][np.abs(I) > 1e-10 * np.max(np.abs(I))]).any()
