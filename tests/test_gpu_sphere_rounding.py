"""Rounding of the sphere quadrature's vector integrals in mixed precision: they are
small differences of large sums, so the way the offsets are combined shows.

The yardstick is the float32 sum of antipodal pairs, weight times the difference of
the two values (the sum for the scalar integral), accumulated with one rounding per
pair, in numpy: its error and the kernel's, both against the FP64 kernel (1e-15),
root mean square over the field.  Both round every term once and the values at most
twice before; the orders of summation differ, which moves the error of one rule by a
few ten per cent either way.  Hence: the geometric mean over the rules at most 1.1
times the pairs' for each integral, no single rule above 1.6.

And an infinite value stays infinite, with the sign of its weight."""
import numpy as np
import pytest

from conftest import to_dev
from oracle.sphere_quad import axis_weights, shell_integrals, sphere_rule
from paper_1407_0674_amd import FLAG_CUBIC, FP64, MIXED

pytestmark = pytest.mark.gpu

H = 0.05


def _cells(r, k, cubic):
    """{offset: (scalar, x, y, z) weights} of the merged stencil, radius r in grid units."""
    theta, wt, phi, wp = sphere_rule(k)
    cells = {}
    for th, a in zip(theta, wt):
        for ph, b in zip(phi, wp):
            nd = np.array([np.cos(th) * np.sin(ph), np.sin(th) * np.sin(ph), np.cos(ph)])
            p = r * nd
            base = np.floor(p).astype(int)
            ax = [axis_weights(p[c] - base[c], cubic) for c in range(3)]
            W = (r * H) ** 2 * np.sin(ph) * a * b
            for ox, wx in zip(*ax[0]):
                for oy, wy in zip(*ax[1]):
                    for oz, wz in zip(*ax[2]):
                        key = (base[0] + int(ox), base[1] + int(oy), base[2] + int(oz))
                        cells[key] = cells.get(key, 0.0) + W * wx * wy * wz * np.array([1.0, *nd])
    top = max(np.max(np.abs(v)) for v in cells.values())
    return {o: v for o, v in cells.items() if np.max(np.abs(v)) > 1e-14 * top}


def _pairs_float32(f, cells):
    f = f.astype(np.float32)
    at = lambda o: np.roll(f, tuple(-v for v in o), axis=(0, 1, 2))
    out = np.zeros((4,) + f.shape, dtype=np.float32)
    for o in sorted(cells):
        m = tuple(-v for v in o)
        if o < m:
            continue
        v = at(o)
        s, d = (v, v) if o == m else (v + at(m), v - at(m))
        for q in range(4):
            w = np.float64(np.float32(cells[o][q]))
            out[q] = (w * (s if q == 0 else d) + out[q]).astype(np.float32)  # one rounding
    return out


@pytest.mark.parametrize("cubic", [False, True])
def test_error_against_antipodal_pairs(ev, cubic):
    f = 1.0 + np.random.default_rng(6000).random((18, 16, 36))
    fd = to_dev(f[None])
    ratios = []
    for k in (4, 6, 8):
        for r in (1.3, 1.7, 2.2, 2.9, 3.6):
            flags = FLAG_CUBIC if cubic else 0
            ref = ev.sphere_quadrature(fd, [r * H], H, k, precision=FP64, flags=flags)[0].cpu().numpy()
            got = ev.sphere_quadrature(fd, [r * H], H, k, precision=MIXED, flags=flags)[0].cpu().numpy()
            pairs = _pairs_float32(f, _cells(r, k, cubic))
            rms = lambda a: np.sqrt(np.mean((a - ref) ** 2, axis=(1, 2, 3)))
            ratios.append(rms(got) / rms(pairs))
    ratios = np.array(ratios)
    mean = np.exp(np.mean(np.log(ratios), axis=0))
    print("geometric means", mean, "largest", ratios.max(axis=0))
    assert (mean < 1.1).all(), mean
    assert (ratios < 1.6).all(), ratios.max(axis=0)


@pytest.mark.parametrize("precision", [FP64, MIXED])
@pytest.mark.parametrize("k,r", [(4, 2.3), (8, 1.6), (8, 3.4), (7, 2.3)])
def test_infinity(ev, precision, k, r):
    f = 1.0 + np.random.default_rng(6100 + k).random((1, 17, 19, 41))
    one = np.zeros(f.shape[1:])
    at = (8, 9, 20)
    one[at] = 1.0
    I, Iv = shell_integrals(one, r * H, H, k)
    w = np.stack([I, *Iv])
    for inf in (np.inf, -np.inf):
        f[0][at] = inf
        got = ev.sphere_quadrature(to_dev(f), [r * H], H, k, precision=precision).cpu().numpy()[0]
        hit = np.abs(w) > 1e-10 * np.max(np.abs(w))
        assert (got[hit] == np.sign(w[hit]) * inf).all()
