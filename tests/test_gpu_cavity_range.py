"""The rigid cavity at the ends of its range: spacings whose squared distances overflow, and
the accuracy of its switch function over its whole argument."""
import numpy as np
import pytest

from paper_1509_00680_amd import gps
from gpu_util import dev, host, empty, plan, require_gpu

pytestmark = pytest.mark.gpu

EPS0 = 78.36


@pytest.mark.parametrize("h", [1e150, 1e154, 1e160, 1e200])
def test_spacing_whose_square_overflows(h):
    """An atom smaller than the spacing on the central point: eps is 1 there and eps0 on every
    other point, also where the squares of the separations overflow (their distance is then
    beyond any atom)."""
    require_gpu()
    shape = (5, 9, 15)
    p = plan(shape, h, "free", "fp64")
    e = empty(shape)
    print("cavity spacing", h, flush=True)
    assert p.rigid_cavity(dev(np.array([[0.0, 0.0, 0.0, 0.1 * h]])), 1e-3 * h, EPS0, e) == gps.GPS_OK
    expect = np.full(shape, EPS0)
    expect[2, 4, 7] = 1.0
    np.testing.assert_allclose(host(e), expect, rtol=1e-15)
    p.close()


def test_switch_function_to_the_last_bits():
    """h = erfc(-t)/2 and h'/h, which the kernel takes from one erfcx and one exp, against 40
    digits over t in [-16, 6.5].  With eps0 = 1e140 the relative error of eps is that of h, and q
    is a sum of its logarithmic derivatives.  Bounds: erfcx 2 units in the last place, exp 1, and
    four roundings, 5 units or 1.1e-15 of eps (rms a fifth of it); h'/h enters q squared, twice
    that for each of its terms, three times the sum at the most: 6.7e-15 of q."""
    mp = pytest.importorskip("mpmath").mp
    require_gpu()
    mp.dps = 40
    shape, h, d, delta, eps0 = (3, 3, 500), 2.0 ** -6, 4.0, 0.25, 1e140
    ax = -3.8671875 + 0.37 * h                          # t from -16 beside the centre to 6.5 and on
    p = plan(shape, h, "free", "fp64")
    e, q = empty(shape), empty(shape)
    print("cavity switch", flush=True)
    assert p.rigid_cavity(dev(np.array([[ax, 0.0, 0.0, d]])), delta, eps0, e, q) == gps.GPS_OK
    p.close()
    e, q = host(e)[1, 1], host(q)[1, 1]
    r = np.abs((np.arange(shape[2]) - 0.5 * (shape[2] - 1)) * h - ax)     # as the kernel forms it
    t = (r - d) * (1.0 / delta)
    use = t <= 6.4
    assert use.sum() > 350 and t.min() < -15.9 and t[use].max() > 6.3
    err_e, err_q = [], []
    a = mp.mpf(eps0) - 1
    for i in np.flatnonzero(use):
        ti, ri, dl = mp.mpf(t[i]), mp.mpf(r[i]), mp.mpf(delta)
        H = mp.erfc(-ti) / 2
        u = 2 * mp.exp(-ti * ti) / (dl * mp.sqrt(mp.pi)) / mp.erfc(-ti)
        ref_e = a * H + 1
        ref_q = a * H * (2 * u / ri - 2 * ti * u / dl) / 2 - (a * H) ** 2 * u * u / (4 * ref_e)
        err_e.append(float((mp.mpf(e[i]) - ref_e) / ref_e))
        # against the larger of q's terms (they cancel where q changes its sign)
        size = a * H * (abs(2 * u / ri) + abs(2 * ti * u / dl) + u * u / 2)
        err_q.append(float((mp.mpf(q[i]) - ref_q) / size) if size else 0.0)
    err_e, err_q = np.abs(err_e), np.abs(err_q)
    print("  eps: max %.2e rms %.2e, q: max %.2e" % (err_e.max(), np.sqrt((err_e ** 2).mean()),
                                                     err_q.max()))
    assert err_e.max() <= 1.1e-15 and np.sqrt((err_e ** 2).mean()) <= 2.2e-16
    assert err_q.max() <= 6.7e-15
