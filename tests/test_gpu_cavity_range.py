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
