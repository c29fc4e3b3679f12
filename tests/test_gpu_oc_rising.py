"""OC update with a volume that rises with the multiplier somewhere: an element
of negative volume and negative density, eta 1.  The volume then meets V* at
three multipliers, the last one above every midpoint of the first halvings, and
the values at the ends of a path do not decide the steps between them: the
sequential loop's path (oracle) has to be taken, by the passes."""
import ctypes

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import oc as OC
from paper_2505_02438_amd import _lib, api

from gpu_util import dev, host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("halvings", [10, 30, 33])
def test_rising_volume_follows_the_loop(halvings):
    first = 1e9 / 2.0 ** halvings  # the first midpoint whose volume is above V*
    rho = np.array([0.5, 0.5, -0.005])
    dv = np.array([13.5, 50.0, -200.0])
    # two drops, at 1.2 and 1.8 times first, and the rise between them
    dc = np.array([-13.5 * 1.2, -50.0 * 1.8, -200.0 * 1.2]) * first
    kw = dict(move=0.01, eta=1.0, tol=1e-3, lmax=1e9, max_steps=200)
    target = OC.volume(dv, OC.oc_candidate(rho, dc, dv, 0.9 * first, 0.01, 1.0)) - 0.05
    above = [OC.volume(dv, OC.oc_candidate(rho, dc, dv, x * first, 0.01, 1.0)) > target for x in (1, 1.5, 1.75, 2)]
    assert above == [True, False, True, False]
    rn, lam, vol, steps, change = OC.oc_update(rho, dc, dv, target, **kw)
    got, info = api.oc_update(dev(rho), dev(dc), dev(dv), target, **kw)
    assert info["lambda"] == lam and info["steps"] == steps and info["change"] == change
    assert np.array_equal(host(got), rn)
    f = ctypes.c_int32()
    assert _lib.lib().soptx_debug_oc_form(ctypes.byref(f)) == 0 and f.value == 0
