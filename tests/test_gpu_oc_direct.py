"""The OC update's predicted and proved bisection (oc.hip, eta 0.5 and 1)
against the sequential oracle: sizes at the edges of a block's elements,
targets in reach and out of it on either side, brackets and step caps of every
kind, the loosest and tightest tolerance it takes, and data that no proof can
hold for (NaN), where the passes take over.  With no step within the device
sum's rounding of V* every result is bitwise the oracle's."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import oc as OC
from paper_2505_02438_amd import api

from gpu_util import dev, host

pytestmark = pytest.mark.gpu


def _inputs(n, seed):
    rng = np.random.default_rng(seed)
    rho = rng.uniform(0.0, 1.0, n)
    rho[::7] = 0.0
    rho[3::11] = 1.0
    dc = -np.exp(rng.normal(0.0, 3.0, n)) * rho
    dc[::13] = 0.0
    dc[5::29] = 1.0     # a positive sensitivity: B = 0
    return rho, dc, rng.uniform(0.5, 1.5, n)


def _tie(rho, dc, dv, target, lam, steps, move, eta, tol, lmax):
    """Whether some step of the path to lam lies within the device sum's rounding of V*."""
    l1, l2 = 0.0, lmax
    for _ in range(steps):
        mid = 0.5 * (l1 + l2)
        vol = OC.volume(dv, OC.oc_candidate(rho, dc, dv, mid, move, eta))
        if abs(vol - target) <= len(rho) * 2.0 ** -53 * vol:
            return True
        if vol > target:
            l1 = mid
        else:
            l2 = mid
    return False


@pytest.mark.parametrize("n", [1, 2, 255, 257, 767, 768, 769, 20011, 262221])
@pytest.mark.parametrize("eta", [0.5, 1.0])
@pytest.mark.parametrize("frac,move,lmax,tol,max_steps", [
    (0.4, 0.2, 1e9, 1e-3, 200), (0.45, 0.2, 1e9, 1e-5, 200), (0.4, 1.0, 1e9, 0.3, 200), (0.5, 0.05, 40.0, 1e-3, 200),
    (0.4, 0.2, 1e9, 1e-3, 1), (0.4, 0.2, 1e9, 1e-3, 7), (0.0, 0.2, 1e9, 1e-3, 200), (3.0, 0.2, 1e9, 1e-3, 200),
    (3.0, 0.2, 1e9, 1e-3, 1000), (0.9, 1.0, 1e-3, 1e-3, 200)])
def test_direct_bisection_matches_oracle(n, eta, frac, move, lmax, tol, max_steps):
    rho, dc, dv = _inputs(n, 1000 + n)
    target = frac * dv.sum()
    kw = dict(move=move, eta=eta, tol=tol, lmax=lmax, max_steps=max_steps)
    rn, lam, vol, steps, change = OC.oc_update(rho, dc, dv, target, **kw)
    got, info = api.oc_update(dev(rho), dev(dc), dev(dv), target, **kw)
    got = host(got)
    assert np.array_equal(got, OC.oc_candidate(rho, dc, dv, info["lambda"], move, eta))
    if _tie(rho, dc, dv, target, lam, steps, move, eta, tol, lmax):
        return
    assert info["steps"] == steps and info["lambda"] == lam
    assert np.array_equal(got, rn) and info["change"] == change
    assert abs(info["volume"] - vol) <= 1e-13 * abs(vol)


@pytest.mark.parametrize("where", ["rho", "dv", "negative dv"])
def test_direct_bisection_with_nan(where):
    """A NaN in the volume fails every comparison with V*, so the loop halves
    l2 to the step cap; the densities elsewhere are the update there."""
    rho, dc, dv = _inputs(3000, 5)
    target = 0.4 * dv.sum()
    if where == "rho":
        rho[17] = np.nan
    elif where == "dv":
        dv[17] = np.nan
    else:
        dv[17], dc[17] = -1.0, -1.0      # sqrt of a negative number
    got, info = api.oc_update(dev(rho), dev(dc), dev(dv), target, max_steps=60)
    lam = 1e9
    for _ in range(60):
        lam = 0.5 * (0.0 + lam)
    assert info["steps"] == 60 and info["lambda"] == lam and np.isnan(info["volume"]) and np.isnan(info["change"])
    ok = np.ones(3000, dtype=bool)
    ok[17] = False
    ref = OC.oc_candidate(rho[ok], dc[ok], dv[ok], lam, 0.2, 0.5)
    got = host(got)
    assert np.isnan(got[17]) and np.array_equal(got[ok], ref)
