"""The FP64 velocity map where its estimate or its Halley steps can fail:
kicks from 1e-20 to 1e20 of the squared speed, perpendicular speeds from far
below to far above the velocity, paths that stop at and turn through zero,
speeds beyond float range, each against the map in 40-digit arithmetic."""
import math

import numpy as np
import pytest

import mp_kick
from parity_util import print_case
from test_gpu_kick import _run

pytestmark = pytest.mark.gpu


def _cases(n, kappa, ratio, scale, turn, seed):
    """vx, c^2 and a of n cases whose integral K = |a| u dt is kappa times the
    squared speed (u dt = 1); c is ratio times |vx|; turn: a against vx."""
    rng = np.random.default_rng(seed)
    vx = scale * rng.uniform(0.5, 2.0, n) * np.sign(rng.normal(size=n))
    c2 = (ratio * vx) ** 2
    a = kappa * rng.uniform(0.9, 1.1, n) * (vx * vx + c2) * np.sign(vx) * np.where(rng.random(n) < turn, -1.0, 1.0)
    return vx, c2, a


@pytest.mark.parametrize("kind", ["step", "smooth"])
@pytest.mark.parametrize("kappa,ratio,scale", [
    (1e-20, 1.0, 1.0), (1e-9, 1e-3, 1.0), (0.11, 1.0, 1.0), (0.2, 0.3, 1.0), (0.5, 1e-9, 1.0), (0.5, 1e-4, 1.0),
    (0.4999999, 1e-7, 1.0), (1.0, 1e6, 1.0), (3.0, 0.1, 1e-6), (1e6, 1.0, 1.0), (1e20, 1e-2, 1.0),
    (0.7, 1.0, 1e25), (0.7, 1e-25, 1.0)])
def test_fp64_map_over_the_range(gpu_lib, kind, kappa, ratio, scale):
    print_case(f"kick f64 {kind} kappa={kappa} c/v={ratio} v={scale}")
    n, u = 40, 1e-3 * scale  # the limit far below the speeds; smooth: c^2 + u^2
    vx, c2, a = _cases(n, kappa, ratio, scale, 0.7, seed=7)
    got, _ = _run(gpu_lib, "f64", kind, u, 1.0 / u, vx, c2, a)
    want = np.array([mp_kick.kick(kind, u, 1.0 / u, vx[i], c2[i], a[i]) for i in range(n)])
    # rounding of the integral (relative to p0^2 + c^2 and K) over the speed
    # at the end, and of the result itself
    cf = c2 + (u * u if kind == "smooth" else 0.0)
    s0, s1 = np.sqrt(vx * vx + cf), np.sqrt(want * want + cf)
    floor = np.maximum(s1, math.sqrt(2.2e-16) * s0)  # a closed form near zero: sqrt(eps) of the speeds
    tol = 16 * 2.2e-16 * ((s0 * s0 + np.abs(a)) / floor + s0 + s1)
    assert np.isfinite(got).all()
    assert (np.abs(got - want) <= tol).all(), np.max(np.abs(got - want) / tol)
