"""Moments of a state with a particle of infinite speed, which only an import
can bring: its beta is zero, so it adds nothing to the density, and its flux
and energy, zero times infinity, show as NaN at its two nodes instead of
getting lost.  Every other node holds what the finite particles give."""
import numpy as np
import pytest

import workloads
from parity_util import print_case

pytestmark = pytest.mark.gpu


def _check(got, want, nodes):
    """Rows of (n, Gamma, energy): NaN where marked, else equal to rounding."""
    for row in (1, 2):
        bad = np.zeros(got[row].shape, bool)
        bad[nodes] = True
        assert np.array_equal(np.isnan(got[row]), bad), row
    for row in range(3):
        ok = ~np.isnan(got[row])
        assert np.abs(got[row][ok] - want[row][ok]).max() <= 1e-11 * np.abs(want[row]).max(), row


@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("beta", ["step", "smooth"])
def test_infinite_speed_shows_in_1d(gpu_lib, prec, beta):
    print_case(f"moments of an infinite speed, 1D {prec} {beta}")
    cfg = workloads.sheath(40, 4, 3.0, beta_kind=beta, seed=1)
    sim = gpu_lib.Sim(cfg, precision=prec, sort_every=1)
    x, vx, vp = np.array([3.25, 20.5, 30.75]), np.array([0.5, np.inf, -0.25]), np.array([0.25, 0.5, 1.0])
    sim.import_particles(0, 0, x, vx, vp)
    sim.import_particles(0, 1, x[:1], vx[:1], vp[:1])
    got = sim.moments(0).cpu().numpy()
    u, w, m = cfg["u"], sim.status(0)["weight"][0], cfg["species"][0]["mass"]
    want = np.zeros((3, 41))
    for i in (0, 2):
        v2 = vx[i] ** 2 + vp[i]
        b = 1 / np.sqrt(1 + v2 / u**2) if beta == "smooth" else min(1.0, u / np.sqrt(v2))
        c, f = int(x[i]), x[i] - int(x[i])
        for row, q in enumerate((1.0, vx[i], 0.5 * m * v2)):
            want[row, c] += w * b * (1 - f) * q / cfg["dx"]
            want[row, c + 1] += w * b * f * q / cfg["dx"]
    _check(got[1:4], want, [20, 21])
    assert np.isfinite(got[4:7]).all()
    sim.close()


@pytest.mark.parametrize("prec", ["f64", "f32"])
def test_infinite_speed_shows_in_2d(gpu_lib, prec):
    print_case(f"moments of an infinite speed, 2D {prec}")
    cfg = workloads.sheath2d(24, 16, 2, 3.0, tile=8, seed=1)
    sim = gpu_lib.Sim2D(cfg, 16, precision=prec, sort_every=8, tile=8, margin=2)
    x, y = np.array([3.25, 20.5]), np.array([2.5, 9.75])
    vx, vy, vz2 = np.array([0.5, np.inf]), np.array([0.25, 0.0]), np.array([0.25, 0.5])
    for s in range(2):
        sim.import_particles(s, x, y, vx, vy, vz2)
    sim.sort_now()  # the windowed pass
    got = sim.moments().cpu().numpy()
    u = cfg["u"]
    for s in range(2):
        w, m = sim.status()["weight"][s], cfg["species"][s]["mass"]
        v2 = vx[0] ** 2 + vy[0] ** 2 + vz2[0]
        b = min(1.0, u / np.sqrt(v2))
        want = np.zeros((3, 25, 16))
        for row, q in enumerate((1.0, vx[0], 0.5 * m * v2)):
            for i, gx in ((3, 0.75), (4, 0.25)):
                for j in (2, 3):
                    want[row, i, j] = w * b * gx * 0.5 * q / cfg["dx"] ** 2
        _check(got[1 + 3 * s:4 + 3 * s], want, (np.array([20, 20, 21, 21]), np.array([9, 10, 9, 10])))
    sim.close()
