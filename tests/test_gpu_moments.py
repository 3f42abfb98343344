"""beta-weighted moments (Eq. 5) at the sizes where the windowed kernels can
go wrong, against the oracle (1D) and against sums written out in NumPy over
the exported particles (2D): ranges of cells beyond the LDS window, rows and
chunks cut short, wavefronts whose chunks cross from one species (or run) to
the next, tile windows left behind by the particles, windows too large for
LDS."""
import math

import numpy as np
import pytest

import oracle
import workloads
from parity_util import print_case, push_oracle_to_gpu, rel_inf

pytestmark = pytest.mark.gpu

# FP64 sums on both sides over the same stored particles; beta of a float
# particle is a reciprocal square root refined in FP64 (1.5e-14 relative), and
# the rows' cancellation (flux) stays below 1e3.
TOL = 1e-11


@pytest.mark.parametrize("nx,ppc,chunk,prec,beta,sort", [
    (4, 3, 64, "f64", "step", 0),       # less than a row of 64 slots
    (127, 5, 64, "f32", "step", 0),     # unsorted: one row spans the window exactly
    (300, 7, 512, "f64", "smooth", 0),  # unsorted: pairs outside the window
    (300, 21, 1024, "f32", "step", 1),  # sorted: several windows per chunk
    (512, 350, 64, "f32", "step", 1),   # more than 4096 wavefronts: grouped chunks, across the species
    (2729, 4, 512, "f64", "step", 1),   # the largest grid
])
def test_moments_match_oracle(gpu_lib, nx, ppc, chunk, prec, beta, sort):
    print_case(f"moments nx={nx} ppc={ppc} chunk={chunk} {prec} {beta} sort={sort}")
    cfg = workloads.sheath(nx, ppc, 5.0, beta_kind=beta, seed=3)
    run = oracle.Run(cfg)
    sim = gpu_lib.Sim(cfg, precision=prec, sort_every=sort, chunk=chunk)
    push_oracle_to_gpu(sim, 0, run, quantize=prec == "f32")
    if sort:
        sim.sort_now()
    want = run.moments()
    got = sim.moments(0).cpu().numpy()
    for _ in range(2):
        sim.moments_sample(-1)
    assert sim.status(0)["moment_samples"] == 2
    win = sim.moments_window(0, reset=True).cpu().numpy()
    for row in range(7):
        assert rel_inf(got[row], want[row]) <= TOL, row
        assert rel_inf(win[row], want[row]) <= TOL, row
    assert sim.status(0)["moment_samples"] == 0 and not sim.moments_window(0).abs().max().item()
    sim.close()


def test_moments_of_ragged_runs_share_a_launch(gpu_lib):
    """Runs of different sizes sampled in one launch, and one of them alone."""
    cfgs = [dict(workloads.sheath(nx, ppc, u, seed=nx), run=r)
            for r, (nx, ppc, u) in enumerate([(64, 9, 2.0), (200, 3, 8.0), (5, 50, math.inf)])]
    sim = gpu_lib.Sim(cfgs, precision="f64", sort_every=1, chunk=128)
    runs = [oracle.Run(c) for c in cfgs]
    for r, run in enumerate(runs):
        push_oracle_to_gpu(sim, r, run, quantize=False)
    sim.moments_sample(-1)
    sim.moments_sample(1)
    for r, run in enumerate(runs):
        want = run.moments()
        win, one = sim.moments_window(r).cpu().numpy(), sim.moments(r).cpu().numpy()
        for row in range(7):
            assert rel_inf(win[row], want[row]) <= TOL, (r, row)
            assert rel_inf(one[row], want[row]) <= TOL, (r, row)
    assert [s["moment_samples"] for s in sim.status()] == [1, 2, 1]
    sim.close()


def _plane_moments(sim, cfg, ny):
    """The six particle rows written out over the exported particles."""
    nx, dx = cfg["nx"], cfg["dx"]
    rows, w = [], sim.status()["weight"]
    for s in range(2):
        x, y, vx, vy, vz2 = sim.export_particles(s)
        live = x >= 0
        x, y, vx, vy, vz2 = (a[live] for a in (x, y, vx, vy, vz2))
        v2 = vx * vx + vy * vy + vz2
        u = cfg["u"]
        b = np.sqrt(1 / (1 + v2 / u**2)) if cfg["beta_kind"] == "smooth" else np.minimum(1.0, u / np.sqrt(v2))
        i, j = x.astype(int), y.astype(int)
        fx, fy = x - i, y - j
        for q in (1.0, vx, 0.5 * cfg["species"][s]["mass"] * v2):
            m = np.zeros((nx + 1, ny))
            for di, gx in ((0, 1 - fx), (1, fx)):
                for dj, gy in ((0, 1 - fy), (1, fy)):
                    np.add.at(m, (i + di, (j + dj) % ny), w[s] * b * gx * gy * q)
            m /= dx * dx
            m[0] *= 2
            m[-1] *= 2
            rows.append(m)
    return rows


@pytest.mark.parametrize("nx,ny,ppc,prec,beta,tile,margin,steps", [
    (24, 16, 11, "f64", "step", 4, 1, 3),    # particles beyond their tile's window
    (24, 16, 11, "f32", "smooth", 4, 2, 2),  # with an unsorted tail
    (9, 4, 7, "f32", "step", 8, 0, 0),       # a window wider than the periodic side, cut tiles
    (70, 64, 3, "f32", "step", 51, 1, 0),    # three window rows beyond 64 KB: the untiled pass
    (70, 64, 3, "f64", "step", 48, 1, 1),    # the largest window that fits
])
def test_moments2d_written_out(gpu_lib, nx, ny, ppc, prec, beta, tile, margin, steps):
    print_case(f"moments2d {nx}x{ny} ppc={ppc} {prec} {beta} tile={tile} margin={margin} steps={steps}")
    cfg = workloads.sheath2d(nx, ny, ppc, 3.0, tile=tile, beta_kind=beta, seed=5)
    sim = gpu_lib.Sim2D(cfg, ny, precision=prec, sort_every=8, tile=tile, margin=margin)
    sim.step(steps)
    got = sim.moments().cpu().numpy()
    want = _plane_moments(sim, cfg, ny)
    assert rel_inf(got[0], sim.grid()["phi"]) == 0.0
    for row in range(6):
        assert rel_inf(got[1 + row], want[row]) <= TOL, row
    sim.close()
