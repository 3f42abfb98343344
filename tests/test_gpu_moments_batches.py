"""The windowed moments' walk over a chunk in batches of 8, 4, 2 and 1
consecutive slots per lane: every length about the batches' ends, cells below
the first batch's, dead slots anywhere, and thin runs whose chunks span more
cells than a window, against sums written out over the imported particles."""
import numpy as np
import pytest

import workloads
from parity_util import print_case, rel_inf

pytestmark = pytest.mark.gpu

# FP64 sums on both sides over the same stored particles; beta of a float
# particle is a reciprocal square root refined in FP64 (1.5e-14 relative), and
# the flux rows' cancellation stays below 1e3
TOL = 1e-11


def _rows(cfg, w, x, vx, vp, s):
    live = x >= 0
    x, vx, vp = x[live], vx[live], vp[live]
    c = np.floor(x).astype(int)
    f, v2, u = x - c, vx * vx + vp, cfg["u"]
    b = 1 / np.sqrt(1 + v2 / u**2) if cfg["beta_kind"] == "smooth" else np.minimum(1.0, u / np.sqrt(v2))
    out = []
    for q in (np.ones(len(x)), vx, 0.5 * cfg["species"][s]["mass"] * v2):
        m = (np.bincount(c, w[s] * b * (1 - f) * q, cfg["nx"] + 1) +
             np.bincount(c + 1, w[s] * b * f * q, cfg["nx"] + 1)) / cfg["dx"]
        m[[0, -1]] *= 2
        out.append(m)
    return out


def _particles(rng, cfg, s, x):
    """Velocities and positions an F32 context stores as they are."""
    vt = np.sqrt(cfg["species"][s]["temperature"] / cfg["species"][s]["mass"])
    vx = (vt * rng.standard_normal(len(x)) + 0.2 * vt).astype(np.float32).astype(np.float64)
    vp = (vt * vt * rng.chisquare(2, len(x))).astype(np.float32).astype(np.float64)
    return np.where(x < 0, -1.0, np.rint(x * 2.0**16) / 2.0**16), vx, vp


def _check(sim, cfg, parts):
    got, w = sim.moments(0).cpu().numpy(), sim.status(0)["weight"]
    for s in range(2):
        want = _rows(cfg, w, *parts[s], s)
        for r in range(3):
            assert rel_inf(got[1 + 3 * s + r], want[r]) <= TOL, (s, r)


@pytest.mark.parametrize("prec,beta", [("f32", "step"), ("f64", "smooth")])
@pytest.mark.parametrize("chunk", [64, 256, 1024])
def test_lengths_about_the_batches(gpu_lib, prec, beta, chunk):
    """A grid that fits the window, so that an import is summed as it lies: two
    cells up and down about a rising trend, a tenth of the slots dead."""
    print_case(f"moment batches {prec} {beta} chunk={chunk}")
    cfg = workloads.sheath(100, 30, 3.0, beta_kind=beta, seed=2)
    sim = gpu_lib.Sim(cfg, precision=prec, sort_every=0, chunk=chunk | gpu_lib.EXACT)
    assert sim.launch_shape()[0] == chunk
    rng = np.random.default_rng(chunk)
    for n in (1, 2, 63, 64, 65, 127, 128, 129, 191, 192, 255, 256, 257, 320, 383, 448, 511, 512, 513, 640, 1023, 1024,
              1025, 1100, 3000):
        parts = []
        for s, m in ((0, n), (1, max(1, n - 3))):
            x = np.clip(np.linspace(5, 95, m) + rng.uniform(-2, 2, m), 0.0, 99.9)
            x[rng.random(m) < 0.1] = -1.0
            parts.append(_particles(rng, cfg, s, x))
            sim.import_particles(0, s, *parts[s])
        if all((p[0] >= 0).any() for p in parts):
            _check(sim, cfg, parts)
    sim.close()


@pytest.mark.parametrize("prec", ["f32", "f64"])
@pytest.mark.parametrize("nx,ppc,chunk,bucket", [
    (500, 40, 1024, 1),    # about 26 cells to a chunk
    (500, 40, 64, 32),     # keys of 32 cells
    (500, 3, 1024, 1),     # thin: 341 cells to a chunk, whole rows
    (500, 9, 512, 1),      # 57
    (500, 200, 256, 100),  # keys about the window's length
])
def test_sorted_chunks_and_thin_runs(gpu_lib, prec, nx, ppc, chunk, bucket):
    print_case(f"moments of sorted chunks {prec} {nx} x {ppc} chunk={chunk} bucket={bucket}")
    cfg = workloads.sheath(nx, ppc, 3.0, seed=3)
    sim = gpu_lib.Sim(cfg, precision=prec, sort_every=8, sort_bucket=bucket, chunk=chunk | gpu_lib.EXACT)
    for steps in (0, 1, 5, 2):
        sim.step(steps)
        _check(sim, cfg, [sim.export_particles(0, s) for s in range(2)])
    sim.close()


def test_cells_below_the_first_batch(gpu_lib):
    """One chunk of 1024 slots whose second half lies 20 and 60 cells below its
    first: within the window's reach below it and beyond."""
    print_case("moments of cells below the first batch")
    cfg = workloads.sheath(100, 30, 3.0, seed=4)
    sim = gpu_lib.Sim(cfg, precision="f64", sort_every=0, chunk=1024 | gpu_lib.EXACT)
    rng = np.random.default_rng(1)
    for down in (20, 60):
        parts = []
        for s in range(2):
            x = np.concatenate([rng.uniform(70, 90, 512), rng.uniform(70, 90, 512) - down])
            parts.append(_particles(rng, cfg, s, x))
            sim.import_particles(0, s, *parts[s])
        _check(sim, cfg, parts)
    sim.close()


@pytest.mark.parametrize("prec,beta", [("f32", "step"), ("f64", "smooth")])
@pytest.mark.parametrize("nx,ppc,chunk", [
    (100, 40, 512),    # fits the window
    (127, 40, 256),    # 128 and 129 nodes: about the window's
    (128, 40, 1024),
    (150, 30, 64),
    (300, 60, 1024),
    (2729, 9, 512),
])
def test_windows_across_the_ends_of_a_box(gpu_lib, prec, beta, nx, ppc, chunk):
    """Particles that crossed the ends since the sort lie in chunks of the other
    end; nodes 0 and nx each keep their own sums."""
    print_case(f"moments of a box {nx} x {ppc} chunk={chunk} {prec} {beta}")
    cfg = workloads.langmuir_box(1.0, nx=nx, ppc=ppc, seed=nx, beta_kind=beta)
    sim = gpu_lib.Sim(cfg, precision=prec, sort_every=16, chunk=chunk | gpu_lib.EXACT)
    for steps in (0, 1, 4, 10, 1):
        sim.step(steps)
        _check(sim, cfg, [sim.export_particles(0, s) for s in range(2)])
    sim.close()


def test_windows_of_boxes_and_sheaths_share_a_launch(gpu_lib):
    cfgs = [dict(workloads.langmuir_box(1.0, nx=200, ppc=30, seed=1), run=0),
            dict(workloads.sheath(300, 20, 4.0, seed=2), run=1),
            dict(workloads.langmuir_box(0.5, nx=90, ppc=20, seed=3), run=2),
            dict(workloads.plates_sheath(0.0158, ppc=300, seed=4), run=3)]
    print_case("moments of boxes, sheaths and plates in one launch")
    sim = gpu_lib.Sim(cfgs, precision="f64", sort_every=8, chunk=256 | gpu_lib.EXACT)
    for steps in (1, 12):
        sim.step(steps)
        sim.moments_sample(-1)
        st = sim.status()
        for r, cfg in enumerate(cfgs):
            win = sim.moments_window(r, reset=True).cpu().numpy()
            for s in range(2):
                want = _rows(cfg, st[r]["weight"], *sim.export_particles(r, s), s)
                for k in range(3):
                    if np.abs(want[k]).max() > 0:
                        assert rel_inf(win[1 + 3 * s + k], want[k]) <= TOL, (r, s, k)
    sim.close()
