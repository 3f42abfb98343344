"""Moments of particles out of cell order, in workgroups that keep the whole
grid's rows in LDS, against the oracle: grids about the 128 nodes of the ordered
kernel's window and the largest, ranges of one chunk and of several across the
species and the runs, rows cut short; and the change from one kernel to the
other as an import, a sort and further steps change the order."""
import math

import numpy as np
import pytest

import oracle
import workloads
from parity_util import oracle_state, print_case, push_oracle_to_gpu, rel_inf

pytestmark = pytest.mark.gpu

# FP64 sums on both sides over the same stored particles; beta of a float
# particle is a reciprocal square root refined in FP64 (1.5e-14 relative), and
# the rows' cancellation (flux) stays below 1e3.
TOL = 1e-11


@pytest.mark.parametrize("nx,ppc,prec,beta,u,kw", [
    (126, 9, "f32", "step", 5.0, {"sort_every": 0}),        # 127 and 128 nodes: one LDS window
    (127, 40, "f64", "smooth", 5.0, {"sort_every": 0}),
    (128, 9, "f32", "step", 5.0, {"sort_every": 0}),        # 129: whole rows
    (300, 7, "f64", "smooth", math.inf, {"sort_every": 0}),
    (300, 70, "f32", "smooth", 5.0, {"sort_every": 0}),     # several workgroups
    (1500, 600, "f32", "step", 5.0, {"sort_every": 0}),     # more than 768: chunks grouped further
    (2729, 3, "f64", "step", 5.0, {"sort_every": 0}),       # the largest grid
    (200, 30, "f32", "step", 5.0, {"sort_every": 1, "sort_bucket": 0}),
    (500, 30, "f64", "step", 5.0, {"sort_every": 1, "sort_bucket": 129}),
])
def test_unordered_moments_match_oracle(gpu_lib, nx, ppc, prec, beta, u, kw):
    print_case(f"unordered moments nx={nx} ppc={ppc} {prec} {beta} {kw}")
    cfg = workloads.sheath(nx, ppc, u, beta_kind=beta, seed=3)
    run = oracle.Run(cfg)
    rng = np.random.default_rng(nx)
    for s in range(2):  # the slots in any order, some of them dead
        x, vx, vp = oracle_state(run, s)
        o = rng.permutation(len(x))
        x = np.where(rng.random(len(x)) < 0.05, -1.0, x[o])
        run.set_particles(s, x, vx[o], np.sqrt(vp[o]), np.zeros(len(x)))
    sim = gpu_lib.Sim(cfg, precision=prec, **kw)
    push_oracle_to_gpu(sim, 0, run, quantize=prec == "f32")
    want = run.moments()
    got = sim.moments(0).cpu().numpy()
    for _ in range(2):
        sim.moments_sample(-1)
    assert sim.status(0)["moment_samples"] == 2
    win = sim.moments_window(0, reset=True).cpu().numpy()
    for row in range(7):
        assert rel_inf(got[row], want[row]) <= TOL, row
        assert rel_inf(win[row], want[row]) <= TOL, row
    sim.close()


def test_unordered_ragged_runs_share_a_launch(gpu_lib):
    cfgs = [dict(workloads.sheath(nx, ppc, u, seed=nx), run=r)
            for r, (nx, ppc, u) in enumerate([(64, 9, 2.0), (700, 3, 8.0), (5, 50, math.inf), (130, 100, 4.0)])]
    sim = gpu_lib.Sim(cfgs, precision="f64", sort_every=0)
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
    assert [s["moment_samples"] for s in sim.status()] == [1, 2, 1, 1]
    sim.close()


@pytest.mark.parametrize("kw", [{"sort_every": 0}, {"sort_every": 8, "graph_steps": 8},
                                {"sort_every": 100, "graph_steps": 100}])
def test_moments_follow_the_order(gpu_lib, kw):
    """The sums do not depend on which kernel the order picks: after a load,
    a sort, steps few and many, an import, and in-step samples of a captured
    block, against sums written out over the exported particles."""
    import torch
    print_case(f"moments by order {kw}")
    cfg = workloads.sheath(300, 40, 4.0, seed=5)
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        sim = gpu_lib.Sim(cfg, precision="f64", **kw)

        def check():
            torch.cuda.synchronize()
            got, w = sim.moments(0).cpu().numpy(), sim.status(0)["weight"]
            for s in range(2):
                x, vx, vp = sim.export_particles(0, s)
                live = x >= 0
                x, vx, vp = x[live], vx[live], vp[live]
                c = np.floor(x).astype(int)
                f, v2 = x - c, vx * vx + vp
                b = np.minimum(1.0, cfg["u"] / np.sqrt(v2))
                for row, q in enumerate((np.ones(len(x)), vx, 0.5 * cfg["species"][s]["mass"] * v2)):
                    m = np.bincount(c, w[s] * b * (1 - f) * q, 301) + np.bincount(c + 1, w[s] * b * f * q, 301)
                    m /= cfg["dx"]
                    m[[0, -1]] *= 2
                    assert rel_inf(got[1 + 3 * s + row], m) <= TOL, (s, row)
        check()
        for act in (sim.sort_now, lambda: sim.step(20), lambda: sim.step(100), sim.sort_now, lambda: sim.step(8)):
            act()
            check()
        for s in range(2):
            p = sim.export_particles(0, s)
            o = np.random.default_rng(1).permutation(len(p[0]))
            sim.import_particles(0, s, *(a[o] for a in p))
        check()
        sim.set_sampling(4 if kw["sort_every"] != 100 else 50)
        sim.step(100)
        torch.cuda.synchronize()
        assert sim.status(0)["moment_samples"] == (25 if kw["sort_every"] != 100 else 2)
        # the window's sum holds the last state's sample: without it, one fewer
        sim.moments_window(0, reset=True)
        sim.moments_sample(-1)
        torch.cuda.synchronize()
        win, one = sim.moments_window(0).cpu().numpy(), sim.moments(0).cpu().numpy()
        for row in range(7):
            assert rel_inf(win[row], one[row]) <= TOL, row
        check()
    sim.close()


@pytest.mark.parametrize("prec", ["f64", "f32"])
def test_unsorted_2d_moments_written_out(gpu_lib, prec):
    """The 2D pass before any sort, after one, and with one species imported
    since, whose slots are then unsorted while the other's tiles are not."""
    from test_gpu_moments import _plane_moments
    ny = 32
    cfg = workloads.sheath2d(70, ny, 60, 3.0, tile=8, seed=5)
    sim = gpu_lib.Sim2D(cfg, ny, precision=prec, sort_every=0, tile=8, margin=2)

    def check(what):
        print_case(f"2D moments {what} {prec}")
        got, want = sim.moments().cpu().numpy(), _plane_moments(sim, cfg, ny)
        for row in range(6):
            assert rel_inf(got[1 + row], want[row]) <= TOL, (what, row)
    check("never sorted")
    sim.sort_now()
    check("sorted")
    sim.step(5)
    check("five steps on")
    p = sim.export_particles(1)
    o = np.random.default_rng(1).permutation(len(p[0]))
    sim.import_particles(1, *(a[o] for a in p))
    check("ions imported")
    sim.sort_now()
    check("sorted again")
    sim.close()
