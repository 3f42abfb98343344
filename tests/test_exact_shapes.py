"""Launch shapes taken exactly (SLPIC_EXACT): the planning on the CPU, and the
comparisons with the oracle that name a push chunk or a sort tile run at that
chunk and tile on the GPU.  A small run set takes smaller ones otherwise, so
that without the flag every shape of a small test is the smallest."""
import ctypes
import math

import numpy as np
import pytest

import oracle
import workloads
from parity_util import oracle_state, print_case, push_oracle_to_gpu, rel_inf


def test_exact_values_are_planned_as_given():
    import torch  # noqa: F401
    from paper_1511_08225_amd import slpic
    L, E = slpic.lib(), slpic.EXACT
    c = slpic.run_config(workloads.small_sheath())

    def ws(**kw):
        return L.slpic_workspace_bytes(ctypes.byref(c), 1, ctypes.byref(slpic.tuning("f32", **kw)))
    # the (key, tile) table grows as the tile shrinks: fitted tiles of a small
    # run are the smallest whatever was asked for, exact ones are not
    assert ws(sort_tile=32768) == ws(sort_tile=1024) == ws(sort_tile=1024 | E) > ws(sort_tile=16384 | E)
    assert ws(sort_tile=0 | E) == ws(sort_tile=16384 | E)  # the default, exactly
    assert ws(chunk=1024) == ws(chunk=64) == ws(chunk=64 | E) > ws(chunk=1024 | E)
    assert ws(chunk=0 | E) == ws(chunk=512 | E)
    for bad in ({"chunk": 100 | E}, {"chunk": 2048 | E}, {"sort_tile": 32769 | E}, {"sort_tile": 65536 | E},
                {"chunk": -64}, {"sort_tile": -1024}):
        assert ws(**bad) == 0, bad
    c2 = slpic.run_config(workloads.sheath2d(nx=64, ny=64, ppc=4))

    def ws2(tile):
        t = slpic.Tuning2D()
        t.sort_tile = tile
        return L.slpic2d_workspace_bytes(ctypes.byref(c2), 64, ctypes.byref(t))
    assert ws2(32768) == ws2(1024) == ws2(1024 | E) > ws2(32768 | E) == ws2(0 | E)
    assert ws2(1536 | E) == ws2(65536 | E) == 0


class _Exact:
    """The library with every context's chunk and sort tile taken exactly, and
    the chunk given where the test names none; the shapes are asserted."""

    def __init__(self, lib, chunk=0):
        self._lib, self._chunk = lib, chunk

    def __getattr__(self, name):
        return getattr(self._lib, name)

    def Sim(self, configs, precision="f32", chunk=0, sort_tile=0, **kw):
        chunk = chunk or self._chunk
        sim = self._lib.Sim(configs, precision=precision, chunk=chunk | self._lib.EXACT,
                            sort_tile=sort_tile | self._lib.EXACT, **kw)
        assert sim.launch_shape() == (chunk or {"f32": 512, "f64": 256}[precision], sort_tile or 16384)
        return sim


@pytest.mark.gpu
def test_fitted_and_exact_shapes(gpu_lib):
    E, cfg = gpu_lib.EXACT, workloads.small_sheath()  # 12800 particles
    for kw, want in (({}, (64, 1024)), ({"chunk": 1024, "sort_tile": 32768}, (64, 1024)),
                     ({"chunk": E, "sort_tile": E}, (512, 16384)),
                     ({"chunk": 128 | E, "sort_tile": 32768 | E}, (128, 32768)),
                     ({"chunk": 1024 | E, "sort_tile": 512}, (1024, 512))):
        sim = gpu_lib.Sim(cfg, precision="f32", **kw)
        assert sim.launch_shape() == want, kw
        sim.close()


# loads are 2 nx ppc particles: a sorting context halves chunks below 2048 of them,
# one that does not below 256
@pytest.mark.gpu
@pytest.mark.parametrize("nx,ppc,prec,kw,chunk", [
    (512, 255, "f32", {"chunk": 128}, 64), (512, 256, "f32", {"chunk": 128}, 128),
    (1024, 511, "f64", {"chunk": 512}, 256), (1024, 512, "f64", {"chunk": 512}, 512),
    (100, 1000, "f32", {}, 64), (100, 1000, "f32", {"sort_bucket": 256}, 64),
    (100, 1000, "f32", {"sort_every": 0}, 512), (100, 1000, "f64", {"sort_every": 0}, 256),
    (100, 1000, "f32", {"sort_bucket": 0}, 512), (100, 1000, "f32", {"sort_bucket": 257}, 512),
    (512, 127, "f32", {"sort_every": 0}, 256), (512, 128, "f32", {"sort_every": 0}, 512),
    (256, 63, "f64", {"sort_every": 0}, 64), (256, 64, "f64", {"sort_every": 0}, 128),
])
def test_fitted_chunk_steps_like_the_oracle(gpu_lib, nx, ppc, prec, kw, chunk):
    print_case(f"fitted chunk {nx} x {ppc} {prec} {kw}")
    cfg = workloads.sheath(nx, ppc, 4.0, seed=6, sort_every=0)
    run = oracle.Run(cfg)
    run.step(2)
    sim = gpu_lib.Sim(cfg, precision=prec, **kw)
    assert sim.launch_shape()[0] == chunk
    push_oracle_to_gpu(sim, 0, run, quantize=prec == "f32")
    sim.step(1)
    run.step(1)
    g, o = sim.grid(0), run.grid()
    for s in range(2):  # the bounds of the other one-step comparisons
        assert rel_inf(g["Q"][s], o["Q"][s]) <= {"f64": 1e-12, "f32": 1e-5}[prec], s
    sim.close()


@pytest.mark.gpu
def test_fitted_chunk_of_unsorted_plates(gpu_lib):
    """Counted by the eighth of its slots that the box fills."""
    for ppc, want in ((500, 64), (2000, 128), (9000, 512)):
        sim = gpu_lib.Sim(workloads.plates_sheath(0.0158, ppc=ppc), precision="f32", sort_every=0)
        assert sim.launch_shape()[0] == want, ppc
        sim.close()


@pytest.mark.gpu
@pytest.mark.parametrize("u,chunk", [(2.0, 0), (10.0, 0), (math.inf, 0), (2.0, 64), (2.0, 128), (2.0, 256),
                                     (2.0, 1024)])
def test_sheath_step_at_every_chunk(gpu_lib, u, chunk):
    import test_gpu_parity
    test_gpu_parity.test_one_step_f32_developed_sheath(_Exact(gpu_lib), u, chunk)


@pytest.mark.gpu
@pytest.mark.parametrize("kind", ["smooth", "limit", "plates", "periodic", "periodic_smooth"])
@pytest.mark.parametrize("chunk", [64, 128, 256, 512, 1024])
def test_other_pushes_f32_at_every_chunk(gpu_lib, kind, chunk):
    """The float pushes beside the step sheath's, one step from the oracle's
    state: the bounds of the other FP32 one-step comparisons."""
    print_case(f"f32 one step {kind} chunk={chunk}")
    if kind == "plates":
        cfg, warm = workloads.plates_sheath(0.0158, ppc=40, sort_every=1, seed=23), 400
    elif kind.startswith("periodic"):
        cfg, warm = workloads.langmuir_box(0.5, nx=150, ppc=40, seed=31, sort_every=8), 20  # none in step 21
        if kind.endswith("smooth"):
            cfg["beta_kind"] = "smooth"
    else:
        cfg, warm = workloads.sheath(200, 60, 3.0, sort_every=1, seed=25), 60
        if kind == "smooth":
            cfg["beta_kind"] = "smooth"
        else:
            cfg["limit_profile"] = cfg["u"] * np.random.default_rng(7).uniform(0.3, 1.7, 201)
    run = oracle.Run(cfg)
    run.step(warm)
    sim = _Exact(gpu_lib).Sim(cfg, precision="f32", sort_every=0, chunk=chunk)
    push_oracle_to_gpu(sim, 0, run, quantize=True)
    g, o = sim.grid(0), run.grid()
    for s in range(2):
        assert rel_inf(g["Q"][s], o["Q"][s]) <= 1e-6, s
    before = [run.nslots(s) for s in range(2)]
    sim.step(1)
    run.step(1)
    g, o = sim.grid(0), run.grid()
    for s in range(2):
        assert rel_inf(g["Q"][s], o["Q"][s]) <= 1e-5, s
        xg, vxg, _ = sim.export_particles(0, s)
        assert before[s] <= len(xg)
        if kind.startswith("periodic"):  # no slot moves: each particle (a wrapped one across the ends)
            xo, vxo, _ = oracle_state(run, s)
            d = np.abs(xg - xo)
            assert np.minimum(d, cfg["nx"] - d).max() <= 1e-5
            assert np.abs(vxg - vxo).max() <= 1e-5 * np.abs(vxo).max()
    sim.close()


@pytest.mark.gpu
@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("nx,ppc,u,chunk", [
    (126, 30, 0.5, 256), (127, 30, 0.5, 256), (128, 30, math.inf, 128), (129, 30, 0.5, 1024),
    (128, 60, 0.5, 512), (300, 40, 2.0, 512), (300, 40, math.inf, 1024), (2729, 5, math.inf, 512)])
def test_ring_windows_at_their_chunks(gpu_lib, prec, nx, ppc, u, chunk):
    import test_gpu_ring_window
    test_gpu_ring_window.test_charge_across_the_ends(_Exact(gpu_lib), prec, nx, ppc, u, chunk)


@pytest.mark.gpu
@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("nx", [96, 100, 110])
@pytest.mark.parametrize("chunk", [64, 512, 1024])
def test_rings_shorter_than_the_window(gpu_lib, prec, nx, chunk):
    """Steps of up to 31 cells: the window starts 32 nodes below the lowest
    cell, and with fewer than 128 nodes goes round the box more than once."""
    print_case(f"short ring nx={nx} chunk={chunk} {prec}")
    cfg = workloads.langmuir_box(1.0, nx=nx, ppc=30, seed=nx, sort_every=8)
    cfg["dt"] *= 31.0
    for sp in cfg["species"]:
        sp["mass"] *= 1e6  # the fields hardly turn the particles
        sp["temperature"] *= 1e6
    run = oracle.Run(cfg)
    sim = _Exact(gpu_lib).Sim(cfg, precision=prec, sort_every=0, chunk=chunk)
    # FP64: sums in another order; FP32: a velocity to 1e-6 moves a particle by
    # 3.1e-5 cells, which shifts at most twice that share of a node's charge
    tol = {"f64": 1e-12, "f32": 1e-4}[prec]
    for k in range(3):
        push_oracle_to_gpu(sim, 0, run, quantize=prec == "f32")
        x0 = oracle_state(run, 0)[0]
        sim.step(1)
        run.step(1)
        d = np.abs(oracle_state(run, 0)[0] - x0)
        assert np.minimum(d, nx - d).max() > 20.0
        g, o = sim.grid(0), run.grid()
        for s in range(2):
            assert rel_inf(g["Q"][s], o["Q"][s]) <= tol, (k, s)
    sim.close()


@pytest.mark.gpu
@pytest.mark.parametrize("nx,ppc,chunk,prec,beta,sort", [
    (300, 7, 512, "f64", "smooth", 0),
    (300, 21, 1024, "f32", "step", 1),     # several windows' cells in a chunk: two passes of 512 slots
    (1200, 3, 1024, "f64", "step", 1),
    (64, 900, 1024, "f32", "smooth", 1),   # about one cell to a chunk
    (2729, 4, 512, "f64", "step", 1)])
def test_moments_at_their_chunks(gpu_lib, nx, ppc, chunk, prec, beta, sort):
    """The six particle rows (phi, a field solve over them, carries 64 x 900's
    systematic 3e-14 of the charge, whatever the chunk, to 1.3e-11)."""
    print_case(f"moments nx={nx} ppc={ppc} chunk={chunk} {prec} {beta} sort={sort}")
    cfg = workloads.sheath(nx, ppc, 5.0, beta_kind=beta, seed=3)
    run = oracle.Run(cfg)
    sim = _Exact(gpu_lib).Sim(cfg, precision=prec, sort_every=sort, chunk=chunk)
    push_oracle_to_gpu(sim, 0, run, quantize=prec == "f32")
    if sort:
        sim.sort_now()
    want, got = run.moments(), sim.moments(0).cpu().numpy()
    for row in range(1, 7):
        assert rel_inf(got[row], want[row]) <= 1e-11, row
    sim.close()


@pytest.mark.gpu
def test_moment_window_placed_by_a_later_pass(gpu_lib):
    """A chunk whose first 512 slots are dead, one whose live particles start
    in the second pass's last row, and one with none."""
    cfg = workloads.sheath(300, 20, 5.0, seed=3)
    run = oracle.Run(cfg)
    for s in range(2):
        x, vx, vp = oracle_state(run, s)
        o = np.argsort(x)
        x, vx, vp = x[o], vx[o], vp[o]
        x[:600] = -1.0
        x[1024:1024 + 1000] = -1.0
        x[2048:3072] = -1.0
        run.set_particles(s, x, vx, np.sqrt(vp), np.zeros(len(x)))
    sim = _Exact(gpu_lib).Sim(cfg, precision="f64", sort_every=1, chunk=1024)
    sim.sort_now()  # the context's slots count as sorted ...
    push_oracle_to_gpu(sim, 0, run, quantize=False)
    tol = 1e-11  # FP64 sums of the same terms in another order, cancelling by less than 1e3
    want = run.moments()
    imported = sim.moments(0).cpu().numpy()
    ckpt = sim.workspace.clone()
    sim.sort_now()
    sim.workspace.copy_(ckpt)  # ... and so do the ones with holes: in order by cell, not compacted
    got = sim.moments(0).cpu().numpy()
    for row in range(7):
        assert rel_inf(imported[row], want[row]) <= tol, row
        assert rel_inf(got[row], want[row]) <= tol, row
    sim.close()


@pytest.mark.gpu
@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("bucket", [1, 4, 5, 0])
@pytest.mark.parametrize("sort_tile", [0, 2048])
def test_sort_permutation_at_their_tiles(gpu_lib, prec, bucket, sort_tile):
    import test_gpu_parity
    test_gpu_parity.test_sort_permutation_bit_exact(_Exact(gpu_lib), prec, bucket, sort_tile)


@pytest.mark.gpu
@pytest.mark.parametrize("bucket", [4, 1])
def test_sort_permutation_production_size_tiles_of_16384(gpu_lib, bucket):
    import test_gpu_parity
    test_gpu_parity.test_sort_permutation_production_size(_Exact(gpu_lib), bucket, 16384)


@pytest.mark.gpu
@pytest.mark.parametrize("nx,ppc,bucket,tile,prec", [
    (2729, 30, 7, 32768, "f32"),
    (700, 150, 0, 32768, "f64"),    # one key: a whole tile in it
    (700, 150, 350, 32768, "f32"),  # two
    (4, 1, 1, 0, "f64"),
])
def test_sort_of_the_largest_tiles(gpu_lib, nx, ppc, bucket, tile, prec):
    import test_gpu_sort_table
    test_gpu_sort_table.test_sort_is_stable_over_table_sizes(_Exact(gpu_lib), nx, ppc, bucket, tile, prec)


@pytest.mark.gpu
def test_2d_sort_of_the_largest_tile(gpu_lib):
    """46080 particles per species, 69120 slots in three tiles (fitted: of 1024)."""
    cfg = workloads.sheath2d(60, 64, 12, 3.0, tile=8, seed=4)
    sims = [gpu_lib.Sim2D(cfg, 64, precision="f32", sort_every=0, tile=8, margin=8, sort_tile=st, record_perm=True)
            for st in (32768 | gpu_lib.EXACT, 0)]
    assert sims[0].workspace_bytes < sims[1].workspace_bytes
    for sim in sims:
        sim.sort_now()
    for s in range(2):
        assert np.array_equal(sims[0].perm(s), sims[1].perm(s)), s
        for a, b in zip(sims[0].export_particles(s), sims[1].export_particles(s)):
            assert np.array_equal(a, b), s
    for sim in sims:
        sim.close()
