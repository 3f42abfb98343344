"""2D sort tiles fitted to the size of the run: the sort's permutation is the
stable order of the tiles' keys on both sides of the sizes where the tile is
halved, from a state with holes, and the charge is the same as with the
smallest tile."""
import numpy as np
import pytest

import workloads
from parity_util import print_case, rel_inf

pytestmark = pytest.mark.gpu


# loads are 2 * nx * ny * ppc particles; a tile of 2048 is halved below 2097152
@pytest.mark.parametrize("nx,ny,ppc,sort_tile,prec", [
    (4, 4, 1, 0, "f64"),           # a few particles
    (60, 64, 5, 32768, "f32"),     # tile 1024
    (64, 64, 255, 2048, "f32"),    # tile 1024
    (64, 64, 256, 2048, "f32"),    # tile 2048
    (100, 64, 20, 3072, "f64"),    # not halved: not a multiple of 2048
    (512, 512, 1, 32768, "f32"),   # 4096 keys: tile 4096
])
def test_fitted_sort_tile(gpu_lib, nx, ny, ppc, sort_tile, prec):
    print_case(f"fit 2d {nx}x{ny} ppc={ppc} sort_tile={sort_tile} {prec}")
    cfg = workloads.sheath2d(nx, ny, ppc, 3.0, seed=4)
    tile = 8
    sims = [gpu_lib.Sim2D(cfg, ny, precision=prec, sort_every=0, tile=tile, margin=8, sort_tile=st, record_perm=True)
            for st in (sort_tile, 1024)]
    for sim in sims:
        sim.step(3)
    nty = -(-ny // tile)
    before = [sims[0].export_particles(s) for s in range(2)]
    for s in range(2):
        sims[1].import_particles(s, *before[s])  # FP64 atomics: the steps agree to rounding only
    for sim in sims:
        sim.sort_now()
        sim.refresh_fields()
    for s in range(2):
        got, other = sims[0].export_particles(s), sims[1].export_particles(s)
        for a, b in zip(got, other):
            assert np.array_equal(a, b)
        x, y = before[s][:2]
        live = np.nonzero(x >= 0)[0]
        key = (np.floor(x[live]) // tile) * nty + np.floor(y[live]) // tile
        order = live[np.argsort(key, kind="stable")]
        for a, b in zip(got, before[s]):
            assert np.array_equal(a, b[order])
        for sim in sims:
            assert np.array_equal(sim.perm(s), order)
    # FP64 sums of the same terms in another order
    for s in range(2):
        assert rel_inf(sims[0].grid()["Q"][s], sims[1].grid()["Q"][s]) <= 1e-12
    for sim in sims:
        sim.close()
