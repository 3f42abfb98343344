"""The cell sort over the sizes of its (key, tile) table: one scan block or
several, written whole by its tiles or zeroed first, one key or thousands.  The
sorted particles are NumPy's stable argsort of the unsorted ones, bit for bit,
and two sorts in a row leave them alone."""
import numpy as np
import pytest

import workloads
from parity_util import print_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,ppc,bucket,tile,prec", [
    (4, 3, 1, 0, "f64"),           # 8 entries
    (64, 40, 0, 1024, "f32"),      # one key
    (128, 120, 1, 1024, "f32"),    # 23 tiles per species: 5888 entries, one scan block
    (256, 120, 1, 1024, "f64"),    # 45 tiles: 23040 entries, three scan blocks
    (1000, 80, 1, 1024, "f32"),    # 118 tiles: 236000 entries, the table written whole
    (1200, 80, 1, 1024, "f32"),    # 141 tiles: 338400 entries, the table zeroed first
    (2729, 30, 7, 32768, "f32"),   # the largest tile: 4 per species at most
])
def test_sort_is_stable_over_table_sizes(gpu_lib, nx, ppc, bucket, tile, prec):
    print_case(f"sort table nx={nx} ppc={ppc} bucket={bucket} tile={tile} {prec}")
    cfg = workloads.sheath(nx, ppc, 4.0, seed=2)
    sim = gpu_lib.Sim(cfg, precision=prec, sort_every=0, sort_bucket=bucket, sort_tile=tile, chunk=1024,
                      record_perm=True)
    sim.step(3)  # holes from the wall, new particles at the end
    before = [sim.export_particles(0, s) for s in range(2)]
    sim.sort_now()
    for s in range(2):
        x, vx, vp = before[s]
        key = np.floor(x) // bucket if bucket else np.zeros(len(x))
        order = np.nonzero(x >= 0)[0]
        order = order[np.argsort(key[order], kind="stable")]
        got = sim.export_particles(0, s)
        for a, b in zip(got, (x[order], vx[order], vp[order])):
            assert np.array_equal(a, b)
        assert np.array_equal(sim.perm(0, s), order)
    after = [sim.export_particles(0, s) for s in range(2)]
    sim.sort_now()
    for s in range(2):
        for a, b in zip(sim.export_particles(0, s), after[s]):
            assert np.array_equal(a, b)
    sim.close()
