"""The scan of the sort table and of a limit change's copy counts on both sides
of the block count (1024 blocks of 8192 entries) from which the block sums are
scanned in a launch of their own: sorts against NumPy's stable argsort, limit
changes over few and over many slots against one another, bit for bit."""
import numpy as np
import pytest

import workloads
from parity_util import print_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("cf", [
    1.5338,  # 2097 tiles of 512 slots per species, 2000 keys: 1024 blocks
    1.534,   # 2098 tiles: 1025 blocks
    4.0,     # 5469 tiles: 2671 blocks
])
def test_sort_of_many_scan_blocks(gpu_lib, cf):
    nx, ppc, tile = 2000, 350, 512
    tiles = -(-int(np.ceil(cf * nx * ppc)) // tile)
    blocks = -(-2 * nx * tiles // 8192)
    print_case(f"sort over {blocks} scan blocks")
    assert blocks == {1.5338: 1024, 1.534: 1025, 4.0: 2671}[cf]
    cfg = workloads.sheath(nx, ppc, 4.0, seed=2, capacity_factor=cf)
    sim = gpu_lib.Sim(cfg, precision="f32", sort_every=0, sort_tile=tile, record_perm=True)
    sim.step(3)  # holes from the wall, new particles at the end
    before = [sim.export_particles(0, s) for s in range(2)]
    sim.sort_now()
    for s in range(2):
        x, vx, vp = before[s]
        order = np.nonzero(x >= 0)[0]
        order = order[np.argsort(np.floor(x[order]), kind="stable")]
        for a, b in zip(sim.export_particles(0, s), (x[order], vx[order], vp[order])):
            assert np.array_equal(a, b), s
        assert np.array_equal(sim.perm(0, s), order), s
    sim.close()


def test_limit_change_over_many_scan_blocks(gpu_lib):
    """The same particles in 2 x 16000 and in 2 x 4.5M slots (1094 scan blocks)."""
    got = []
    for cf in (2.5, 7000.0):
        print_case(f"limit change, capacity factor {cf}")
        cfg = workloads.sheath(64, 100, 2.0, seed=3, capacity_factor=cf)
        sim = gpu_lib.Sim(cfg, precision="f64", sort_every=0)
        sim.set_speed_limit(0, 2.0 * cfg["u"], 0.5 * cfg["dt"])
        got.append([sim.export_particles(0, s) for s in range(2)])
        assert sim.status(0)["error_flags"] == 0
        sim.close()
    for s in range(2):
        assert len(got[0][s][0]) > 0
        for a, b in zip(got[0][s], got[1][s]):
            assert np.array_equal(a, b), s
