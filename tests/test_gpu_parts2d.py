"""2D pushes with sorted tiles split over several workgroups, at tile lengths
where a part is empty, one row, cut short or several rows: one step from the
oracle's sorted state, and the counts of the step."""
import pytest

import oracle
import workloads
from parity_util import print_case
from test_gpu_parity2d import _compare, _push_to_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("nx,ny,ppc,tile,per_thread,kind", [
    (16, 16, 4, 8, 1, "step"),      # parts of less than a row
    (12, 8, 64, 8, 1, "smooth"),    # tiles of 4096 and of half a tile
    (8, 8, 300, 8, 4, "step"),      # one tile a species, rows of 1024
    (24, 32, 40, 8, 2, "step"),     # several tiles, several parts
    (40, 32, 3, 4, 1, "step"),      # 160 workgroups of 48: not split
    (4, 4, 1, 1, 8, "step"),        # tiles of one particle
])
def test_split_tiles_match_oracle(gpu_lib, prec, nx, ny, ppc, tile, per_thread, kind):
    print_case(f"2d parts {nx}x{ny} ppc={ppc} tile={tile} per_thread={per_thread} {kind} {prec}")
    cfg = workloads.sheath(nx=nx, ppc=ppc, u_over_vti=3.0, beta_kind=kind, seed=8, sort_every=0)
    run = oracle.Run2D(cfg, ny, tile=tile)
    run.step(2)
    sim = gpu_lib.Sim2D(cfg, ny, precision=prec, sort_every=0, tile=tile, margin=8, per_thread=per_thread)
    _push_to_gpu(sim, run, quantize=prec == "f32")
    sim.sort_now()
    run.sort()
    sim.refresh_fields()
    run.refresh_fields()
    before = sim.status()
    sim.step(1)
    run.step(1)
    after = sim.status()
    assert after["pushed_total"] - before["pushed_total"] == sum(before["nslots"])
    # the bounds of the other one-step comparisons with the oracle
    if prec == "f64":
        _compare(sim, run, tol_q=1e-12, tol_x=1e-11, tol_v=1e-11)
    else:
        _compare(sim, run, tol_q=1e-5, tol_x=1e-5, tol_v=1e-5, exact_counts=False)
    sim.close()
