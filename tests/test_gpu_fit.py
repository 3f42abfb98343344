"""Push chunks and sort tiles fitted to the size of a run set, against the
oracle on both sides of the sizes where they are halved: one step's charge and
potential, and the sort's permutation, whatever was requested."""
import numpy as np
import pytest

import oracle
import workloads
from parity_util import print_case, push_oracle_to_gpu, rel_inf

pytestmark = pytest.mark.gpu


# loads are 2 * nx * ppc particles; chunks of 128 are halved below 262144 and of
# 1024 below 2097152, tiles of 2048 below 1048576
@pytest.mark.parametrize("nx,ppc,cf,chunk,tile", [
    (4, 1, 1.5, 1024, 32768),      # a few particles: the smallest chunk and tile
    (512, 255, 1.5, 128, 2048),    # chunk 64, tile 1024
    (512, 256, 1.5, 128, 2048),    # chunk 128, tile 1024
    (1024, 511, 1.5, 1024, 2048),  # tile 1024
    (1024, 512, 1.5, 1024, 2048),  # tile 2048
    (64, 50, 40.0, 1024, 16384),   # slots counted: ten times the load
    (64, 50, 1.5, 64, 512),        # nothing to halve
])
def test_fitted_launch_matches_oracle(gpu_lib, nx, ppc, cf, chunk, tile):
    print_case(f"fit nx={nx} ppc={ppc} cf={cf} chunk={chunk} tile={tile}")
    cfg = workloads.sheath(nx, ppc, 4.0, seed=6, sort_every=0, capacity_factor=cf)
    run = oracle.Run(cfg)
    run.step(2)
    sim = gpu_lib.Sim(cfg, precision="f64", sort_every=0, sort_bucket=1, chunk=chunk, sort_tile=tile,
                      record_perm=True)
    push_oracle_to_gpu(sim, 0, run, quantize=False)
    sim.step(1)
    run.step(1)
    g, o = sim.grid(0), run.grid()
    # FP64 sums of the same terms in another order, and a solve over them: the
    # bounds the other FP64 one-step comparisons with the oracle use
    for s in range(2):
        assert rel_inf(g["Q"][s], o["Q"][s]) <= 1e-12, s
    assert rel_inf(g["phi"], o["phi"]) <= 1e-9
    # the sort moves the stored particles: from the oracle's state on both sides
    push_oracle_to_gpu(sim, 0, run, quantize=False)
    sim.sort_now()
    perms = run.sort()
    for s in range(2):
        assert np.array_equal(sim.perm(0, s), perms[s]), s
    sim.close()
