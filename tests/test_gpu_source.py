"""New particles of a step at source sizes from none to several rounds of the
workgroup, mostly of one species: counts, places and charge against the oracle,
one step from the oracle's state."""
import numpy as np
import pytest

import oracle
import workloads
from parity_util import oracle_state, print_case, push_oracle_to_gpu, rel_inf

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,ppc,u,beta,least", [
    (64, 100, 3.0, "step", 0),       # none or a few
    (16, 2000, 10.0, "smooth", 64),  # more than a wave
    (12, 9000, 10.0, "step", 500),
    (12, 40000, 10.0, "step", 1100),  # more than the workgroup's 1024 threads
])
def test_source_matches_oracle(gpu_lib, nx, ppc, u, beta, least):
    print_case(f"source nx={nx} ppc={ppc} u={u} {beta}")
    cfg = workloads.sheath(nx, ppc, u, beta_kind=beta, seed=3, sort_every=0)
    run = oracle.Run(cfg)
    run.step(3)
    sim = gpu_lib.Sim(cfg, precision="f64", sort_every=0)
    push_oracle_to_gpu(sim, 0, run, quantize=False)
    before = [len(oracle_state(run, s)[0]) for s in range(2)]
    sim.step(1)
    run.step(1)
    made = 0
    for s in range(2):
        got, want = sim.export_particles(0, s), oracle_state(run, s)
        assert len(got[0]) == len(want[0]), s
        made += len(got[0]) - before[s]
        new = slice(before[s], None)
        assert np.array_equal(got[0][new], want[0][new]), s
        for a, b in zip(got[1:], want[1:]):  # libm's last bits in the normal draws
            assert np.allclose(a[new], b[new], rtol=1e-12, atol=0), s
    assert made >= least, made
    g, o = sim.grid(0), run.grid()
    for s in range(2):
        assert rel_inf(g["Q"][s], o["Q"][s]) <= 1e-12, s
    sim.close()
