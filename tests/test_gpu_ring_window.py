"""Charge of a periodic box whose deposit windows lie across its ends, at box
lengths about the window's and far from it: the charge of every node (0 and nx
each their own) against the oracle, one step from the oracle's state some steps
after a sort, when chunks at both ends hold particles that crossed."""
import math

import pytest

import oracle
import workloads
from parity_util import print_case, push_oracle_to_gpu, rel_inf

pytestmark = pytest.mark.gpu

# the bounds of the other one-step comparisons with the oracle: FP64 sums of the
# same terms in another order; FP32 particles a step away from quantised ones
TOL = {"f64": 1e-12, "f32": 1e-5}


@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("nx,ppc,u,chunk", [
    (4, 40, 1.0, 64),             # the ring inside the window several times
    (5, 200, math.inf, 512),
    (126, 30, 0.5, 256),          # nodes 127, 128, 129, 130: about the window's 128
    (127, 30, 0.5, 256),
    (128, 30, math.inf, 128),
    (129, 30, 0.5, 1024),
    (300, 40, 2.0, 512),          # windows of part of the ring
    (2729, 5, math.inf, 64),
])
def test_charge_across_the_ends(gpu_lib, prec, nx, ppc, u, chunk):
    print_case(f"ring window nx={nx} ppc={ppc} u={u} chunk={chunk} {prec}")
    cfg = workloads.langmuir_box(u, nx=nx, ppc=ppc, seed=nx, sort_every=8)
    run = oracle.Run(cfg)
    run.step(13)  # the last sort five steps ago
    sim = gpu_lib.Sim(cfg, precision=prec, sort_every=0, chunk=chunk)
    push_oracle_to_gpu(sim, 0, run, quantize=prec == "f32")
    sim.refresh_fields()  # the deposit alone
    g0, o0 = sim.grid(0), run.grid()
    sim.step(1)
    run.step(1)
    g, o = sim.grid(0), run.grid()
    for s in range(2):
        assert rel_inf(g0["Q"][s], o0["Q"][s]) <= TOL[prec], s
        assert rel_inf(g["Q"][s], o["Q"][s]) <= TOL[prec], s
    sim.close()
