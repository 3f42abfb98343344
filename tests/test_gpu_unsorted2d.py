"""2D steps of slots that no sort has put in order, pushed without tile
workgroups: the same step as from sorted slots, whichever of the two the host
counts (a restored workspace may hold the other), with and without a graph."""
import pytest

import workloads
from parity_util import print_case, rel_inf

pytestmark = pytest.mark.gpu

# one step moves each particle alike; only the order of FP64 sums differs (in F32 a
# field value may round to the neighbouring float: 1e-6)
TOL = 1e-12


@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("nx,ny,ppc", [(60, 64, 16), (24, 16, 3)])
def test_step_of_unsorted_slots(gpu_lib, prec, nx, ny, ppc):
    cfg = workloads.sheath2d(nx, ny, ppc, 3.0, tile=8, seed=7)

    def make():
        return gpu_lib.Sim2D(cfg, ny, precision=prec, sort_every=0, tile=8, margin=2)
    want = make()  # sorted, and counted as such
    want.sort_now()
    want.refresh_fields()
    ckpt = want.workspace.clone()
    q0 = want.grid()["Q"]
    want.step(1)
    q1 = want.grid()["Q"]
    got = []
    sim = make()  # unsorted, and counted as such
    got.append(("unsorted", sim))
    sim = make()  # sorted in the workspace, counted as unsorted
    sim.workspace.copy_(_aligned(ckpt, want, sim))
    got.append(("restored sorted", sim))
    sim = make()  # unsorted in the workspace, counted as sorted
    raw = sim.workspace.clone()
    sim.sort_now()
    sim.workspace.copy_(raw)
    got.append(("restored unsorted", sim))
    for what, sim in got:
        print_case(f"2D unsorted step {nx}x{ny}x{ppc} {prec}: {what}")
        sim.refresh_fields()
        for s in range(2):
            assert rel_inf(sim.grid()["Q"][s], q0[s]) <= TOL, (what, s)
        sim.step(1)
        st = sim.status()
        assert st["nslots"] == want.status()["nslots"] and st["pushed_total"] == want.status()["pushed_total"], what
        for s in range(2):
            assert rel_inf(sim.grid()["Q"][s], q1[s]) <= (TOL if prec == "f64" else 1e-6), (what, s)
        sim.close()
    want.close()


def _aligned(ckpt, src, dst):
    """A checkpoint moved to where dst's workspace starts in its tensor."""
    out = dst.workspace.clone()
    a, b = src._ws_ptr - src.workspace.data_ptr(), dst._ws_ptr - dst.workspace.data_ptr()
    out[b:b + src.workspace_bytes] = ckpt[a:a + src.workspace_bytes]
    return out


def test_graph_steps_of_unsorted_slots(gpu_lib):
    """Captured blocks replayed before a sort, after one and after an import."""
    import torch
    print_case("2D unsorted graph steps")
    cfg = workloads.sheath2d(60, 64, 8, 3.0, tile=8, seed=8)
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        sims = [gpu_lib.Sim2D(cfg, 64, precision="f64", sort_every=0, tile=8, margin=2, graph_steps=g)
                for g in (4, 0)]
        for act in ("steps", "sort", "steps", "import", "steps"):
            for sim in sims:
                if act == "steps":
                    sim.step(8)
                elif act == "sort":
                    sim.sort_now()
                else:
                    for s in range(2):
                        sim.import_particles(s, *sims[1].export_particles(s))
                torch.cuda.synchronize()
            a, b = (sim.grid()["Q"] for sim in sims)
            for s in range(2):
                assert rel_inf(a[s], b[s]) <= 1e-9, (act, s)  # rounding, amplified over the steps
            assert sims[0].status()["nslots"] == sims[1].status()["nslots"], act
        for sim in sims:
            sim.close()
