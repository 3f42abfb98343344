"""The network's backward scratch holds the three hidden layers' gradients and
nothing else (the output layer's are rounded as they are read): its size, and
a backward pass in just that much, with what lies around it left alone."""
import pytest

from parity_util import print_case


@pytest.mark.parametrize("batch", [16, 256, 4096])
def test_work_bytes(batch):
    import torch  # noqa: F401
    from paper_1511_08225_amd import slpic
    L = slpic.lib()
    assert L.slpic_mlp_work_bytes(batch) == batch * 3 * slpic.MLP_HIDDEN * 2
    assert L.slpic_mlp_work_bytes(0) == L.slpic_mlp_work_bytes(-16) == 0


@pytest.mark.gpu
@pytest.mark.parametrize("batch", [16, 48, 256])
def test_backward_stays_in_its_scratch(gpu_lib, batch):
    import torch
    from test_gpu_mlp import _data
    print_case(f"mlp backward scratch, batch {batch}")
    n = gpu_lib.lib().slpic_mlp_work_bytes(batch)
    assert n == batch * 3 * gpu_lib.MLP_HIDDEN * 2
    p, x, t = _data(batch, 5)
    dy = torch.randn(batch, gpu_lib.MLP_OUT, generator=torch.Generator().manual_seed(1))
    grads = []
    for fill in (0, 0xA5):
        net = gpu_lib.Mlp(p, batch)
        pad = torch.full((n + 2048,), fill, dtype=torch.uint8, device="cuda")
        net.work = pad[1024:1024 + n]
        net.forward(x)
        grads.append(net.backward(dy).clone())
        assert bool((pad[:1024] == fill).all()) and bool((pad[1024 + n:] == fill).all())
    assert torch.equal(*grads)  # nothing is read before it is written
