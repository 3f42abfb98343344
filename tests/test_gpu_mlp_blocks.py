"""The network's kernels at the batch sizes where their blocks are cut: fewer
rows than a 32-row block or a 64-deep product step (16), rows that end inside
them (48, 80), many blocks (1024), against the NumPy oracle; and the mean
squared error over lengths that end inside its strided passes."""
import numpy as np
import pytest
import torch

from oracle import mlp
from parity_util import print_case
from test_gpu_mlp import _data, _rel

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B", [16, 48, 80, 1024])
def test_forward_and_backward_match_oracle(gpu_lib, B):
    p, x, t = _data(B, 21)
    net = gpu_lib.Mlp(p, B)
    y = net.forward(x).cpu().numpy().astype(np.float64)
    yo, cache = mlp.forward(p, x.astype(np.float64), bf16=True)
    # FP32 sums on identical BF16 operands: a hidden value now and then lands on
    # the other side of a BF16 rounding boundary (2^-8 of it)
    assert np.abs(y - yo).max() / np.abs(yo).max() < 2e-3
    assert _rel(y, yo) < 1e-3
    _, dy = mlp.mse(y, t.astype(np.float64))
    g = net.backward(dy.astype(np.float32)).cpu().numpy().astype(np.float64)
    go = mlp.backward(p, cache, dy, bf16=True)
    for name, shape, off in mlp.layout():
        n = int(np.prod(shape))
        e = _rel(g[off:off + n], go[off:off + n])
        print_case(f"mlp grad {name} B={B}: rel Frobenius {e:.2e}")
        assert e < 0.02, name


@pytest.mark.parametrize("n", [1, 255, 65536, 65537, 262145])
def test_mse_lengths(gpu_lib, n):
    print_case(f"mlp mse n={n}")
    gen = torch.Generator().manual_seed(n)
    y, t = torch.randn(n, generator=gen), torch.randn(n, generator=gen)
    yd, td = y.cuda(), t.cuda()
    dy, loss = torch.full((n + 8,), 7.0, device="cuda"), torch.zeros(1, device="cuda")
    P = gpu_lib._P
    stream = P(torch.cuda.current_stream().cuda_stream)
    rc = gpu_lib.lib().slpic_mlp_mse(P(yd.data_ptr()), P(td.data_ptr()), P(dy.data_ptr()), n, P(loss.data_ptr()),
                                     stream)
    assert rc == 0
    d = y.double() - t.double()
    # a difference, a doubling and a division in FP32
    np.testing.assert_allclose(dy[:n].cpu().numpy(), (2.0 * d / n).numpy(), rtol=1e-6, atol=1e-7 / n)
    assert float((dy[n:] - 7.0).abs().max()) == 0.0  # nothing past the end
    # non-negative FP32 terms in a tree of partial sums and at most 256 atomics
    assert loss.item() == pytest.approx(float((d * d).mean()), rel=3e-5)
