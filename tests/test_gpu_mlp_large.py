"""The network's forward pass on both sides of the batch sizes where its launch
changes: the outputs and the activations kept for the backward pass are those of
the same rows in batches of 256, bit for bit (a row's sums do not depend on the
launch), and the first rows agree with the NumPy oracle."""
import numpy as np
import pytest
import torch

from oracle import mlp
from parity_util import print_case
from test_gpu_mlp import _data, _rel

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B", [576, 592, 1152, 1168, 4096, 4112, 8208])
def test_forward_is_the_same_in_every_launch(gpu_lib, B):
    print_case(f"mlp forward B={B}")
    p, x, _ = _data(B, 5)
    net, small = gpu_lib.Mlp(p, B), gpu_lib.Mlp(p, 256)
    y = net.forward(x).cpu()
    act = net.act.cpu().view(torch.int16).flatten()
    kin, hid = gpu_lib.MLP_IN, gpu_lib.MLP_HIDDEN
    parts = [act[:B * kin].view(B, kin)] + [act[B * (kin + k * hid):B * (kin + (k + 1) * hid)].view(B, hid)
                                            for k in range(3)]
    for b in sorted({0, 256, B // 2 // 16 * 16, B - 256}):  # rows b..b+255
        ys = small.forward(x[b:b + 256]).cpu()
        assert torch.equal(y[b:b + 256], ys), b
        a = small.act.cpu().view(torch.int16).flatten()
        o = 0
        for part in parts:
            n = 256 * part.shape[1]
            assert torch.equal(part[b:b + 256].flatten(), a[o:o + n]), b
            o += n
    yo, _ = mlp.forward(p, x[:256].astype(np.float64), bf16=True)
    # the bounds of the other comparisons with the oracle
    yf = y[:256].numpy().astype(np.float64)
    assert np.abs(yf - yo).max() / np.abs(yo).max() < 2e-3 and _rel(yf, yo) < 1e-3
