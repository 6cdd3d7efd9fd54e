"""Loss and gradient of the warm-start network where its split changes: the
last tile ragged, as many partials as the reduction has waves, one
more, a full batch of its loads, one more, and workgroups that take a second
tile; and weights at an address that is only a multiple of two bytes.

The bound per parameter block is that of the whole-network comparison: the
backward pass rounds its deltas to bfloat16 (4e-3 per operand), 2e-2 of the
block's norm.  The residual itself is taken at the forward pass's bfloat16
rounding (the FP64 network's targets are shifted by the difference of the two
forward passes): a residual near zero has no relative accuracy against the
FP64 forward.  (A single record is in the whole-network comparison.)  Weights at another address give the same bits."""
from __future__ import annotations

import numpy as np
import pytest

from oracle import wsn_forward_bf16, wsnet
from test_gpu_wsn import _net, _records

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [17, 16 * 16, 16 * 17, 16 * 128, 16 * 129 + 1, 16 * 520 + 5])
def test_loss_gradient_at_the_edges_of_the_split(n):
    import torch
    print("case wsn tiles, n =", n, flush=True)
    net = _net(4)
    R = _records(n, seed=n)
    Rd = torch.tensor(R, device="cuda")
    L, g = (t.clone() for t in net.loss_grad(Rd))
    wb, R64 = net.weights_bf16_as_float(), R.astype(np.float64)
    shift = wsnet.forward(wb, R64[:, :7]) - wsn_forward_bf16(wb, R64)
    Lr, gr = wsnet.loss_grad(wb, R64[:, :7], R64[:, 7:10] + shift)
    assert abs(float(L.item()) - Lr) <= 1e-2 * Lr
    g64 = g.cpu().numpy().astype(np.float64)
    offs = [0, 448, 512, 4608, 4672, 4864, 4867]
    for a, b in zip(offs[:-1], offs[1:]):
        assert np.linalg.norm(g64[a:b] - gr[a:b]) <= 2e-2 * np.linalg.norm(gr[a:b]) + 1e-9, (a, b)
    buf = torch.empty(net.wb.numel() + 1, dtype=net.wb.dtype, device="cuda")
    buf[1:] = net.wb
    net.wb = buf[1:]
    L2, g2 = net.loss_grad(Rd)
    assert torch.equal(L2, L) and torch.equal(g2, g)
