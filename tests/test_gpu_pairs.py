"""The network's forward pass two layers a launch against one layer a launch
(which a cap on the single-layer kernels' workgroups asks for): activations,
prediction, gradients and rollouts bit for bit."""
import pytest
import torch

from paper_1107_2157_amd import surrogate, sw
from swtest import announce

pytestmark = pytest.mark.gpu


# widths of one to four column groups; heights of one row, of less than a run and of several runs with a remainder
@pytest.mark.parametrize("B,H,W", [(1, 1, 64), (2, 3, 64), (3, 64, 64), (2, 40, 128), (40, 33, 192), (5, 219, 256),
                                   (70, 64, 64)])
def test_two_layers_a_launch_equal_one(B, H, W):
    announce(f"network two layers a launch: {B} x {H} x {W}")
    net = sw.Surrogate(H, W, B, seed=9)
    net.set_norm(surrogate.IN_OFFSET, surrogate.IN_SCALE, (0.05, 0.05, 0.05))
    net.set_fused(0)
    u = surrogate.initial_states(B, H, W, 300)
    gen = torch.Generator().manual_seed(B * H + W)
    u[:, 1:] += 0.05 * (torch.rand((B, 2, H, W), generator=gen).cuda() - 0.5)
    u8 = u + 0.01 * torch.rand((B, 3, H, W), generator=gen).cuda()
    batch = sw.Batch([(W, H)] * B)
    got = []
    for cap in (0, 1024):
        net.set_block_cap(cap)
        out = [net.forward(u)] + [net.activation(k, B) for k in range(7)]
        g, loss = net.grad(u, u8)
        out += [g.clone(), loss.clone()]
        batch.load(u)
        net.advance(batch, 16)
        out.append(batch.export().clone())
        got.append(out)
    for k, (x, y) in enumerate(zip(*got)):
        assert torch.equal(x, y), f"output {k} differs"
