"""What sw_surrogate_activation shows after a rollout by layers: the hidden
layers and the prediction of the rollout's last network pass, whichever number
of layers a launch takes (a cap on the single-layer kernels' workgroups asks
for one)."""
import pytest
import torch

from paper_1107_2157_amd import surrogate, sw
from swtest import announce

pytestmark = pytest.mark.gpu


# widths of one to four column groups, one run of rows and several
@pytest.mark.parametrize("B,H,W", [(1, 5, 64), (3, 64, 128), (40, 33, 192), (5, 219, 256)])
@pytest.mark.parametrize("steps,graph,judge", [(8, True, False), (24, True, False), (16, False, False), (16, True, True)])
def test_activations_after_a_rollout(B, H, W, steps, graph, judge):
    announce(f"activations after a rollout: {B} x {H} x {W}, {steps} steps, graph={graph} judge={judge}")
    net = sw.Surrogate(H, W, B, seed=9)
    net.set_norm(surrogate.IN_OFFSET, surrogate.IN_SCALE, (0.05, 0.05, 0.05))
    net.set_fused(0)
    net.set_graph(graph)
    u = surrogate.initial_states(B, H, W, 300)
    other = u.flip(0).flip(3).contiguous() * 1.1
    batch = sw.Batch([(W, H)] * B)
    got = []
    for cap in (0, 1024):
        net.set_block_cap(cap)
        for _ in range(2):                       # captured, then replayed
            net.forward(other)                   # what an earlier pass left behind
            batch.load(u)
            net.advance(batch, steps, judge=judge)
            got.append([net.activation(k, B) for k in range(1, 7)] + [batch.export().clone()])
    for out in got[:-1]:
        for k, (x, y) in enumerate(zip(out, got[-1])):
            assert torch.equal(x, y), f"layer {k + 1} differs"
