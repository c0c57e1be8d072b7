"""The backward pass where its kernels' runs of rows begin, end and cross from
one image to the next, and where batches go row by row or tile by tile: every
entry of the gradient against the oracle's backward pass fed the GPU's forward
pass, within the bound of the same comparison in test_gpu_surrogate.py."""
import numpy as np
import pytest

from swtest import announce
from test_gpu_surrogate import KAPPA_FROM_GPU_FORWARD, check_grad, grad_case, make_net, oracle_grad_from_gpu_forward

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,H,W,cap", [(1, 3, 64, 0), (5, 1, 64, 2), (3, 7, 128, 0), (2, 13, 192, 0), (1, 300, 192, 0),
                                       (2, 5, 256, 0), (4, 200, 256, 0), (3, 11, 320, 5), (2, 9, 512, 0),
                                       (10, 241, 256, 0), (10, 241, 256, 7), (60, 20, 512, 0)])
def test_gradient_at_run_edges(B, H, W, cap):
    p, out_scale, u, u8 = grad_case(B, H, W, 16)
    announce(f"surrogate gradient at run edges B={B} {H}x{W} cap={cap}")
    net = make_net(H, W, B, p, out_scale)
    net.set_block_cap(cap)
    g, _ = net.grad(u, u8)
    _, ref, S = oracle_grad_from_gpu_forward(net, p, B, u, u8, out_scale)
    check_grad(g.cpu().numpy().astype(np.float64), ref, S, KAPPA_FROM_GPU_FORWARD, B * H * W, "run edges")
