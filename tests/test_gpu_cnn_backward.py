"""Weight and bias gradients of the corrector around the edges of the backward kernels'
tiles (8 and 16 rows x 32 pixels): heights that leave remainders, images of one row or one
tile column, batches small and large enough for both tile heights, against the CPU reference
with bfloat16 rounding where the GPU rounds: inputs, weights, hidden activations and the
gradient of every layer's output.  (On images of few pixels the roundings do not average
out: a reference without those of the activations is 3.8e-2 off at one row of 32 pixels.)
Tolerances as in test_gpu_cnn.py (2^-8 sqrt(K) relative)."""
import numpy as np
import pytest

from gpu_helpers import rel_l2
from oracle import conv_ref
from test_gpu_cnn import make

pytestmark = pytest.mark.gpu


def ref_loss_and_grads(layers, x, target):
    acts, h = [conv_ref.to_bf16(x)], conv_ref.to_bf16(x)
    for k, (w, b) in enumerate(layers):
        h = conv_ref.conv3x3(h, w, b)
        if k < 3:
            h = conv_ref.to_bf16(conv_ref.relu(h))
            acts.append(h)
    g = conv_ref.to_bf16(2.0 * (h - target) / h.size)
    grads = [None] * 4
    for k in range(3, -1, -1):
        dx, dw, db = conv_ref.conv3x3_backward(acts[k], layers[k][0], g)
        grads[k] = (dw, db)
        g = conv_ref.to_bf16(dx * (acts[k] > 0))
    return conv_ref.mse(h, target), grads


@pytest.mark.parametrize("batch,H,W", [(1, 1, 32), (2, 7, 32), (3, 8, 64), (1, 9, 96), (5, 17, 32), (2, 48, 64),
                                       (86, 33, 64), (256, 32, 32)])
def test_gradients_tile_edges(batch, H, W):
    import torch
    net, x, t, xd, td = make(batch, H=H, W=W, seed=31)
    layers = [(conv_ref.to_bf16(w), b) for w, b in net.get_weights()]
    g = net.gradients(xd, td)
    torch.cuda.synchronize()
    flat = g.cpu().numpy().copy()
    got = net.unpack(flat)
    loss_ref, grads_ref = ref_loss_and_grads(layers, x.transpose(0, 3, 1, 2), t.transpose(0, 3, 1, 2))
    assert abs(net.loss.item() - loss_ref) < 1e-2 * loss_ref
    for l in range(4):
        print(f"layer {l}: {rel_l2(got[l][0], grads_ref[l][0]):.2e} {rel_l2(got[l][1], grads_ref[l][1]):.2e}")
        assert rel_l2(got[l][0], grads_ref[l][0]) < 3e-2, l
        assert rel_l2(got[l][1], grads_ref[l][1]) < 3e-2, l
    net.set_weights(got)  # the padding of the gradient is exactly zero
    assert np.all(flat[net.params.cpu().numpy() == 0] == 0)
    net.close()


def test_gradients_unaligned_input():
    """An input that is not 16-byte aligned is packed element by element: the same bits."""
    import torch
    net, x, t, xd, td = make(2, seed=8)
    a = net.gradients(xd, td).clone()
    buf = torch.empty(xd.numel() + 1, dtype=torch.float32, device="cuda")
    view = buf[1:].view(xd.shape)
    view.copy_(xd)
    b = net.gradients(view, td).clone()
    assert torch.equal(a, b)
    net.close()
