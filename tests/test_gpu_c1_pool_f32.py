"""The launch that pads, convolves and pools the first layer of an fp32 inference plan, against the plan that keeps every layer
(padding, convolution and pool as launches of their own, tested against the oracle): same operations in the same order, so equal
bit for bit."""
import numpy as np
import pytest
import torch

import sk_synth as S
from paper_1509_03371_amd import binding as B

pytestmark = pytest.mark.gpu

# k, maps, images, h, w, padded, relu: two rows a thread and four, maps that leave half a pair, groups of maps, ragged last groups,
# the smallest map (2 x 4 pooled samples), borders wider than a window
CASES = [(4, 8, 1, 96, 96, True, True), (4, 48, 1, 64, 61, True, True), (3, 5, 2, 33, 47, True, False), (3, 17, 1, 200, 131, False, True),
         (4, 48, 2, 301, 258, True, True), (4, 1, 1, 6, 8, False, True), (3, 2, 3, 5, 7, False, False), (4, 48, 1, 515, 402, False, False)]


@pytest.mark.parametrize("k,maps,n,h,w,pad,relu", CASES)
@pytest.mark.parametrize("pad_mode", [0, 1])
def test_first_layer_with_its_pool(k, maps, n, h, w, pad, relu, pad_mode):
    layers = [{"type": "conv", "f_out": maps, "k": k, "d": 1, "relu": relu}, {"type": "pool", "k": 2, "d": 1, "s": 1},
              {"type": "conv", "f_out": 2, "k": 1, "d": 1, "relu": False}]
    ws, bs = S.he_normal_weights(layers, 1, 77 + k)
    img = torch.from_numpy(S.uniform_image(n, 1, h, w, 5)).cuda()
    net = B.SKNet(layers, 1, 2, pad_mode=pad_mode)
    for i, (wt, b) in enumerate(zip(ws, bs)):
        net.set_weights(i, wt, b + np.float32(0.1) * np.arange(len(b), dtype=np.float32))
    got = {}
    for keep in (True, False):
        net.plan(n, h, w, pad=pad, keep=keep)
        names = [net.step_name(i) for i in range(net.num_steps())]
        assert ("conv0_k%d_d1_o%d_pool" % (k, maps) in names) == (not keep)
        net.forward(img)
        got[keep] = [net.get_activation(i) for i in (-1, 1, 0, 2)]
    net.close()
    for a, b in zip(got[True], got[False]):
        assert np.array_equal(a, b)
