"""The fp32 inference head that takes the maxima of the pool in front of it, against the layers one by one (the plan that keeps every layer):
the pool's values bit for bit, the probabilities within the sums' rounding -- 48 + 200 products of a class sum and the exponential, whose
error is below 300 * 2^-24 of the largest logit's size in either plan."""
import numpy as np
import pytest
import torch

import sk_synth as S
from paper_1509_03371_amd import binding as B

pytestmark = pytest.mark.gpu

# maps, hidden, classes, d, images, h, w: rows shorter and longer than a group of 64 pixels, ends of rows at every phase of a lane's four
# pixels, groups that move back, one image and several, the smallest plane, 3 and 4 classes
CASES = [(16, 32, 2, 2, 1, 97, 99), (8, 16, 2, 1, 1, 17, 5), (12, 40, 3, 4, 2, 33, 71), (48, 64, 4, 8, 1, 40, 130), (5, 16, 1, 3, 3, 20, 67),
         (48, 200, 2, 8, 3, 161, 201), (16, 32, 2, 16, 1, 50, 84)]


@pytest.mark.parametrize("maps,hidden,classes,d,n,h,w", CASES)
def test_head_with_its_pool(maps, hidden, classes, d, n, h, w):
    layers = [S.conv(maps, 1, 1), S.conv(maps, 1, 1, relu=False), S.pool(2, d), S.conv(hidden, 1, 1), S.conv(classes, 1, 1, relu=False)]
    ws, bs = S.he_normal_weights(layers, 1, 31 * maps + d, bias_scale=0.2)
    img = torch.from_numpy(S.uniform_image(n, 1, h, w, 9)).cuda()
    net = B.SKNet(layers, 1, classes)
    for i, (wt, b) in enumerate(zip(ws, bs)):
        net.set_weights(i, wt, b)
    got = {}
    for keep in (True, False):
        net.plan(n, h, w, pad=False, keep=keep)
        names = [net.step_name(i) for i in range(net.num_steps())]
        assert any(s.startswith("pool2") for s in names) == keep, names
        prob = net.forward(img).cpu().numpy().astype(np.float64)
        got[keep] = prob, net.get_activation(1), net.get_activation(2)
        if keep:
            size = np.abs(net.get_activation(4)).max()
    net.close()
    assert np.array_equal(got[True][1], got[False][1]) and np.array_equal(got[True][2], got[False][2])
    assert np.abs(got[True][0] - got[False][0]).max() <= 300 * 2.0 ** -24 * max(1.0, size)
