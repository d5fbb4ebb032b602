"""GPU check of the fp32 4x4 weight gradient that keeps input rows in LDS: against fp64 sums over the very tensors the GPU holds (the
layer's input and the gradient of its output).  Ragged rows and columns, maps off the tiles of 8 and 16, one to six input maps
a wave, walks shorter than the ring of rows, kernel strides with either slot pitch up to the widest that fits, and sizes next to the
dispatch's lines; in test_walks many steps and several walks a workgroup.  An element's sum is a chain of at most pixels / 4 + copies fp32 additions, so
its error stays below (pixels / 4 + 512) * 2^-24 of the sum of magnitudes."""
import numpy as np
import pytest
import torch

import exact_wgrad
import sk_synth as S

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("c_in,c_out,d,n,h,w", [
    (48, 48, 1, 1, 70, 131), (48, 48, 8, 2, 90, 90), (16, 16, 2, 1, 7, 7), (24, 20, 1, 2, 40, 67), (33, 48, 4, 1, 77, 140), (47, 7, 3, 3, 35, 201),
    (40, 33, 16, 1, 120, 118), (48, 48, 16, 1, 60, 115), (16, 1, 1, 1, 4, 4), (48, 16, 2, 1, 300, 7), (8, 48, 1, 1, 259, 66), (9, 17, 2, 2, 150, 130),
    (8, 24, 1, 1, 60, 60), (12, 48, 16, 1, 111, 300), (48, 48, 1, 1, 330, 323), (49, 48, 1, 1, 40, 40), (48, 49, 1, 1, 40, 40),
])
def test_gradient(c_in, c_out, d, n, h, w):
    from paper_1509_03371_amd import binding as B
    layers = [S.conv(c_in, 1, 1, relu=False), S.conv(c_out, 4, d, relu=False), S.conv(2, 1, 1, relu=False)]
    rng = np.random.default_rng(c_in + h * w)
    net = B.SKNet(layers, 3, 2)
    for i in range(3):
        s = net.conv_shape(i)
        net.set_weights(i, (rng.standard_normal(s) / np.sqrt(np.prod(s[1:]))).astype(np.float32), rng.standard_normal(s[0]).astype(np.float32))
    net.plan(n, h, w, pad=False, training=True)
    net.forward(torch.from_numpy(rng.standard_normal((n, 3, h, w)).astype(np.float32)).cuda())
    ho, wo = h - 3 * d, w - 3 * d
    labels = torch.from_numpy(rng.integers(-1, 2, (n, ho, wo)).astype(np.int32)).cuda()
    dy = torch.from_numpy(net.get_activation_grad(1, labels)).double()
    net.backward(labels)
    dw, db = net.get_grad(1)
    x = torch.from_numpy(net.get_activation(0)).double()
    net.close()
    bound = (n * ho * wo / 4 + 512) * 2.0 ** -24
    for i in range(4):
        for j in range(4):
            xs = x[:, :, i * d:i * d + ho, j * d:j * d + wo].permute(1, 0, 2, 3).reshape(c_in, -1)
            ys = dy.permute(1, 0, 2, 3).reshape(c_out, -1)
            ref, mag = ys @ xs.T, ys.abs() @ xs.abs().T
            assert bool(((torch.from_numpy(dw[:, :, i, j]).double() - ref).abs() <= bound * mag).all()), (i, j)
    ref, mag = dy.sum(dim=(0, 2, 3)), dy.abs().sum(dim=(0, 2, 3))
    assert bool(((torch.from_numpy(db).double() - ref).abs() <= bound * mag).all())


# A workgroup (one a CU, 256) walks at least twice round its ring of five rows, over ends of strips, residue classes and images; nothing rounds,
# so a row, column or buffer taken wrongly shows in the last bit.
@pytest.mark.parametrize("c_in,c_out,d,n,h,w", [
    (48, 48, 1, 3, 310, 205), (16, 16, 3, 4, 369, 140), (33, 20, 2, 5, 287, 137), (48, 33, 8, 2, 699, 150), (8, 24, 1, 7, 409, 66), (21, 48, 16, 3, 500, 177),
])
def test_walks(c_in, c_out, d, n, h, w):
    assert -(-(w - 3 * d) // 64) * (h - 3 * d) * n >= 2 * 5 * 256
    exact_wgrad.check(c_in, c_out, 4, d, n, h, w, "f32")
