"""GPU check of the 16-bit 1x1 weight gradient around its rules: tile groups that do not divide the workgroups the GPU runs at once (their
copies are rounded down), four and twelve column tiles a wave, several rounds of groups.  Against fp64 sums over the very tensors the GPU
holds; an element's sum takes at most pixels + 512 fp32 additions, so its error stays below (pixels + 512) * 2^-24 of the sum of magnitudes."""
import numpy as np
import pytest
import torch

import sk_synth as S

pytestmark = pytest.mark.gpu


# 3 and 6 groups of column tiles; a last group of one tile; 192 groups of four tiles against 64 of twelve; more groups than places
@pytest.mark.parametrize("c_in,c_out,n,h,w", [(768, 19, 2, 40, 131), (1536, 64, 1, 30, 67), (784, 48, 1, 33, 65), (3072, 768, 1, 9, 70), (2304, 1200, 1, 5, 13)])
def test_gradient(c_in, c_out, n, h, w):
    from paper_1509_03371_amd import binding as B
    layers = [S.conv(c_in, 1, 1, relu=False), S.conv(c_out, 1, 1, relu=False), S.conv(2, 1, 1, relu=False)]
    rng = np.random.default_rng(c_in + h * w)
    net = B.SKNet(layers, 3, 2, dtype="bf16")
    for i in range(3):
        s = net.conv_shape(i)
        net.set_weights(i, (rng.standard_normal(s) / np.sqrt(np.prod(s[1:]))).astype(np.float32), rng.standard_normal(s[0]).astype(np.float32))
    net.plan(n, h, w, pad=False, training=True)
    net.forward(torch.from_numpy(rng.standard_normal((n, 3, h, w)).astype(np.float32)).cuda())
    labels = torch.from_numpy(rng.integers(-1, 2, (n, h, w)).astype(np.int32)).cuda()
    dy = torch.from_numpy(net.get_activation_grad(1, labels)).double()
    net.backward(labels)
    dw, db = net.get_grad(1)
    x = torch.from_numpy(net.get_activation(0)).double()
    net.close()
    bound = (n * h * w + 512) * 2.0 ** -24
    xs, ys = (t.permute(1, 0, 2, 3).reshape(t.shape[1], -1) for t in (x, dy))
    assert bool(((torch.from_numpy(dw[:, :, 0, 0]).double() - ys @ xs.T).abs() <= bound * (ys.abs() @ xs.abs().T)).all())
    assert bool(((torch.from_numpy(db).double() - ys.sum(1)).abs() <= bound * ys.abs().sum(1)).all())
