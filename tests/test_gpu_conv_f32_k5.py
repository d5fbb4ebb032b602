"""GPU parity of the fp32 5x5 convolutions on the prefetching kernel: ragged tiles and map groups, kernel strides up to the widest it
takes (16; 17 stays on the generic kernel), zero borders and ReLU masks of the data gradient.

An fp32 sum of K products errs by at most K * 2^-24 of the sum of their magnitudes; the error maps start from a softmax in fp32
(1e-6)."""
import numpy as np
import pytest
import torch

import sk_synth as S
from oracle import layers as OL

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,c_in,c_out,n,h,w", [
    (1, 3, 8, 1, 5, 5), (1, 8, 16, 2, 23, 70), (2, 7, 20, 1, 41, 133), (3, 16, 33, 2, 34, 80), (4, 5, 50, 1, 90, 84), (8, 12, 64, 1, 77, 97),
    (16, 9, 70, 1, 101, 131), (17, 9, 16, 1, 100, 134), (2, 48, 128, 1, 150, 165),
])
def test_forward(d, c_in, c_out, n, h, w):
    from paper_1509_03371_amd import binding as B
    rng = np.random.default_rng(h * w)
    img = rng.standard_normal((n, c_in, h, w)).astype(np.float32)
    w0, b0 = rng.standard_normal((c_out, c_in, 5, 5)).astype(np.float32), rng.standard_normal(c_out).astype(np.float32)
    net = B.SKNet([S.conv(c_out, 5, d, relu=True), S.conv(2, 1, 1, relu=False)], c_in, 2)
    net.set_weights(0, w0, b0)
    net.set_weights(1, np.ones((2, c_out, 1, 1), np.float32), np.zeros(2, np.float32))
    net.plan(n, h, w, pad=False, keep=True)
    net.forward(torch.from_numpy(img).cuda())
    ref, size = OL.conv_sk(img, w0, b0, d, relu=True), OL.conv_sk(np.abs(img), np.abs(w0), np.abs(b0), d)
    assert np.all(np.abs(net.get_activation(0) - ref) <= (25 * c_in + 1) * 2.0 ** -24 * size)
    net.close()


@pytest.mark.parametrize("relu", [False, True])
@pytest.mark.parametrize("d,maps,classes,n,h,w", [
    (1, 8, 2, 2, 19, 71), (2, 20, 3, 1, 47, 66), (3, 40, 2, 1, 30, 131), (16, 50, 2, 1, 85, 90), (17, 16, 2, 1, 85, 90), (4, 64, 5, 1, 60, 64),
])
def test_data_gradient(d, maps, classes, n, h, w, relu):
    from paper_1509_03371_amd import binding as B
    rng = np.random.default_rng(h + w)
    w1 = rng.standard_normal((classes, maps, 5, 5)).astype(np.float32) * 0.2
    net = B.SKNet([S.conv(maps, 1, 1, relu=relu), S.conv(classes, 5, d, relu=False)], 2, classes)
    net.set_weights(0, rng.standard_normal((maps, 2, 1, 1)).astype(np.float32), rng.standard_normal(maps).astype(np.float32))
    net.set_weights(1, w1, np.zeros(classes, np.float32))
    net.plan(n, h, w, pad=False, training=True)
    prob = net.forward(torch.from_numpy(rng.standard_normal((n, 2, h, w)).astype(np.float32)).cuda()).cpu().numpy().astype(np.float64)
    labels = rng.integers(-1, classes, (n,) + prob.shape[2:]).astype(np.int32)
    got = net.get_activation_grad(0, torch.from_numpy(labels).cuda())
    kept = labels >= 0
    dz = (prob - np.eye(classes)[np.maximum(labels, 0)].transpose(0, 3, 1, 2)) * kept[:, None] / max(1, kept.sum())
    ref, size = OL.conv_sk_bwd_data(dz, w1, d, (h, w)), OL.conv_sk_bwd_data(np.abs(dz), np.abs(w1), d, (h, w))
    if relu:
        ref = ref * (net.get_activation(0) > 0)
    bound = 25 * classes * 2.0 ** -24 * size + 1e-6 / max(1, kept.sum()) * np.abs(w1).sum(axis=(0, 2, 3))[None, :, None, None]
    assert np.abs(ref).max() > 1e-5 and np.all(np.abs(got - ref) <= bound)
    net.close()
