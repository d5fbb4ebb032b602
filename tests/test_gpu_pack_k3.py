"""Weights of 16-bit 3x3 layers packed again after a step of SGD, on tiles of 16 x 32 maps that are whole and those that are not: the same net planned
afresh with these weights, which packs them with another kernel, gives the same probabilities and gradients bit for bit."""
import numpy as np
import pytest
import torch

import sk_synth as S

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("maps", [(32, 48, 32), (16, 32, 96), (64, 64, 80), (40, 33, 24), (7, 100, 130)])
def test_repacked(maps):
    from paper_1509_03371_amd import binding as B
    rng = np.random.default_rng(sum(maps))
    layers = [S.conv(f, 3, 1) for f in maps] + [S.conv(2, 1, 1, relu=False)]
    img = torch.from_numpy(rng.standard_normal((2, 1, 30, 41)).astype(np.float32)).cuda()
    lab = torch.from_numpy(rng.integers(-1, 2, (2, 24, 35)).astype(np.int32)).cuda()
    first, second = B.SKNet(layers, 1, 2, dtype="bf16"), B.SKNet(layers, 1, 2, dtype="bf16")
    for i in range(4):
        s = first.conv_shape(i)
        first.set_weights(i, (rng.standard_normal(s) / np.sqrt(np.prod(s[1:]))).astype(np.float32), rng.standard_normal(s[0]).astype(np.float32))
    first.plan(2, 30, 41, pad=False, training=True)
    first.forward(img)
    first.backward(lab)
    first.sgd_step(lr=0.5)
    for i in range(4):
        second.set_weights(i, *first.get_weights(i))
    second.plan(2, 30, 41, pad=False, training=True)
    got = []
    for net in (first, second):
        prob = net.forward(img).cpu().numpy().copy()
        net.backward(lab)
        got.append([prob] + [net.get_grad(i)[0] for i in range(4)])
        net.close()
    for a, b in zip(*got):
        assert np.array_equal(a, b)
