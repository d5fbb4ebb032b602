"""16-bit 3-D nets after a step of SGD, which packs all layers' weights in one launch (two for more forms than a launch takes): the same net planned afresh
with these weights, layer by layer, gives the same probabilities and gradients bit for bit."""
import numpy as np
import pytest
import torch

import sk_synth as S

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("maps,ks", [((16, 40, 7), (3, 2, 1)), ((5,) + (16,) * 17, (3,) + (1,) * 17)])
def test_repacked(maps, ks):
    from paper_1509_03371_amd import binding as B
    rng = np.random.default_rng(len(maps))
    layers = [S.conv(f, k, 1) for f, k in zip(maps, ks)] + [S.conv(2, 1, 1, relu=False)]
    img = torch.from_numpy(rng.standard_normal((9, 1, 20, 23)).astype(np.float32)).cuda()
    first, second = (B.SKNet3D(layers, 1, 2, dtype="bf16") for _ in range(2))
    count = first.num_convs()
    for i in range(count):
        s = first.conv_shape(i)
        first.set_weights(i, (rng.standard_normal(s) * np.sqrt(2 / np.prod(s[1:]))).astype(np.float32), (rng.random(s[0]) * 0.2).astype(np.float32))
    first.plan(9, 20, 23, training=True)
    _, _, ho, wo = first.out_shape()
    lab = torch.from_numpy(rng.integers(-1, 2, (first.out_shape()[0], ho, wo)).astype(np.int32)).cuda()
    first.forward(img)
    first.backward(lab)
    first.sgd_step(lr=0.3)
    for i in range(count):
        second.set_weights(i, *first.get_weights(i))
    second.plan(9, 20, 23, training=True)
    got = []
    for net in (first, second):
        prob = net.forward(img).cpu().numpy().copy()
        net.backward(lab)
        got.append([prob] + [net.get_grad(i)[0] for i in range(count)])
        net.close()
    assert any(np.abs(g).max() > 0 for g in got[0][1:2])
    for a, b in zip(*got):
        assert np.array_equal(a, b)
