"""Training plans with the head in one kernel: a step of SGD packs the head's weights with those of the other layers, also where these fill a launch or are
too many for one.  The same net planned afresh with these weights gives the same probabilities and gradients bit for bit."""
import numpy as np
import pytest
import torch

import sk_synth as S

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("convs,maps,hidden", [(1, 48, 200), (1, 13, 17), (13, 16, 40), (14, 16, 65), (15, 8, 16), (17, 8, 30)])
def test_repacked(convs, maps, hidden):
    from paper_1509_03371_amd import binding as B
    rng = np.random.default_rng(convs + maps)
    layers = [S.conv(maps, 4, 1)] + [S.conv(maps, 2, 1) for _ in range(convs - 1)] + [S.pool(2, 1), S.conv(hidden, 1, 1), S.conv(2, 1, 1, relu=False)]
    size = 40 + 4 + convs
    img = torch.from_numpy(rng.standard_normal((1, 1, size, size)).astype(np.float32)).cuda()
    first, second = (B.SKNet(layers, 1, 2, dtype="bf16") for _ in range(2))
    count = convs + 2
    for i in range(count):
        s = first.conv_shape(i)
        first.set_weights(i, (rng.standard_normal(s) * np.sqrt(2 / np.prod(s[1:]))).astype(np.float32), (0.1 * rng.random(s[0])).astype(np.float32))
    first.plan(1, size, size, pad=False, training=True, fused_head=True)
    lab = torch.from_numpy(rng.integers(-1, 2, (1,) + tuple(first.out_shape()[2:])).astype(np.int32)).cuda()
    before = first.forward(img).cpu().numpy().copy()
    first.backward(lab)
    first.sgd_step(lr=0.3)
    for i in range(count):
        second.set_weights(i, *first.get_weights(i))
    second.plan(1, size, size, pad=False, training=True, fused_head=True)
    got = []
    for net in (first, second):
        prob = net.forward(img).cpu().numpy().copy()
        net.backward(lab)
        got.append([prob] + [net.get_grad(i)[0] for i in range(count)])
        net.close()
    assert not np.array_equal(before, got[0][0])
    for a, b in zip(*got):
        assert np.array_equal(a, b)
