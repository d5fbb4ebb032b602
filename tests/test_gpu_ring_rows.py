"""GPU: 16-bit 4x4 layers on tiles of 4, 6 and 8 rows, which the launch picks by how many rounds of tiles the output is.  Layers copy their input
shifted by one tap and every value is a multiple of 1/16, so maps and pooled maps are known exactly: seams between tiles, row phases of unequal
length, ragged columns, overlapping and carried rows of pooled outputs."""
import numpy as np
import pytest
import torch

import sk_synth as S

pytestmark = pytest.mark.gpu

# 256 compute units: one round of 4-row tiles, two rounds of 6, one or four of 8; the last ones walk long runs of tiles
SIZES = [(1, 1, 60, 70), (2, 1, 117, 137), (8, 1, 90, 200), (2, 1, 562, 550), (4, 1, 548, 140), (1, 5, 253, 260), (2, 2, 294, 327), (16, 2, 210, 150),
         (2, 8, 700, 380)]


def tap_weights(c_out, c_in, tap):
    w = np.zeros((c_out, c_in, 4, 4), np.float32)
    w[np.arange(c_out), np.arange(c_out) % c_in, tap[0], tap[1]] = 1.0
    return w


def make(layers, c_in, ws, dtype):
    from paper_1509_03371_amd import binding as B
    net = B.SKNet(layers, c_in, 2, dtype=dtype)
    for i, w in enumerate(ws):
        net.set_weights(i, w, np.zeros(w.shape[0], np.float32))
    return net


def image(n, c, h, w):
    return (np.random.default_rng(h + w).integers(-16, 48, (n, c, h, w)) / 16.0).astype(np.float32)


def shifted(x, maps, tap, d):
    h, w = x.shape[2] - 3 * d, x.shape[3] - 3 * d
    return np.maximum(x[:, np.arange(maps) % x.shape[1], tap[0] * d:tap[0] * d + h, tap[1] * d:tap[1] * d + w], 0)


@pytest.mark.parametrize("maps", [16, 48])
@pytest.mark.parametrize("d,n,h,w", SIZES)
def test_layer(d, n, h, w, maps):
    c_in = 16
    x = image(n, c_in, h + 3 * d, w + 3 * d)
    net = make([S.conv(maps, 4, d, relu=True), S.conv(2, 1, 1, relu=False)], c_in, [tap_weights(maps, c_in, (2, 1)), np.ones((2, maps, 1, 1), np.float32)], "bf16")
    net.plan(n, x.shape[2], x.shape[3], pad=False, keep=True)
    net.forward(torch.from_numpy(x).cuda())
    assert np.array_equal(net.get_activation(0), shifted(x, maps, (2, 1), d))
    net.close()


@pytest.mark.parametrize("d,n,h,w", SIZES)
def test_layer_behind_and_in_front_of_pools(d, n, h, w):
    maps, c_in = 32, 16
    x = image(n, c_in, h + 10 * d, w + 10 * d)
    layers = [S.conv(maps, 4, d, relu=True), S.pool(2, d), S.conv(maps, 4, d, relu=True), S.pool(2, d), S.conv(maps, 4, d, relu=True), S.conv(24, 1, 1, relu=True),
              S.conv(2, 1, 1, relu=False)]
    ws = [tap_weights(maps, c_in, (1, 2)), tap_weights(maps, maps, (3, 0)), tap_weights(maps, maps, (0, 3)), np.ones((24, maps, 1, 1), np.float32),
          np.ones((2, 24, 1, 1), np.float32)]
    net = make(layers, c_in, ws, "f16")
    net.plan(n, x.shape[2], x.shape[3], pad=False)
    assert [net.step_name(i).split("_")[-1] for i in range(net.num_steps())][1:3] == ["vpool", "vpool"]
    net.forward(torch.from_numpy(x).cuda())
    ref = x
    for tap in ((1, 2), (3, 0)):
        y = shifted(ref, maps, tap, d)
        ref = np.maximum(np.maximum(y[:, :, :-d, :-d], y[:, :, :-d, d:]), np.maximum(y[:, :, d:, :-d], y[:, :, d:, d:]))
    assert np.array_equal(net.get_activation(4), shifted(ref, maps, (0, 3), d))
    net.close()
