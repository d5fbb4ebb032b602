"""GPU parity on degenerate and ragged shapes: single-pixel outputs, images barely larger than the
context, wide-and-short images, odd batch sizes, maps that do not fill an octet or an MFMA tile."""
import numpy as np
import pytest
import torch

import sk_synth as S
from oracle import nets as ON

pytestmark = pytest.mark.gpu

TOL = {"f32": 1e-4, "bf16": 2e-2, "f16": 2e-2}


def make_net(layers, c_in, classes, ws, bs, dtype):
    from paper_1509_03371_amd import binding as B
    net = B.SKNet(layers, c_in, classes, dtype=dtype)
    for i, (w, b) in enumerate(zip(ws, bs)):
        net.set_weights(i, w, b)
    return net


def compare(layers, c_in, classes, img, dtype, pad, seed):
    ws, bs = S.he_normal_weights(layers, c_in, seed, bias_scale=0.1)
    net = make_net(layers, c_in, classes, ws, bs, dtype)
    n, _, h, w = img.shape
    net.plan(n, h, w, pad=pad)
    got = net.forward(torch.from_numpy(img).cuda()).cpu().numpy()
    ref = ON.sknet_forward(img, layers, ws, bs, pad=pad)
    assert got.shape == ref.shape
    assert np.abs(got - ref).max() <= TOL[dtype]
    net.close()
    return got


@pytest.mark.parametrize("dtype", ["f32", "bf16", "f16"])
def test_single_output_pixel_without_padding(dtype):
    # an image of exactly context + 1 samples per side, unpadded: the net of configs C2-C4 yields one pixel
    layers = S.sknet_layers(width=48, hidden=200)
    got = compare(layers, 1, 2, S.uniform_image(2, 1, 61, 61, 40), dtype, False, 41)
    assert got.shape == (2, 2, 1, 1)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_smallest_image_that_reflect_padding_accepts(dtype):
    # reflect padding by 30 needs 31 samples; 31 x 37 -> padded 91 x 97
    layers = S.sknet_layers(width=48, hidden=200)
    got = compare(layers, 1, 2, S.uniform_image(1, 1, 31, 37, 42), dtype, True, 43)
    assert got.shape == (1, 2, 31, 37)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_wide_short_image_odd_batch_ragged_maps(dtype):
    # 3 images, 3 input maps, 20 / 9 / 5 maps (no octet or 16-map tile is full), 35 x 301 pixels
    layers = [S.conv(20, 4, 1), S.pool(2, 1), S.conv(9, 3, 2), S.pool(2, 2), S.conv(5, 1, 1, relu=False)]
    got = compare(layers, 3, 5, S.uniform_image(3, 3, 35, 301, 44), dtype, True, 45)
    assert got.shape == (3, 5, 35, 301)
    assert np.abs(got.sum(1) - 1).max() < 1e-3


def test_image_too_small_for_reflect_padding_is_rejected():
    from paper_1509_03371_amd import binding as B
    layers = S.sknet_layers()
    net = B.SKNet(layers, 1, 2)
    with pytest.raises(B.SknetError):
        net.plan(1, 30, 64, pad=True)          # context 60 -> 30 rows of border need 31 rows
    with pytest.raises(B.SknetError):
        net.plan(1, 60, 60, pad=False)         # unpadded: the map vanishes
    net.close()


def test_fp32_5x5_map_of_more_than_2_to_the_29_samples():
    # byte offsets inside such a map leave 32 bits: the layer runs on the generic kernel.  fp32 sums of 25 products, softmax
    # of two logits below 8: 1e-5
    from paper_1509_03371_amd import binding as B
    side = 23171
    assert side * side >= 2 ** 29
    rng = np.random.default_rng(46)
    w, b = (rng.standard_normal((2, 1, 5, 5)) * 0.5).astype(np.float32), rng.standard_normal(2).astype(np.float32)
    net = B.SKNet([S.conv(2, 5, 1, relu=False)], 1, 2)
    net.set_weights(0, w, b)
    net.plan(1, side, side, pad=False)
    img = torch.rand((1, 1, side, side), generator=torch.Generator("cuda").manual_seed(47), device="cuda")
    prob = net.forward(img)
    out = side - 4
    assert tuple(prob.shape) == (1, 2, out, out)
    for y, x in ((0, 0), (0, out - 40), (out - 40, 0), (out - 40, out - 40), (out // 2, out // 3), (17000, 22001)):
        ref = torch.nn.functional.conv2d(img[:, :, y:y + 44, x:x + 44].cpu().double(), torch.from_numpy(w).double(), torch.from_numpy(b).double())
        got = prob[:, :, y:y + 40, x:x + 40].cpu().double()
        assert (got - ref.softmax(1)).abs().max() <= 1e-5, (y, x)
    net.close()
