"""GPU parity of the fp32 4x4 weight gradient on the 16-bit matrix unit, and of how the row-streaming gradients deal out their rows: phases that
are no equal share, strips with one half beyond the image, several images, operands whose magnitudes rise and fall from row to row.

Both operands are pairs of fp16 values, a product is within 2^-19 of its magnitude, and a sum of K products (hundreds at least) within
(K + 9) * 2^-24 of the sum of magnitudes of the very products that make it, whatever else is in their rows; the reference takes the maps and error
maps of the pass itself."""
import numpy as np
import pytest
import torch

import sk_synth as S

pytestmark = pytest.mark.gpu


def gradient(c_in, c_out, d, n, h, w, dtype="f32", scale=None, maps=None, map_scale=None, error_scale=None, masked=None):
    """(gradient of a 4x4 layer, its bias gradient, the layer's input, its error map); map_scale, error_scale: of the input's and the error
    map's maps; masked: rows and columns without labels"""
    from paper_1509_03371_amd import binding as B
    rng = np.random.default_rng(h + w)
    net = B.SKNet([S.conv(c_in, 1, 1, relu=True), S.conv(c_out, 4, d, relu=False), S.conv(2, 1, 1, relu=False)], 3, 2, dtype=dtype)
    for i in range(3):
        s = net.conv_shape(i)
        net.set_weights(i, (rng.standard_normal(s) / np.sqrt(np.prod(s[1:]))).astype(np.float32), rng.standard_normal(s[0]).astype(np.float32) * np.float32(i != 0))
    if map_scale is not None or error_scale is not None:
        s0, s2 = net.conv_shape(0), net.conv_shape(2)
        net.set_weights(0, rng.standard_normal(s0).astype(np.float32) * (1 if map_scale is None else map_scale[:, None, None, None]), np.zeros(s0[0], np.float32))
        net.set_weights(2, rng.standard_normal(s2).astype(np.float32) * (1 if error_scale is None else error_scale[None, :, None, None]), np.zeros(2, np.float32))
    if maps is not None:                                    # every map of the layer's input is this image
        w0 = np.zeros(net.conv_shape(0), np.float32)
        w0[:, 0] = 1
        net.set_weights(0, w0, np.zeros(c_in, np.float32))
    net.plan(n, h, w, pad=False, training=True)
    img = rng.standard_normal((n, 3, h, w)).astype(np.float32)
    if maps is not None:
        img[:, 0] = maps
    if scale is not None:
        img *= scale
    net.forward(torch.from_numpy(img).cuda())
    lab = rng.integers(-1, 2, (n, h - 3 * d, w - 3 * d)).astype(np.int32)
    if masked is not None:
        lab[:, masked[0], masked[1]] = -1
    lab = torch.from_numpy(lab).cuda()
    net.backward(lab)
    dw, db = net.get_grad(1)
    x, dy = net.get_activation(0), net.get_activation_grad(1, lab)
    net.close()
    return dw, db, x, dy


def sums(x, dy, d):
    x, dy = torch.from_numpy(x).double(), torch.from_numpy(dy).double()
    n, c_out, ho, wo = dy.shape
    out = torch.zeros(c_out, x.shape[1], 4, 4, dtype=torch.double)
    for i in range(4):
        for j in range(4):
            win = x[:, :, i * d:i * d + ho, j * d:j * d + wo]
            for b in range(n):
                out[:, :, i, j] += dy[b].reshape(c_out, -1) @ win[b].reshape(win.shape[1], -1).T.contiguous()
    return out.numpy(), dy.sum(dim=(0, 2, 3)).numpy()


@pytest.mark.parametrize("c_in,c_out,d,n,h,w", [
    (48, 48, 2, 1, 180, 300), (48, 48, 8, 1, 207, 217), (32, 16, 1, 3, 103, 99), (40, 24, 3, 2, 209, 140), (48, 40, 7, 1, 721, 50), (16, 48, 1, 2, 303, 310),
    (32, 32, 4, 12, 100, 40),
])
def test_gradient(c_in, c_out, d, n, h, w):
    check_gradient(c_in, c_out, d, n, h, w)


def check_gradient(c_in, c_out, d, n, h, w, **scales):
    dw, db, x, dy = gradient(c_in, c_out, d, n, h, w, **scales)
    ref, rb = sums(x, dy, d)
    size, sb = sums(np.abs(x), np.abs(dy), d)
    products = dy.size // c_out
    assert np.abs(ref).max() > 1e-4
    assert np.all(np.abs(dw - ref) <= (products + 9) * 2.0 ** -24 * size) and np.all(np.abs(db - rb) <= (products + 9) * 2.0 ** -24 * sb)
    # sums of random signs: what the bound allows all of them at once, a right kernel shows a hundredth of
    assert np.linalg.norm(dw - ref) <= 3e-7 * np.linalg.norm(ref)


# every kernel: (output map tiles, input map tiles); the last two stay on the fp32 matrix unit
@pytest.mark.parametrize("c_in,c_out,d,n,h,w,tiles", [
    (16, 24, 1, 1, 303, 700, (2, 1)), (16, 48, 2, 1, 306, 650, (3, 1)), (32, 16, 1, 1, 203, 230, (1, 2)), (24, 32, 2, 2, 260, 390, (2, 2)),
    (32, 40, 3, 1, 250, 200, (3, 2)), (48, 16, 4, 1, 200, 270, (1, 3)), (40, 24, 1, 1, 180, 260, (2, 3)), (48, 40, 8, 1, 250, 230, (3, 3)),
    (48, 48, 1, 1, 703, 7, (3, 3)), (48, 48, 1, 1, 710, 6, (0, 0)), (16, 16, 1, 1, 303, 700, (0, 0)),
])
@pytest.mark.parametrize("wide", [False, True])
def test_every_kernel(c_in, c_out, d, n, h, w, tiles, wide):
    from paper_1509_03371_amd import binding as B
    assert B.sk_probe_pairs_path(4, d, c_in, c_out, n, h - 3 * d, w - 3 * d, 2)[:2] == tiles
    check_gradient(c_in, c_out, d, n, h, w, map_scale=np.float32(10.0) ** -np.linspace(0, 20, c_in).astype(np.float32) if wide else None)


@pytest.mark.parametrize("way", ["rising", "falling", "dark half"])
def test_magnitudes(way):
    h, w, d = 180, 300, 2
    ramp = np.float32(2.0) ** np.linspace(-12, 12, h).astype(np.float32)[:, None]
    scale = {"rising": ramp, "falling": ramp[::-1], "dark half": np.where(np.arange(w) < 150, np.float32(1e-7), np.float32(1))[None, :]}[way]
    dw, db, x, dy = gradient(48, 48, d, 1, h, w, scale=scale.astype(np.float32))
    ref, _ = sums(x, dy, d)
    assert np.linalg.norm(dw - ref) <= 1e-6 * np.linalg.norm(ref)


# A gradient whose products do not meet the large samples of its rows is as right as if they were not there
@pytest.mark.parametrize("d,h,w", [(2, 180, 300), (8, 207, 217)])
@pytest.mark.parametrize("case", ["input maps", "error maps", "both", "outlier", "outliers in every row", "dark columns"])
def test_magnitudes_far_apart(case, d, h, w):
    # (both: products of 1e-24, beside labels' 1e-5, stay above 2^-126, where fp32 has all its bits)
    down = (np.float32(10.0) ** -np.linspace(0, 12 if case == "both" else 24, 48).astype(np.float32)).astype(np.float32)
    args = {}
    if case in ("input maps", "both"):
        args["map_scale"] = down[::-1] if case == "both" else down
    if case in ("error maps", "both"):
        args["error_scale"] = down
    if case.startswith("outlier"):
        maps = np.random.default_rng(3).uniform(0.1, 1.5, (1, h, w)).astype(np.float32)
        maps[:, 90 if case == "outlier" else slice(None), 70] = np.float32(1e22)
        args["maps"], args["masked"] = maps, (slice(None), slice(70 - 3 * d, 71))     # every error that meets an outlier is zero
    if case == "dark columns":
        args["scale"] = np.where(np.arange(w) % 64 < 32, np.float32(1e-18), np.float32(1))[None, :].astype(np.float32)
    dw, db, x, dy = gradient(48, 48, d, 1, h, w, **args)
    ref, rb = sums(x, dy, d)
    size, sb = sums(np.abs(x), np.abs(dy), d)
    products = dy.size // 48
    assert np.isfinite(ref).all() and np.abs(dy).max() > 0
    assert np.all(np.abs(dw - ref) <= (products + 9) * 2.0 ** -24 * size) and np.all(np.abs(db - rb) <= (products + 9) * 2.0 ** -24 * sb)
    # (sums of random signs: a hundredth of that)
    big = np.abs(ref) > 1e-3 * size
    assert np.sqrt(np.mean(((dw - ref)[big] / ref[big]) ** 2)) <= 3e-5


def test_samples_just_below_a_power_of_two():
    # rows behind the first four are eight times as large and end an ulp below 16: as far as the scale of the first ones reaches
    h, w, d = 180, 300, 1
    maps = np.random.default_rng(9).uniform(0.1, 1.5, (1, h, w)).astype(np.float32)
    maps[:, 4:] *= 8
    maps[:, 4::3, ::5] = np.nextafter(np.float32(16), np.float32(0))
    dw, db, x, dy = gradient(48, 48, d, 1, h, w, maps=maps)
    assert x.max() == maps.max()
    ref, _ = sums(x, dy, d)
    assert np.linalg.norm(dw - ref) <= 1e-6 * np.linalg.norm(ref)


# Both backward calls have scratch for 256 copies of any of these and take the same kernel
@pytest.mark.parametrize("c_in,c_out,h,w", [(16, 16, 300, 700), (16, 32, 300, 700), (48, 16, 180, 260), (32, 48, 180, 300)])
def test_both_backward_calls_agree_bit_for_bit(c_in, c_out, h, w):
    from paper_1509_03371_amd import binding as B
    rng = np.random.default_rng(c_in + c_out)
    net = B.SKNet([S.conv(c_in, 1, 1, relu=True), S.conv(c_out, 4, 1, relu=False), S.conv(2, 1, 1, relu=False)], 3, 2)
    for i in range(3):
        s = net.conv_shape(i)
        net.set_weights(i, (rng.standard_normal(s) / np.sqrt(np.prod(s[1:]))).astype(np.float32), rng.standard_normal(s[0]).astype(np.float32))
    net.plan(1, h, w, pad=False, training=True)
    img = torch.from_numpy(rng.standard_normal((1, 3, h, w)).astype(np.float32)).cuda()
    lab = torch.from_numpy(rng.integers(-1, 2, (1, h - 3, w - 3)).astype(np.int32)).cuda()
    got = []
    for noalloc in (False, True):
        net.forward(img)
        net.backward(lab, loss=torch.zeros(1, device="cuda"), noalloc=noalloc)
        got.append(net.get_grad(1))
    net.close()
    assert np.abs(got[0][0]).max() > 0
    np.testing.assert_array_equal(got[0][0], got[1][0])
    np.testing.assert_array_equal(got[0][1], got[1][1])


@pytest.mark.parametrize("c_in,c_out,d,n,h,w", [(48, 48, 2, 1, 568, 568), (16, 24, 8, 1, 100, 300), (24, 8, 5, 2, 61, 81), (48, 48, 21, 1, 90, 130), (8, 16, 3, 1, 700, 70)])
def test_rows_of_16_bit_gradients(c_in, c_out, d, n, h, w):
    dw, db, x, dy = gradient(c_in, c_out, d, n, h, w, dtype="bf16")
    ref, rb = sums(x, dy, d)
    size, sb = sums(np.abs(x), np.abs(dy), d)
    products = dy.size // c_out
    # operands are the stored bf16 values themselves; only the fp32 sums are rounded
    assert np.all(np.abs(dw - ref) <= (products + 2) * 2.0 ** -24 * size) and np.all(np.abs(db - rb) <= (products + 2) * 2.0 ** -24 * sb)
    assert np.linalg.norm(dw - ref) <= 2e-6 * np.linalg.norm(ref)
