"""GPU parity of the fp32 3x3 and 4x4 convolutions on the 16-bit matrix unit: every tile, ragged tiles, maps and map groups, kernel
strides up to the widest they take (a halo of 24; one more stays on the fp32 matrix unit), zero borders and ReLU masks of the data gradient,
samples and weights of any magnitude.

A value is a pair of fp16 values to 2^-21 of its magnitude or better, of three products the fourth partial one is below 2^-22, so a product is
within 2^-19 and the fp32 sum of K products (at least 216) within (K + 9) * 2^-24 of the sum of magnitudes of the very products that make an
output, whatever else is in its tile."""
import numpy as np
import pytest
import torch

import sk_synth as S
from oracle import layers as OL

pytestmark = pytest.mark.gpu


def forward(k, d, img, w0, b0, relu=True):
    from paper_1509_03371_amd import binding as B
    n, c_in, h, w = img.shape
    c_out = w0.shape[0]
    net = B.SKNet([S.conv(c_out, k, d, relu=relu), S.conv(2, 1, 1, relu=False)], c_in, 2)
    net.set_weights(0, w0, b0)
    net.set_weights(1, np.ones((2, c_out, 1, 1), np.float32), np.zeros(2, np.float32))
    net.plan(n, h, w, pad=False, keep=True)
    net.forward(torch.from_numpy(img).cuda())
    out = net.get_activation(0)
    net.close()
    return out


def check(k, d, img, w0, b0):
    got = forward(k, d, img, w0, b0)
    ref, size = OL.conv_sk(img, w0, b0, d, relu=True), OL.conv_sk(np.abs(img), np.abs(w0), np.abs(b0), d)
    products = k * k * img.shape[1]
    assert np.all(np.abs(got - ref) <= (products + 9) * 2.0 ** -24 * size + 1e-44)
    return got, ref


@pytest.mark.parametrize("k,d,c_in,c_out,n,h,w", [
    (4, 1, 24, 16, 1, 4, 4), (4, 1, 23, 16, 1, 30, 40), (4, 1, 25, 20, 2, 23, 70), (4, 2, 24, 48, 1, 150, 165), (4, 8, 48, 48, 1, 90, 97),
    (4, 9, 24, 48, 1, 60, 60), (4, 4, 40, 96, 1, 140, 141), (4, 3, 24, 33, 4, 160, 150), (4, 1, 24, 130, 1, 67, 66), (4, 5, 31, 64, 1, 260, 270),
    (4, 1, 48, 48, 1, 515, 530), (4, 2, 24, 32, 2, 300, 310), (4, 1, 24, 16, 1, 100, 40), (4, 2, 24, 16, 2, 330, 340),
    (3, 1, 24, 16, 1, 34, 36), (3, 1, 24, 16, 1, 10, 12), (3, 2, 26, 50, 2, 45, 71), (3, 12, 24, 32, 1, 80, 77), (3, 13, 24, 32, 1, 80, 77),
    (3, 4, 64, 96, 1, 100, 131), (3, 1, 64, 64, 1, 300, 290), (3, 1, 24, 144, 1, 142, 130), (3, 6, 33, 48, 3, 160, 170), (3, 1, 128, 128, 1, 68, 66),
    (3, 1, 24, 48, 2, 330, 310), (3, 2, 24, 20, 3, 300, 310),
])
def test_forward(k, d, c_in, c_out, n, h, w):
    rng = np.random.default_rng(h * w + c_in)
    img = rng.standard_normal((n, c_in, h, w)).astype(np.float32)
    w0, b0 = rng.standard_normal((c_out, c_in, k, k)).astype(np.float32), rng.standard_normal(c_out).astype(np.float32)
    check(k, d, img, w0, b0)


# (kernel, d, output maps, output height: of 24 maps, ten columns more) and the tile it picks (map tiles, rows, waves side by side): every tile at every
# pitch of the staged rows that kernel strides lead to
TILES = [
    (3, 1, 16, 36, (1, 2, 2)), (3, 8, 16, 36, (1, 2, 2)), (3, 1, 96, 60, (1, 4, 2)), (3, 8, 64, 72, (1, 4, 2)), (3, 2, 32, 168, (1, 4, 4)),
    (3, 8, 32, 156, (1, 4, 4)), (3, 4, 64, 200, (2, 4, 2)), (3, 8, 64, 200, (2, 4, 2)), (3, 1, 64, 350, (2, 6, 4)), (3, 8, 32, 410, (2, 6, 4)),
    (3, 1, 32, 440, (2, 8, 4)), (3, 8, 32, 440, (2, 8, 4)), (3, 1, 48, 320, (3, 4, 2)), (3, 8, 48, 320, (3, 4, 2)), (3, 1, 48, 350, (3, 5, 4)),
    (3, 8, 48, 350, (3, 5, 4)),
    (4, 1, 16, 24, (1, 2, 2)), (4, 4, 16, 24, (1, 2, 2)), (4, 8, 16, 30, (1, 2, 2)), (4, 1, 96, 60, (1, 4, 2)), (4, 4, 96, 60, (1, 4, 2)),
    (4, 8, 64, 72, (1, 4, 2)), (4, 2, 32, 168, (1, 4, 4)), (4, 4, 16, 560, (1, 4, 4)), (4, 8, 32, 156, (1, 4, 4)), (4, 1, 96, 180, (2, 4, 2)),
    (4, 4, 64, 200, (2, 4, 2)), (4, 8, 64, 200, (2, 4, 2)), (4, 1, 64, 180, (2, 6, 4)), (4, 4, 64, 168, (2, 6, 4)), (4, 8, 64, 168, (2, 6, 4)),
    (4, 1, 32, 440, (2, 8, 4)), (4, 4, 32, 440, (2, 8, 4)), (4, 8, 32, 440, (2, 8, 4)), (4, 1, 48, 200, (3, 4, 2)), (4, 4, 96, 132, (3, 4, 2)),
    (4, 8, 96, 132, (3, 4, 2)), (4, 1, 48, 350, (3, 5, 4)), (4, 4, 48, 350, (3, 5, 4)), (4, 8, 48, 350, (3, 5, 4)),
]


@pytest.mark.parametrize("wide", [False, True])
@pytest.mark.parametrize("k,d,c_out,ho,tile", TILES)
def test_every_tile(k, d, c_out, ho, tile, wide):
    from paper_1509_03371_amd import binding as B
    wo, halo = ho + 10, (k - 1) * d
    assert B.sk_probe_pairs_path(k, d, 24, c_out, 1, ho, wo) == tile
    rng = np.random.default_rng(ho)
    img = rng.standard_normal((1, 24, ho + halo, wo + halo)).astype(np.float32)
    if wide:                                                 # half of the tiles, all of them where there are few, on the fp32 matrix unit
        img[0, rng.integers(24, size=40), rng.integers(ho + halo, size=40), rng.integers(wo + halo, size=40)] = np.float32(1e-20)
    check(k, d, img, rng.standard_normal((c_out, 24, k, k)).astype(np.float32), rng.standard_normal(c_out).astype(np.float32))


@pytest.mark.parametrize("case", ["tiny", "huge", "rising", "falling", "zero chunk", "bright corner", "small weights", "large weights"])
def test_magnitudes(case):
    rng = np.random.default_rng(5)
    img = rng.standard_normal((1, 40, 70, 130)).astype(np.float32)
    w0 = rng.standard_normal((48, 40, 4, 4)).astype(np.float32)
    steps = np.float32(2.0) ** np.repeat(np.arange(-16, 17, 8), 8).astype(np.float32)[None, :, None, None]
    if case == "tiny":
        img *= np.float32(1e-30)
    elif case == "huge":
        img *= np.float32(1e30)
    elif case == "rising":                                  # the scale of the sums falls from chunk to chunk
        img *= steps
    elif case == "falling":
        img *= steps[:, ::-1]
    elif case == "zero chunk":
        img[:, :8] = 0
        img[:, 16:24] = 0
    elif case == "bright corner":
        img[:, 3, :9, :9] *= np.float32(1e6)
    elif case == "small weights":
        w0 *= np.float32(1e-25)
    else:
        w0 *= np.float32(1e20)
    check(4, 2, img, w0, np.zeros(48, np.float32))


# Magnitudes far apart, finite: a sum of products that does not meet the large ones is as right as if they were not there
@pytest.mark.parametrize("k,d", [(3, 1), (4, 2), (3, 8)])
@pytest.mark.parametrize("case", ["1e9", "1e30", "outlier in the last chunk", "dark half", "maps", "pixels", "log-uniform"])
def test_samples_far_apart(case, k, d):
    rng = np.random.default_rng(11)
    img = rng.standard_normal((1, 40, 70, 130)).astype(np.float32)
    w0 = rng.standard_normal((48, 40, k, k)).astype(np.float32)
    if case in ("1e9", "1e30"):
        img[0, 3, 20, 50] = np.float32(case)
    elif case == "outlier in the last chunk":                # sums of four chunks follow the scale down
        img[0, 39, 33, 70] = np.float32(1e22)
    elif case == "dark half":
        img[..., 64:] *= np.float32(1e-11)
    elif case == "maps":                                     # half of the output maps meet the small ones alone
        img *= (np.float32(10.0) ** -np.arange(40, dtype=np.float32))[None, :, None, None] * np.float32(1e6)
        w0[::2, :20] = 0
    elif case == "pixels":
        img[:, :, ::3, ::5] *= np.float32(1e-14)
        w0[::2, :, 0, 0] = 0
    else:
        img *= np.exp2(rng.uniform(-40, 40, img.shape)).astype(np.float32)
    check(k, d, img, w0, np.zeros(48, np.float32))


@pytest.mark.parametrize("k", [3, 4])
@pytest.mark.parametrize("case", ["output maps", "output maps, falling", "one large weight", "input maps", "log-uniform", "pruned"])
def test_weights_far_apart(case, k):
    rng = np.random.default_rng(12)
    img = rng.standard_normal((1, 40, 70, 130)).astype(np.float32)
    w0 = rng.standard_normal((50, 40, k, k)).astype(np.float32)
    steps = np.float32(2.0) ** -np.linspace(0, 80, 50).astype(np.float32)[:, None, None, None]
    if case == "output maps":
        w0 *= steps
    elif case == "output maps, falling":
        w0 *= steps[::-1]
    elif case == "one large weight":                         # of output map 7; the others don't know it
        w0[7, 11, 1, 1] = np.float32(1e28)
        img[:, 11, :, 70:] = 0
    elif case == "input maps":                               # where the samples of the first twenty are zero, the small weights decide
        w0[:, 20:] *= np.float32(1e-12)
        img[:, :20, :, 60:] = 0
    elif case == "log-uniform":
        w0 *= np.exp2(rng.uniform(-40, 40, w0.shape)).astype(np.float32)
    else:
        w0[3:40] = 0
        w0[41, 5:] *= np.float32(1e-33)
    check(k, 1, img, w0, np.zeros(50, np.float32))


# Ordinary samples: no further from 64 bits than on the fp32 matrix unit, whose sums are rounded after every four products
@pytest.mark.parametrize("c_in", [24, 48])
@pytest.mark.parametrize("k", [3, 4])
def test_error_of_ordinary_sums(k, c_in):
    rng = np.random.default_rng(13)
    img = np.maximum(rng.standard_normal((1, c_in, 90, 140)), 0).astype(np.float32)
    w0 = (rng.standard_normal((48, c_in, k, k)) / (7 * k)).astype(np.float32)
    got = forward(k, 1, img, w0, np.zeros(48, np.float32), relu=False)
    ref = OL.conv_sk(img, w0, np.zeros(48), 1)
    ho, wo = ref.shape[2:]
    fp32 = np.zeros(ref.shape[1:], np.float32)
    for c in range(0, c_in, 4):
        for i in range(k):
            for j in range(k):
                four = np.tensordot(w0[:, c:c + 4, i, j].astype(np.float64), img[0, c:c + 4, i:i + ho, j:j + wo].astype(np.float64), 1)
                fp32 = (fp32 + four).astype(np.float32)
    assert np.linalg.norm(got[0] - ref[0]) <= np.linalg.norm(fp32 - ref[0])


def test_infinities_and_nan_stay_where_they_are():
    rng = np.random.default_rng(6)
    img = rng.standard_normal((1, 24, 60, 120)).astype(np.float32)
    w0 = rng.standard_normal((48, 24, 4, 4)).astype(np.float32)
    clean = forward(4, 1, img, w0, np.zeros(48, np.float32), relu=False)
    bad = img.copy()
    bad[0, 2, 20, 30] = np.inf
    bad[0, 9, 40, 90] = np.nan
    got = forward(4, 1, bad, w0, np.zeros(48, np.float32), relu=False)
    hit = np.zeros(clean.shape, bool)
    hit[:, :, 17:21, 27:31] = True
    hit[:, :, 37:41, 87:91] = True
    assert not np.isfinite(got[hit]).any()
    size = OL.conv_sk(np.abs(img), np.abs(w0), np.zeros(48), 1)
    assert np.all(np.abs(got - clean)[~hit] <= 2 * (384 + 9) * 2.0 ** -24 * size[~hit])


@pytest.mark.parametrize("k", [3, 4])
def test_samples_just_below_a_power_of_two(k):
    # the maps behind the first eight are eight times as large and end an ulp below 16: as far as the scale of the first ones reaches
    rng = np.random.default_rng(7)
    img = rng.uniform(-1.5, 1.5, (1, 40, 70, 130)).astype(np.float32)
    img[:, 8:] *= 8
    img[:, 8:, ::3, ::5] = np.nextafter(np.float32(16), np.float32(0))
    w0 = rng.standard_normal((48, 40, k, k)).astype(np.float32)
    w0[::5] = np.nextafter(np.float32(4), np.float32(0))
    check(k, 2, img, w0, np.zeros(48, np.float32))


@pytest.mark.parametrize("which", ["samples", "weights"])
def test_infinities_keep_their_sign(which):
    # as on the fp32 matrix unit: ReLU drops minus infinity and keeps plus infinity
    rng = np.random.default_rng(8)
    img = rng.uniform(0.5, 1.5, (1, 24, 60, 120)).astype(np.float32)
    w0 = rng.standard_normal((48, 24, 4, 4)).astype(np.float32)
    w0 += np.sign(w0) * np.float32(0.01)
    if which == "samples":
        img[0, 2, 20, 30], img[0, 13, 40, 90] = np.inf, -np.inf
    else:
        w0[3, 5, 1, 2], w0[17, 20, 0, 3] = np.inf, -np.inf
    got = forward(4, 1, img, w0, np.zeros(48, np.float32))
    ref = OL.conv_sk(img, w0, np.zeros(48), 1, relu=True)
    assert np.isinf(ref).any() and np.array_equal(np.isinf(got), np.isinf(ref))
    clean = OL.conv_sk(np.where(np.isinf(img), 0, img), np.where(np.isinf(w0), 0, w0), np.zeros(48), 1, relu=False)
    dropped = (ref == 0) & (clean > 1)                       # minus infinity
    assert dropped.any() and not got[dropped].any()


@pytest.mark.parametrize("which", ["samples", "weights", "both"])
@pytest.mark.parametrize("k,d,c_in", [(3, 1, 24), (3, 4, 26), (3, 1, 31), (4, 1, 24), (4, 3, 29), (4, 2, 31)])
def test_infinities_meet_real_taps_and_maps_alone(k, d, c_in, which):
    # every kernel column meets one, the last map among them; an infinite sample meets an infinite weight; later chunks add finite products
    rng = np.random.default_rng(9 * k + c_in)
    img = rng.uniform(0.5, 1.5, (1, c_in, 50, 110)).astype(np.float32)
    w0 = rng.standard_normal((40, c_in, k, k)).astype(np.float32)
    w0 += np.sign(w0) * np.float32(0.01)
    if which != "weights":
        img[0, 2, 20, 30], img[0, c_in - 1, 33, 90], img[0, 12, 40, 5] = np.inf, -np.inf, np.inf
    if which != "samples":
        w0[3, 2, 1, 2], w0[17, c_in - 1, 0, k - 1], w0[39, 5, k - 1, 0] = np.inf, -np.inf, np.inf
    got = forward(k, d, img, w0, np.zeros(40, np.float32), relu=False)
    with np.errstate(invalid="ignore"):
        ref, size = OL.conv_sk(img, w0, np.zeros(40), d, relu=False), OL.conv_sk(np.abs(img), np.abs(w0), np.zeros(40), d)
    assert np.isposinf(ref).any() and np.isneginf(ref).any()
    assert np.array_equal(np.isposinf(got), np.isposinf(ref)) and np.array_equal(np.isneginf(got), np.isneginf(ref)) and np.array_equal(np.isnan(got), np.isnan(ref))
    finite = np.isfinite(ref)
    assert np.all(np.abs(got[finite] - ref[finite]) <= (k * k * c_in + 9) * 2.0 ** -24 * size[finite])


def check_data_gradient(k, d, maps, classes, n, h, w, relu):
    from paper_1509_03371_amd import binding as B
    rng = np.random.default_rng(h + w)
    w1 = rng.standard_normal((classes, maps, k, k)).astype(np.float32) * np.float32(0.2)
    net = B.SKNet([S.conv(maps, 1, 1, relu=relu), S.conv(classes, k, d, relu=False)], 2, classes)
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
    products = k * k * classes
    bound = (products + 9) * 2.0 ** -24 * size + 1e-6 / max(1, kept.sum()) * np.abs(w1).sum(axis=(0, 2, 3))[None, :, None, None]
    assert np.abs(ref).max() > 1e-6 and np.all(np.abs(got - ref) <= bound)
    net.close()


@pytest.mark.parametrize("relu", [False, True])
@pytest.mark.parametrize("k,d,maps,classes,n,h,w", [
    (4, 1, 8, 24, 2, 19, 71), (4, 2, 20, 25, 1, 47, 66), (4, 8, 48, 48, 1, 70, 131), (4, 9, 16, 24, 1, 70, 80), (3, 1, 40, 32, 1, 40, 131),
    (3, 12, 48, 24, 1, 85, 90), (3, 4, 64, 26, 1, 60, 64), (3, 2, 130, 24, 1, 40, 70), (4, 2, 96, 40, 1, 300, 250),
])
def test_data_gradient(k, d, maps, classes, n, h, w, relu):
    check_data_gradient(k, d, maps, classes, n, h, w, relu)


@pytest.mark.parametrize("k,d,maps,h,tile", TILES)
def test_every_tile_of_data_gradients(k, d, maps, h, tile):
    from paper_1509_03371_amd import binding as B
    assert B.sk_probe_pairs_path(k, d, 24, maps, 1, h, h + 10, 1) == tile
    check_data_gradient(k, d, maps, 24, 1, h, h + 10, True)


# Layers of volumes: the depth taps' maps in one launch (d = 1) or a launch each, whose sums are added to what is there (d = 2)
@pytest.mark.parametrize("d", [1, 2])
@pytest.mark.parametrize("case", ["plain", "weights far apart", "samples far apart", "infinity"])
def test_volumes(case, d):
    from oracle import nd as OND
    from paper_1509_03371_amd import binding as B
    rng = np.random.default_rng(d)
    vol = rng.standard_normal((32, 7, 45, 83)).astype(np.float32)
    w0 = rng.standard_normal((40, 32, 3, 3, 3)).astype(np.float32)
    if case == "weights far apart":
        w0 *= np.exp2(-np.linspace(0, 60, 40)).astype(np.float32)[:, None, None, None, None]
        w0[::3, :16] *= np.float32(1e-15)
    if case == "samples far apart":
        vol[5, 3, 20, 40] = np.float32(1e20)
    if case == "infinity":
        vol[5, 3, 20, 40] = np.float32(np.inf)
    net = B.SKNet3D([S.conv(40, 3, d, relu=False), S.conv(2, 1, 1, relu=False)], 32, 2)
    net.set_weights(0, w0, np.zeros(40, np.float32))
    net.set_weights(1, np.zeros((2, 40, 1, 1, 1), np.float32), np.zeros(2, np.float32))
    net.plan(7, 45, 83, keep=True)
    net.forward(torch.from_numpy(np.ascontiguousarray(vol.transpose(1, 0, 2, 3))).cuda())
    got = net.get_activation(0).transpose(1, 0, 2, 3)
    net.close()
    with np.errstate(invalid="ignore"):
        ref, size = OND.conv_sk3d(vol, w0, np.zeros(40), d), OND.conv_sk3d(np.abs(vol), np.abs(w0), np.zeros(40), d)
    finite = np.isfinite(ref)
    assert np.array_equal(got[~finite], ref[~finite].astype(np.float32)) and (case == "infinity") == (not finite.all())
    assert np.all(np.abs(got[finite] - ref[finite]) <= (27 * 32 + 9) * 2.0 ** -24 * size[finite])
