"""GPU parity of the 16-bit convolutions for many maps (1x1, 3x3, 5x5, 6x6, 8x8, 10x10): every tile shape and dispatch branch at sizes that leave
remainders (pixels, rows, map groups, input maps off the chunk of 32), the widest kernel strides, fp32 output planes, and,
through a U-Net small enough that its deep layers split their input maps, partial sums, masks and zero borders.

The layer tests round image and weights to the storage type first, so that against fp64 only the sum's fp32 rounding (below
K * 2^-24 of the sum of magnitudes, K <= 64*100: 2e-4) and the one rounding of the stored result (half a unit: 2^-8 bf16, 2^-11
fp16, relative) are left."""
import numpy as np
import pytest
import torch

import sk_synth as S
from oracle import layers as OL, nets as ON

pytestmark = pytest.mark.gpu

HALF_ULP = {"bf16": 2.0 ** -8, "f16": 2.0 ** -11}      # 8 and 11 significant bits: spacing 2^-7, 2^-10 of the power of two below


def rounded(a, dtype):
    return torch.from_numpy(a).to(torch.bfloat16 if dtype == "bf16" else torch.float16).float().numpy()


NARROW = (0, 0, 1, 0)                                  # conv_h_kernel: small images, or maps that would pack with too much waste


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("k,d,c_in,c_out,n,h,w,path", [
    # 3x3, tiles of 8 rows x 32 pixels: remainders everywhere; strides 1, 2 and 6 (three and four input loads a wave)
    (3, 1, 64, 64, 1, 36, 35, NARROW), (3, 2, 40, 112, 2, 33, 64, (1, 0, 1, 3)), (3, 18, 32, 64, 1, 56, 69, NARROW),
    (3, 6, 96, 128, 1, 20, 50, (1, 0, 1, 4)), (3, 1, 33, 64, 1, 3, 3, NARROW), (3, 1, 72, 64, 1, 36, 35, (1, 0, 1, 3)),
    # ... the widest stride (one octet row of 68 units; d > rows), and one pixel
    (3, 18, 72, 64, 1, 56, 69, (1, 0, 1, 8)), (3, 1, 65, 64, 1, 3, 3, (1, 0, 1, 3)),
    # ... 16 rows x 32: more tiles than CUs; strides 1 and 6 (five / eight input loads a wave)
    (3, 1, 64, 128, 2, 262, 182, (1, 1, 1, 5)), (3, 6, 96, 64, 2, 312, 302, (1, 1, 1, 8)),
    # ... 12 rows x 64
    (3, 1, 64, 64, 2, 402, 391, (1, 2, 1, 8)),
    # 1x1: 128 x 128 pixels on eight waves; on four; 128 x 256; 64 x 256 (an odd number of 64-map groups in the first three)
    (1, 1, 40, 112, 2, 23, 60, (1, 0, 1, 1)), (1, 1, 64, 320, 1, 17, 30, (1, 0, 1, 1)), (1, 1, 33, 512, 2, 90, 101, (1, 1, 1, 2)),
    (1, 1, 320, 448, 1, 150, 150, (1, 2, 1, 4)), (1, 1, 64, 64, 2, 300, 300, (1, 3, 1, 4)), (1, 1, 32, 64, 1, 1, 1, (1, 0, 1, 1)),
    # large kernels on images too small for large tiles, and 70 maps
    (5, 1, 40, 70, 2, 37, 41, NARROW), (6, 1, 33, 112, 1, 22, 39, NARROW), (6, 3, 64, 64, 1, 49, 50, NARROW), (8, 8, 40, 64, 2, 93, 90, NARROW),
    (10, 8, 64, 64, 1, 107, 130, NARROW), (10, 10, 32, 64, 1, 100, 122, NARROW), (8, 18, 40, 64, 1, 130, 149, NARROW), (5, 2, 32, 512, 1, 72, 136, NARROW),
    # more maps than the LDS holds biases for at this kernel stride
    (5, 18, 32, 7184, 1, 75, 81, NARROW),
    # large kernels, 16 rows x 32 pixels: two, four and six input loads a wave; odd input maps, ragged map groups
    (5, 1, 40, 64, 9, 61, 45, (2, 2, 1, 2)), (5, 9, 37, 64, 9, 82, 79, (2, 2, 1, 4)), (5, 16, 40, 64, 5, 138, 104, (2, 2, 1, 6)),
    (6, 1, 33, 64, 9, 65, 76, (2, 2, 1, 2)), (6, 8, 40, 64, 9, 81, 106, (2, 2, 1, 4)), (6, 16, 40, 64, 5, 158, 145, (2, 2, 1, 6)),
    (8, 1, 40, 112, 5, 56, 76, (2, 2, 1, 2)), (8, 8, 40, 112, 5, 93, 128, (2, 2, 1, 4)), (8, 12, 33, 112, 3, 145, 154, (2, 2, 1, 6)),
    (10, 4, 40, 208, 5, 56, 109, (2, 2, 1, 4)), (10, 8, 40, 192, 3, 111, 139, (2, 2, 1, 6)), (10, 1, 40, 256, 9, 38, 10, (2, 2, 1, 4)),
    # ... 8 rows x 64
    (5, 1, 40, 208, 16, 9, 146, (2, 4, 1, 2)), (5, 10, 40, 112, 9, 71, 80, (2, 4, 1, 4)), (5, 18, 40, 64, 5, 154, 112, (2, 4, 1, 6)),
    (6, 2, 40, 112, 16, 20, 155, (2, 4, 1, 2)), (6, 9, 40, 64, 16, 72, 90, (2, 4, 1, 4)), (6, 18, 40, 64, 9, 148, 131, (2, 4, 1, 6)),
    (8, 10, 40, 208, 5, 100, 110, (2, 4, 1, 4)), (8, 16, 33, 112, 5, 161, 154, (2, 4, 1, 6)),
    (10, 2, 40, 512, 9, 25, 58, (2, 4, 1, 4)), (10, 8, 40, 208, 5, 96, 118, (2, 4, 1, 6)), (10, 10, 40, 192, 5, 91, 92, (2, 4, 1, 6)),
])
def test_layer(dtype, k, d, c_in, c_out, n, h, w, path):
    from paper_1509_03371_amd import binding as B
    assert B.sk_probe_conv_path(k, d, c_in, c_out, n, h - (k - 1) * d, w - (k - 1) * d) == path
    layers = [S.conv(c_out, k, d, relu=True), S.conv(2, 1, 1, relu=False)]
    rng = np.random.default_rng(k * h + w)
    img = rounded(rng.standard_normal((n, c_in, h, w)).astype(np.float32), dtype)
    ws = [rounded((rng.standard_normal((c_out, c_in, k, k)) / np.sqrt(c_in * k * k)).astype(np.float32), dtype), np.ones((2, c_out, 1, 1), np.float32)]
    bs = [rng.standard_normal(c_out).astype(np.float32), np.zeros(2, np.float32)]
    net = B.SKNet(layers, c_in, 2, dtype=dtype)
    for i in range(2):
        net.set_weights(i, ws[i], bs[i])
    net.plan(n, h, w, pad=False, keep=True)
    net.forward(torch.from_numpy(img).cuda())
    ref = OL.conv_sk(img, ws[0], bs[0], d, relu=True)
    got = net.get_activation(0)
    assert got.shape == ref.shape
    # fp16's subnormal results carry an absolute half unit of 2^-25
    assert np.all(np.abs(got - ref) <= HALF_ULP[dtype] * np.abs(ref) + 2e-4 + 2.0 ** -25)
    net.close()


@pytest.mark.parametrize("k,c_in,c_out,h,w", [(3, 64, 70, 21, 40), (1, 40, 112, 19, 33)])
def test_many_class_planes(k, c_in, c_out, h, w):
    # the last layer leaves fp32 planes; 112 classes pack without waste, 70 stay on the narrow kernel
    from paper_1509_03371_amd import binding as B
    layers = [S.conv(c_in, 1, 1, relu=True), S.conv(c_out, k, 1, relu=False)]
    rng = np.random.default_rng(5)
    ws = [np.eye(c_in, dtype=np.float32).reshape(c_in, c_in, 1, 1), rounded((rng.standard_normal((c_out, c_in, k, k)) * 0.1).astype(np.float32), "bf16")]
    bs = [np.zeros(c_in, np.float32), rng.standard_normal(c_out).astype(np.float32)]
    img = rounded(rng.random((2, c_in, h, w)).astype(np.float32), "bf16")
    net = B.SKNet(layers, c_in, c_out, dtype="bf16")
    for i in range(2):
        net.set_weights(i, ws[i], bs[i])
    net.plan(2, h, w, pad=False, keep=True)
    net.forward(torch.from_numpy(img).cuda())
    assert np.abs(net.get_activation(1) - OL.conv_sk(img, ws[1], bs[1], 1, relu=False)).max() <= 2e-4
    net.close()


def test_usknet_data_gradients():
    # 64..512 maps: the data gradients of the 6x6, 4x4, 8x8 and 1x1 layers read zero borders around the error maps.  Tolerances as
    # in the 16-bit training tests, which hold the nets of few maps to them
    from paper_1509_03371_amd import binding as B
    base, h, w, n = 64, 206, 214, 2
    params = S.usknet_params(2, 2, 550, base=base, bias_scale=0.1)
    net = B.USKNet(2, 2, base_ch=base, dtype="bf16")
    for i, name in enumerate(S.USKNET_PARAM_NAMES):
        net.set_weights(i, *params[name])
    img = np.stack([np.stack([S.em_like_image(h, w, 551 + 7 * i + c) for c in range(2)]) for i in range(n)]).astype(np.float32)
    net.plan(n, h, w, training=True)
    ho, wo = net.output_size(h, w)
    lab = np.random.default_rng(552).integers(0, 2, (n, ho, wo)).astype(np.int32)
    net.forward(torch.from_numpy(img).cuda())
    net.backward(torch.from_numpy(lab).cuda())
    p64 = {k: (a.astype(np.float64), b.astype(np.float64)) for k, (a, b) in params.items()}
    _, ref = ON.usknet_backward(img, p64, lab, base=base)
    for i, name in enumerate(S.USKNET_PARAM_NAMES):
        err = np.abs(net.get_grad(i)[0] - ref[name][0]).max() / np.abs(ref[name][0]).max()
        print("%s %.2e" % (name, err), flush=True)
        assert err <= 8e-2, name
    net.close()


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
def test_unet_with_split_layers(dtype):
    # 128..512 maps on maps of 4 to 28 pixels: the deep layers and their data gradients split the input maps.  Tolerances as in
    # the 16-bit training tests (a dozen rounded tensors between input and gradient)
    from paper_1509_03371_amd import binding as B
    depth, base, h, w, n = 2, 128, 60, 76, 2
    params = S.unet_params(1, 2, 540, depth=depth, base=base, bias_scale=0.05)
    names = S.unet_param_names(depth)
    net = B.UNet(1, 2, depth=depth, base_ch=base, dtype=dtype)
    for i, name in enumerate(names):
        net.set_weights(i, *params[name])
    img = np.stack([S.em_like_image(h, w, 541 + i)[None] for i in range(n)]).astype(np.float32)
    net.plan(n, h, w, training=True)
    ho, wo = net.output_size(h, w)
    rng = np.random.default_rng(542)
    lab = rng.integers(0, 2, (n, ho, wo)).astype(np.int32)
    lab[rng.random(lab.shape) < 0.25] = -1
    image, labels = torch.from_numpy(img).cuda(), torch.from_numpy(lab).cuda()
    prob = net.forward(image).cpu().numpy()
    loss = float(net.backward(labels).item())
    p64 = {k: (a.astype(np.float64), b.astype(np.float64)) for k, (a, b) in params.items()}
    assert np.abs(prob - ON.unet_forward(img, p64, depth=depth)).max() <= 2e-2
    ref_loss, ref = ON.unet_backward(img, p64, lab, depth=depth)
    assert abs(loss - ref_loss) <= 2e-2 * abs(ref_loss)
    tol = {"bf16": 8e-2, "f16": 3e-2}[dtype]
    grads = [net.get_grad(i) for i in range(len(names))]
    for name, (dw, _) in zip(names, grads):
        err = np.abs(dw - ref[name][0]).max() / np.abs(ref[name][0]).max()
        print("%s %.2e" % (name, err), flush=True)
        assert err <= tol, name
    net.forward(image)                                   # partial sums are added in a fixed order
    net.backward(labels)
    for i, (dw, db) in enumerate(grads):
        again = net.get_grad(i)
        assert np.array_equal(dw, again[0]) and np.array_equal(db, again[1])
    net.close()


def store(t, dtype):
    return t.to(torch.bfloat16 if dtype == "bf16" else torch.float16).double()


def sparse_labels(shape, classes, kept, rng):
    """Labels of about `kept` samples, half of them on the border of the map; -1 elsewhere."""
    labels = np.full(shape, -1, np.int32)
    for i in range(kept):
        at = [int(rng.integers(0, s)) for s in shape]
        if i % 2:
            axis = int(rng.integers(1 if len(shape) == 3 and shape[0] < 3 else 0, len(shape)))
            at[axis] = 0 if i % 4 == 1 else shape[axis] - 1
        labels[tuple(at)] = rng.integers(0, classes)
    return labels


def error_map(prob, labels, dtype):
    """dz = (p - onehot) / P of the labelled samples, rounded to the storage type; prob [n, classes, ...]."""
    kept = labels >= 0
    onehot = torch.nn.functional.one_hot(labels.clamp(min=0).long(), prob.shape[1]).movedim(-1, 1)
    dz = (prob - onehot) * kept.unsqueeze(1) / max(1, int(kept.sum()))
    return store(dz.float(), dtype)


def gradient_bound(ref, dz, w, dtype):
    """The stored result's half unit, the fp32 sum (2e-4 of the magnitudes, as above), and two samples of dz that the GPU, which
    forms the softmax in fp32, rounds to the other side of a boundary."""
    ulp = HALF_ULP[dtype]
    return ulp * ref.abs() + (2e-4 + 4 * ulp) * float(dz.abs().max()) * float(w.abs().max()) + 2.0 ** -25


@pytest.mark.parametrize("relu", [False, True])
@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("k,d,maps,classes,n,h,w,path", [
    # the data gradient of a k x k layer to `classes` maps: zeros around the error map, ReLU mask of the layer below, ragged sizes
    (3, 1, 112, 40, 2, 33, 37, (1, 0, 1, 3)), (3, 4, 64, 72, 1, 41, 66, (1, 0, 1, 4)), (3, 18, 64, 64, 1, 333, 303, (1, 0, 1, 8)),
    # sizes kept on conv_h_kernel: padded loads, one chunk, up to 64 columns, the 32 x 16 tile at stride 6
    (3, 18, 64, 64, 1, 110, 71, (0, 0, 1, 0)), (3, 4, 64, 32, 1, 105, 110, (0, 0, 1, 0)), (3, 1, 64, 96, 1, 42, 64, (0, 0, 1, 0)),
    (3, 6, 128, 40, 1, 162, 167, (0, 0, 1, 0)),
    (3, 1, 128, 40, 2, 262, 182, (1, 1, 1, 5)), (3, 6, 64, 40, 2, 310, 303, (1, 1, 1, 8)), (3, 1, 64, 40, 2, 402, 391, (1, 2, 1, 8)),
    (1, 1, 112, 40, 2, 23, 61, (1, 0, 1, 1)), (1, 1, 512, 33, 2, 90, 101, (1, 1, 1, 2)), (1, 1, 64, 40, 2, 301, 300, (1, 3, 1, 4)),
])
def test_data_gradient(dtype, relu, k, d, maps, classes, n, h, w, path):
    from paper_1509_03371_amd import binding as B
    assert B.sk_probe_conv_path(k, d, classes, maps, n, h, w, data_gradient=True) == path
    rng = np.random.default_rng(h + w)
    net = B.SKNet([S.conv(maps, 1, 1, relu=relu), S.conv(classes, k, d, relu=False)], 2, classes, dtype=dtype)
    w1 = rounded((rng.standard_normal((classes, maps, k, k)) / np.sqrt(maps * k * k)).astype(np.float32), dtype)
    net.set_weights(0, rng.standard_normal((maps, 2, 1, 1)).astype(np.float32), rng.standard_normal(maps).astype(np.float32))
    net.set_weights(1, w1, np.zeros(classes, np.float32))
    net.plan(n, h, w, pad=False, training=True)
    prob = net.forward(torch.from_numpy(rng.standard_normal((n, 2, h, w)).astype(np.float32)).cuda()).cpu().double()
    labels = sparse_labels((n,) + tuple(prob.shape[2:]), classes, 400, rng)
    got = torch.from_numpy(net.get_activation_grad(0, torch.from_numpy(labels).cuda())).double()
    dz = error_map(prob, torch.from_numpy(labels), dtype)
    ref = torch.from_numpy(OL.conv_sk_bwd_data(dz.numpy(), w1, d, (h, w)))
    if relu:
        ref = ref * (torch.from_numpy(net.get_activation(0)) > 0)
    assert float(ref.abs().max()) > 1e-5
    assert bool(((got - ref).abs() <= gradient_bound(ref, dz, torch.from_numpy(w1), dtype)).all())
    net.close()


# 3-D nets hand the kernels slices as images and (depth tap, octet) pairs as input octets: at d > 1 groups of octets with slices
# between them, of any size against the chunk of four
@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("k,d,c_in,c_out,size,path", [
    (3, 1, 16, 112, (4, 21, 40), (1, 0, 1, 3)), (3, 2, 16, 112, (3, 21, 40), (1, 0, 1, 3)), (3, 2, 24, 128, (3, 20, 33), (1, 0, 1, 3)),
    (3, 4, 40, 112, (2, 18, 35), (1, 0, 1, 4)), (3, 2, 48, 64, (3, 30, 33), (1, 0, 1, 3)), (3, 3, 8, 112, (3, 19, 34), (0, 0, 1, 0)),
    (3, 2, 72, 64, (2, 16, 20), (1, 0, 1, 3)), (5, 2, 8, 64, (16, 61, 45), (2, 2, 1, 2)), (5, 1, 24, 64, (16, 61, 45), (2, 2, 1, 2)),
    (5, 3, 24, 112, (9, 40, 60), (2, 2, 1, 4)), (5, 4, 16, 112, (9, 50, 62), (2, 2, 1, 4)), (5, 2, 8, 64, (4, 20, 20), (0, 0, 1, 0)),
])
def test_volume_layer(dtype, k, d, c_in, c_out, size, path):
    from paper_1509_03371_amd import binding as B
    octets = (c_in + 7) // 8
    assert B.sk_probe_conv_path(k, d, k * octets * 8, c_out, *size) == path
    rng = np.random.default_rng(k * size[1] + c_in)
    net = B.SKNet3D([S.conv(c_out, k, d, relu=True), S.conv(2, 1, 1, relu=False)], c_in, 2, dtype=dtype)
    full = tuple(s + (k - 1) * d for s in size)
    img = rounded(rng.standard_normal((full[0], c_in) + full[1:]).astype(np.float32), dtype)
    w0 = rounded((rng.standard_normal((c_out, c_in, k, k, k)) / np.sqrt(c_in * k ** 3)).astype(np.float32), dtype)
    b0 = rng.standard_normal(c_out).astype(np.float32)
    net.set_weights(0, w0, b0)
    net.set_weights(1, np.ones((2, c_out, 1, 1, 1), np.float32), np.zeros(2, np.float32))
    net.plan(*full)
    net.forward(torch.from_numpy(img).cuda())
    volume = torch.from_numpy(img).double().transpose(0, 1).unsqueeze(0)
    ref = torch.nn.functional.conv3d(volume, torch.from_numpy(w0).double(), torch.from_numpy(b0).double(), dilation=d).clamp(min=0)[0].transpose(0, 1).numpy()
    got = net.get_activation(0)
    assert got.shape == ref.shape
    assert np.all(np.abs(got - ref) <= HALF_ULP[dtype] * np.abs(ref) + 2e-4 + 2.0 ** -25)
    net.close()


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("k,d,maps,classes,size,relu,path", [
    (3, 1, 112, 12, (3, 19, 36), True, (1, 0, 1, 3)), (3, 2, 112, 20, (5, 20, 37), True, (1, 0, 1, 3)), (3, 2, 112, 20, (5, 20, 37), False, (1, 0, 1, 3)),
    (3, 4, 64, 44, (9, 24, 67), True, (1, 0, 1, 4)), (3, 4, 64, 44, (9, 24, 39), True, (0, 0, 1, 0)),
    (5, 1, 64, 2, (16, 49, 45), False, (2, 2, 1, 2)), (5, 2, 64, 20, (16, 49, 47), False, (2, 2, 1, 2)),
    (5, 3, 112, 2, (13, 40, 62), False, (2, 2, 1, 4)), (5, 2, 64, 2, (9, 20, 20), False, (0, 0, 1, 0)),
])
def test_volume_data_gradient(dtype, k, d, maps, classes, size, relu, path):
    # A 1x1x1 layer on input maps that are each one sample of 1: its weight gradient [map][input map] is the stored error map of
    # `map` at that sample, mask included (no sum is left: one product each)
    from paper_1509_03371_amd import binding as B
    octets = (classes + 7) // 8
    assert B.sk_probe_conv_path(k, d, k * octets * 8, maps, *size, data_gradient=True) == path
    rng = np.random.default_rng(k * size[1] + classes)
    probes, halo = 32, (k - 1) * d
    spots = [tuple(int(rng.choice([0, 1, halo, s // 2, s - 1 - halo, s - 2, s - 1])) for s in size) for _ in range(probes - 1)] + [(0, 0, 0)]
    img = np.zeros((size[0], probes) + size[1:], np.float32)
    out = tuple(s - halo for s in size)
    labels = np.full(out, -1, np.int32)
    for j, at in enumerate(spots):
        img[at[0], j, at[1], at[2]] = 1.0
        for _ in range(10):                                  # label some of the outputs that read this sample
            o = [a - d * int(rng.integers(0, k)) for a in at]
            if all(0 <= v < s for v, s in zip(o, out)):
                labels[tuple(o)] = rng.integers(0, classes)
    labels[0, 0, 0] = 0
    net = B.SKNet3D([S.conv(maps, 1, 1, relu=relu), S.conv(classes, k, d, relu=False)], probes, classes, dtype=dtype)
    w1 = rounded((rng.standard_normal((classes, maps, k, k, k)) / np.sqrt(maps)).astype(np.float32), dtype)
    net.set_weights(0, rng.standard_normal((maps, probes, 1, 1, 1)).astype(np.float32), rng.standard_normal(maps).astype(np.float32))
    net.set_weights(1, w1, np.zeros(classes, np.float32))
    net.plan(*size, training=True)
    prob = net.forward(torch.from_numpy(img).cuda()).cpu().double()
    prob = prob.reshape((out[0], classes) + out[1:]).transpose(0, 1).unsqueeze(0)
    net.backward(torch.from_numpy(labels).cuda())
    got = torch.from_numpy(net.get_grad(0)[0].reshape(maps, probes)).double()
    dz = error_map(prob, torch.from_numpy(labels).unsqueeze(0), dtype)
    ref = torch.nn.functional.conv_transpose3d(dz, torch.from_numpy(w1).double(), dilation=d)[0]
    hidden = torch.from_numpy(net.get_activation(0)).transpose(0, 1) if relu else None
    at = tuple(torch.tensor([s[i] for s in spots]) for i in range(3))
    ref = ref[:, at[0], at[1], at[2]]
    if relu:
        ref = ref * (hidden[:, at[0], at[1], at[2]] > 0)
    assert float(ref.abs().max()) > 1e-4
    # several maps may share a spot: each still reads its own product
    assert bool(((got - ref).abs() <= gradient_bound(ref, dz, torch.from_numpy(w1), dtype)).all())
    net.close()


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
def test_unet_split_layers_forward(dtype):
    # a bottom level small enough to split its input maps, and an up-convolution that splits: against the GPU's own stored inputs.
    # The 3x3 layers' pair has one stored map between them, where a value may fall to the other side of a rounding boundary (one in
    # a hundred: fp32 sums err by 2e-5 of a unit): four times their rms share in a sum is allowed
    from paper_1509_03371_amd import binding as B
    base, h, w = 128, 36, 44
    params = S.unet_params(1, 2, 560, depth=1, base=base, bias_scale=0.1)
    names = S.unet_param_names(1)
    net = B.UNet(1, 2, depth=1, base_ch=base, dtype=dtype)
    for i, name in enumerate(names):
        net.set_weights(i, *params[name])
    img = S.em_like_image(h, w, 561)[None, None].astype(np.float32)
    net.plan(1, h, w)
    net.forward(torch.from_numpy(img).cuda())
    bh, bw = (h - 4) // 2, (w - 4) // 2
    assert B.sk_probe_conv_path(3, 1, 2 * base, 2 * base, 1, bh - 4, bw - 4, scratch=True)[2] > 1
    assert B.sk_probe_conv_path(1, 1, 2 * base, 4 * base, 1, bh - 4, bw - 4, scratch=True)[0] == 1
    r = {name: (rounded(params[name][0], dtype).astype(np.float64), params[name][1].astype(np.float64)) for name in names}
    pooled, _ = OL.maxpool_sk(net.get_activation("down0").astype(np.float64), 2, 1, 2)
    a = OL.conv_sk(pooled, *r["down1a"], d=1, relu=True)
    a = rounded(a.astype(np.float32), dtype).astype(np.float64)
    ref = OL.conv_sk(a, *r["down1b"], d=1, relu=True)
    got = net.get_activation("down1")
    flips = 4 * 2 * HALF_ULP[dtype] * np.sqrt(9 * 2 * base / 100.0) * np.sqrt((a ** 2).mean() * (r["down1b"][0] ** 2).mean())
    assert np.all(np.abs(got - ref) <= HALF_ULP[dtype] * np.abs(ref) + 2e-4 + flips)
    up = OL.upconv2x2(got.astype(np.float64), *r["up0"])
    assert np.all(np.abs(net.get_activation("up0") - up) <= HALF_ULP[dtype] * np.abs(up) + 2e-4)
    net.close()


class RoundedLayers:
    """The oracle's layers with every stored map and error map, and the weights of every product, rounded to a 16-bit type."""

    def __init__(self, dtype):
        self.r = lambda a: rounded(np.asarray(a, np.float32), dtype).astype(np.float64)

    def __getattr__(self, name):
        return getattr(OL, name)

    def conv_sk(self, x, w, b=None, d=1, relu=False):
        y = OL.conv_sk(x, self.r(w), b, d, relu)
        return self.r(y) if relu else y                          # the layer without a ReLU is the last: fp32 logits

    def upconv2x2(self, x, w, b):
        return self.r(OL.upconv2x2(x, self.r(w), b))

    def softmax_loss(self, z, labels):
        loss, g = OL.softmax_loss(z, labels)
        return loss, self.r(g)

    def conv_sk_bwd_data(self, g, w, d, in_hw):
        return self.r(OL.conv_sk_bwd_data(g, self.r(w), d, in_hw))

    def maxpool_bwd(self, g, am, in_hw):
        return self.r(OL.maxpool_bwd(g, am, in_hw))

    def upconv2x2_bwd(self, x, w, g):
        dx, dw, db = OL.upconv2x2_bwd(x, self.r(w), g)
        return self.r(dx), dw, db


def whole_number_params(shapes, seed):
    """Weights of -1, 0 and 1, three taps per output, biases of -1, 0 and 1 (the last layer: 64ths): maps and products of whole
    numbers that 16 bits hold exactly, so that no sum depends on its order and no value on a rounding."""
    rng = np.random.default_rng(seed)
    out = {}
    for name, (w, b) in shapes.items():
        w = np.zeros_like(w)
        up = w.shape[2] == 2
        flat = w.transpose(1, 2, 3, 0).reshape(-1, w.shape[0]) if up else w.reshape(w.shape[0], -1)     # [outputs][taps]
        for row in flat:
            row[rng.choice(row.size, 3, replace=False)] = rng.choice([-1.0, 1.0], 3)
        if up:
            w = np.ascontiguousarray(flat.reshape(w.shape[1], 2, 2, w.shape[0]).transpose(3, 0, 1, 2))
        else:
            w = flat.reshape(w.shape)
        b = rng.integers(-1, 2, b.shape).astype(np.float32)
        out[name] = (w, b)
    last = list(shapes)[-1]
    head = shapes[last][0].shape
    out[last] = ((rng.integers(-2, 3, head) / 64.0).astype(np.float32), out[last][1] / 64)
    return out


@pytest.mark.parametrize("net_kind,dtype", [("unet", "bf16"), ("unet", "f16"), ("usknet", "bf16")])
def test_whole_number_nets(net_kind, dtype, monkeypatch):
    # Whole-net gradients of nets whose every stored value is exact: U-Net layers with split input maps (partial sums, zero borders
    # and ReLU masks in the reduction), USK-Net 6x6 and 8x8 layers.  The border of the labels is kept whole, the rest sparse.
    # Error maps are rounded where the GPU stores them; their sums are exact in fp32.  Left: the softmax in fp32 (1e-6) and the fp32
    # sums of the weight gradients, and one error value in 30000 that rounds to the other side (2^-8 of itself)
    from paper_1509_03371_amd import binding as B
    if net_kind == "unet":
        n, base, h, w = 1, 128, 36, 44
        names = S.unet_param_names(1)
        params = whole_number_params({k: S.unet_params(1, 2, 570, depth=1, base=base)[k] for k in names}, 574)
        net = B.UNet(1, 2, depth=1, base_ch=base, dtype=dtype)
        bh, bw = (h - 4) // 2, (w - 4) // 2
        for c, hh, ww in ((2 * base, bh - 2, bw - 2), (base, bh, bw)):
            assert B.sk_probe_conv_path(3, 1, 2 * base, c, 1, hh, ww, data_gradient=True, scratch=True)[2] > 1
    else:
        n, base, h, w = 3, 64, 230, 262
        names = S.USKNET_PARAM_NAMES
        params = whole_number_params({k: S.usknet_params(1, 2, 571, base=base)[k] for k in names}, 575)
        net = B.USKNet(1, 2, base_ch=base, dtype=dtype)
        bh, bw = (h - 4) // 2, (w - 4) // 2
        assert B.sk_probe_conv_path(6, 1, 2 * base, base, n, bh, bw, data_gradient=True)[0] == 2
        assert B.sk_probe_conv_path(8, 8, 8 * base, 2 * base, n, bh - 30, bw - 30, data_gradient=True)[0] == 2
    for i, name in enumerate(names):
        net.set_weights(i, *params[name])
    rng = np.random.default_rng(576)
    img = rng.integers(0, 3, (n, 1, h, w)).astype(np.float32)
    net.plan(n, h, w, training=True)
    ho, wo = net.output_size(h, w)
    lab = np.full((n, ho, wo), -1, np.int32)
    keep = rng.random(lab.shape) < 0.1
    keep[:, [0, -1], :] = keep[:, :, [0, -1]] = True
    lab[keep] = rng.integers(0, 2, int(keep.sum()))
    prob = net.forward(torch.from_numpy(img).cuda()).cpu().numpy()
    loss = float(net.backward(torch.from_numpy(lab).cuda()).item())
    monkeypatch.setattr(ON, "L", RoundedLayers(dtype))
    p64 = {name: (a.astype(np.float64), b.astype(np.float64)) for name, (a, b) in params.items()}
    forward, backward, kind = (ON.unet_forward, ON.unet_backward, {"depth": 1}) if net_kind == "unet" else (ON.usknet_forward, ON.usknet_backward, {"base": base})
    assert np.abs(prob - forward(img, p64, **kind)).max() <= 1e-5
    ref_loss, ref = backward(img, p64, lab, **kind)
    assert abs(loss - ref_loss) <= 1e-5 * abs(ref_loss)
    for i, name in enumerate(names):
        dw, db = net.get_grad(i)
        size = np.linalg.norm(ref[name][0])
        assert size > 1e-3, name
        e, eb = np.linalg.norm(dw - ref[name][0]) / size, np.linalg.norm(db - ref[name][1]) / max(np.linalg.norm(ref[name][1]), size * 1e-2)
        print("%s dW %.2e db %.2e" % (name, e, eb), flush=True)
        assert e <= 1e-4 and eb <= 1e-4, name
    net.close()
