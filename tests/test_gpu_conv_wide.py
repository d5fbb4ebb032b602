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
