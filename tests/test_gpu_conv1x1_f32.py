"""GPU check of the fp32 1x1 kernels (forward, data gradient with and without ReLU mask, weight and bias gradient, fused head): against fp64
results of the very tensors the GPU holds.  Planes below, at and just past the 64 pixels of a wave and off every multiple of four,
maps off the tiles of 16 and the steps of four, both sides of the 48 maps one side may have and of the 208 of the other, more
tiles than one half of a weight gradient's waves takes, maps shared out over workgroups, several images.

An fp32 sum of K products errs by at most (K + 2) * 2^-24 of the sum of magnitudes; a gradient's chains are at most pixels / 4 + 512
additions long.  A class probability moves by at most the largest error of a class sum (the softmax's slope is at most 1/4 a class, four
classes and more add up to less than 1) and a few roundings."""
import numpy as np
import pytest
import torch

import sk_synth as S

pytestmark = pytest.mark.gpu

U = 2.0 ** -24


def double(a):
    return torch.from_numpy(np.ascontiguousarray(a)).double()


@pytest.mark.parametrize("c_in,c_hid,classes,n,h,w", [
    (48, 200, 2, 1, 65, 75), (48, 200, 3, 2, 14, 16), (16, 208, 2, 1, 33, 40), (17, 209, 2, 1, 33, 40), (49, 50, 2, 1, 30, 31), (1, 33, 1, 1, 9, 9),
    (5, 16, 8, 3, 9, 9), (8, 17, 5, 1, 8, 8), (9, 112, 2, 2, 40, 41), (20, 113, 4, 1, 41, 43), (33, 48, 2, 1, 9, 10), (48, 49, 6, 2, 60, 61),
    (24, 64, 2, 4, 257, 66), (48, 200, 2, 1, 260, 262), (200, 48, 2, 1, 50, 47), (12, 65, 2, 1, 4, 5),
])
def test_layers(c_in, c_hid, classes, n, h, w):
    from paper_1509_03371_amd import binding as B
    layers = [S.conv(c_in, 2, 1, relu=True), S.conv(c_hid, 1, 1, relu=True), S.conv(classes, 1, 1, relu=False)]
    rng = np.random.default_rng(c_in + h * w)
    net, head = B.SKNet(layers, 2, classes), B.SKNet(layers, 2, classes)
    ws, bs = [], []
    for i in range(3):
        s = net.conv_shape(i)
        ws.append((rng.standard_normal(s) / np.sqrt(np.prod(s[1:]))).astype(np.float32))
        bs.append(rng.standard_normal(s[0]).astype(np.float32))
        net.set_weights(i, ws[i], bs[i])
        head.set_weights(i, ws[i], bs[i])
    net.plan(n, h, w, pad=False, training=True)
    head.plan(n, h, w, pad=False)
    image = torch.from_numpy(rng.standard_normal((n, 2, h, w)).astype(np.float32)).cuda()
    labels = torch.from_numpy(rng.integers(-1, classes, (n, h - 1, w - 1)).astype(np.int32)).cuda()
    labels[0, 0, 0] = 0
    net.forward(image)
    x, hid, z = (double(net.get_activation(i)) for i in range(3))
    dx, dh, dz = (double(net.get_activation_grad(i, labels)) for i in range(3))
    net.backward(labels)
    grads = [net.get_grad(i) for i in range(3)]
    prob = head.forward(image).cpu().double()
    net.close()
    head.close()

    def mix(w, t):                                          # sum over maps: w [o, c], t [n, c, y, x]
        return torch.einsum("oc,ncyx->noyx", w, t)

    def close(got, ref, mag, terms):
        assert bool(((got - ref).abs() <= (terms + 2) * U * mag).all())

    w1, w2, b1, b2 = double(ws[1].reshape(c_hid, c_in)), double(ws[2].reshape(classes, c_hid)), double(bs[1]), double(bs[2])
    add = lambda t, b: t + b[:, None, None]
    ref = add(mix(w1, x), b1)
    close(hid, ref.clamp(min=0), add(mix(w1.abs(), x.abs()), b1.abs()), c_in)
    close(z, add(mix(w2, hid), b2), add(mix(w2.abs(), hid), b2.abs()), c_hid)
    close(dh, mix(w2.T, dz) * (hid > 0), mix(w2.T.abs(), dz.abs()), classes)
    close(dx, mix(w1.T, dh) * (x > 0), mix(w1.T.abs(), dh.abs()), c_hid)
    pixels = n * (h - 1) * (w - 1)
    for i, (a, g) in ((1, (x, dh)), (2, (hid, dz))):
        dw, db = double(grads[i][0][:, :, 0, 0]), double(grads[i][1])
        close(dw, torch.einsum("noyx,ncyx->oc", g, a), torch.einsum("noyx,ncyx->oc", g.abs(), a.abs()), pixels / 4 + 512)
        close(db, g.sum((0, 2, 3)), g.abs().sum((0, 2, 3)), pixels / 4 + 512)
    hid64 = ref.clamp(min=0)
    slack = (c_in + 2) * U * mix(w2.abs(), add(mix(w1.abs(), x.abs()), b1.abs())) + (c_hid + 2) * U * add(mix(w2.abs(), hid64), b2.abs())
    p = torch.softmax(add(mix(w2, hid64), b2), 1)
    assert bool(((prob - p).abs() <= slack.amax(1, keepdim=True) + 16 * U).all())
