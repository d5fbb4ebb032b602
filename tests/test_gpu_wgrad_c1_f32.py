"""fp32 weight gradient of a layer with one input map: every kernel size, blocks of 32 pixels that end inside a row and rows shorter than one, maps off the
tiles of sixteen, several images, more blocks than waves, a column of the image that one column of taps alone meets.

The chains of a sum are at most blocks / 2048 + 1 times 32 products and 256 copies long and a tree of partial sums, so that K = 4096 bounds the roundings;
the reference takes the image and the error map of the pass itself."""
import numpy as np
import pytest
import torch

import sk_synth as S

pytestmark = pytest.mark.gpu


def step(k, d, c_out, n, h, w, img):
    from paper_1509_03371_amd import binding as B
    rng = np.random.default_rng(h * w + c_out)
    net = B.SKNet([S.conv(c_out, k, d, relu=False), S.conv(2, 1, 1, relu=False)], 1, 2)
    for i in range(2):
        s = net.conv_shape(i)
        net.set_weights(i, (rng.standard_normal(s) / np.sqrt(np.prod(s[1:]))).astype(np.float32), rng.standard_normal(s[0]).astype(np.float32))
    net.plan(n, h, w, pad=False, training=True)
    net.forward(torch.from_numpy(img).cuda())
    lab = torch.from_numpy(rng.integers(-1, 2, (n, h - (k - 1) * d, w - (k - 1) * d)).astype(np.int32)).cuda()
    net.backward(lab)
    dw, db = net.get_grad(0)
    dy = net.get_activation_grad(0, lab)
    net.close()
    return dw, db, dy


@pytest.mark.parametrize("k,d,c_out,n,h,w", [
    (4, 1, 48, 1, 260, 259), (4, 1, 8, 1, 99, 99), (3, 1, 64, 1, 70, 130), (2, 3, 17, 2, 33, 36), (4, 2, 1, 3, 41, 23), (3, 5, 33, 1, 12, 43), (4, 1, 16, 1, 4, 5),
    (2, 1, 49, 1, 300, 33), (4, 9, 30, 1, 28, 700),
])
def test_gradient(k, d, c_out, n, h, w):
    img = np.random.default_rng(w).standard_normal((n, 1, h, w)).astype(np.float32)
    dw, db, dy = step(k, d, c_out, n, h, w, img)
    x, dy = torch.from_numpy(img).double()[:, 0], torch.from_numpy(dy).double()
    ho, wo = dy.shape[2:]
    for i in range(k):
        for j in range(k):
            win = x[:, i * d:i * d + ho, j * d:j * d + wo].reshape(-1)
            e = dy.permute(1, 0, 2, 3).reshape(c_out, -1)
            ref, size = (e @ win).numpy(), (e.abs() @ win.abs()).numpy()
            assert np.all(np.abs(dw[:, 0, i, j] - ref) <= 4096 * 2.0 ** -24 * size)
    assert np.all(np.abs(db - dy.sum((0, 2, 3)).numpy()) <= 4096 * 2.0 ** -24 * dy.abs().sum((0, 2, 3)).numpy())


def test_last_column():
    # the last column of the image meets the last tap column alone
    img = np.random.default_rng(3).standard_normal((1, 1, 50, 53)).astype(np.float32)
    from paper_1509_03371_amd import binding as B
    net = B.SKNet([S.conv(20, 3, 1, relu=True), S.conv(2, 1, 1, relu=False)], 1, 2)
    w0 = np.zeros((20, 1, 3, 3), np.float32)
    w0[:, 0, :, :2] = np.random.default_rng(4).standard_normal((20, 3, 2))
    net.set_weights(0, w0, np.ones(20, np.float32))
    net.set_weights(1, np.stack([np.full((20, 1, 1), 0.01), np.full((20, 1, 1), -0.01)]).astype(np.float32), np.zeros(2, np.float32))   # (equal rows have no gradient)
    net.plan(1, 50, 53, pad=False, training=True)
    img[0, 0, :, 52] = 1e30
    net.forward(torch.from_numpy(img).cuda())
    net.backward(torch.from_numpy(np.zeros((1, 48, 51), np.int32)).cuda())
    dw, _ = net.get_grad(0)
    net.close()
    assert np.abs(dw[:, 0, :, :2]).max() < 1e3 and np.abs(dw[:, 0, :, 2]).max() > 1e20
