"""Weight and bias gradients of one layer with nothing to round: inputs, output gradients and all partial sums are integers (times one power of two)
that fp32 and the storage type hold, so a kernel's result must be the exact one bit for bit, in whatever order it adds."""
import numpy as np
import torch

import sk_synth as S


def check(c_in, c_out, k, d, n, h, w, dtype, labelled=None):
    """The layer c_in -> c_out between a 1x1 layer with small integers and one to four classes.  Its own weights are zero: all logits are 0,
    every probability is 1/4, and the loss gradient of a labelled pixel is (1, 1, 1, -3) / (4 * labelled) in some order."""
    from paper_1509_03371_amd import binding as B
    layers = [S.conv(c_in, 1, 1, relu=False), S.conv(c_out, k, d, relu=False), S.conv(4, 1, 1, relu=False)]
    rng = np.random.default_rng(c_in * 1000 + h * w)
    ho, wo = h - (k - 1) * d, w - (k - 1) * d
    if labelled is None:
        labelled = 1 << ((n * ho * wo).bit_length() - 1)
    net = B.SKNet(layers, 3, 4, dtype=dtype)
    net.set_weights(0, rng.integers(-1, 2, (c_in, 3, 1, 1)).astype(np.float32), rng.integers(-1, 2, c_in).astype(np.float32))
    net.set_weights(1, np.zeros((c_out, c_in, k, k), np.float32), np.zeros(c_out, np.float32))
    net.set_weights(2, rng.integers(-3, 4, (4, c_out, 1, 1)).astype(np.float32), np.zeros(4, np.float32))
    net.plan(n, h, w, pad=False, training=True)
    net.forward(torch.from_numpy(rng.integers(-2, 3, (n, 3, h, w)).astype(np.float32)).cuda())
    labels = np.full(n * ho * wo, -1, np.int32)
    labels[rng.permutation(n * ho * wo)[:labelled]] = rng.integers(0, 4, labelled)
    labels = torch.from_numpy(labels.reshape(n, ho, wo)).cuda()
    dy = torch.from_numpy(net.get_activation_grad(1, labels)).double() * (4 * labelled)
    net.backward(labels)
    dw, db = net.get_grad(1)
    x = torch.from_numpy(net.get_activation(0)).double()
    net.close()
    for t in (x, dy):
        assert bool((t == t.round()).all()) and float(t.abs().max()) <= 18 and float((t != 0).double().mean()) > 0.05 * labelled / (n * ho * wo)
    ys = dy.permute(1, 0, 2, 3).reshape(c_out, -1)
    for i in range(k):
        for j in range(k):
            xs = x[:, :, i * d:i * d + ho, j * d:j * d + wo].permute(1, 0, 2, 3).reshape(c_in, -1)
            assert float((ys.abs() @ xs.abs().T).max()) < 2 ** 24               # no partial sum leaves the integers of fp32
            assert torch.equal(torch.from_numpy(dw[:, :, i, j]).double() * (4 * labelled), ys @ xs.T), (i, j)
    assert torch.equal(torch.from_numpy(db).double() * (4 * labelled), ys.sum(1))
