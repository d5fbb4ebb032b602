"""GPU check of the 16-bit weight gradient that loads input rows straight into LDS: against fp64 sums over the very tensors the GPU holds (the
layer's input and the gradient of its output, both in the 16-bit type, whose products are exact in fp32).  Segments of one column to
two segments and an odd rest (half a segment skipped at 32 and below), residue classes of unequal length and empty ones, maps off the
tiles, kernels of two to four rows with one tile group and several, windows up to the widest; in test_gradient a workgroup has one step, or
two, in test_walks many.
An element's sum takes at most pixels + 512 fp32 additions, so its error stays below (pixels + 512) * 2^-24 of the sum of magnitudes."""
import numpy as np
import pytest
import torch

import exact_wgrad
import sk_synth as S

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("c_in,c_out,k,d,n,h,w", [
    (16, 16, 3, 1, 1, 3, 3), (64, 64, 3, 1, 1, 30, 30), (64, 64, 3, 1, 2, 34, 34), (64, 72, 3, 1, 1, 5, 35), (128, 64, 3, 1, 1, 33, 66),
    (40, 24, 3, 2, 2, 9, 71), (96, 128, 3, 4, 1, 30, 137), (33, 33, 3, 1, 1, 70, 67), (24, 80, 2, 1, 2, 40, 90), (16, 48, 2, 5, 1, 8, 50),
    (64, 64, 4, 1, 1, 40, 100), (56, 100, 4, 3, 2, 25, 48), (20, 64, 3, 16, 1, 50, 130), (64, 16, 3, 12, 1, 70, 130), (80, 1, 3, 1, 3, 4, 66),
])
@pytest.mark.parametrize("dtype", ["bf16", "f16"])
def test_gradient(c_in, c_out, k, d, n, h, w, dtype):
    from paper_1509_03371_amd import binding as B
    layers = [S.conv(c_in, 1, 1, relu=False), S.conv(c_out, k, d, relu=False), S.conv(2, 1, 1, relu=False)]
    rng = np.random.default_rng(c_in + h * w)
    net = B.SKNet(layers, 3, 2, dtype=dtype)
    for i in range(3):
        s = net.conv_shape(i)
        net.set_weights(i, (rng.standard_normal(s) / np.sqrt(np.prod(s[1:]))).astype(np.float32), rng.standard_normal(s[0]).astype(np.float32))
    net.plan(n, h, w, pad=False, training=True)
    net.forward(torch.from_numpy(rng.standard_normal((n, 3, h, w)).astype(np.float32)).cuda())
    ho, wo = h - (k - 1) * d, w - (k - 1) * d
    labels = rng.integers(-1, 2, (n, ho, wo)).astype(np.int32)
    labels[0, 0, 0] = 1
    labels = torch.from_numpy(labels).cuda()
    dy = torch.from_numpy(net.get_activation_grad(1, labels)).double()
    net.backward(labels)
    dw, db = net.get_grad(1)
    x = torch.from_numpy(net.get_activation(0)).double()
    net.close()
    bound = (n * ho * wo + 512) * 2.0 ** -24
    for i in range(k):
        for j in range(k):
            xs = x[:, :, i * d:i * d + ho, j * d:j * d + wo].permute(1, 0, 2, 3).reshape(c_in, -1)
            ys = dy.permute(1, 0, 2, 3).reshape(c_out, -1)
            ref, mag = ys @ xs.T, ys.abs() @ xs.abs().T
            assert bool(((torch.from_numpy(dw[:, :, i, j]).double() - ref).abs() <= bound * mag).all()), (i, j)
    ref, mag = dy.sum(dim=(0, 2, 3)), dy.abs().sum(dim=(0, 2, 3))
    assert bool(((torch.from_numpy(db).double() - ref).abs() <= bound * mag).all())


# A workgroup walks at least twice round its ring of k + 2 (one team) or k + 3 (two) rows, over ends of strips, residue classes and images: the
# gradient's tile groups share at most 512 workgroups, two teams at most 256, so steps (64-column segments of output rows) / that is the
# least a workgroup gets.  Nothing rounds, so a row, column or buffer taken wrongly shows in the last bit.
@pytest.mark.parametrize("c_in,c_out,k,d,n,h,w,workgroups,ring", [
    (16, 16, 3, 1, 5, 522, 131, 512, 5), (24, 48, 3, 2, 9, 611, 94, 512, 5), (16, 64, 2, 3, 6, 700, 66, 512, 4), (64, 16, 3, 4, 3, 905, 70, 171, 5),
    (64, 64, 4, 3, 3, 500, 100, 128, 6),                                      # one team (the last one: more than 36 tiles a wave)
    (96, 64, 3, 1, 3, 301, 141, 128, 6), (128, 48, 3, 3, 5, 203, 97, 128, 6), (64, 48, 4, 2, 3, 379, 135, 128, 7), (200, 32, 3, 1, 2, 701, 66, 64, 6),
])
@pytest.mark.parametrize("dtype", ["bf16", "f16"])
def test_walks(c_in, c_out, k, d, n, h, w, workgroups, ring, dtype):
    ho, wo = h - (k - 1) * d, w - (k - 1) * d
    assert -(-wo // 64) * ho * n >= 2 * ring * workgroups
    # (fp16: loss gradients of 1 / (4 * 4096) are still normal numbers)
    exact_wgrad.check(c_in, c_out, k, d, n, h, w, dtype, None if dtype == "bf16" else 4096)
