"""GPU check of the k = 2, s = 1 pool gradient: the gradient at the pool's input must be the gradient at its output routed to
the recorded winners, summed in fp32 in the order of the winner codes, rounded once to the storage type, and zero where the
layer below gave nothing positive -- bit for bit, from the tensors the GPU itself holds.  Sizes around the kernels' edges:
maps narrower than the four columns of the fp32 kernel, row ends at every remainder of four, kernel strides wider than the
output, chains and segments that end early, ties and a layer below without ReLU."""
import numpy as np
import pytest
import torch

import sk_synth as S

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["f32", "bf16", "f16"])
@pytest.mark.parametrize("relu", [True, False])
@pytest.mark.parametrize("maps,d,n,h,w", [
    (8, 1, 1, 2, 2), (8, 1, 2, 9, 4), (16, 3, 1, 5, 6), (8, 1, 1, 6, 5), (8, 2, 1, 11, 8), (12, 5, 2, 7, 12), (16, 9, 1, 12, 13),
    (8, 4, 1, 75, 67), (24, 1, 1, 38, 261), (48, 8, 1, 140, 130), (48, 2, 2, 300, 301),
    (64, 5, 4, 97, 33), (48, 1, 4, 300, 47), (16, 7, 1, 20, 300), (128, 1, 1, 12, 90),
])
def test_pool_gradient(dtype, relu, maps, d, n, h, w):
    from paper_1509_03371_amd import binding as B
    layers = [S.conv(maps, 1, 1, relu=relu), S.pool(2, d), S.conv(2, 1, 1, relu=False)]
    ws, bs = S.he_normal_weights(layers, 1, 7, bias_scale=0.1)
    net = B.SKNet(layers, 1, 2, dtype=dtype)
    for i, (wt, b) in enumerate(zip(ws, bs)):
        net.set_weights(i, wt, b)
    net.plan(n, h, w, pad=False, training=True)
    rng = np.random.default_rng(h * w)
    img = (rng.integers(-8, 8, (n, 1, h, w)) / 8.0).astype(np.float32)                                # ties included
    labels = torch.from_numpy(rng.integers(-1, 2, (n, h - d, w - d)).astype(np.int32)).cuda()
    net.forward(torch.from_numpy(img).cuda())
    below, idx = net.get_activation(0), net.get_pool_argmax(0).reshape(n, maps, h - d, w - d)
    above = net.get_activation_grad(1, labels).astype(np.float32)
    got = net.get_activation_grad(0, labels).astype(np.float32)
    net.close()
    ho, wo = h - d, w - d
    corner = np.arange(ho)[:, None] * w + np.arange(wo)[None, :]
    ref = np.zeros((n, maps, h, w), np.float32)
    for i in range(2):
        for j in range(2):
            won = idx == corner + i * d * w + j * d
            ref[:, :, i * d:i * d + ho, j * d:j * d + wo] += np.where(won, above, np.float32(0))
    if relu:
        ref = np.where(below > 0, ref, np.float32(0))
    if dtype != "f32":
        ref = torch.from_numpy(ref).to(torch.bfloat16 if dtype == "bf16" else torch.float16).float().numpy()
    assert np.abs(ref).max() > 0
    assert np.array_equal(got, ref)
