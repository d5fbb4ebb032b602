"""GPU parity of the k = 2, s = 1 pool kernels where their cut into chains and row blocks changes: widths around one row
block (64, 128, 256 threads), row counts around one chain (4, 8, 16, 32 windows), few and many maps.  Values and winner
codes must equal the oracle's pool of the activation the GPU itself holds, bit for bit (pooling is exact)."""
import numpy as np
import pytest
import torch

import sk_synth as S
from oracle import layers as OL

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("training", [False, True])
@pytest.mark.parametrize("maps,d,n,h,w", [
    (8, 1, 1, 6, 64), (8, 1, 1, 10, 66), (16, 1, 2, 18, 130), (8, 2, 1, 36, 259), (24, 4, 1, 133, 131), (48, 2, 1, 67, 258),
    (48, 4, 2, 140, 300), (8, 1, 1, 7, 7),
    # narrow rows: several residue classes and segments a workgroup, some of them empty; chains of one, two and more windows
    (8, 1, 1, 40, 21), (16, 3, 2, 61, 36), (64, 5, 4, 97, 33), (48, 1, 4, 300, 47), (128, 2, 8, 180, 66), (16, 7, 1, 20, 300), (48, 8, 1, 45, 1030),
])
def test_pool_chains(dtype, training, maps, d, n, h, w):
    from paper_1509_03371_amd import binding as B
    layers = [S.conv(maps, 1, 1, relu=True), S.pool(2, d), S.conv(2, 1, 1, relu=False)]
    ws, bs = S.he_normal_weights(layers, 1, 7, bias_scale=0.1)
    net = B.SKNet(layers, 1, 2, dtype=dtype)
    for i, (wt, b) in enumerate(zip(ws, bs)):
        net.set_weights(i, wt, b)
    net.plan(n, h, w, pad=False, training=training, keep=not training)
    img = (np.random.default_rng(h * w).integers(-8, 8, (n, 1, h, w)) / 8.0).astype(np.float32)     # ties included
    net.forward(torch.from_numpy(img).cuda())
    ref, arg = OL.maxpool_sk(net.get_activation(0).astype(np.float64), 2, d, 1)
    assert np.array_equal(net.get_activation(1).astype(np.float64), ref)
    if training:
        assert np.array_equal(net.get_pool_argmax(0).reshape(-1), arg.reshape(-1))
    net.close()
