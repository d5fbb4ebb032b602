"""GPU check of the 16-bit 3-D pools (k = 2, s = 1): values and winners against the oracle on the activation the GPU holds, bit for bit, and the
gradient through them.  Volumes around the kernels' edges: planes off the blocks of 256 positions, chains and segments of slices that end
early, kernel strides wider than the output, ties.

Error maps of the layer below are read through a 1x1x1 layer whose input maps are each one sample of 1: its weight gradient [map][input
map] is the stored error map of `map` at that sample, ReLU mask included."""
import numpy as np
import pytest
import torch

import sk_synth as S
import test_gpu_conv_wide as wide

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("relu", [True, False])
@pytest.mark.parametrize("maps,d,size", [(8, 1, (2, 3, 4)), (16, 1, (34, 17, 16)), (8, 3, (5, 9, 20)), (24, 2, (41, 18, 30)), (8, 5, (12, 7, 21)), (16, 1, (9, 40, 70))])
def test_pool(dtype, relu, maps, d, size):
    from paper_1509_03371_amd import binding as B
    rng = np.random.default_rng(size[0] * size[2])
    out = tuple(s - d for s in size)
    spots = [tuple(int(rng.choice([0, min(d, s - 1), s // 2, max(0, s - 1 - d), s - 1])) for s in size) for _ in range(32)]
    img = np.zeros((size[0], 33) + size[1:], np.float32)
    for j, at in enumerate(spots):
        img[at[0], j, at[1], at[2]] = 1.0
    img[:, 32] = rng.integers(-8, 8, size) / 8.0                                            # (ties included)
    net = B.SKNet3D([S.conv(maps, 1, 1, relu=relu), S.pool(2, d), S.conv(3, 1, 1, relu=False)], 33, 3, dtype=dtype)
    w0 = np.zeros((maps, 33, 1, 1, 1), np.float32)
    w0[:, 32, 0, 0, 0] = rng.choice([-2.0, -1.0, 0.5, 1.0], maps)
    w1 = wide.rounded(rng.standard_normal((3, maps, 1, 1, 1)).astype(np.float32), dtype)
    net.set_weights(0, w0, (rng.integers(-4, 5, maps) / 8.0).astype(np.float32))
    net.set_weights(1, w1, np.zeros(3, np.float32))
    net.plan(*size, training=True)
    prob = net.forward(torch.from_numpy(img).cuda()).cpu().double()
    labels = rng.integers(-1, 3, out).astype(np.int32)
    labels[0, 0, 0] = 0
    net.backward(torch.from_numpy(labels).cuda())
    below, got = net.get_activation(0), torch.from_numpy(net.get_grad(0)[0].reshape(maps, 33)[:, :32]).double()
    pooled, idx = net.get_activation(1), torch.from_numpy(net.get_pool_argmax(0).astype(np.int64))
    net.close()
    # the windows in scan order: the first maximum wins
    taps = [(a, i, j) for a in range(2) for i in range(2) for j in range(2)]
    shifted = np.stack([below[a * d:a * d + out[0], :, i * d:i * d + out[1], j * d:j * d + out[2]] for a, i, j in taps])
    assert np.array_equal(pooled, shifted.max(0))
    first = torch.from_numpy(shifted.argmax(0))
    corner = (torch.arange(out[0])[:, None, None, None] * size[1] + torch.arange(out[1])[None, None, :, None]) * size[2] + torch.arange(out[2])[None, None, None, :]
    offset = torch.tensor([(a * d * size[1] + i * d) * size[2] + j * d for a, i, j in taps])
    assert torch.equal(idx.reshape(out[0], maps, out[1], out[2]), corner + offset[first])
    prob = prob.reshape((out[0], 3) + out[1:]).transpose(0, 1).unsqueeze(0)
    dz = wide.error_map(prob, torch.from_numpy(labels).unsqueeze(0), dtype)[0]                # [3, z, y, x]
    above = wide.store(torch.einsum("cm,czyx->zmyx", torch.from_numpy(w1.reshape(3, maps)).double(), dz).float(), dtype)
    ref = torch.zeros((size[0], maps) + size[1:], dtype=torch.float64)
    for t, (a, i, j) in enumerate(taps):
        ref[a * d:a * d + out[0], :, i * d:i * d + out[1], j * d:j * d + out[2]] += torch.where(first == t, above, torch.zeros_like(above))
    if relu:
        ref = ref * (torch.from_numpy(below) > 0)
    at = tuple(torch.tensor([s[i] for s in spots]) for i in range(3))
    ref = ref[at[0], :, at[1], at[2]].T
    # up to eight stored gradients meet in a sample; each may have been rounded to the other side, as may the sum
    assert float(ref.abs().max()) > 1e-5
    assert bool(((got - ref).abs() <= 8 * wide.gradient_bound(ref, dz, torch.from_numpy(w1), dtype)).all())
