"""16-bit 1x1 layers of at most sixteen maps to fp32 sums, against fp64 results of the very maps the GPU holds.  Planes below and off the sixteen pixels of
a run, sizes on both sides of the lines between one, two and four runs a wave, maps off the octets and the chunks of 32, one chunk to more than a batch
and more than 48 KB of weights, several images.  A sum of K products and a bias errs by at most (K + 2) * 2^-24 of the sum of magnitudes."""
import numpy as np
import pytest
import torch

import sk_synth as S

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("c_in,c_out,n,h,w", [
    (1, 1, 1, 3, 4), (8, 2, 1, 4, 4), (9, 16, 3, 5, 7), (31, 5, 1, 9, 31), (33, 2, 2, 33, 17), (64, 2, 1, 257, 256), (40, 3, 5, 111, 119), (64, 2, 1, 388, 389),
    (24, 13, 3, 211, 213), (257, 2, 1, 128, 127), (512, 2, 1, 40, 41), (1600, 2, 1, 19, 23), (1600, 2, 1, 263, 259),
])
@pytest.mark.parametrize("dtype", ["bf16", "f16"])
def test_sums(c_in, c_out, n, h, w, dtype):
    from paper_1509_03371_amd import binding as B
    rng = np.random.default_rng(c_in + h * w)
    net = B.SKNet([S.conv(c_in, 2, 1, relu=True), S.conv(c_out, 1, 1, relu=False)], 2, c_out, dtype=dtype)
    to = torch.bfloat16 if dtype == "bf16" else torch.float16
    w0 = (rng.standard_normal((c_in, 2, 2, 2)) / np.sqrt(8)).astype(np.float32)
    w1 = torch.from_numpy(rng.standard_normal((c_out, c_in, 1, 1)).astype(np.float32)).to(to)
    b1 = rng.standard_normal(c_out).astype(np.float32)
    net.set_weights(0, w0, np.zeros(c_in, np.float32))
    net.set_weights(1, w1.float().numpy(), b1)
    net.plan(n, h + 1, w + 1, pad=False, keep=True)
    net.forward(torch.from_numpy(rng.standard_normal((n, 2, h + 1, w + 1)).astype(np.float32)).cuda())
    x, got = torch.from_numpy(net.get_activation(0)).cuda().double(), torch.from_numpy(net.get_activation(1)).cuda().double()
    wm = w1.double().cuda()[:, :, 0, 0]
    x = x.permute(0, 2, 3, 1).reshape(-1, c_in)
    bias = torch.from_numpy(b1).double().cuda()
    ref, size = x @ wm.t() + bias, x.abs() @ wm.abs().t() + bias.abs()
    got = got.permute(0, 2, 3, 1).reshape(-1, c_out)
    assert bool(((got - ref).abs() <= (c_in + 2) * 2.0 ** -24 * size).all())
    net.close()
