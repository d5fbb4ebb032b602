"""GPU check of the 16-bit 4x4 layers with pools inside them on tall images, whose table of row tiles grows with the height: tiles that overlap by a
row (few tiles a workgroup) need more entries than plain ones, and up to about 19000 rows (48 maps, d = 8) the table still fits the LDS beside the
weights, so the pools stay inside.  Copying convolutions on values that 16 bits hold: the maps must be exactly the image's pooled, shifted ones."""
import numpy as np
import pytest
import torch

import sk_synth as S
from test_gpu_fused_pool import exact_image, make_net, tap_weights

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,h,w", [(1, 700, 40), (2, 2500, 30), (4, 9000, 33), (8, 16100, 57), (8, 18900, 60), (1, 40000, 14)])
def test_pools_inside_their_neighbours(d, h, w):
    maps = 48
    layers = [S.conv(maps, 4, d), S.pool(2, d), S.conv(maps, 4, d), S.conv(24, 1, 1), S.conv(2, 1, 1, relu=False)]
    ws, bs = S.he_normal_weights(layers, maps, 41, bias_scale=0.1)
    ws[0], ws[1] = tap_weights(maps, (1, 2)), tap_weights(maps, (3, 1))
    bs[0][:], bs[1][:] = 0, 0
    img = exact_image(1, maps, h, w, d + h)
    net = make_net(layers, maps, ws, bs, "bf16")
    net.plan(1, h, w, pad=False)
    assert [net.step_name(i) for i in range(net.num_steps())][1:3] == ["conv0_k4_d%d_o%d_vpool" % (d, maps), "conv2_k4_d%d_o%d_hpool" % (d, maps)]
    net.forward(torch.from_numpy(img).cuda())
    got = net.get_activation(2)
    net.close()
    a = np.maximum(img[:, :, d:h - 2 * d, 2 * d:w - d], 0)
    a = np.maximum(a[:, :, :-d], a[:, :, d:])
    a = np.maximum(a[..., :-d], a[..., d:])
    assert np.array_equal(got, a[:, :, 3 * d:, d:a.shape[3] - 2 * d])
