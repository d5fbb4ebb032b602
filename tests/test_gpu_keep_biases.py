"""set_weights without biases keeps the current ones (b = NULL in the C ABI): after SGD steps those are the trained ones,
whether or not the weights have been read back since."""
import numpy as np
import pytest
import torch

import sk_synth as S

pytestmark = pytest.mark.gpu


def trained_net(family, dtype):
    from paper_1509_03371_amd import binding as B
    if family in ("unet", "usknet"):
        if family == "unet":
            net, names, params, (c, h, w) = B.UNet(1, 2, depth=1, base_ch=8, dtype=dtype), S.unet_param_names(1), S.unet_params(1, 2, 3, depth=1, base=8), (1, 28, 36)
        else:
            net, names, params, (c, h, w) = B.USKNet(2, 2, base_ch=8, dtype=dtype), S.USKNET_PARAM_NAMES, S.usknet_params(2, 2, 4, base=8), (2, 184, 186)
        values = [params[name] for name in names]
        net_plan = lambda: net.plan(1, h, w, training=True)
        shape, label_shape = (1, c, h, w), lambda: (1,) + tuple(net.output_size(h, w))
    else:
        layers = [S.conv(8, 3, 1), S.conv(2, 1, 1, relu=False)]
        net = B.SKNet(layers, 1, 2, dtype=dtype) if family == "sknet" else B.SKNet3D(layers, 1, 2, dtype=dtype)
        rng = np.random.default_rng(5)
        values = [(rng.standard_normal(net.conv_shape(i)).astype(np.float32) * 0.3, np.full(net.conv_shape(i)[0], 0.25, np.float32)) for i in range(2)]
        if family == "sknet":
            net_plan, shape, label_shape = lambda: net.plan(1, 12, 14, pad=False, training=True), (1, 1, 12, 14), lambda: (1, 10, 12)
        else:
            net_plan, shape, label_shape = lambda: net.plan(6, 12, 14, training=True), (6, 1, 12, 14), lambda: (4, 10, 12)
    for i, (w0, b0) in enumerate(values):
        net.set_weights(i, w0, b0)
    net_plan()
    gen = torch.Generator().manual_seed(6)
    net.forward(torch.rand(shape, generator=gen).cuda())
    net.backward(torch.randint(0, 2, label_shape(), generator=gen, dtype=torch.int32).cuda())
    net.sgd_step(lr=0.5)
    return net, values


@pytest.mark.parametrize("read_first", [False, True])
@pytest.mark.parametrize("family,dtype", [("unet", "f32"), ("unet", "bf16"), ("usknet", "f32"), ("sknet", "f32"), ("sknet", "bf16"), ("sknet3d", "f32")])
def test_set_weights_keeps_trained_biases(family, dtype, read_first):
    kept, values = trained_net(family, dtype)
    ref, _ = trained_net(family, dtype)                  # the same step, its biases read and never written
    if read_first:
        for i in range(len(values)):
            kept.get_weights(i)
    moved = 0
    for i, (w0, b0) in enumerate(values):
        kept.set_weights(i, w0)
        w1, b1 = kept.get_weights(i)
        trained = ref.get_weights(i)[1]
        moved += not np.array_equal(trained, b0)
        assert np.array_equal(w1, w0) and np.array_equal(b1, trained), i
    assert moved > len(values) // 2                      # the step changed what a stale copy would bring back
    kept.close()
    ref.close()
