"""Reading a U-Net's parameters back from a training plan: every tensor, from a bias to one of many pieces of the reader's
(2 MB each; 37.7 MB here, and 8.4 MB of an up-convolution, which the device keeps as four stacked 1x1 layers), must be the one that was set,
bit for bit; a net with maps off the 32 x 32 blocks that the stacked form is turned in, too."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("depth,base,size", [(4, 64, 188), (1, 40, 44)])
def test_weights_come_back(dtype, depth, base, size):
    from paper_1509_03371_amd import binding as B
    net = B.UNet(1, 2, depth=depth, base_ch=base, dtype=dtype)
    net.plan(1, size, size, training=True)
    rng = np.random.default_rng(base)
    kept = []
    for i in range(net.num_params()):
        s = net.param_shape(i)
        w = rng.standard_normal(s, dtype=np.float32)
        b = rng.standard_normal(net.get_weights(i)[1].shape, dtype=np.float32)
        net.set_weights(i, w, b)
        kept.append((w, b))
    for i, (w, b) in enumerate(kept):
        got = net.get_weights(i)
        assert np.array_equal(got[0], w) and np.array_equal(got[1], b), i
    net.close()
