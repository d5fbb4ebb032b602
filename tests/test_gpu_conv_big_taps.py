"""Large kernels to many maps (5x5, 6x6, 10x10) whose last one or two columns share fragments of the matrix unit: every kernel row and column meets
the sample that it should and no other.  An infinity in the image turns exactly the outputs infinite (or NaN) whose windows hold it, also next to
taps that do not exist; elsewhere the fp64 sum, to the storage type's half unit and the fp32 sum (K <= 40*100 products: 2e-4)."""
import numpy as np
import pytest
import torch

import sk_synth as S
from oracle import layers as OL

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("k,d,c_in,c_out,n,h,w,path", [
    # 16 x 32 and 8 x 64 pixel tiles; rows at the pitch of the bank rule and, at small strides, as wide as whole column steps
    (5, 1, 40, 64, 9, 61, 45, (2, 2, 1, 2)), (5, 18, 40, 64, 5, 154, 112, (2, 4, 1, 6)), (6, 1, 33, 64, 9, 65, 76, (2, 2, 1, 2)),
    (6, 8, 40, 64, 9, 81, 106, (2, 2, 1, 4)), (6, 9, 40, 64, 16, 72, 90, (2, 4, 1, 4)), (10, 4, 40, 208, 5, 56, 109, (2, 2, 1, 4)),
    (10, 10, 40, 192, 5, 91, 92, (2, 4, 1, 6)),
    # layers that this kernel takes since its tiles are shorter
    (5, 2, 32, 512, 1, 270, 247, (2, 2, 1, 2)), (6, 1, 64, 512, 4, 73, 216, (2, 2, 1, 2)),
])
def test_taps(k, d, c_in, c_out, n, h, w, path):
    from paper_1509_03371_amd import binding as B
    ho, wo = h - (k - 1) * d, w - (k - 1) * d
    assert B.sk_probe_conv_path(k, d, c_in, c_out, n, ho, wo) == path
    rng = np.random.default_rng(k * h + w)
    rounded = lambda a: torch.from_numpy(a.astype(np.float32)).to(torch.bfloat16).float().numpy()
    img = rounded(rng.standard_normal((n, c_in, h, w)))
    w0 = rounded(rng.standard_normal((c_out, c_in, k, k)) / np.sqrt(c_in * k * k))
    b0 = rng.standard_normal(c_out).astype(np.float32)
    net = B.SKNet([S.conv(c_out, k, d, relu=False), S.conv(2, 1, 1, relu=False)], c_in, 2, dtype="bf16")
    net.set_weights(0, w0, b0)
    net.set_weights(1, np.ones((2, c_out, 1, 1), np.float32), np.zeros(2, np.float32))
    net.plan(n, h, w, pad=False, keep=True)
    bad = [(int(rng.integers(0, n)), int(rng.integers(0, c_in)), int(rng.integers(0, h)), int(rng.integers(0, w))) for _ in range(3)]
    holed = img.copy()
    for at in bad:
        holed[at] = np.inf
    net.forward(torch.from_numpy(holed).cuda())
    got = net.get_activation(0)
    meets = np.zeros((n, ho, wo), bool)
    for b, _, y, x in bad:
        for i in range(k):
            for j in range(k):
                if 0 <= y - i * d < ho and 0 <= x - j * d < wo:
                    meets[b, y - i * d, x - j * d] = True
    assert np.array_equal(~np.isfinite(got).all(1), meets) and not np.isfinite(got).all(1)[meets].any()
    rows = rng.choice(c_out, 24, replace=False)
    ref = OL.conv_sk(img, w0[rows], b0[rows], d, relu=False)
    keep = np.broadcast_to(~meets[:, None], ref.shape)
    assert np.all((np.abs(got[:, rows] - ref) <= 2.0 ** -8 * np.abs(ref) + 2e-4)[keep])
    net.close()
