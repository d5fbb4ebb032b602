"""GPU parity of the 16-bit 3x3 kernel for 17 to 32 maps (32 maps x 64 x 12 pixels a tile), at sizes that its dispatch rule gives it: ragged
maps, rows, columns and chunks of input maps, kernel strides 1 to 4, one tile and several a CU, slices of a volume; and next to
them sizes that the rule keeps on the kernel of smaller tiles.  Tolerances as derived for the layers of more maps."""
import pytest

import test_gpu_conv_wide as wide

pytestmark = pytest.mark.gpu

HERE, KEPT = (1, 3, 1, 8), (0, 0, 1, 0)


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("d,c_in,c_out,n,h,w,path", [
    (1, 40, 32, 2, 262, 264, HERE), (4, 72, 24, 2, 270, 270, HERE), (3, 33, 17, 2, 267, 263, HERE), (2, 64, 32, 8, 215, 197, HERE),
    (1, 64, 32, 1, 100, 90, KEPT), (1, 24, 32, 2, 262, 264, KEPT), (5, 40, 32, 2, 270, 270, KEPT), (1, 64, 16, 8, 215, 197, KEPT),
])
def test_layer(dtype, d, c_in, c_out, n, h, w, path):
    wide.test_layer(dtype, 3, d, c_in, c_out, n, h, w, path)


@pytest.mark.parametrize("relu", [False, True])
@pytest.mark.parametrize("d,maps,classes,n,h,w,path", [
    (1, 32, 40, 2, 262, 263, HERE), (4, 24, 72, 2, 265, 263, HERE), (3, 17, 100, 3, 250, 211, HERE), (1, 32, 64, 1, 70, 65, KEPT),
])
def test_data_gradient(relu, d, maps, classes, n, h, w, path):
    wide.test_data_gradient("bf16", relu, 3, d, maps, classes, n, h, w, path)


@pytest.mark.parametrize("d,c_in,h", [(1, 16, 100), (2, 16, 100), (4, 24, 96), (3, 40, 100)])
def test_volume(d, c_in, h):
    wide.test_volume_layer("bf16", 3, d, c_in, 32, (16, h, 130), HERE)
    wide.test_volume_data_gradient("bf16", 3, d, 32, c_in, (16, h, 130), c_in == 16, HERE)
