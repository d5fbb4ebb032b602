"""GPU check of the 16-bit 4x4 weight gradient, whose loads to LDS the compiler does not see and which waits for them by count: many steps and several
walks a workgroup, over ends of strips, residue classes and images, at one to six input octets and kernel strides to the widest.  Nothing
rounds, so the result must be exact."""
import pytest

import exact_wgrad

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("c_in,c_out,d,n,h,w", [
    (48, 48, 8, 3, 530, 150), (48, 48, 1, 4, 333, 140), (1, 48, 1, 5, 515, 131), (17, 33, 5, 3, 601, 90), (48, 16, 2, 4, 403, 70), (8, 48, 4, 3, 500, 205),
    (40, 9, 3, 2, 700, 100), (24, 24, 16, 3, 477, 180),
])
@pytest.mark.parametrize("dtype", ["bf16", "f16"])
def test_walks(c_in, c_out, d, n, h, w, dtype):
    # (fp16: loss gradients of 1 / (4 * 4096) are still normal numbers)
    exact_wgrad.check(c_in, c_out, 4, d, n, h, w, dtype, None if dtype == "bf16" else 4096)
