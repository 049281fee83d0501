"""GPU parity of the row-band weight gradient at widths that start rows inside
a 16- or a 4-byte unit (W mod 8 = 1 .. 7), with rows of fewer voxels than a
unit, odd planes (rows and planes change parity), several bands and the ends
of the tensors."""
import pytest

from tests.test_gpu_ops import _id, test_conv3d as check_conv3d

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("case", [
    (2, 16, 64, 5, 9, 9, 3, 1, 1, False, "bf16"),
    (1, 32, 64, 4, 11, 10, 3, 1, 1, False, "bf16"),
    (3, 16, 64, 3, 7, 11, 3, 1, 1, False, "bf16"),
    (1, 16, 64, 5, 5, 13, 3, 1, 1, False, "bf16"),
    (1, 32, 128, 3, 13, 22, 3, 1, 1, False, "bf16"),
    (2, 16, 64, 3, 9, 31, 3, 1, 1, False, "bf16"),
    (1, 16, 64, 5, 31, 5, 3, 1, 1, False, "bf16"),
    (1, 16, 64, 6, 40, 3, 3, 1, 1, False, "bf16"),
    (1, 16, 64, 12, 16, 1, 3, 1, 1, False, "bf16"),
    (2, 64, 64, 7, 19, 46, 3, 1, 1, True, "bf16"),
    (1, 32, 64, 3, 8, 55, 3, 1, 1, False, "bf16"),
    (1, 16, 64, 3, 8, 54, 3, 1, 1, False, "bf16"),
], ids=_id)
def test_band_wgrad(case):
    check_conv3d(case)


# maps of 96 to 127 voxels and rows of 5 to 7: from 2^18 volumes times channel
# pairs on this kernel, below that the gather kernel
@pytest.mark.parametrize("case", [
    (16, 128, 128, 4, 4, 6, 3, 1, 1, False, "bf16"),
    (64, 64, 64, 4, 4, 7, 3, 1, 1, False, "bf16"),
    (16, 128, 128, 5, 4, 5, 3, 1, 1, True, "bf16"),
    (15, 128, 128, 5, 5, 5, 3, 1, 1, False, "bf16"),
    (2, 64, 64, 5, 5, 5, 3, 1, 1, False, "bf16"),
], ids=_id)
def test_band_small(case):
    check_conv3d(case)
