"""GPU parity of the pipelined gather convolutions: one, two, three and more K
steps in each direction, strides 2 and 3 with taps outside the volume on every
side, classes that no tap reaches, odd sizes, several samples in one tile, 7^3."""
import pytest

from tests.test_gpu_ops import _id, test_conv3d as check_conv3d

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("case", [
    (2, 32, 32, 5, 7, 9, 1, 2, 0, False, "bf16"),
    (2, 64, 64, 5, 7, 9, 1, 2, 0, True, "bf16"),
    (1, 96, 96, 4, 4, 4, 1, 3, 0, False, "bf16"),
    (1, 128, 96, 4, 5, 4, 1, 2, 0, False, "bf16"),
    (5, 32, 64, 3, 3, 3, 3, 2, 1, False, "bf16"),
    (2, 64, 96, 7, 5, 11, 3, 2, 1, True, "bf16"),
    (1, 32, 32, 8, 8, 8, 3, 3, 2, False, "bf16"),
    (1, 32, 33, 6, 7, 5, 3, 2, 1, False, "bf16"),
    (1, 33, 32, 6, 7, 5, 3, 2, 1, False, "bf16"),
    (2, 256, 256, 3, 4, 3, 3, 1, 1, False, "bf16"),
    (1, 5, 7, 6, 6, 6, 5, 1, 2, False, "bf16"),
    (1, 32, 32, 9, 8, 9, 7, 2, 3, False, "bf16"),
    (1, 2, 32, 9, 8, 9, 8, 2, 3, False, "bf16"),
], ids=_id)
def test_gather_pipe(case):
    check_conv3d(case)


# few live rows of a tile over 320000 voxels and more, where the weight gradient
# is the plain kernel's, and just below either line
@pytest.mark.parametrize("case", [
    (5, 3, 4, 40, 40, 41, 1, 1, 0, True, "bf16"),
    (6, 1, 2, 38, 38, 38, 3, 1, 1, False, "bf16"),
    (5, 3, 4, 39, 40, 41, 1, 1, 0, False, "bf16"),
    (6, 1, 24, 38, 38, 38, 3, 1, 1, False, "bf16"),
], ids=_id)
def test_gather_few_rows(case):
    check_conv3d(case)
