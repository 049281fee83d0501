"""GPU parity of the float32 voxel-box convolutions: small layers (boxes that
divide the map or leave a remainder on each axis, several samples in one box, K
split over waves, K entries past the end, 7^3, residue classes with different
tap counts and with none; some passes of them take the gather kernels), and
layers that take every built shape of workgroup in the forward and input
gradient and the larger ones of the weight gradient (asserted on the host in
tests/test_box_plan.py, and again here)."""
import pytest

from tests.test_box_plan import COVER, box_plan
from tests.test_gpu_ops import _id, test_conv3d as check_conv3d

pytestmark = pytest.mark.gpu

CASES = [
    # N, Ci, Co, D, H, W, k, s, p, bias, dtype
    (1, 17, 33, 9, 11, 13, 3, 1, 1, True, "f32"),
    (2, 64, 65, 6, 7, 9, 3, 1, 1, False, "f32"),
    (1, 64, 64, 17, 16, 24, 3, 1, 1, False, "f32"),
    (1, 8, 16, 25, 23, 31, 3, 1, 1, True, "f32"),
    (9, 32, 48, 3, 4, 3, 3, 1, 1, False, "f32"),
    (5, 256, 256, 2, 2, 2, 3, 1, 1, False, "f32"),
    (1, 40, 1, 5, 6, 40, 3, 1, 1, False, "f32"),
    (2, 1, 32, 20, 22, 19, 7, 2, 3, False, "f32"),
    (1, 3, 16, 9, 10, 11, 7, 1, 3, False, "f32"),
    (1, 2, 32, 15, 12, 13, 7, 2, 3, True, "f32"),
    (1, 6, 20, 9, 8, 10, 5, 1, 2, True, "f32"),
    (2, 5, 7, 8, 9, 10, 2, 1, 0, False, "f32"),
    (2, 64, 128, 7, 8, 9, 1, 1, 0, True, "f32"),
    (2, 32, 64, 9, 10, 11, 3, 2, 1, False, "f32"),
    (2, 20, 24, 10, 11, 12, 3, 3, 1, False, "f32"),
    (2, 32, 64, 9, 8, 7, 1, 2, 0, False, "f32"),
    (1, 4, 4, 1, 1, 200, 3, 1, 1, False, "f32"),
    (1, 2, 2, 3, 4, 5, 3, 1, 2, False, "f32"),
]


@pytest.mark.parametrize("case", CASES, ids=_id)
def test_conv3d_box(case):
    check_conv3d(case)


@pytest.mark.parametrize("case,pass_,a,b,c", COVER, ids=str)
def test_conv3d_box_shapes(case, pass_, a, b, c):
    assert box_plan(case, pass_)[:3] == [a, b, c]
    check_conv3d(case + ("f32",))
