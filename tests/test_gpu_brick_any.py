"""GPU parity of the brick convolutions at widths that are not a multiple of 8:
every remainder, rows shorter than a staging group, odd planes (rows change
parity), the narrowest rows, tiles that end inside the map, input gradients plain and
accumulating, sources split over workgroups and not, 1^3."""
import pytest

from tests.test_gpu_ops import _id, test_conv3d as check_conv3d

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("c", [32, 64])  # one chunk of channels (never split) and two
@pytest.mark.parametrize("w", [2, 3, 4, 5, 6, 7, 9, 10, 12, 13, 14, 15, 17, 18, 22, 31, 33, 46])
def test_brick_any_width(w, c):
    check_conv3d((2, c, c, 5, 9, w, 3, 1, 1, c == 32, "bf16"))


@pytest.mark.parametrize("case", [
    (1, 32, 32, 9, 17, 18, 3, 1, 1, True, "bf16"),
    (1, 32, 96, 4, 8, 23, 3, 1, 1, False, "bf16"),
    (2, 64, 32, 5, 9, 13, 1, 1, 0, True, "bf16"),
    (2, 64, 64, 5, 9, 14, 1, 1, 0, False, "bf16"),
    (1, 128, 128, 3, 7, 7, 3, 1, 1, True, "bf16"),
], ids=_id)
def test_brick_any_case(case):
    check_conv3d(case)


# Even widths with several tiles per workgroup (more than 256 tiles): results
# leave through LDS, in 16-byte units and 4-byte ones at a row's end; with 32
# source channels and rows whose last tile holds four columns (W = 4, 20), and
# with one tile per workgroup (above), straight from the lanes.
@pytest.mark.parametrize("w,c", [(4, 32), (6, 32), (10, 32), (12, 32), (14, 32), (18, 32), (20, 32),
                                 (22, 32), (6, 64), (14, 64), (20, 64)])
def test_brick_even_many_tiles(w, c):
    check_conv3d((140, c, c, 5, 3, w, 3, 1, 1, c == 32, "bf16"))
