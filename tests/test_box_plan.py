"""Plans of the float32 voxel-box convolutions (host side, no GPU needed): the
layout and the launches they ask for stay within what the kernels assume."""
import ctypes

import pytest

from paper_2104_05035_amd import rat3d as R


def box_plan(case, pass_):
    """None, or {CT, VT, WK (weight gradient: CT, JT, PR), grid x, y, z, LDS
    bytes, LDS offset of the rows read 16 bytes at a time} of a float32 pass;
    case as in tests/test_gpu_ops.py."""
    out = (ctypes.c_int64 * 8)()
    fn = R.lib().rat3d_box_plan
    fn.restype, fn.argtypes = ctypes.c_int, [ctypes.POINTER(R.ConvDesc), ctypes.c_int,
                                             ctypes.POINTER(ctypes.c_int64)]
    desc = R.conv_desc(*case[:9], case[9], R.F32)
    return list(out) if fn(ctypes.byref(desc), pass_, out) else None


@pytest.mark.parametrize("case", [
    # C_in k^3 no multiple of 16 (a channel of zeros in front of the weights) and
    # regions of 350, 243, 210 positions; the last has no such channel
    (1, 24, 48, 30, 33, 31, 3, 1, 1, False), (1, 4, 8, 7, 7, 7, 3, 1, 1, False),
    (1, 4, 8, 9, 11, 10, 3, 1, 1, False), (1, 8, 16, 25, 23, 31, 3, 1, 1, True),
    (2, 3, 5, 7, 9, 11, 3, 1, 1, False), (1, 1, 1, 5, 5, 5, 3, 1, 1, False),
    (1, 6, 20, 9, 8, 10, 5, 1, 2, True), (2, 16, 16, 7, 7, 7, 3, 1, 1, False),
], ids=str)
def test_forward_rows_are_16_byte_aligned(case):
    plan = box_plan(case, 0)
    assert plan is not None and plan[7] > 0 and plan[7] % 16 == 0, plan
