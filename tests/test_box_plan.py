"""Plans of the float32 voxel-box convolutions (host side, no GPU needed): the
layout and the launches they ask for stay within what the kernels assume."""
import ctypes
import time

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


@pytest.mark.parametrize("case,pass_", [
    ((33372, 3, 16, 64, 25, 146, 2, 2, 1, False), 0),   # 19.5 M ragged boxes
    ((36, 4, 2, 1755, 14, 4979, 5, 1, 1, False), 1),    # 17.5 M
    ((3606, 8, 1, 123, 78, 116, 2, 1, 1, False), 2),    # few weights: 83436 splits
    ((93669, 1, 1, 41, 154, 41, 2, 1, 1, False), 2),    # 635321
    ((2, 4, 8, 9, 11, 10, 3, 1, 1, False), 0), ((2, 4, 8, 9, 11, 10, 3, 1, 1, False), 1),
    ((2, 4, 8, 9, 11, 10, 3, 1, 1, False), 2),
], ids=str)
def test_launches_within_limits(case, pass_):
    """Less than 2^32 work-items along x and 2^16 workgroups along y and z, or
    the general kernels."""
    plan = box_plan(case, pass_)
    assert plan is None or (plan[3] * 256 < 2 ** 32 and max(plan[4:6]) <= 65535), plan
    assert plan is not None or case[0] > 2


@pytest.mark.parametrize("c_in,k,taken", [
    (97720, 7, False), (36506, 7, True), (36507, 7, False), (600, 7, True), (60000, 3, True)])
def test_forward_division_range(c_in, k, taken):
    """A K entry's channel comes from i * ceil(2^32 / k^3) >> 32, exact while
    i k^3 < 2^32; entries up to 96 past the last are divided too."""
    nt = k ** 3
    plan = box_plan((1, c_in, 1, 7, 7, 7, k, 1, k // 2, False), 0)
    assert (plan is not None) == taken
    if taken:
        m = -(-2 ** 32 // nt)
        last = c_in * nt + 96
        for i in [*range(max(0, last - 2 * nt), last), *range(0, last, max(1, last // 4096))]:
            assert i * m >> 32 == i // nt, i


@pytest.mark.parametrize("case", [
    (33049, 96, 69, 5, 9, 9, 3, 1, 2, True),
    (28968, 48, 75, 4, 4, 7, 3, 1, 0, True)], ids=str)
def test_noalloc_keeps_what_it_took(case):
    """Batches whose bias-gradient sums leave less than 24 MiB for the partial
    sums: the weight gradient without a workspace argument still takes them."""
    desc = R.conv_desc(*case[:9], case[9], R.F32)
    assert box_plan(case, 2) is not None
    need = R.rat3d_conv3d_workspace_size(desc, 2)
    assert need <= R.lib().rat3d_conv3d_wgrad_noalloc_max_bytes(), need


def test_plans_of_long_axes_take_little_time():
    """A plan looks at no more boxes than one has voxels, so an axis of a
    million voxels costs a first call (three plans) well under the 0.2 to 0.8 s of
    a search over every number of cuts."""
    t0 = time.perf_counter()
    for i, size in enumerate([(1, 2000000, 14), (4, 700001, 10), (3, 1000003, 9)]):
        for pass_ in range(3):
            assert box_plan((1, 2, 3, *size, 3, 1, 1, False), pass_) is not None, (i, pass_)
    assert time.perf_counter() - t0 < 0.1


# us measured on one box: gather kernel, box kernel
@pytest.mark.parametrize("case,pass_,gather,box", [
    ((8, 32, 32, 60, 50, 77, 1, 1, 0, False), 0, 271.1, 1100.3),
    ((1, 192, 192, 67, 72, 52, 1, 1, 0, False), 0, 405.1, 708.4),
    ((2, 48, 128, 53, 73, 64, 3, 3, 2, False), 1, 276.5, 489.8),
    ((8, 32, 32, 60, 50, 77, 1, 1, 0, False), 1, 300.6, 866.5),
    ((4, 96, 128, 27, 21, 35, 7, 3, 3, False), 2, 622.6, 1068.8),
    ((16, 8, 96, 48, 55, 64, 3, 3, 1, False), 2, 200.1, 445.4),
    ((1, 64, 96, 74, 56, 93, 1, 2, 0, False), 2, 50.7, 179.5),
    ((16, 4, 64, 3, 3, 2, 7, 2, 3, False), 2, 12.0, 33.8),
    ((2, 64, 64, 24, 28, 24, 3, 1, 1, False), 0, 232.0, 78.0),
    ((2, 64, 64, 24, 28, 24, 3, 1, 1, False), 1, 310.0, 83.0),
    ((2, 64, 64, 24, 28, 24, 3, 1, 1, False), 2, 168.0, 107.0),
    ((8, 64, 64, 46, 55, 46, 3, 1, 1, False), 2, 5009.0, 2504.0),
    ((2, 256, 256, 6, 7, 6, 3, 1, 1, False), 0, 770.0, 105.0),
], ids=str)
def test_the_faster_kernel_is_taken(case, pass_, gather, box):
    assert (box_plan(case, pass_) is not None) == (box < gather)


# Layers whose plans take every built shape of workgroup: (case, pass, CT, VT, WK)
# or, weight gradients, (case, 2, CT, JT, PR).  Channel counts that leave a
# remainder of the tiles; run against the oracle in tests/test_gpu_box.py.
COVER = [
    ((3, 16, 48, 25, 27, 29, 3, 1, 1, False), 0, 4, 2, 1),
    ((1, 4, 33, 31, 33, 30, 3, 1, 1, True), 0, 4, 2, 1),
    ((2, 16, 48, 20, 21, 23, 3, 1, 1, False), 0, 2, 2, 1),
    ((1, 4, 17, 31, 33, 30, 3, 1, 1, True), 0, 2, 2, 1),
    ((3, 16, 64, 25, 27, 29, 3, 2, 1, False), 0, 2, 1, 1),
    ((3, 4, 33, 13, 15, 17, 3, 1, 1, True), 0, 2, 1, 1),
    ((1, 4, 8, 31, 33, 30, 3, 1, 1, False), 0, 1, 4, 1),
    ((1, 17, 33, 9, 11, 13, 3, 1, 1, True), 0, 1, 1, 1),
    ((3, 48, 16, 25, 27, 29, 3, 2, 1, False), 1, 4, 4, 1),
    ((3, 33, 8, 25, 27, 29, 3, 2, 1, False), 1, 4, 4, 1),
    ((3, 33, 33, 20, 21, 23, 3, 2, 1, False), 1, 4, 2, 1),
    ((3, 33, 8, 20, 21, 23, 3, 2, 1, False), 1, 2, 4, 1),
    ((2, 33, 8, 13, 15, 17, 3, 2, 1, False), 1, 2, 2, 1),
    ((2, 4, 8, 20, 21, 23, 3, 2, 1, False), 1, 1, 4, 1),
    ((2, 17, 8, 13, 15, 17, 3, 2, 1, False), 1, 2, 2, 4),
    ((2, 4, 8, 13, 15, 17, 3, 2, 1, False), 1, 1, 2, 4),
    ((1, 17, 33, 9, 11, 13, 3, 1, 1, True), 1, 1, 1, 4),
    ((2, 33, 8, 13, 15, 17, 3, 1, 1, True), 2, 1, 4, 2),
    ((1, 24, 8, 25, 27, 29, 3, 1, 1, False), 2, 1, 7, 2),
    ((1, 12, 17, 25, 27, 29, 3, 1, 1, False), 2, 2, 4, 2),
    ((1, 48, 17, 31, 33, 30, 3, 1, 1, False), 2, 2, 7, 2),
    ((1, 17, 65, 13, 15, 17, 3, 1, 1, True), 2, 4, 2, 2),
    ((2, 33, 65, 13, 15, 17, 3, 1, 1, False), 2, 4, 4, 2),
    ((1, 48, 33, 31, 33, 30, 3, 1, 1, False), 2, 4, 7, 2),
    ((1, 1, 70, 3, 14, 4, 5, 1, 2, False), 2, 4, 2, 4),
    ((3, 1, 101, 1, 4, 6, 6, 1, 3, False), 2, 4, 4, 4),
    ((3, 1, 40, 3, 5, 5, 7, 1, 3, False), 2, 4, 7, 16),
    ((2, 1, 17, 15, 25, 1, 7, 2, 3, False), 2, 2, 7, 16),
]


@pytest.mark.parametrize("case,pass_,a,b,c", COVER, ids=str)
def test_cover_takes_its_shape(case, pass_, a, b, c):
    plan = box_plan(case, pass_)
    assert plan is not None and plan[:3] == [a, b, c], plan


def test_cover_has_every_forward_and_input_gradient_shape():
    assert {c[2:] for c in COVER if c[1] == 0} == {(4, 2, 1), (2, 2, 1), (2, 1, 1), (1, 4, 1),
                                                   (1, 1, 1)}
    assert {c[2:] for c in COVER if c[1] == 1} == {(4, 4, 1), (4, 2, 1), (2, 4, 1), (2, 2, 1),
                                                   (1, 4, 1), (2, 2, 4), (1, 2, 4), (1, 1, 4)}
