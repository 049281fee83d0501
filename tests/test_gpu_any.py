"""GPU parity of the passes for maps of any size at the places where their
blocks and vectors end: planes that start and end inside a 16-byte unit, one
or several chunks of a plane, volumes of several blocks with a short last
one, resampling by less than 1, to the same size and by almost 3, planes too
large for the staged kernels."""
import pytest

from tests import gpu_util as U
from tests.test_gpu_ops import test_bn as check_bn
from tests.test_gpu_ops import test_maxpool as check_maxpool
from tests.test_gpu_ops import test_trilinear as check_trilinear

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("case", [
    (2, 3, 7, 9, 11, "bf16"), (3, 5, 1, 1, 1, "bf16"), (2, 3, 1, 1, 9, "bf16"),
    (2, 2, 13, 15, 23, "bf16"), (1, 3, 19, 21, 25, "bf16"), (2, 3, 7, 9, 11, "f32"),
    (2, 2, 13, 15, 23, "f32"), (3, 3, 1, 1, 5, "f32"), (5, 1, 1, 2, 1, "f32"),
], ids=lambda c: "%dx%dx%dx%dx%d_%s" % c)
@pytest.mark.parametrize("relu,resid", [(1, False), (0, False), (1, True), (0, True)])
def test_bn_odd(case, relu, resid):
    check_bn(case, relu, resid)


@pytest.mark.parametrize("case", [
    (1, 3, 9, 11, 13, "bf16"), (2, 2, 46, 55, 46, "bf16"), (1, 1, 7, 70, 70, "bf16"),
    (2, 3, 12, 14, 12, "f32"), (1, 2, 5, 41, 39, "f32"), (1, 1, 3, 80, 90, "f32"),
    (3, 1, 1, 1, 2, "f32"), (1, 1, 4, 16, 24, "f32"),
], ids=lambda c: "%dx%dx%dx%dx%d_%s" % c)
def test_maxpool_any(case):
    check_maxpool(case)


# The kernels form an axis position as (o + 1/2) * (in / out) - 1/2 in float32:
# with an inexact ratio its error is up to |position| 2^-23, which moves the
# weights by as much and an output by that times the difference of neighbouring
# inputs -- more than 2^-16 of the sum of |terms| where the heavier terms happen
# to be small.  The float32 cases therefore have ratios that float32 holds
# exactly; the others are small maps in bf16, whose outputs are coarser than
# this error except next to zero.
EXACT = [((23, 28, 23), (46, 56, 46)), ((6, 5, 9), (8, 8, 12)), ((4, 6, 10), (2, 3, 5)),
         ((3, 3, 3), (3, 3, 3)), ((5, 5, 15), (8, 8, 16)), ((1, 1, 1), (3, 2, 3)),
         ((2, 60, 50), (4, 120, 100)),
         # rows of one voxel, planes of an odd number of them, more than the 512
         # outputs that a block forms at a time
         ((1, 601, 1), (2, 601, 1)), ((3, 2402, 1), (3, 1201, 1)),
         # columns beyond 15 and 16 bits
         ((1, 1, 40000), (1, 1, 256)), ((2, 3, 65536), (4, 4, 64)), ((1, 1, 80000), (1, 1, 256))]
ANY = [((23, 28, 23), (46, 55, 46)), ((7, 5, 9), (13, 10, 17)), ((4, 6, 5), (2, 3, 4)),
       ((2, 3, 5), (6, 8, 14)), ((9, 4, 2), (10, 5, 2))]


@pytest.mark.parametrize("sizes,dt", [(s, d) for s in EXACT for d in ("f32", "bf16")] +
                         [(s, "bf16") for s in ANY],
                         ids=lambda v: v if isinstance(v, str) else "%s_to_%s" % v)
def test_trilinear_any(sizes, dt):
    check_trilinear(sizes, dt)


# More blocks than one launch takes (2^24 of 256 threads): the general kernels.
# The planes are copies of a few, so the result is that of the few; dy holds small
# integers, whose pooled sums are exact in any order.
def _planes(t, c):
    return t.repeat(1, -(-c // t.shape[1]), 1, 1, 1)[:, :c].contiguous()


def test_maxpool_many_planes():
    from paper_2104_05035_amd import rat3d as R
    torch = U.torch_mod()
    few, many = 4096, 2 ** 24 + 8
    torch.manual_seed(1)
    x = torch.randn(1, few, 1, 4, 8, device="cuda")
    y, am = torch.empty(1, few, 1, 2, 4, device="cuda"), \
        torch.empty(1, few, 1, 2, 4, dtype=torch.uint8, device="cuda")
    R.rat3d_softmask_down_fwd(R.PoolDesc(1, few, 1, 4, 8, 3, 2, 1, R.F32), x, y, am)
    dy = torch.randint(-8, 9, y.shape, device="cuda").float()
    dx = {}
    for c in (few, many):
        dx[c] = torch.full((1, c, 1, 4, 8), 7.0, device="cuda")
        R.rat3d_softmask_down_bwd(R.PoolDesc(1, c, 1, 4, 8, 3, 2, 1, R.F32), _planes(dy, c),
                                  _planes(am, c), dx[c], 0)
    U.sync()
    assert torch.equal(dx[many], _planes(dx[few], many))


def test_trilinear_many_planes():
    """8193 fine planes of one voxel from 2731: sums of up to three products,
    to within their roundings."""
    from paper_2104_05035_amd import rat3d as R
    torch = U.torch_mod()
    few, many = 64, 12288
    torch.manual_seed(2)
    dy = torch.randn(1, few, 8193, 1, 1, device="cuda")
    dx = {}
    for c in (few, many):
        dx[c] = torch.full((1, c, 2731, 1, 1), 7.0, device="cuda")
        R.rat3d_softmask_up_bwd(R.UpDesc(1, c, 2731, 1, 1, 8193, 1, 1, R.F32), _planes(dy, c), dx[c], 0)
    U.sync()
    ref = _planes(dx[few], many)
    assert float((dx[many] - ref).abs().max()) <= 8 * 2.0 ** -24 * 6 * float(dy.abs().max())
