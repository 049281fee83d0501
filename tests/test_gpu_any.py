"""GPU parity of the passes for maps of any size at the places where their
blocks and vectors end: planes that start and end inside a 16-byte unit, one
or several chunks of a plane, volumes of several blocks with a short last
one, resampling by less than 1, to the same size and by almost 3, planes too
large for the staged kernels."""
import numpy as np
import pytest

from oracle import ops
from tests import gpu_util as U
from tests.test_gpu_ops import test_bn as check_bn
from tests.test_gpu_ops import test_maxpool as check_maxpool
from tests.test_gpu_ops import test_trilinear as check_trilinear

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("case", [
    (2, 3, 7, 9, 11, "bf16"), (3, 5, 1, 1, 1, "bf16"), (2, 3, 1, 1, 9, "bf16"),
    (2, 2, 13, 15, 23, "bf16"), (1, 3, 19, 21, 25, "bf16"), (2, 3, 7, 9, 11, "f32"),
    (2, 2, 13, 15, 23, "f32"), (3, 3, 1, 1, 5, "f32"), (5, 1, 1, 2, 1, "f32"),
    # in vectors: 400000 elements (bf16) and 200000 (float32) in planes of 1024 or more
    (7, 55, 5, 11, 19, "bf16"), (3, 31, 13, 15, 23, "bf16"), (1, 5, 43, 45, 47, "bf16"),
    (9, 22, 5, 11, 19, "f32"), (1, 3, 41, 43, 45, "f32"),
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
         ((2, 60, 50), (4, 120, 100))]
ANY = [((23, 28, 23), (46, 55, 46)), ((7, 5, 9), (13, 10, 17)), ((4, 6, 5), (2, 3, 4)),
       ((2, 3, 5), (6, 8, 14)), ((9, 4, 2), (10, 5, 2))]


@pytest.mark.parametrize("sizes,dt", [(s, d) for s in EXACT for d in ("f32", "bf16")] +
                         [(s, "bf16") for s in ANY],
                         ids=lambda v: v if isinstance(v, str) else "%s_to_%s" % v)
def test_trilinear_any(sizes, dt):
    check_trilinear(sizes, dt)


# The staged kernels need enough volumes to fill the chip: seven (an odd number,
# so that odd planes meet both alignments) against the oracle, repeated to c.
def _planes(t, c):
    return t.repeat(1, -(-c // t.shape[1]), 1, 1, 1)[:, :c].contiguous()


def _tags(run):
    """The measurement tags of what run launches."""
    from paper_2104_05035_amd import rat3d as R
    R.rat3d_profile_reset()
    R.rat3d_profile_filter(None)
    R.rat3d_profile_enable(1)
    try:
        run()
        U.sync()
    finally:
        R.rat3d_profile_enable(0)
    return [R.rat3d_profile_read(i)[0] for i in range(R.rat3d_profile_count())]


STAGED_UP = [
    # sizes, volumes, whether forward and transpose are staged
    ((23, 28, 23), (46, 56, 46), 70, 1, 1), ((5, 17, 17), (10, 17, 17), 700, 1, 0),
    ((9, 18, 15), (12, 24, 20), 700, 1, 0), ((3, 40, 40), (3, 40, 80), 700, 1, 1),
    ((12, 16, 20), (8, 16, 32), 700, 1, 0), ((2, 60, 50), (4, 120, 100), 700, 1, 0),
    # rows of one voxel, planes of an odd number of them, more than the 512
    # outputs that a block forms at a time
    ((1, 601, 1), (2, 601, 1), 2100, 1, 0), ((3, 2402, 1), (3, 1201, 1), 700, 1, 0),
    # columns beyond 15 and 16 bits
    ((1, 1, 40000), (1, 1, 256), 700, 1, 0), ((2, 3, 65536), (4, 4, 64), 70, 1, 0),
    ((1, 1, 80000), (1, 1, 256), 700, 0, 0),
]
STAGED_UP_BF16 = [
    ((23, 28, 23), (46, 55, 46), 70, 1, 1), ((9, 20, 13), (17, 41, 27), 700, 1, 1),
    ((7, 23, 31), (21, 40, 50), 70, 1, 1),
]


@pytest.mark.parametrize("case,dt", [(c, d) for c in STAGED_UP for d in ("f32", "bf16")] +
                         [(c, "bf16") for c in STAGED_UP_BF16],
                         ids=lambda v: v if isinstance(v, str) else "%s_to_%s_c%d" % v[:3])
def test_trilinear_staged(case, dt):
    from paper_2104_05035_amd import rat3d as R
    si, so, c, up, down = case
    rng = np.random.default_rng(si[1] * 7 + so[1])
    rnd = ops.round_bf16 if dt == "bf16" else ops.identity
    x, xr = U.dev_input(rng.standard_normal((1, 7, *si)), dt)
    dy, dyr = U.dev_input(rng.standard_normal((1, 7, *so)), dt)
    base0, baser = U.dev_input(rng.standard_normal((1, 7, *si)), dt)
    desc = R.UpDesc(1, c, *si, *so, U.code(dt))
    out = [U.guarded((1, c, *sz), dt) for sz in (so, si, si)]
    (y, dx, base) = (t for t, _ in out)
    base.copy_(_planes(base0, c))
    assert _tags(lambda: R.rat3d_softmask_up_fwd(desc, _planes(x, c), y)) == \
        ["up_fwd_any" if up else "up_fwd"]
    assert _tags(lambda: (R.rat3d_softmask_up_bwd(desc, _planes(dy, c), dx, 0),
                          R.rat3d_softmask_up_bwd(desc, _planes(dy, c), base, 1))) == \
        ["up_bwd_any" if down else "up_bwd"]
    for t, buf in out:
        U.guard_intact(buf)
        assert U.torch_mod().equal(t, _planes(t[:, :7], c))
    U.check(U.f64(y[:, :7]), rnd(ops.trilinear_fwd(xr, so)), dt, "y",
            terms=ops.trilinear_fwd(np.abs(xr), so))
    dxr, tdx = ops.trilinear_bwd(dyr, si), ops.trilinear_bwd(np.abs(dyr), si)
    U.check(U.f64(dx[:, :7]), rnd(dxr), dt, "dx", terms=tdx)
    U.check(U.f64(base[:, :7]), rnd(baser + dxr), dt, "dx accumulate", terms=tdx + np.abs(baser))


@pytest.mark.parametrize("case", [
    (46, 55, 46, 7, "bf16", 1), (46, 55, 46, 7, "f32", 1), (9, 11, 13, 700, "bf16", 1),
    (9, 11, 13, 700, "f32", 1), (5, 41, 39, 700, "bf16", 1), (12, 14, 12, 700, "f32", 1),
    (4, 16, 24, 700, "f32", 1), (9, 11, 13, 70, "f32", 0), (6, 7, 6, 2100, "bf16", 0),
], ids=lambda c: "%dx%dx%d_c%d_%s" % c[:5])
def test_maxpool_staged(case):
    from paper_2104_05035_amd import rat3d as R
    D, H, W, c, dt, staged = case
    rng = np.random.default_rng(D * H + W)
    rnd = ops.round_bf16 if dt == "bf16" else ops.identity
    x, xr = U.dev_input(rng.standard_normal((1, 7, D, H, W)), dt)
    yref, amref = ops.maxpool3d_fwd(xr)
    am = U.to_dev(U.torch_mod().from_numpy(amref.astype(np.uint8)))
    dy, dyr = U.dev_input(rng.standard_normal(yref.shape), dt)
    base0, baser = U.dev_input(rng.standard_normal((1, 7, D, H, W)), dt)
    desc = R.PoolDesc(1, c, D, H, W, 3, 2, 1, U.code(dt))
    out = [U.guarded((1, c, D, H, W), dt) for _ in range(2)]
    (dx, base) = (t for t, _ in out)
    base.copy_(_planes(base0, c))
    assert _tags(lambda: (R.rat3d_softmask_down_bwd(desc, _planes(dy, c), _planes(am, c), dx, 0),
                          R.rat3d_softmask_down_bwd(desc, _planes(dy, c), _planes(am, c), base, 1))) \
        == ["pool_bwd_any" if staged else "pool_bwd"]
    for t, buf in out:
        U.guard_intact(buf)
        assert U.torch_mod().equal(t, _planes(t[:, :7], c))
    dxr = ops.maxpool3d_bwd(dyr, amref, xr.shape)
    tdx = ops.maxpool3d_bwd(np.abs(dyr), amref, xr.shape)
    U.check(U.f64(dx[:, :7]), rnd(dxr), dt, "dx", terms=tdx)
    U.check(U.f64(base[:, :7]), rnd(baser + dxr), dt, "dx accumulate", terms=tdx + np.abs(baser))


# More blocks than one launch takes (2^24 of 256 threads): the general kernels.
# The planes are copies of a few, so the result is that of the few; dy holds small
# integers, whose pooled sums are exact in any order.
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
