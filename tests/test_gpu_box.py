"""GPU parity of the float32 voxel-box convolutions: small layers (boxes that
divide the map or leave a remainder on each axis, several samples in one box, K
split over waves, K entries past the end, 7^3, residue classes with different
tap counts and with none; some passes of them take the gather kernels), and
layers that take every built shape of workgroup in the forward and input
gradient and the larger ones of the weight gradient (asserted on the host in
tests/test_box_plan.py, and again here); and the rounding of the weight gradient's
sums over many voxels."""
import pytest
import torch

from paper_2104_05035_amd import rat3d as R
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


@pytest.mark.parametrize("case", [
    # a box's sum apart from the range's, of 7 to 40 boxes of up to 128 voxels
    (4, 128, 32, 38, 52, 40, 3, 2, 1, False), (2, 64, 64, 31, 26, 32, 3, 1, 1, False),
    (2, 128, 128, 20, 17, 20, 3, 1, 1, False), (8, 32, 8, 35, 30, 28, 3, 2, 1, False),
    (8, 32, 64, 14, 15, 14, 3, 1, 1, False),
    # one running sum over a short range
    (2, 4, 32, 34, 12, 20, 7, 1, 3, False), (4, 8, 64, 20, 12, 8, 7, 1, 3, False),
], ids=str)
def test_wgrad_box_rounding(case):
    """No more rounding than the general kernel's ranges of R voxels, S of them:
    rounding a running sum of n independent terms n times leaves a relative error
    of about c sqrt(n / 2), with c = 2^-23 / sqrt(12) * sqrt(3 / (8 ln 2)) for
    mantissas spread evenly over their logarithm; the ranges' sums add S more."""
    N, Ci, Co, D, H, W, k, s, p, _ = case
    assert box_plan(case, 2) is not None
    gen = torch.Generator().manual_seed(11)
    x = torch.randn(N, Ci, D, H, W, generator=gen)
    Do, Ho, Wo = ((v + 2 * p - k) // s + 1 for v in (D, H, W))
    dy = torch.randn(N, Co, Do, Ho, Wo, generator=gen)
    x, dy = x.cuda(), dy.cuda()
    desc = R.conv_desc(*case[:9], False, R.F32)
    n = R.rat3d_conv3d_workspace_size(desc, 2)
    ws = torch.empty(max(n, 1), dtype=torch.uint8, device="cuda")
    dw = torch.empty(Co, Ci, k, k, k, device="cuda")
    R.rat3d_conv3d_wgrad(desc, x, dy, dw, None, 0, ws, n)

    ref = torch.zeros(Co, Ci, k, k, k, dtype=torch.float64, device="cuda")
    xp = torch.nn.functional.pad(x.double(), (p, p + s) * 3)
    sl = lambda t, m: slice(t, t + (m - 1) * s + 1, s)
    for a in range(k):
        for b in range(k):
            for c in range(k):
                for i in range(N):
                    v = xp[i, :, sl(a, Do), sl(b, Ho), sl(c, Wo)].reshape(Ci, -1)
                    ref[:, :, a, b, c] += dy[i].double().reshape(Co, -1) @ v.t().contiguous()
    err = float((dw.double() - ref).norm() / ref.norm())
    voxels = N * Do * Ho * Wo
    S = max(1, min(-(-2048 // (-(-Co // 64) * -(-Ci * k ** 3 // 64))), -(-voxels // 256), 4096))
    c = 2.0 ** -23 * (3 / (8 * 12 * 0.6931)) ** 0.5
    bound = 1.1 * c * ((voxels / S + S) / 2) ** 0.5
    print(case, "error %.2e of %.2e" % (err, bound), flush=True)
    assert err < bound
