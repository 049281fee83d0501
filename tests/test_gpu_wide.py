"""Strided bf16 convolutions of tensors of 2^30 elements and more, which the
gather kernels address with 64 bits: equal bit for bit to the same samples one by
one, which are below the line and take the 32-bit kernels, and these right at
the tensors' far corner.  Weight gradients (another kernel above the line) are
within the rounding of float32 sums of the samples' own."""
import pytest

from tests import gpu_util as U

pytestmark = pytest.mark.gpu

LINE = 2 ** 30


def _run(n, ci, co, size, inputs=None):
    """(x, w, dy, y, dx, dw) of a 3^3 stride-2 pad-1 convolution of n cubes."""
    from paper_2104_05035_amd import rat3d as R
    torch = U.torch_mod()
    so = (size - 1) // 2 + 1
    if inputs is None:
        torch.manual_seed(ci + co)
        x = torch.empty(n, ci, size, size, size, dtype=torch.bfloat16, device="cuda").normal_()
        dy = torch.empty(n, co, so, so, so, dtype=torch.bfloat16, device="cuda").normal_()
        w = torch.randn(co, ci, 3, 3, 3, device="cuda").mul_((2 / (27 * ci)) ** 0.5).bfloat16()
    else:
        x, w, dy = inputs
    desc = R.conv_desc(n, ci, co, size, size, size, 3, 2, 1, False, R.BF16)
    nbytes = max(R.rat3d_conv3d_workspace_size(desc, i) for i in range(3))
    ws = U.workspace(nbytes)
    y, dx = torch.full_like(dy, 7.0), torch.full_like(x, 7.0)
    dw = torch.full(w.shape, 7.0, device="cuda")
    R.rat3d_conv3d_fwd(desc, x, w, None, y, ws, nbytes)
    R.rat3d_conv3d_dgrad(desc, dy, w, dx, 0, ws, nbytes)
    R.rat3d_conv3d_wgrad(desc, x, dy, dw, None, 0, ws, nbytes)
    U.sync()
    return x, w, dy, y, dx, dw


# x past the line (its samples a third of it each); dy past the line
@pytest.mark.parametrize("ci,co,size", [(32, 32, 225), (4, 64, 356)])
def test_tensors_past_the_line(ci, co, size):
    torch = U.torch_mod()
    x, w, dy, y, dx, dw = _run(3, ci, co, size)
    assert max(x.numel(), dy.numel()) >= LINE and max(x.numel(), dy.numel()) // 3 < LINE
    total, terms = torch.zeros_like(dw, dtype=torch.float64), torch.zeros_like(dw, dtype=torch.float64)
    for n in range(3):
        one = tuple(t[n:n + 1] for t in (x, dy))
        r = _run(1, ci, co, size, (one[0], w, one[1]))
        assert torch.equal(r[3], y[n:n + 1]) and torch.equal(r[4], dx[n:n + 1]), n
        total += r[5].double()
        terms += _run(1, ci, co, size, (one[0].abs(), w, one[1].abs()))[5].double()
    # float32 sums of up to 16.9 M products, as in gpu_util: 2^-12 of the sum of
    # |terms| on either side
    assert bool(((dw.double() - total).abs() <= 2 * 2.0 ** -12 * terms).all())
    # the last four outputs of each axis of the last sample: taps 2 o - 1 .. 2 o + 1
    so = dy.shape[-1]
    i0 = 2 * (so - 4) - 1
    pad = 2 * (so - 1) + 2 - size  # zeros behind the map that the last tap reads
    c = x[2:, :, i0:, i0:, i0:].cpu().double()
    ref = torch.nn.functional.conv3d(torch.nn.functional.pad(c, (0, pad) * 3), w.cpu().double(),
                                     stride=2)
    U.check(U.f64(y[2:, :, -4:, -4:, -4:]), ref.bfloat16().double().numpy(), "bf16", "y corner",
            terms=torch.nn.functional.conv3d(torch.nn.functional.pad(c.abs(), (0, pad) * 3),
                                             w.cpu().double().abs(), stride=2).numpy())
    # and the last four inputs': output o reaches 2 o - 1 .. 2 o + 1
    g = dy[2:, :, -4:, -4:, -4:].cpu().double()
    j0 = size - 4 - i0
    dref, dterms = (torch.nn.functional.conv_transpose3d(a, b, stride=2)[..., j0:j0 + 4, j0:j0 + 4, j0:j0 + 4]
                    for a, b in ((g, w.cpu().double()), (g.abs(), w.cpu().double().abs())))
    U.check(U.f64(dx[2:, :, -4:, -4:, -4:]), dref.bfloat16().double().numpy(), "bf16", "dx corner",
            terms=dterms.numpy())
