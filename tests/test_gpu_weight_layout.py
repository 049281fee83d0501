"""GPU parity of convolutions whose weight layouts are staged in blocks: target
channel counts of one block and several, both directions, 1^3 and 3^3, and a
weight tensor that is not 16-byte aligned."""
import pytest

from tests import gpu_util as U
from tests.test_gpu_ops import _id, test_conv3d as check_conv3d

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("case", [
    (1, 32, 32, 3, 5, 8, 3, 1, 1, False, "bf16"),
    (1, 96, 32, 3, 5, 8, 3, 1, 1, False, "bf16"),
    (1, 32, 160, 3, 5, 8, 3, 1, 1, False, "bf16"),
    (1, 96, 32, 3, 5, 8, 1, 1, 0, False, "bf16"),
    (1, 32, 160, 3, 5, 8, 1, 1, 0, False, "bf16"),
    # one thread per unit up to 128 x 128 channel pairs, staged beyond
    (1, 128, 128, 3, 5, 8, 3, 1, 1, False, "bf16"),
    (1, 96, 192, 3, 5, 8, 3, 1, 1, False, "bf16"),
    (1, 192, 96, 3, 5, 8, 3, 1, 1, False, "bf16"),
], ids=_id)
def test_weight_layout(case):
    check_conv3d(case)


@pytest.mark.parametrize("k,c", [(1, 96), (3, 96), (3, 288)])
def test_unaligned_weights(k, c):
    """The same weights 2 bytes past a 16-byte boundary: the same outputs."""
    from paper_2104_05035_amd import rat3d as R
    torch = U.torch_mod()
    desc = R.conv_desc(1, 64, c, 3, 5, 8, k, 1, k // 2, False, R.BF16)
    n = c * 64 * k ** 3
    flat = torch.randn(n + 1, device="cuda").to(torch.bfloat16)
    ws = U.workspace(max(R.rat3d_conv3d_workspace_size(desc, i) for i in range(3)))
    x = torch.randn(1, 64, 3, 5, 8, device="cuda").to(torch.bfloat16)
    dy = torch.randn(1, c, 3, 5, 8, device="cuda").to(torch.bfloat16)
    got = []
    for w in (flat[1:], flat[1:].clone()):
        w = w.view(c, 64, k, k, k)
        y, dx = torch.empty_like(dy), torch.empty_like(x)
        R.rat3d_conv3d_fwd(desc, x, w, None, y, ws, ws.numel())
        R.rat3d_conv3d_dgrad(desc, dy, w, dx, 0, ws, ws.numel())
        U.sync()
        got.append((y, dx))
    assert torch.equal(got[0][0], got[1][0]) and torch.equal(got[0][1], got[1][1])
