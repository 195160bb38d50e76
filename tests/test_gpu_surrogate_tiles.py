"""The order in which the convolution blocks take their tiles: patches of 4 x 8
tiles per XCD where the image divides into them, a remainder past the last full
round of blocks, and images that do not divide.  With a cap on the blocks every
tile is taken in plain order, and the results are the same bits."""
import pytest
import torch

from paper_1908_05232_amd import fps, surrogate as SG
from tests.gpu_util import say

pytestmark = pytest.mark.gpu


# tiles of 16 x 32 pixels: 288 = 256 + 32 in patches, 512 in patches, 300 not in
# patches, 257 in one row, 35 (fewer than the blocks)
@pytest.mark.parametrize("n,H,W", [(3, 192, 256), (2, 512, 256), (3, 160, 320), (1, 16, 32 * 257), (1, 112, 160)])
def test_tile_order_does_not_change_the_results(n, H, W):
    g = torch.Generator(device="cuda").manual_seed(n * H + W)
    x = torch.zeros(n, H, W, 16, device="cuda", dtype=torch.bfloat16)
    x[..., :6] = (torch.rand(n, H, W, 6, device="cuda", generator=g) * 2 - 1).bfloat16()
    t = torch.zeros(n, H, W, 4, device="cuda")
    t[..., :3] = torch.randn(n, H, W, 3, device="cuda", generator=g)
    p = torch.tensor(SG.init_params(5), device="cuda")
    p = p + 0.01 * torch.randn(p.shape, device="cuda", generator=g) * (p != 0)
    out = []
    for cap in (0, 7):
        sur = fps.Surrogate(n, H, W)
        sur.set_params(p)
        sur.set_blocks(conv_blocks=cap)
        y = sur.forward(x).clone()
        loss, grad = sur.gradients(x, t)
        out.append((y, loss.clone(), grad))
        sur.close()
    say(f"{n} x {H} x {W}: {n * H * W // 512} tiles, max|y| {float(out[0][0].abs().max()):.3f}")
    assert torch.isfinite(out[0][0]).all() and float(out[0][0].abs().max()) > 0
    for a, b in zip(*out):
        assert torch.equal(a, b)
