"""The order in which the convolution blocks take their tiles: patches of 4 x 8
tiles per XCD where the image divides into them, a remainder past the last full
round of blocks, and images that do not divide.  With a cap on the blocks every
tile is taken in plain order, and the results are the same bits.  And the
weight gradient's runs of 4-row bands: with a batch that is no multiple of eight
a run ends inside an image or past the last band."""
import numpy as np
import pytest
import torch

from oracle import surrogate_oracle as S
from paper_1908_05232_amd import fps, surrogate as SG
from tests.gpu_util import say
from tests.test_gpu_surrogate import ELEM_TOL, cosine, make_case, rel_l2, to_dev, unpack

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


# bands of the batch: 4 (four empty slots), 8 (one each), 12 (runs of 2, two
# slots empty), 20 (runs of 3 over image borders, the last slot 2 short of
# full), 60 (runs of 8 in images of 12), with the bars of the other gradient tests
@pytest.mark.parametrize("n,H,W", [(1, 16, 32), (2, 16, 32), (3, 16, 64), (5, 16, 32), (5, 48, 32)])
def test_weight_gradient_of_ragged_batches_matches_oracle(n, H, W):
    params, x, target = make_case(40 + n, n, H, W)
    sur = fps.Surrogate(n, H, W)
    p, xt, tt = to_dev(params, x, target)
    sur.set_params(p)
    _, g = sur.gradients(xt, tt)
    _, gb = S.loss_and_grads(params, x, target, bf16=True)
    gg = unpack(g.cpu().numpy().astype(np.float64), params)
    sur.close()
    for li in range(len(gg)):
        (dw, db), (dwb, dbb) = gg[li], gb[li]
        if li == 0:
            dw, dwb = dw[..., :5], dwb[..., :5]       # zero input channels carry no gradient
        ew = float(np.abs(dw - dwb).max() / np.abs(dwb).max())
        eb = float(np.abs(db - dbb).max() / np.abs(dbb).max())
        say(f"{n} x {H} x {W}, layer {li + 1}: dW max|d| / max|ref| {ew:.2e}, db {eb:.2e}")
        assert ew <= ELEM_TOL and eb <= ELEM_TOL
        assert cosine(dw, dwb) >= 0.9999 and rel_l2(dw, dwb) <= 1e-2


# 9 bands of 12 tiles: 14 tiles an XCD (the last 10), and grids capped to both orders
def test_weight_gradient_blocks_only_group_the_sums():
    params, x, target = make_case(71, 3, 96, 96)
    p, xt, tt = to_dev(params, x, target)
    out = []
    for cap in (0, 8, 16, 7, 100):
        sur = fps.Surrogate(3, 96, 96)
        sur.set_params(p)
        sur.set_blocks(0, cap)
        out.append(sur.gradients(xt, tt)[1].cpu().numpy().astype(np.float64))
        sur.close()
    assert np.abs(out[0]).max() > 0
    for g in out[1:]:
        d = float(np.abs(g - out[0]).max() / np.abs(out[0]).max())
        say(f"max|dg| / max|g| = {d:.2e}")
        assert d <= 1e-5
