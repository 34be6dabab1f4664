"""Factor gradients of convolutions with windows three pixels wide and many pixels: whole numbers of a size that every
product and sum holds exactly (dT up to 256 in bf16, sums below 2^24 in fp32), so the results have to be equal."""
import pytest
import torch

from paper_2405_01067_amd import binding as abt

pytestmark = pytest.mark.gpu

BF = torch.bfloat16


def whole(g, shape, lo, hi):
    return torch.randint(lo, hi + 1, shape, generator=g).float()


# grids of just the positions of a slab (128 up to r = 64, 64 at r = 96) and odd ones, heights of one, three and five rows, channels in one to three blocks of 64, half and whole
# tiles of dA, numbers of rows that are no multiple of a slab
@pytest.mark.parametrize("N,H,W,C,m,r,kh,stride", [
    (66, 16, 8, 64, 64, 32, 3, 1), (81, 11, 12, 64, 128, 64, 3, 1), (53, 13, 13, 128, 192, 64, 3, 1), (137, 8, 8, 192, 64, 96, 3, 1),
    (13, 29, 27, 64, 256, 96, 5, 1), (41, 15, 14, 128, 64, 32, 1, 1), (3, 3, 1025, 64, 64, 64, 3, 1), (70, 23, 24, 64, 128, 64, 3, 2),
    (64, 22, 23, 128, 64, 32, 5, 2), (140, 16, 15, 64, 64, 96, 3, 2), (40, 29, 29, 64, 192, 64, 1, 2)])
@pytest.mark.parametrize("with_dA,accumulate", [(True, False), (False, False), (True, True)])
def test_factor_gradients_are_exact(N, H, W, C, m, r, kh, stride, with_dA, accumulate):
    g = torch.Generator().manual_seed(H * W + r + kh)
    act = whole(g, (N, H, W, C), 0, 3)
    Ho, Wo = -(-H // stride), -(-W // stride)
    rows = N * Ho * Wo
    assert rows > 8192                                   # fewer pixels take other kernels
    dY = whole(g, (rows, m), -1, 1) * (whole(g, (rows, m), 0, 9) < 2)    # mostly zeros: |dT| is held exactly for any m here
    A, T = whole(g, (m, r), -1, 1), whole(g, (rows, r), -2, 2)
    B = torch.zeros((r, kh * 3 * C))
    dT = dY @ A
    assert float(dT.abs().max()) <= 256
    # Infinities all along an edge of every image, in a channel of their own: no tap that looks away from that edge comes to one, in whatever slab or
    # split the pixel beside it lies, and a zero gradient in its place would make a NaN
    edges = {5: (slice(None), W - 1), 6: (slice(None), 0), 7: (H - 1, slice(None)), 8: (0, slice(None))}
    clean = act.clone()
    for c, (y, x) in edges.items():
        act[:, y, x, c] = float("inf")
        clean[:, y, x, c] = 0
    patches = torch.nn.functional.unfold(clean.permute(0, 3, 1, 2), (kh, 3), padding=(kh // 2, 1), stride=stride)
    patches = patches.view(N, C, kh * 3, Ho * Wo)
    want = torch.einsum("nctl,nlr->rtc", patches.double(), dT.view(N, Ho * Wo, r).double())
    dev = [t.to("cuda:0").to(BF) for t in (dY, act, T, A, B)]
    given = {"dA": torch.full((m, r), 3.0, device="cuda:0"), "dB": torch.full((r, kh * 3 * C), 5.0, device="cuda:0")} if accumulate else {}
    _, dA, dB = abt.lr_conv_bwd(dev[0], dev[1], dev[2], dev[3], dev[4], kh, 3, stride=stride, need_dAct=False, need_dA=with_dA, accumulate=accumulate, **given)
    got = dB.cpu().double().view(r, kh * 3, C) - (5 if accumulate else 0)
    keep = [c for c in range(C) if c not in edges]
    assert torch.equal(got[:, :, keep], want[:, :, keep])
    tap = torch.arange(kh * 3)
    away = {5: tap % 3 == 0, 6: tap % 3 == 2, 7: tap // 3 < kh // 2, 8: tap // 3 > kh // 2}
    for c, taps in away.items():
        assert torch.equal(got[:, taps, c], want[:, taps, c])
        assert not torch.isfinite(got[:, 3 * (kh // 2) + 1, c]).all() or (c == 5 and stride == 2 and W % 2 == 0) or (c == 7 and stride == 2 and H % 2 == 0)
    if with_dA:
        assert torch.equal(dA.cpu().double() - (3 if accumulate else 0), dY.double().T @ T.double())
