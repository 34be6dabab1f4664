"""Infinite inputs: they reach the rows and pixels that depend on them and no others, and stay infinities where every term
of the exact sum that is not finite has the same sign."""
import pytest

torch = pytest.importorskip("torch")
from paper_2405_01067_amd import binding as abt

pytestmark = pytest.mark.gpu
BF = torch.bfloat16


# ranks whose kernel computes 32 columns more than there are, and others; few rows and many
@pytest.mark.parametrize("r", [96, 192, 224, 256, 288, 320, 352, 384])
@pytest.mark.parametrize("M,m,n", [(300, 128, 192), (300, 1024, 192), (12000, 128, 192)])
def test_rows_of_a_linear_layer(r, M, m, n):
    g = torch.Generator(device="cuda").manual_seed(r + M)
    rn = lambda *s: (torch.rand(s, generator=g, device="cuda") + 0.5).to(BF)
    X, A, B, dY = rn(M, n), rn(m, r), rn(r, n), rn(M, m)
    X[33, 5] = float("inf")
    dY[34, 7] = float("-inf")
    Y, T = abt.lr_linear_fwd(X, A, B)
    dX = abt.lr_linear_bwd(dY, X, T, A, B, need_dA=False, need_dB=False)[0]
    for out, row, value in ((T, 33, float("inf")), (Y, 33, float("inf")), (dX, 34, float("-inf"))):
        assert bool((out[row] == value).all())
        out[row] = 0
        assert bool(torch.isfinite(out).all())


# one pixel, through the window in LDS (one block of channels, several), gathered, and as two products
@pytest.mark.parametrize("N,H,W,C,r,stride", [(90, 14, 14, 64, 64, 1), (90, 14, 14, 128, 96, 1), (30, 26, 64, 64, 192, 1), (60, 15, 13, 64, 64, 2), (2, 14, 14, 256, 256, 1)])
def test_pixels_of_a_convolution(N, H, W, C, r, stride):
    g = torch.Generator(device="cuda").manual_seed(r + N)
    rn = lambda *s: (torch.rand(s, generator=g, device="cuda") + 0.5).to(BF)
    act, A, B = rn(N, H, W, C), rn(64, r), rn(r, 9 * C)
    act[1, 4, 6, C - 1] = float("inf")
    Y, T = abt.lr_conv_fwd(act, A, B, 3, 3, stride=stride)
    Ho, Wo = -(-H // stride), -(-W // stride)
    hit = torch.zeros((N, Ho, Wo), dtype=torch.bool, device="cuda")
    for y in range(Ho):
        for x in range(Wo):
            hit[1, y, x] = abs(y * stride - 4) <= 1 and abs(x * stride - 6) <= 1
    hit = hit.view(-1)
    for out in (T, Y):
        assert bool((out[hit] == float("inf")).all()) and bool(torch.isfinite(out[~hit]).all())
    # dAct: pixels within reach of an infinite dY
    dY = rn(N * Ho * Wo, 64)
    at = (1 * Ho + 3) * Wo + 2
    dY[at, 9] = float("-inf")
    dAct = abt.lr_conv_bwd(dY, act, T, A, B, 3, 3, stride=stride, need_dA=False, need_dB=False)[0]
    hit = torch.zeros((N, H, W), dtype=torch.bool, device="cuda")
    hit[1, 3 * stride - 1:3 * stride + 2, 2 * stride - 1:2 * stride + 2] = True
    assert bool((dAct[hit] == float("-inf")).all()) and bool(torch.isfinite(dAct[~hit]).all())


# A merge of a rank-32 layer, whose sorted values must be those of this call and no others.  Every column of the core is then not finite, or, with
# the fault in B, one is zero; the stages for all sizes, taken when a layer of another rank is in the batch, do the same.
@pytest.mark.parametrize("side", ["A", "B"])
@pytest.mark.parametrize("value", [float("nan"), float("inf"), float("-inf")])
@pytest.mark.parametrize("row,col", [(0, 0), (17, 31), (31, 5)])
def test_merge_of_a_core_of_32(side, value, row, col):
    g = torch.Generator(device="cuda").manual_seed(row + col)
    rn = lambda *s: torch.randn(s, generator=g, device="cuda")
    lay = lambda k, scale: {"A_copies": [scale * rn(96, k) for _ in range(2)], "B_copies": [rn(k, 80) for _ in range(2)], "tau": 0.3}
    bad, other = lay(32, 1.0), lay(64, 1.0)
    bad[side + "_copies"][1][row, col] = value
    runs = []
    for scale in (1.0, 1e3):                              # what merges before it leave behind
        abt.ab_merge_batched([lay(32, scale) for _ in range(300)])
        runs.append(abt.ab_merge_batched([bad])[0])
    for out in runs + [abt.ab_merge_batched([bad, other])[0]]:
        assert not bool((torch.isfinite(out["S"]) & (out["S"] != 0)).any())
        assert int(out["k"]) == 1                         # no value passes the comparison with the largest
    first, again = runs
    for name in ("S", "k", "A", "B"):
        assert torch.equal(first[name].view(torch.int32), again[name].view(torch.int32))
    # a layer beside it is not touched
    good = lay(32, 1.0)
    alone = abt.ab_merge_batched([good])[0]
    beside = abt.ab_merge_batched([bad, good])[1]
    assert all(torch.equal(alone[name], beside[name]) for name in ("S", "k", "A", "B"))
