"""The kernels for few rows at the edges of their tiles (32 rows, 64 columns of the rank and of the factors), of the
contraction that eight waves share, and of the rule that takes them (2048 or 4096 rows), against fp64.

Tolerance: bf16 has eight significant bits, so a value is off by 2^-8 of itself at most after one rounding: dB carries that of dT, dX
that of dT and its own, T its own, Y its own beside that of the T it is compared with; dA only carries fp32 sums of exact products, (M + 1) 2^-24 of the sum of their sizes at most."""
import pytest

torch = pytest.importorskip("torch")
from paper_2405_01067_amd import binding as abt

pytestmark = pytest.mark.gpu
BF = torch.bfloat16


def rel(a, b):
    return float((a.double() - b).norm() / b.norm())


@pytest.mark.parametrize("M,m,n,r", [(1, 64, 64, 32), (31, 64, 128, 96), (32, 576, 64, 64), (33, 1088, 320, 160), (129, 2304, 768, 96),
                                     (197, 768, 768, 384), (700, 128, 1920, 192), (2048, 64, 64, 32), (2049, 64, 64, 32),
                                     (2100, 960, 64, 352), (4096, 768, 256, 32), (4097, 768, 256, 32)])
@pytest.mark.parametrize("accumulate", [False, True])
def test_backward_of_few_rows(M, m, n, r, accumulate):
    g = torch.Generator(device="cuda").manual_seed(M + m + n + r)
    rn = lambda std, *s: (torch.randn(s, generator=g, device="cuda") * std)
    X, dY, A, B, T = (rn(s, *sh).to(BF) for s, sh in ((1, (M, n)), (1e-2, (M, m)), (r ** -0.5, (m, r)), (n ** -0.5, (r, n)), (1, (M, r))))
    dA0, dB0 = rn(1e-2, m, r), rn(1e-2, r, n)
    Xd, dYd, Ad, Bd, Td = (t.double() for t in (X, dY, A, B, T))
    dT = dYd @ Ad
    want = (dT @ Bd, dYd.T @ Td + (dA0.double() if accumulate else 0), dT.T @ Xd + (dB0.double() if accumulate else 0))
    run = lambda **kw: abt.lr_linear_bwd(dY, X, T, A, B, accumulate=accumulate, **{
        k: v.clone() for k, v in (("dA", dA0), ("dB", dB0)) if accumulate and kw.get("need_" + k, True)}, **kw)
    got = run()
    assert rel(got[0], want[0]) < 2 ** -7 and rel(got[1], want[1]) < 1e-5 and rel(got[2], want[2]) < 2 ** -8
    # the same bits whatever else is asked for, and again
    for which in ((True, True, True), (True, True, False), (True, False, True), (False, True, False), (False, False, True), (True, False, False)):
        again = run(need_dX=which[0], need_dA=which[1], need_dB=which[2])
        for a, b, w in zip(got, again, which):
            assert torch.equal(a, b) if w else b is None


# one work-group of the gradients per compute unit, and two, next to each limit: rows (1400, ten times the rank), tiles of dA and dB (120), work-groups (640)
@pytest.mark.parametrize("M,m,n,r", [(1400, 128, 1920, 96), (1401, 128, 1920, 96), (1920, 128, 1920, 192), (1921, 128, 1920, 192), (4063, 256, 1280, 288),
                                     (4063, 320, 1280, 288), (3300, 64, 2560, 96), (3700, 64, 2560, 96)])
def test_gradients_that_share_a_compute_unit_and_that_do_not(M, m, n, r):
    test_backward_of_few_rows(M, m, n, r, False)


@pytest.mark.parametrize("M,m,n,r", [(5, 1600, 64, 32), (2048, 1984, 64, 128), (2049, 1088, 320, 128), (2720, 576, 64, 96), (2721, 2112, 512, 96)])
def test_tiles_of_dT_of_either_width(M, m, n, r):
    # 32 columns up to 256 tiles, 64 beyond; contractions that end at every one of the slabs in flight
    g = torch.Generator(device="cuda").manual_seed(M + m)
    rn = lambda std, *s: (torch.randn(s, generator=g, device="cuda") * std).to(BF)
    X, dY, A, B = rn(1, M, n), rn(1e-2, M, m), rn(r ** -0.5, m, r), rn(n ** -0.5, r, n)
    dX, _, dB = abt.lr_linear_bwd(dY, X, None, A, B, need_dA=False)
    dT = dY.double() @ A.double()
    assert rel(dX, dT @ B.double()) < 2 ** -7 and rel(dB, dT.T @ X.double()) < 2 ** -8


def test_not_finite_rows_stay_in_their_rows():
    M, m, n, r = 70, 128, 192, 64
    g = torch.Generator(device="cuda").manual_seed(1)
    rn = lambda *s: torch.randn(s, generator=g, device="cuda").to(BF)
    X, dY, A, B, T = rn(M, n), rn(M, m), rn(m, r), rn(r, n), rn(M, r)
    ref = abt.lr_linear_bwd(dY, X, T, A, B)[0]
    dY[33, 5] = float("inf")
    dX = abt.lr_linear_bwd(dY, X, T, A, B, need_dA=False, need_dB=False)[0]
    keep = torch.arange(M, device="cuda") != 33
    assert torch.equal(dX[keep], ref[keep]) and not bool(torch.isfinite(dX[33]).any())


def conv_patches(act, kh, kw, stride):
    N, H, W, C = act.shape
    p = torch.nn.functional.pad(act, (0, 0, kw // 2, kw // 2, kh // 2, kh // 2))
    cols = [p[:, y:y + H:stride, x:x + W:stride] for y in range(kh) for x in range(kw)]
    return torch.cat(cols, dim=-1).reshape(-1, kh * kw * C).contiguous()


# rows / 32 times r / 32 tiles of T: up to 256, 512, 1024, more; Y in tiles of 64 x 64 or 64 x 128; rows 4096 and, at r = 224, 288 and 352,
# 10240; beyond, those ranks and 320 in 128-row work-groups, whose last 32 columns of T may be padding
@pytest.mark.parametrize("M,m,n,r", [(1, 64, 768, 32), (31, 192, 320, 96), (33, 64, 64, 256), (65, 2304, 768, 384), (197, 768, 3072, 352), (1000, 320, 576, 288),
                                     (1025, 128, 192, 352), (2000, 64, 128, 384), (4096, 1088, 64, 384), (4096, 1024, 1920, 32), (4097, 576, 192, 224),
                                     (10240, 64, 192, 288), (10241, 64, 192, 288), (10241, 192, 64, 224), (12345, 128, 320, 352),
                                     (20001, 192, 128, 320), (1, 960, 64, 256), (31, 192, 1920, 96), (33, 64, 960, 256), (1000, 320, 768, 288),
                                     (1024, 64, 768, 128), (1025, 960, 64, 352), (2000, 64, 1024, 384), (10240, 64, 960, 288), (10241, 64, 960, 288)])
def test_forward_of_few_rows(M, m, n, r):
    g = torch.Generator(device="cuda").manual_seed(M + m + n + r)
    rn = lambda std, *s: (torch.randn(s, generator=g, device="cuda") * std).to(BF)
    X, A, B, dY = rn(1, M, n), rn(r ** -0.5, m, r), rn(n ** -0.5, r, n), rn(1e-2, M, m)
    Y, T = abt.lr_linear_fwd(X, A, B)
    assert rel(T, X.double() @ B.double().T) < 2 ** -8 and rel(Y, T.double() @ A.double().T) < 2 ** -8
    # T in a workspace, and again for the factor gradient: the same bits; without a place for it the other kernels
    assert torch.equal(abt.lr_linear_fwd(X, A, B, save_T=False)[0], Y)
    kept, again = (abt.lr_linear_bwd(dY, X, t, A, B, need_dX=False, need_dB=False)[1] for t in (T, None))
    assert torch.equal(kept, again)
    bare = torch.empty_like(Y)
    lib, stream = abt.load(), torch.cuda.current_stream().cuda_stream
    assert lib.lr_linear_fwd(X.data_ptr(), A.data_ptr(), B.data_ptr(), bare.data_ptr(), None, M, m, n, r, abt.ABT_BF16, None, 0, stream) == 0
    assert rel(bare, T.double() @ A.double().T) < 2 ** -7
    # an output over the input: Y may lie there, and T sends the call to the other kernels
    if m == n:
        over = X.clone()
        assert torch.equal(abt.lr_linear_fwd(over, A, B, Y=over)[0], Y)
    # groups of it, each with inputs of its own
    groups = [dict(X=X, A=A, B=B), dict(X=X * 2, A=A, B=B), dict(X=X, A=A, B=B * 2)]
    for save in (True, False):
        outs = abt.lr_linear_fwd_grouped(groups, save_T=save)
        for k, (Yg, Tg) in zip((1, 2, 2), outs):
            assert rel(Yg, k * (X.double() @ B.double().T) @ A.double().T) < 2 ** -6.5      # T and Y rounded: 2^-7, and its square
            assert not save or rel(Tg, k * (X.double() @ B.double().T)) < 2 ** -8


# grids of one pixel, odd sides, windows without a tap for some parity, and 4096 rows and their surroundings
@pytest.mark.parametrize("N,H,W,C,kh,kw,stride,m,r", [(1, 1, 1, 64, 3, 3, 1, 64, 256), (2, 7, 7, 512, 3, 3, 1, 512, 64), (3, 14, 13, 128, 3, 3, 2, 64, 96),
                                                      (1, 9, 5, 64, 5, 5, 2, 128, 384), (20, 14, 14, 256, 3, 3, 1, 256, 32), (2, 28, 28, 64, 3, 3, 1, 64, 320),
                                                      (4, 7, 9, 192, 1, 1, 2, 64, 160), (5, 6, 11, 64, 1, 3, 2, 192, 64), (2, 1, 8, 128, 3, 1, 2, 64, 96),
                                                      (21, 14, 14, 64, 3, 3, 1, 64, 128), (17, 31, 31, 64, 3, 3, 2, 64, 64), (32, 16, 16, 64, 3, 3, 1, 64, 192)])
def test_convolution_of_few_pixels(N, H, W, C, kh, kw, stride, m, r):
    g = torch.Generator(device="cuda").manual_seed(N + H + C + r)
    rn = lambda std, *s: (torch.randn(s, generator=g, device="cuda") * std).to(BF)
    n = kh * kw * C
    act, A, B = rn(1, N, H, W, C), rn(r ** -0.5, m, r), rn(n ** -0.5, r, n)
    P = conv_patches(act, kh, kw, stride)
    Y, T = abt.lr_conv_fwd(act, A, B, kh, kw, stride=stride)
    assert rel(T, P.double() @ B.double().T) < 2 ** -8 and rel(Y.reshape(len(P), m), T.double() @ A.double().T) < 2 ** -8
    dY = rn(1e-2, len(P), m)
    dT = dY.double() @ A.double()
    pixels = act.double().requires_grad_()
    want = torch.autograd.grad(conv_patches(pixels, kh, kw, stride), pixels, dT @ B.double())[0]
    got = abt.lr_conv_bwd(dY, act, T, A, B, kh, kw, stride=stride)
    assert rel(got[0], want) < 2 ** -7 and rel(got[1], dY.double().T @ T.double()) < 1e-5 and rel(got[2], dT.T @ P.double()) < 2 ** -8
    for which in ((True, False, False), (False, True, False), (False, False, True), (False, True, True)):
        again = abt.lr_conv_bwd(dY, act, T, A, B, kh, kw, stride=stride, need_dAct=which[0], need_dA=which[1], need_dB=which[2])
        for a, b, w in zip(got, again, which):
            assert torch.equal(a, b) if w else b is None
    twice = abt.lr_conv_bwd(dY, act, T, A, B, kh, kw, stride=stride, dA=got[1].clone(), dB=got[2].clone(), accumulate=True)
    assert rel(twice[1], 2 * got[1].double()) < 1e-6 and rel(twice[2], 2 * got[2].double()) < 1e-6


# Which backward it is shows in the order of dA's fp32 sums: with the column parts named, the kernels for many rows.
# Sizes on both sides of every limit: rows, products, a wide dX, a long contraction of dT.
@pytest.mark.parametrize("M,m,n,r,few", [(2048, 64, 64, 32, True), (2049, 64, 64, 32, False), (4096, 768, 256, 32, True), (4097, 768, 256, 32, False),
                                         (4096, 3072, 768, 192, True), (4096, 3072, 768, 256, False), (4096, 1024, 4096, 384, False), (2048, 4096, 4096, 384, False),
                                         (2048, 64, 8192, 96, True), (2048, 64, 8192, 192, False), (1024, 128, 16384, 160, False), (1024, 64, 16384, 64, True),
                                         (197, 7168, 64, 96, True), (197, 7232, 64, 96, False), (197, 8192, 64, 64, True), (1024, 8192, 64, 64, False),
                                         (197, 8256, 64, 32, False), (100, 8320, 7232, 32, True), (4055, 768, 3072, 352, True)])
def test_which_backward_a_linear_layer_takes(M, m, n, r, few):
    g = torch.Generator(device="cuda").manual_seed(M + m + n + r)
    rn = lambda std, *s: (torch.randn(s, generator=g, device="cuda") * std).to(BF)
    X, dY, A, B, T = rn(1, M, n), rn(1e-2, M, m), rn(r ** -0.5, m, r), rn(n ** -0.5, r, n), rn(1, M, r)
    dA = lambda: abt.lr_linear_bwd(dY, X, T, A, B, need_dX=False, need_dB=False)[1]
    got = dA()
    prev = abt.set_chain_parts(1)
    try:
        want = dA()
    finally:
        abt.set_chain_parts(prev)
    assert rel(got, want.double()) < 1e-5 and torch.equal(got, want) != few
    if (M, m) == (4055, 768):                            # with dB they are too many products
        assert torch.equal(abt.lr_linear_bwd(dY, X, T, A, B, need_dX=False)[1], want)


# the same for convolutions: rows, products, columns of the patch matrix, pixels, products with A
@pytest.mark.parametrize("N,side,C,kh,stride,m,r,few", [(1, 45, 512, 3, 1, 64, 384, True), (20, 14, 576, 3, 1, 64, 384, False), (20, 14, 512, 3, 1, 64, 192, True),
                                                        (20, 14, 1024, 3, 1, 64, 32, True), (1, 60, 1344, 3, 1, 64, 128, False), (83, 14, 1024, 1, 2, 64, 64, False),
                                                        (187, 7, 2048, 1, 2, 64, 64, True), (256, 7, 2048, 1, 2, 64, 192, False), (256, 7, 2048, 1, 2, 64, 256, True),
                                                        (2, 57, 64, 3, 1, 1472, 160, True), (2, 57, 64, 3, 1, 1600, 160, False), (169, 7, 64, 3, 1, 64, 64, False)])
def test_which_backward_a_convolution_takes(N, side, C, kh, stride, m, r, few):
    g = torch.Generator(device="cuda").manual_seed(N + C + r)
    rn = lambda std, *s: (torch.randn(s, generator=g, device="cuda") * std).to(BF)
    rows = N * (-(-side // stride)) ** 2
    act, A, B, dY, T = rn(1, N, side, side, C), rn(r ** -0.5, m, r), rn(0.01, r, kh * kh * C), rn(1e-2, rows, m), rn(1, rows, r)
    dA = lambda: abt.lr_conv_bwd(dY, act, T, A, B, kh, kh, stride=stride, need_dAct=False, need_dB=False)[1]
    got = dA()
    prev = abt.set_chain_parts(1)
    try:
        want = dA()
    finally:
        abt.set_chain_parts(prev)
    assert rel(got, want.double()) < 1e-5 and torch.equal(got, want) != few
