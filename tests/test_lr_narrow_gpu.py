"""The narrow-rank chain kernel (r <= 192, several work-groups per compute unit) where its dispatch takes it:
small batches whose row blocks are shared by output tiles, large ones with evenly shared rows, and the
factored convolution, whose activation gradient is taken parity by parity with stride 2.

Against the CPU oracle with the layer's tolerance (1e-2: bf16 storage, fp32 accumulation), and against the
kernels for all ranks (forced by set_chain_rows): the same products summed in fp32 in another order and
rounded to bf16 twice (T or dT, then the result), so two results differ by single roundings of a few entries:
below 2^-8 = 4e-3 in norm."""
import numpy as np
import pytest
import torch

from oracle import ab_oracle as orc
from paper_2405_01067_amd import binding as abt
from paper_2405_01067_amd import inputs as gen

pytestmark = pytest.mark.gpu

TOL, TOL_ORDER = 1e-2, 4e-3
BF = torch.bfloat16


def rel(a, b):
    a = np.asarray(a, dtype=np.float64)
    b = np.asarray(b, dtype=np.float64)
    return float(np.linalg.norm(a - b) / max(np.linalg.norm(b), 1e-300))


def dev(x):
    return torch.from_numpy(np.ascontiguousarray(x)).to("cuda:0").to(BF)


def host(t):
    return t.detach().float().cpu().numpy().astype(np.float64)


@pytest.mark.parametrize("M,m,n,r", [
    (1, 64, 64, 32),            # one row, one slab, one output tile
    (33, 448, 64, 96),          # one slab; seven tiles, shared by as many work-groups
    (129, 192, 128, 64),        # ragged second row block
    (700, 640, 320, 192),       # odd numbers of slabs and tiles at the widest rank
    (8192, 128, 64, 128),       # the largest small batch
    (32769, 64, 64, 96),        # the smallest large one: two work-groups per compute unit
    (40001, 128, 192, 64),      # rows that do not divide evenly among the work-groups
    (33333, 64, 128, 160),
])
def test_linear_step(M, m, n, r):
    c = gen.lr_case(M=M, m=m, n=n, r=r, seed=M + m + n + r)
    X, dY, A, B = (dev(c[k]) for k in ("X", "dY", "A", "B"))
    Y, T = abt.lr_linear_fwd(X, A, B, save_T=True)
    dX, dA, dB = abt.lr_linear_bwd(dY, X, T, A, B)
    torch.cuda.synchronize()
    Yo, To = orc.lr_linear_fwd(c["X"], c["A"], c["B"])
    dXo, dAo, dBo, _ = orc.lr_linear_bwd(c["dY"], c["X"], c["A"], c["B"])
    errs = {k: rel(host(a), b) for k, a, b in (("Y", Y, Yo), ("T", T, To), ("dX", dX, dXo), ("dA", dA, dAo), ("dB", dB, dBo))}
    assert all(e < TOL for e in errs.values()), errs


@pytest.mark.parametrize("N,H,W,C,m,r,kh,kw,stride", [
    (2, 7, 9, 64, 64, 96, 3, 3, 2),       # odd sides: the parities have grids of different sizes
    (3, 6, 5, 128, 64, 32, 1, 1, 2),      # 1 x 1: three parities without a tap
    (2, 9, 6, 192, 64, 64, 5, 3, 2),      # 3 + 2 taps by 2 + 1
    (1, 1, 11, 64, 64, 64, 7, 7, 2),      # height 1: two parities without a row
    (5, 12, 12, 320, 64, 160, 3, 3, 1),   # channel blocks of 160
    (3, 10, 10, 512, 64, 32, 3, 3, 2),    # four blocks of 128 channels x four parities: two launches
    (86, 14, 14, 64, 192, 64, 3, 3, 1),   # more than 128 row blocks: the forward too
])
def test_convolution_agrees_with_the_kernels_for_all_ranks(N, H, W, C, m, r, kh, kw, stride):
    c = gen.conv_case(N, H, W, C, m, r, kh, kw, seed=N + 10 * H + W + C + r, stride=stride)
    act, dY, A, B = (dev(c[k]) for k in ("act", "dY", "A", "B"))

    def step():
        Y, T = abt.lr_conv_fwd(act, A, B, kh, kw, save_T=True, stride=stride)
        out = (Y, T) + tuple(abt.lr_conv_bwd(dY, act, T, A, B, kh, kw, stride=stride))
        torch.cuda.synchronize()
        return out

    got = step()
    prev = abt.set_chain_rows(64)
    try:
        want = step()
    finally:
        abt.set_chain_rows(prev)
    for name, a, b in zip(("Y", "T", "dAct", "dA", "dB"), got, want):
        assert rel(host(a), host(b)) < TOL_ORDER, name
    # pixels that no window reaches get exact zeros from both
    assert torch.equal(got[2] == 0, want[2] == 0)


@pytest.mark.parametrize("C", [1 << 19, 1 << 20])
def test_activation_gradient_of_many_tiny_images_with_wide_rows(C):
    # 3 x 3 images, 1 x 1 window, stride 2: a row block of the odd pixels spans as many images as it has rows, and at 2^20
    # channels 128 of them are beyond 32-bit offsets (the kernels for all ranks take the call)
    N, side, m, r = 128, 3, 64, 32
    g = torch.Generator(device="cuda").manual_seed(9)
    rnd = lambda shape, std: (torch.randn(shape, generator=g, device="cuda") * std).to(BF)
    B, A, dY = rnd((r, C), r ** -0.5), rnd((m, r), r ** -0.5), rnd((N * 4, m), 1.0)
    act = torch.zeros((N, side, side, C), dtype=BF, device="cuda")
    dAct = torch.full_like(act, 7.0)
    abt.lr_conv_bwd(dY, act, None, A, B, 1, 1, need_dA=False, need_dB=False, dAct=dAct, stride=2)
    even = dAct[:, ::2, ::2, :].reshape(N * 4, C)
    dT = (dY.float() @ A.float()).to(BF).float()
    for i in range(0, N * 4, 64):                        # in slices: the product in fp32 is 2 GB
        want = dT[i:i + 64] @ B.float()
        assert float((even[i:i + 64].float() - want).norm() / want.norm()) < TOL
    assert not dAct[:, 1].any() and not dAct[:, :, 1].any()


@pytest.mark.parametrize("r", [32, 64, 96, 128, 160, 192])
@pytest.mark.parametrize("M", [1, 197, 4000, 8192])
def test_first_stage_alone_repeats_the_saved_product(M, r):
    # T again, without a second stage: its columns are shared among work-groups, by 32, 64 or not at all
    m, n = 640, 320
    c = gen.lr_case(M=M, m=m, n=n, r=r, seed=M + r)
    X, dY, A, B = (dev(c[k]) for k in ("X", "dY", "A", "B"))
    T = abt.lr_linear_fwd(X, A, B)[1]
    with_T = abt.lr_linear_bwd(dY, X, T, A, B, need_dX=False)
    again = abt.lr_linear_bwd(dY, X, None, A, B, need_dX=False)
    assert torch.equal(again[1], with_T[1]) and torch.equal(again[2], with_T[2])
    # dT alone, p = m: 64 -> 64 and wider
    dX, _, dB = abt.lr_linear_bwd(dY, X, T, A, B, need_dA=False)
    assert torch.equal(dB, with_T[2])
    assert rel(host(dX), orc.lr_linear_bwd(c["dY"], c["X"], c["A"], c["B"])[0]) < TOL


def test_first_stage_of_several_groups_repeats_the_saved_products():
    M, m, n, r = 500, 640, 320, 96
    groups, outs = [], []
    for g in range(3):
        c = gen.lr_case(M=M, m=m, n=n, r=r, seed=70 + g)
        groups.append({k: dev(c[k]) for k in ("X", "dY", "A", "B")})
    for e, (_, T) in zip(groups, abt.lr_linear_fwd_grouped([{k: e[k] for k in ("X", "A", "B")} for e in groups])):
        e["T"] = T
    with_T = abt.lr_linear_bwd_grouped([dict(e, dA=True) for e in groups])
    again = abt.lr_linear_bwd_grouped([dict(e, T=None, dA=True) for e in groups])
    for a, b in zip(again, with_T):
        assert torch.equal(a[1], b[1])


@pytest.mark.parametrize("N", [28, 30, 48])       # splits of six tiles: 42 (rows for no more), 42 instead of 45, 64
def test_convolution_gradients_between_one_and_two_work_groups_per_unit(N):
    H, C, m, r = 28, 64, 64, 32
    c = gen.conv_case(N, H, H, C, m, r, 3, 3, seed=N)
    act, dY, A, B = (dev(c[k]) for k in ("act", "dY", "A", "B"))
    T = abt.lr_conv_fwd(act, A, B, 3, 3)[1]
    dAct, dA, dB = abt.lr_conv_bwd(dY, act, T, A, B, 3, 3)
    pt = torch.nn.functional.pad(act.float(), (0, 0, 1, 1, 1, 1)).unfold(1, 3, 1).unfold(2, 3, 1)      # [N, H, W, C, ky, kx]
    patches = pt.permute(0, 1, 2, 4, 5, 3).reshape(N * H * H, 9 * C)
    dT = (dY.float() @ A.float()).to(BF).float()
    assert rel(host(dB), (dT.t() @ patches).cpu()) < TOL
    assert rel(host(dA), (dY.float().t() @ T.float()).cpu()) < TOL


# More than 8192 output pixels, beyond the kernels for few pixels: the activation gradient with a window of several taps in this kernel,
# parity by parity with stride 2 (a parity's window of the image in LDS, or gathered), and with stride 1.
@pytest.mark.parametrize("N,H,W,C,m,r,kh,kw,stride", [
    (34, 31, 33, 64, 64, 64, 3, 3, 2),       # odd sides, one block of 64 ranks: parities of 4, 2, 2 and 1 taps through windows in one launch
    (34, 31, 33, 64, 64, 96, 3, 3, 2),       # two blocks of ranks with fewer than nine taps: gathered
    (40, 29, 30, 64, 64, 64, 5, 3, 2),       # 3 + 2 taps by 1 + 2
    (9, 63, 65, 192, 64, 64, 3, 3, 2),       # blocks of 192 channels
    (34, 31, 31, 512, 64, 32, 3, 3, 2),      # four blocks of 128 channels x four parities: two launches
    (2100, 3, 3, 64, 64, 64, 3, 3, 2),       # the odd pixels of tiny images, an image each: no window holds a row block's
    (1100, 1, 15, 64, 64, 64, 3, 3, 2),      # height 1: two parities without a row
    (150, 15, 16, 64, 64, 32, 1, 1, 2),      # 1 x 1: three parities without a tap
    (60, 13, 11, 64, 64, 64, 5, 3, 1),       # stride 1, a window of 15 taps
    (60, 12, 12, 320, 64, 160, 3, 3, 1),     # three blocks of ranks, channel blocks of 160
])
def test_many_pixels_against_the_kernels_for_all_ranks(N, H, W, C, m, r, kh, kw, stride):
    assert N * -(-H // stride) * -(-W // stride) > 8192
    g = torch.Generator(device="cuda").manual_seed(N + H + C + r)
    rn = lambda std, *s: (torch.randn(s, generator=g, device="cuda") * std).to(BF)
    act, A, B = rn(1, N, H, W, C), rn(r ** -0.5, m, r), rn((kh * kw * C) ** -0.5, r, kh * kw * C)
    dY = rn(1e-2, N * -(-H // stride) * -(-W // stride), m)

    def step():
        Y, T = abt.lr_conv_fwd(act, A, B, kh, kw, stride=stride)
        return (Y, T) + tuple(abt.lr_conv_bwd(dY, act, T, A, B, kh, kw, stride=stride))

    got = step()
    prev = abt.set_chain_rows(64)
    try:
        want = step()
    finally:
        abt.set_chain_rows(prev)
    for name, a, b in zip(("Y", "T", "dAct", "dA", "dB"), got, want):
        assert rel(host(a), host(b)) < TOL_ORDER, name
    assert torch.equal(got[2] == 0, want[2] == 0)
    # dAct itself, in fp32 from the same dT: the sum over taps of shifted products
    dT = (dY.float() @ A.float()).to(BF).float().view(N, -(-H // stride), -(-W // stride), r)
    dAct = torch.nn.functional.conv_transpose2d(dT.permute(0, 3, 1, 2).cpu(), B.float().cpu().view(r, kh, kw, C).permute(0, 3, 1, 2),
                                                stride=stride, padding=(kh // 2, kw // 2),
                                                output_padding=((H - 1) % stride, (W - 1) % stride)).permute(0, 2, 3, 1)
    assert rel(host(got[2]), dAct) < TOL
