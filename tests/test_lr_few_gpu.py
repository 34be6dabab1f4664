"""The forward of a few rows in one launch, at the edges of its work-groups (32 rows, 256 or 128 columns, contractions of fewer pieces than waves and with
a remainder) and of the rule that takes it, against fp64.

Tolerance: bf16 has eight significant bits, so a value is off by 2^-8 of itself at most after one rounding."""
import pytest

torch = pytest.importorskip("torch")
from paper_2405_01067_amd import binding as abt

pytestmark = pytest.mark.gpu
BF = torch.bfloat16


def rel(a, b):
    return float((a.double() - b).norm() / b.norm())


def layer(M, m, n, r):
    g = torch.Generator(device="cuda").manual_seed(M + m + n + r)
    rn = lambda std, *s: (torch.randn(s, generator=g, device="cuda") * std).to(BF)
    return rn(1, M, n), rn(r ** -0.5, m, r), rn(n ** -0.5, r, n), rn(1e-2, M, m)


@pytest.mark.parametrize("M,m,n,r", [(1, 64, 64, 32), (31, 320, 128, 64), (32, 256, 320, 96), (33, 192, 64, 128), (197, 2304, 768, 96), (100, 1088, 896, 160),
                                     (65, 64, 704, 192), (4096, 512, 3072, 96), (4096, 960, 64, 32), (4096, 1088, 64, 32), (4095, 256, 1088, 128),
                                     (2048, 1024, 3072, 64), (2049, 1024, 3072, 64), (4097, 64, 64, 64), (130, 64, 3136, 32)])
def test_one_launch(M, m, n, r):
    X, A, B, dY = layer(M, m, n, r)
    Y, T = abt.lr_linear_fwd(X, A, B)
    assert rel(T, X.double() @ B.double().T) < 2 ** -8 and rel(Y, T.double() @ A.double().T) < 2 ** -8
    assert torch.equal(abt.lr_linear_fwd(X, A, B, save_T=False)[0], Y)
    Yg, Tg = abt.lr_linear_fwd_grouped([dict(X=X, A=A, B=B)])[0]
    assert torch.equal(Yg, Y) and torch.equal(Tg, T)
    # T again for the factor gradient: the same bits
    kept, again = (abt.lr_linear_bwd(dY, X, t, A, B, need_dX=False, need_dB=False)[1] for t in (T, None))
    assert torch.equal(kept, again)


@pytest.mark.parametrize("r", [96, 128])
def test_outputs_over_inputs_and_rows_that_are_not_finite(r):
    M, n = 70, 576
    X, A, B, _ = layer(M, n, n, r)
    Y, T = abt.lr_linear_fwd(X, A, B)
    over = X.clone()
    assert rel(abt.lr_linear_fwd(over, A, B, Y=over)[0], Y.double()) < 2 ** -7
    X[M - 1, 5] = float("inf")
    Y2, T2 = abt.lr_linear_fwd(X, A, B)
    assert torch.equal(Y2[:-1], Y[:-1]) and bool(torch.isinf(T2[-1]).all()) and not bool(torch.isfinite(Y2[-1]).any())


@pytest.mark.parametrize("G,M,m,n,r", [(2, 33, 512, 320, 96), (8, 65, 640, 192, 32), (3, 100, 320, 768, 128), (4, 197, 2304, 768, 96), (5, 197, 2304, 768, 96)])
def test_groups_in_one_launch(G, M, m, n, r):
    layers = [layer(M, m, n, r) for _ in range(G)]
    groups = [dict(X=X + g, A=A, B=B) for g, (X, A, B, _) in enumerate(layers)]
    outs = abt.lr_linear_fwd_grouped(groups)
    for e, (Y, T) in zip(groups, outs):
        assert rel(T, e["X"].double() @ e["B"].double().T) < 2 ** -8 and rel(Y, T.double() @ e["A"].double().T) < 2 ** -8
    for (Y, _), (Y2, _) in zip(outs, abt.lr_linear_fwd_grouped(groups, save_T=False)):
        assert torch.equal(Y, Y2)
    grad = lambda keep: abt.lr_linear_bwd_grouped([dict(e, dY=l[3], T=o[1] if keep(i) else None, dA=True) for i, (e, l, o) in enumerate(zip(groups, layers, outs))])
    for a, b in zip(grad(lambda i: True), grad(lambda i: i == 0)):
        assert torch.equal(a[1], b[1])


def patches(act, w, stride):
    N, H, W, C = act.shape
    h = w // 2
    pad = torch.nn.functional.pad(act.double(), (0, 0, h, h, h, h))
    cols = [pad[:, ky:ky + H:stride, kx:kx + W:stride] for ky in range(w) for kx in range(w)]
    return torch.cat(cols, 3).reshape(-1, w * w * C)


# one row to whole images of rows, odd sides, both strides, a row block over several images, all numbers of waves
@pytest.mark.parametrize("N,H,W,C,m,r,w,stride", [(1, 1, 1, 64, 64, 32, 3, 1), (3, 7, 5, 128, 192, 64, 3, 1), (2, 9, 8, 64, 320, 96, 3, 2), (5, 3, 2, 64, 64, 160, 3, 1),
                                                  (7, 6, 13, 256, 128, 32, 1, 2), (4, 28, 28, 64, 64, 64, 3, 1), (1, 15, 29, 64, 256, 192, 3, 2)])
def test_convolution_in_one_launch(N, H, W, C, m, r, w, stride):
    g = torch.Generator(device="cuda").manual_seed(N + H + C + r)
    rn = lambda std, *s: (torch.randn(s, generator=g, device="cuda") * std).to(BF)
    act, A, B = rn(1, N, H, W, C), rn(r ** -0.5, m, r), rn((w * w * C) ** -0.5, r, w * w * C)
    Y, T = abt.lr_conv_fwd(act, A, B, w, w, stride=stride)
    X = patches(act, w, stride)
    assert rel(T, X @ B.double().T) < 2 ** -8 and rel(Y, T.double() @ A.double().T) < 2 ** -8
    assert torch.equal(abt.lr_conv_fwd(act, A, B, w, w, stride=stride, save_T=False)[0], Y)
    dY = rn(1e-2, Y.shape[0], m)
    kept, again = (abt.lr_conv_bwd(dY, act, t, A, B, w, w, stride=stride)[1] for t in (T, None))
    assert torch.equal(kept, again)
