"""The two products for many rows at the edges of what their work-groups take (8 to 256 rows, 256 columns, ranks that are padded to the
next 64), of the rows where another split of the contraction begins (64 and 128 per work-group) and of the rule that takes them, against fp64.

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


# rows per work-group: 32 (the least), 64, more in one round; a last work-group of one row, of all; one and two rounds of the compute units;
# a result of 256 columns and one more block, of half a block of columns; an odd and an even number of slabs
@pytest.mark.parametrize("M,m,n,r", [(4609, 1344, 320, 96), (6000, 1088, 1920, 192), (8192, 1344, 256, 128), (10239, 1408, 256, 288), (10240, 1344, 640, 64),
                                     (10241, 2304, 256, 160), (12800, 2304, 1152, 192),
                                     (12345, 128, 1152, 288), (16384, 1024, 256, 352), (16385, 1344, 512, 224), (17001, 512, 960, 160),
                                     (20000, 1344, 512, 256), (22528, 1344, 256, 384), (32769, 448, 256, 320), (33333, 2304, 256, 64),
                                     (40000, 1088, 256, 128), (40960, 512, 768, 96), (49152, 128, 768, 384), (50433, 768, 768, 384), (65537, 768, 832, 160)])
def test_two_products_of_many_rows(M, m, n, r):
    X, A, B, dY = layer(M, m, n, r)
    assert abt.load().lr_linear_fwd_wants_T(1, M, m, n, r, abt.ABT_BF16) == 1
    Y, T = abt.lr_linear_fwd(X, A, B)
    assert rel(T, X.double() @ B.double().T) < 2 ** -8 and rel(Y, T.double() @ A.double().T) < 2 ** -8
    # without T, and with T again for the factor gradient: the same bits; with no place for T the fused kernel
    assert torch.equal(abt.lr_linear_fwd(X, A, B, save_T=False)[0], Y)
    kept, again = (abt.lr_linear_bwd(dY, X, t, A, B, need_dX=False, need_dB=False)[1] for t in (T, None))
    assert torch.equal(kept, again)
    # the backward: the same dT with dX and without
    dX, dA, dB = abt.lr_linear_bwd(dY, X, T, A, B)
    dT = dY.double() @ A.double()
    assert rel(dX, dT @ B.double()) < 2 ** -7 and rel(dB, dT.T @ X.double()) < 2 ** -8
    assert torch.equal(abt.lr_linear_bwd(dY, X, T, A, B, need_dX=False)[2], dB)


@pytest.mark.parametrize("G,M,m,n,r", [(2, 2310, 1344, 1344, 96), (3, 11000, 1344, 512, 192), (4, 8200, 448, 256, 352), (8, 5000, 768, 768, 160)])
def test_groups_of_many_rows_together(G, M, m, n, r):
    layers = [layer(M + g, m, n, r) for g in range(G)]
    groups = [dict(X=X[:M], A=A, B=B) for X, A, B, _ in layers]
    assert abt.load().lr_linear_fwd_wants_T(G, M, m, n, r, abt.ABT_BF16) == 1
    outs = abt.lr_linear_fwd_grouped(groups)
    for g, (Y, T) in zip(groups, outs):
        assert rel(T, g["X"].double() @ g["B"].double().T) < 2 ** -8 and rel(Y, T.double() @ g["A"].double().T) < 2 ** -8
    for (Y, _), (Y2, _) in zip(outs, abt.lr_linear_fwd_grouped(groups, save_T=False)):
        assert torch.equal(Y, Y2)
    # (shapes whose backward is in the rule too) dT of some of the groups alone, and T again for some: the order of the sums is that of the whole call
    every = [dict(g, dY=l[3][:M], T=o[1], dX=True, dB=True) for g, l, o in zip(groups, layers, outs)]
    full = abt.lr_linear_bwd_grouped(every)
    some = [dict(e, dX=True if i else None) for i, e in enumerate(every)]
    for a, b in zip(full, abt.lr_linear_bwd_grouped(some)):
        assert torch.equal(a[2], b[2])
    grad = lambda keep: abt.lr_linear_bwd_grouped([dict(X=e["X"], A=e["A"], B=e["B"], dY=e["dY"], T=e["T"] if keep(i) else None, dA=True) for i, e in enumerate(every)])
    for a, b in zip(grad(lambda i: True), grad(lambda i: i == 0)):
        assert torch.equal(a[1], b[1])


def test_a_result_over_its_input_and_rows_that_are_not_finite():
    M, m, r = 33001, 768, 224                             # padded to 256 columns of T
    X, A, B, _ = layer(M, m, m, r)
    Y = abt.lr_linear_fwd(X, A, B)[0]
    over = X.clone()
    assert torch.equal(abt.lr_linear_fwd(over, A, B, Y=over)[0], Y)
    X[M - 1, 5] = float("inf")
    Y2, T2 = abt.lr_linear_fwd(X, A, B)
    assert torch.equal(Y2[:-1], Y[:-1]) and bool(torch.isinf(T2[-1]).all()) and not bool(torch.isfinite(Y2[-1]).any())
