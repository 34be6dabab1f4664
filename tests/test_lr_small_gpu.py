"""The backward kernels for few rows at the edges of their tiles (32 rows, 64 columns of the rank and of the factors), of the
contraction that eight waves share, and of the rule that takes them (2048 or 4096 rows), against fp64.

Tolerance: bf16 has eight significant bits, so a value is off by 2^-8 of itself at most after one rounding: dB carries that of dT, dX
that of dT and its own; dA only carries fp32 sums of exact products, (M + 1) 2^-24 of the sum of their sizes at most."""
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
