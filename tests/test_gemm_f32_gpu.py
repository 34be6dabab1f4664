"""The fp32 matrix product behind the fp32 layer path and ab_reconstruct, at the edges of its tiles
(32 and 64), of its slabs (32 and 64 columns of the contraction), of the 16-byte load path (sizes that
are not multiples of four) and of the split contraction (batches from 512 rows).

Bound: a sum of K products in fp32 in any order is off by at most (K + 2) 2^-24 sum |a| |b| (K roundings of
partial sums, one of the product, one of the output)."""
import pytest

torch = pytest.importorskip("torch")
from paper_2405_01067_amd import binding as abt

pytestmark = pytest.mark.gpu
EPS = 2.0 ** -24


def close(out, a, b):
    """out = a b, a and b fp64 on the GPU."""
    assert bool(torch.isfinite(out).all())
    assert bool(((out.double() - a @ b).abs() <= (a.shape[1] + 2) * EPS * (a.abs() @ b.abs())).all())


def rnd(g, *shape):
    return torch.randn(shape, generator=g, device="cuda")


@pytest.mark.parametrize("m,n,k", [(1, 1, 1), (31, 33, 5), (32, 32, 64), (33, 64, 65), (64, 65, 128), (4, 4, 3), (63, 100, 31),
                                   (130, 68, 36), (1024, 1025, 33), (1023, 1028, 96), (1088, 1024, 192)])
def test_reconstruct_edges(m, n, k):
    g = torch.Generator(device="cuda").manual_seed(m * 7 + n * 3 + k)
    A, B = rnd(g, m, k), rnd(g, k, n)
    close(abt.ab_reconstruct(A, B), A.double(), B.double())


@pytest.mark.parametrize("M,m,n,r", [(1, 24, 36, 8), (5, 33, 7, 3), (64, 256, 256, 32), (63, 66, 130, 34), (511, 64, 68, 32),
                                     (512, 65, 64, 31), (1030, 200, 96, 36), (3152, 768, 192, 96), (2049, 1028, 1024, 64)])
@pytest.mark.parametrize("keep_T,accumulate", [(True, False), (False, True)])
def test_layer_edges(M, m, n, r, keep_T, accumulate):
    g = torch.Generator(device="cuda").manual_seed(M + m + n + r)
    X, dY, A, B = rnd(g, M, n), rnd(g, M, m), rnd(g, m, r), rnd(g, r, n)
    Xd, dYd, Ad, Bd = (t.double() for t in (X, dY, A, B))
    Y, T = abt.lr_linear_fwd(X, A, B, save_T=keep_T)
    dA0, dB0 = rnd(g, m, r), rnd(g, r, n)
    dA, dB = (dA0.clone(), dB0.clone()) if accumulate else (None, None)
    dX, dA, dB = abt.lr_linear_bwd(dY, X, T, A, B, dA=dA, dB=dB, accumulate=accumulate)
    again = abt.lr_linear_bwd(dY, X, T, A, B, dA=dA0.clone() if accumulate else None,
                              dB=dB0.clone() if accumulate else None, accumulate=accumulate)
    for a, b in zip((dX, dA, dB), again):
        assert torch.equal(a, b)                      # fixed order of summation
    if keep_T:
        close(T, Xd, Bd.T)
    # second products: T and dT carry the error of the first ones, bounded through |X| |B|^T and |dY| |A|
    Td, dTd = Xd @ Bd.T, dYd @ Ad
    Tm, dTm = (Xd.abs() @ Bd.abs().T) * (n + 2) * EPS, (dYd.abs() @ Ad.abs()) * (m + 2) * EPS
    for out, a, b, am, bm, base in ((Y, Td, Ad.T, Tm, None, None), (dX, dTd, Bd, dTm, None, None),
                                    (dA, dYd.T, Td, None, Tm, dA0 if accumulate else None),
                                    (dB, dTd.T, Xd, dTm.T, None, dB0 if accumulate else None)):
        ref, mag = a @ b, a.abs() @ b.abs()
        err = (a.shape[1] + 4) * EPS * mag + (am @ b.abs() if am is not None else a.abs() @ bm) * (1 + 1e-3)
        if base is not None:
            ref, err = ref + base.double(), err + 2 * EPS * (base.double().abs() + ref.abs())
        assert bool(torch.isfinite(out).all())
        assert bool(((out.double() - ref).abs() <= err).all())


def test_split_fits_the_static_scratch():
    """A shape whose dT and T alone fill the 64 MiB of lr_linear_bwd_static is still served by it."""
    M, m, n, r = 65536, 32, 36, 128
    g = torch.Generator(device="cuda").manual_seed(3)
    X, dY, A, B = rnd(g, M, n), rnd(g, M, m), rnd(g, m, r), rnd(g, r, n)
    dB = torch.empty_like(B)
    abt.lr_linear_bwd_static(dY, X, None, A, B, dB=dB)
    Xd, dYd, Ad = X.double(), dY.double(), A.double()
    dT, dT_err = dYd @ Ad, (dYd.abs() @ Ad.abs()) * (m + 2) * EPS
    err = (M + 4) * EPS * (dT.abs().T @ Xd.abs()) + (dT_err.T @ Xd.abs()) * (1 + 1e-3)
    assert bool(((dB.double() - dT.T @ Xd).abs() <= err).all())


@pytest.mark.parametrize("M", [24575, 28000, 32767, 32768, 32769])
def test_split_beside_the_static_scratch(M):
    """256 x 256 x 256: up to 24575 rows the partial sums of 32 splits fit the 64 MiB beside dT and T, at 28000 those of
    16, at 32767 none, and 32769 rows do not fit; a caller's workspace always has room for 32."""
    m = n = r = 256
    g = torch.Generator(device="cuda").manual_seed(M)
    X, dY, A, B = rnd(g, M, n), rnd(g, M, m), rnd(g, m, r), rnd(g, r, n)
    dX, dA, dB = abt.lr_linear_bwd(dY, X, None, A, B)
    out = [torch.full_like(t, 7.0) for t in (dX, dA, dB)]
    if M > 32768:
        with pytest.raises(abt.AbtError):
            abt.lr_linear_bwd_static(dY, X, None, A, B, *out)
    else:
        abt.lr_linear_bwd_static(dY, X, None, A, B, *out)
        assert torch.equal(out[0], dX)
        if M <= 24575:
            assert torch.equal(out[1], dA) and torch.equal(out[2], dB)
    Xd, dYd, Ad, Bd = (t.double() for t in (X, dY, A, B))
    T, dT = Xd @ Bd.T, dYd @ Ad
    T_err, dT_err = (Xd.abs() @ Bd.abs().T) * (n + 2) * EPS, (dYd.abs() @ Ad.abs()) * (m + 2) * EPS
    for got in ((dA, dB), out[1:]) if M <= 32768 else ((dA, dB),):
        for o, a, b, err in ((got[0], dYd, T, dYd.abs().T @ T_err), (got[1], dT, Xd, dT_err.T @ Xd.abs())):
            bound = (M + 4) * EPS * (a.abs().T @ b.abs()) + err * (1 + 1e-3)
            assert bool(((o.double() - a.T @ b).abs() <= bound).all())


# T and dT with a split contraction: one to 3152 rows, tiles of either size, contractions that are not multiples of 4, 64 or the splits, both split, and
# where the static scratch has no room for all of the partial sums of dT (16385 rows: of two of four)
@pytest.mark.parametrize("M,m,n,r", [(1, 1024, 64, 32), (65, 3071, 96, 33), (800, 2304, 1500, 64), (3152, 3072, 64, 192), (3152, 2304, 64, 384), (16385, 3072, 64, 255)])
def test_split_products_of_the_rows(M, m, n, r):
    g = torch.Generator(device="cuda").manual_seed(M + m + n + r)
    X, dY, A, B = rnd(g, M, n), rnd(g, M, m), rnd(g, m, r), rnd(g, r, n)
    dX, dA, dB = abt.lr_linear_bwd(dY, X, None, A, B)
    out = [torch.full_like(t, 7.0) for t in (dX, dA, dB)]
    abt.lr_linear_bwd_static(dY, X, None, A, B, *out)
    Xd, dYd, Ad, Bd = (t.double() for t in (X, dY, A, B))
    T, dT = Xd @ Bd.T, dYd @ Ad
    T_err, dT_err = (Xd.abs() @ Bd.abs().T) * (n + 2) * EPS, (dYd.abs() @ Ad.abs()) * (m + 2) * EPS
    for got in ((dX, dA, dB), out):
        for o, a, b, err in ((got[0], dT, Bd, dT_err @ Bd.abs()), (got[1], dYd.T, T, dYd.abs().T @ T_err), (got[2], dT.T, Xd, dT_err.T @ Xd.abs())):
            assert bool(((o.double() - a @ b).abs() <= (a.shape[1] + 4) * EPS * (a.abs() @ b.abs()) + err * (1 + 1e-3)).all())


# one launch each way: blocks of 32 rows, 128 columns of the widths, chunks of 256 of the contraction, widths that are not multiples of four, and
# the sizes next to its limits
@pytest.mark.parametrize("M,m,n,r", [(1, 1, 1, 1), (31, 127, 129, 32), (32, 512, 511, 5), (33, 256, 512, 32), (64, 255, 257, 31), (64, 257, 256, 32),
                                     (64, 512, 512, 32), (65, 256, 256, 32), (64, 256, 513, 32), (64, 256, 256, 33)])
@pytest.mark.parametrize("accumulate", [False, True])
def test_smallest_layers(M, m, n, r, accumulate):
    g = torch.Generator(device="cuda").manual_seed(M + m + n + r)
    X, dY, A, B = rnd(g, M, n), rnd(g, M, m), rnd(g, m, r), rnd(g, r, n)
    Xd, dYd, Ad, Bd = (t.double() for t in (X, dY, A, B))
    Y, T = abt.lr_linear_fwd(X, A, B)
    close(T, Xd, Bd.T), close(Y, T.double(), Ad.T)        # of the T that was kept, Y is one product
    assert torch.equal(abt.lr_linear_fwd(X, A, B, save_T=False)[0], Y)
    dA0, dB0 = rnd(g, m, r), rnd(g, r, n)
    run = lambda **kw: abt.lr_linear_bwd(dY, X, T, A, B, accumulate=accumulate, **{
        k: v.clone() for k, v in (("dA", dA0), ("dB", dB0)) if accumulate and kw.get("need_" + k, True)}, **kw)
    dX, dA, dB = run()
    base = lambda out, b: out - b if accumulate else out
    slack = lambda b: 4 * EPS * b.double().abs() if accumulate else 0.0
    assert bool(((base(dA, dA0).double() - dYd.T @ T.double()).abs() <= (M + 3) * EPS * (dYd.abs().T @ T.double().abs()) + slack(dA0)).all())
    # dT carries (m + 2) EPS |dY| |A|, which the products that follow pass on
    dT, mag = dYd @ Ad, dYd.abs() @ Ad.abs()
    bound = lambda a, b, K: ((m + 2) + (K + 4)) * EPS * (a @ b) * 1.001
    assert bool(((dX.double() - dT @ Bd).abs() <= bound(mag, Bd.abs(), r)).all())
    assert bool(((base(dB, dB0).double() - dT.T @ Xd).abs() <= bound(mag.T, Xd.abs(), M) + slack(dB0)).all())
    # the same bits whatever else is asked for
    for which in ((True, False, True), (False, True, False), (False, False, True), (True, False, False)):
        for a, b, w in zip(run(need_dX=which[0], need_dA=which[1], need_dB=which[2]), (dX, dA, dB), which):
            assert torch.equal(a, b) if w else a is None


# T again is the T of the forward, bit for bit, whatever is asked for with it: one launch each way, tiles of either size alone and beside dT, a
# contraction that is long against the rows
@pytest.mark.parametrize("M,m,n,r", [(64, 256, 256, 32), (33, 130, 511, 7), (64, 512, 512, 32), (100, 64, 1024, 32), (800, 64, 3072, 64), (3152, 3072, 768, 192),
                                     (3152, 768, 2304, 384), (1030, 200, 96, 36), (300, 131, 512, 36)])
def test_T_again_is_the_T_of_the_forward(M, m, n, r):
    g = torch.Generator(device="cuda").manual_seed(M + m + n + r)
    X, dY, A, B = rnd(g, M, n), rnd(g, M, m), rnd(g, m, r), rnd(g, r, n)
    T = abt.lr_linear_fwd(X, A, B)[1]
    # (rows of dY with a single one: dA is then rows of T, whose sum has one term)
    pick = torch.zeros_like(dY)
    rows = torch.randperm(M, generator=g, device="cuda")[:m]
    pick[rows, torch.arange(len(rows), device="cuda")] = 1.0
    for kw in ({"need_dX": False, "need_dB": False}, {"need_dX": False}, {}):
        dA = abt.lr_linear_bwd(pick, X, None, A, B, **kw)[1]
        assert torch.equal(dA[:len(rows)], T[rows])
    if M <= 64 and m <= 512 and n <= 512 and r <= 32:     # and nothing else depends on whether it was kept
        for a, b in zip(abt.lr_linear_bwd(dY, X, None, A, B), abt.lr_linear_bwd(dY, X, T, A, B)):
            assert torch.equal(a, b)


# dX is that of lr_linear_bwd: dT is split no further than the static scratch has room for the parts
def test_static_scratch_gives_the_same_dX():
    M, m, n, r = 16385, 3072, 64, 255
    g = torch.Generator(device="cuda").manual_seed(M)
    X, dY, A, B = rnd(g, M, n), rnd(g, M, m), rnd(g, m, r), rnd(g, r, n)
    dX, out = abt.lr_linear_bwd(dY, X, None, A, B)[0], torch.empty_like(X)
    abt.lr_linear_bwd_static(dY, X, None, A, B, dX=out)
    assert torch.equal(out, dX)


# one tile per work-group and several: tiles on both sides of three and of four work-groups per compute unit, one slab to many, ragged edges
@pytest.mark.parametrize("m,n,k", [(1664, 1664, 32), (1700, 1820, 64), (2048, 2048, 96), (2049, 2052, 32), (3150, 3068, 192), (64 * 257, 64, 160), (64 * 300 + 4, 4, 320),
                                   (4100, 4, 320)])       # (the last one has too few tiles: 32 x 32)
def test_work_groups_that_stay(m, n, k):
    g = torch.Generator().manual_seed(m + k)
    A, B = torch.randn((m, k), generator=g).to("cuda:0"), torch.randn((k, n), generator=g).to("cuda:0")
    W = abt.ab_reconstruct(A, B)
    want = A.double() @ B.double()
    # k products and their sum in fp32, each rounded once: k 2^-24 of the sum of their magnitudes at most
    bound = (k + 1) * 2.0 ** -24 * (A.double().abs() @ B.double().abs())
    assert bool(((W.double() - want).abs() <= bound).all())


# three unlike problems in a launch, two of them split, added to what is there; an odd number of slabs, ragged edges of the outputs
@pytest.mark.parametrize("M,m,n,r", [(3136, 1024, 512, 192), (2016, 1472, 1984, 64), (3168, 1028, 516, 96),
                                       (2000, 1472, 1984, 64)])       # (the last one's rows are no whole slabs: one tile after the other)
def test_gradients_by_work_groups_that_stay(M, m, n, r):
    g = torch.Generator().manual_seed(M + r)
    make = lambda *s: torch.randn(s, generator=g).to("cuda:0")
    X, dY, A, B = make(M, n), make(M, m), make(m, r), make(r, n)
    T = abt.lr_linear_fwd(X, A, B)[1]
    dA, dB = torch.ones_like(A), torch.ones_like(B)
    dX, _, _ = abt.lr_linear_bwd(dY, X, T, A, B, dA=dA, dB=dB, accumulate=True)
    d = lambda t: t.double()
    dT = d(dY) @ d(A)
    for got, want in ((dX, dT @ d(B)), (dA - 1, d(dY).T @ d(T)), (dB - 1, dT.T @ d(X))):
        # sums of up to 3136 products, rounded some sqrt(3136) 2^-24 in the norm, dT once before
        assert float((d(got) - want).norm() / want.norm()) < 6e-6
