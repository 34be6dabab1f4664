"""Outputs that lie over inputs which the call has finished with: the results are those of separate buffers, bit for
bit (the order of the sums does not depend on where a result goes)."""
import pytest
import torch

from paper_2405_01067_amd import binding as abt

pytestmark = pytest.mark.gpu

BF = torch.bfloat16


def rnd(seed, *shape, dtype=BF, std=1.0):
    g = torch.Generator(device="cuda").manual_seed(seed)
    return (torch.randn(shape, generator=g, device="cuda") * std).to(dtype)


def over(t, shape):
    """An fp32 tensor of this shape at the start of t's memory."""
    return t.view(-1).view(torch.float32)[:shape[0] * shape[1]].view(shape)


@pytest.mark.parametrize("M,m,n,r", [(64, 1024, 64, 32), (192, 64, 1920, 32), (500, 1024, 1024, 96)])
def test_factor_gradient_over_an_activation(M, m, n, r):
    # fewer than 1024 rows: one split, whose sums are the result
    X, dY, A, B = rnd(1, M, n), rnd(2, M, m, std=1e-2), rnd(3, m, r, std=r ** -0.5), rnd(4, r, n, std=n ** -0.5)
    T = abt.lr_linear_fwd(X, A, B)[1]
    for what, src in (("dA", dY), ("dB", X)):
        shape = (m, r) if what == "dA" else (r, n)
        if shape[0] * shape[1] * 4 > src.numel() * 2:
            continue
        kw = dict(need_dX=False, need_dA=what == "dA", need_dB=what == "dB")
        want = abt.lr_linear_bwd(dY, X, T, A, B, **kw)
        buf = src.clone()
        args = (buf, X) if what == "dA" else (dY, buf)
        got = abt.lr_linear_bwd(*args, T, A, B, **kw, **{what: over(buf, shape)})
        i = 1 if what == "dA" else 2
        assert torch.equal(got[i], want[i]), what


def test_convolution_gradient_over_the_activation():
    N, side, C, m, r = 4, 14, 128, 64, 32
    act, dY, A, B = rnd(5, N, side, side, C), rnd(6, N * side * side, m, std=1e-2), rnd(7, m, r), rnd(8, r, 9 * C, std=0.03)
    T = abt.lr_conv_fwd(act, A, B, 3, 3)[1]
    kw = dict(need_dAct=False, need_dA=False)
    want = abt.lr_conv_bwd(dY, act, T, A, B, 3, 3, **kw)[2]
    buf = act.clone()
    got = abt.lr_conv_bwd(dY, buf, T, A, B, 3, 3, dB=over(buf, (r, 9 * C)), **kw)[2]
    assert torch.equal(got, want)


def near(a, b, terms=2000):
    # The same fp32 products in a launch of another tile form.  Sums of up to `terms` products in another order: the
    # roundings of the partial sums walk at random, sqrt(terms) 2^-24 in norm per product; two products and both sides: 4.
    assert float((a - b).norm() / b.norm()) < 4 * terms ** 0.5 * 2.0 ** -24


@pytest.mark.parametrize("M,m,n,r", [(64, 256, 256, 32), (300, 130, 130, 20), (2000, 256, 256, 32)])
def test_fp32_backward_over_its_inputs(M, m, n, r):
    f32 = torch.float32
    X, dY, A, B = rnd(1, M, n, dtype=f32), rnd(2, M, m, dtype=f32), rnd(3, m, r, dtype=f32), rnd(4, r, n, dtype=f32)
    T = abt.lr_linear_fwd(X, A, B)[1]
    want = abt.lr_linear_bwd(dY, X, T, A, B)
    # dB over B: dX is computed from B first; and added to it in place, a step of plain descent
    Bc = B.clone()
    got = abt.lr_linear_bwd(dY, X, T, A, Bc, dB=Bc)
    near(got[0], want[0]), near(got[1], want[1]), near(Bc, want[2])
    Bc = B.clone()
    near(abt.lr_linear_bwd(dY, X, T, A, Bc, dB=Bc, accumulate=True, need_dA=False)[0], want[0])
    near(Bc, B + want[2])
    # dA over A, dX over dY (no dA) and over X (no dB)
    Ac = A.clone()
    got = abt.lr_linear_bwd(dY, X, T, Ac, B, dA=Ac)
    near(got[0], want[0]), near(Ac, want[1]), near(got[2], want[2])
    d = dY.clone()
    got = abt.lr_linear_bwd(d, X, T, A, B, dX=d, need_dA=False)
    near(d, want[0]), near(got[2], want[2])
    x = X.clone()
    got = abt.lr_linear_bwd(dY, x, T, A, B, dX=x, need_dB=False)
    near(x, want[0]), near(got[1], want[1])


def close16(a, b):
    # bf16 results of the same products summed in fp32 in another order: T and the result differ by single roundings
    # of a few entries, below 2^-8 in norm
    assert float((a.double() - b.double()).norm() / b.double().norm()) < 2.0 ** -8


@pytest.mark.parametrize("M", [40, 700, 8192])
@pytest.mark.parametrize("m,r", [(128, 32), (768, 96)])
def test_layer_in_place(M, m, r):
    # up to 8192 rows several work-groups share a row block; not when the block's input is overwritten
    X, dY, A, B = rnd(1, M, m), rnd(2, M, m, std=1e-2), rnd(3, m, r, std=r ** -0.5), rnd(4, r, m, std=m ** -0.5)
    Y, T = abt.lr_linear_fwd(X, A, B)
    x = X.clone()
    close16(abt.lr_linear_fwd(x, A, B, Y=x, save_T=False)[0], Y)
    xs = [X.clone(), X.clone()]
    for (y, t) in abt.lr_linear_fwd_grouped([dict(X=x, Y=x, A=A, B=B) for x in xs]):
        close16(y, Y), close16(t, T)
    want = abt.lr_linear_bwd(dY, X, T, A, B, need_dA=False)
    d = dY.clone()
    got = abt.lr_linear_bwd(d, X, T, A, B, need_dA=False, dX=d)
    close16(d, want[0]), close16(got[2], want[2])


def test_saved_product_over_the_input():
    M, m, r = 700, 1024, 64                      # T and X have the same shape
    X, A, B = rnd(1, M, r), rnd(2, m, r, std=r ** -0.5), rnd(3, r, r, std=r ** -0.5)
    Y, T = abt.lr_linear_fwd(X, A, B)
    x = X.clone()
    y, t = abt.lr_linear_fwd(x, A, B, T=x)
    close16(y, Y), close16(t, T)
