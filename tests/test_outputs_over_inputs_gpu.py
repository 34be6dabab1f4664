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
