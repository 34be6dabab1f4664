"""The native code of the single-layer calls: what it takes gives the bits of the Python path, and what it leaves to it
is answered or refused as there (a workspace in the arguments is one of those, which gives the test its other side)."""
import pytest
import torch

from paper_2405_01067_amd import binding as abt

pytestmark = pytest.mark.gpu


def layer(dtype, M=70, m=128, n=64, r=32, seed=0):
    g = torch.Generator().manual_seed(seed)
    make = lambda *s: torch.randn(s, generator=g).to("cuda:0").to(dtype)
    return make(M, m), make(M, n), make(m, r), make(r, n)


def workspace():
    return torch.empty(1 << 22, dtype=torch.uint8, device="cuda:0")


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("M", [1, 70, 5000])
def test_same_bits_as_the_python_path(dtype, M):
    dY, X, A, B = layer(dtype, M)
    for save in (True, False):
        got, want = abt.lr_linear_fwd(X, A, B, save_T=save), abt.lr_linear_fwd(X, A, B, save_T=save, workspace=workspace())
        assert torch.equal(got[0], want[0]) and ((got[1] is None and want[1] is None) if not save else torch.equal(got[1], want[1]))
    T = got[1] if got[1] is not None else abt.lr_linear_fwd(X, A, B)[1]
    for kw in ({}, {"need_dX": False}, {"need_dA": False}, {"need_dB": False, "need_dA": False}):
        for t in (T, None):
            got, want = abt.lr_linear_bwd(dY, X, t, A, B, **kw), abt.lr_linear_bwd(dY, X, t, A, B, workspace=workspace(), **kw)
            for a, b in zip(got, want):
                assert (a is None) == (b is None) and (a is None or (torch.equal(a, b) and a.dtype == b.dtype and not a.requires_grad))


def test_results_in_tensors_of_the_caller():
    dY, X, A, B = layer(torch.float32)
    T = abt.lr_linear_fwd(X, A, B)[1]
    dA, dB, dX = torch.ones_like(A), torch.ones_like(B), torch.empty_like(X)
    got = abt.lr_linear_bwd(dY, X, T, A, B, dX=dX, dA=dA, dB=dB, accumulate=True)
    assert got[0] is dX and got[1] is dA and got[2] is dB
    want = abt.lr_linear_bwd(dY, X, T, A, B)
    assert torch.equal(dX, want[0])
    # ones added to sums of 70 products: half an ulp of the total each
    assert float((dA - 1 - want[1]).abs().max()) < 1e-4 and float((dB - 1 - want[2]).abs().max()) < 1e-4
    assert abt.lr_linear_bwd(dY, X, T, A, B, need_dX=False, dX=dX)[0] is None
    P = torch.nn.Parameter(A)
    y = abt.lr_linear_fwd(X, P, B)[0]
    assert not y.requires_grad and torch.equal(y, abt.lr_linear_fwd(X, A, B)[0])


def test_refused_as_before():
    dY, X, A, B = layer(torch.float32)
    T = abt.lr_linear_fwd(X, A, B)[1]
    with pytest.raises(abt.AbtError, match="contiguous"):
        abt.lr_linear_fwd(X.T.contiguous().T, A, B)
    with pytest.raises(abt.AbtError, match="on the GPU"):
        abt.lr_linear_fwd(X.cpu(), A, B)
    with pytest.raises(abt.AbtError, match="shape/dtype"):
        abt.lr_linear_fwd(X, A, B.bfloat16())
    with pytest.raises(abt.AbtError, match="unsupported dtype"):
        abt.lr_linear_fwd(X.double(), A.double(), B.double())
    with pytest.raises(abt.AbtError, match="ABT_ESHAPE"):
        abt.lr_linear_fwd(X.bfloat16()[:, :63].contiguous(), A.bfloat16(), B.bfloat16()[:, :63].contiguous())
    with pytest.raises(abt.AbtError, match="needs existing dA"):
        abt.lr_linear_bwd(dY, X, T, A, B, accumulate=True)
    with pytest.raises(abt.AbtError, match="dA must be"):
        abt.lr_linear_bwd(dY, X, T, A, B, dA=A.double())
    with pytest.raises(abt.AbtError, match="T must be"):
        abt.lr_linear_bwd(dY, X, T[:-1], A, B)
    with pytest.raises(RuntimeError):                    # a batched tensor has no memory of its own
        torch.func.vmap(lambda x: abt.lr_linear_fwd(x, A, B)[0])(X.view(2, 35, 64))


def test_what_torch_refuses_is_refused_before_the_launch():
    dY, X, A, B = layer(torch.float32)
    T = abt.lr_linear_fwd(X, A, B)[1]
    dA, dB = torch.ones_like(A), torch.ones_like(B)
    torch._C._set_throw_on_mutable_data_ptr(dB)          # an address that may not be asked for
    with pytest.raises(RuntimeError):
        abt.lr_linear_bwd(dY, X, T, A, B, dA=dA, dB=dB, accumulate=True)
    torch.cuda.synchronize()
    assert bool((dA == 1).all())                         # nothing was added, once or twice
    Z = X.clone()
    torch._C._set_throw_on_mutable_data_ptr(Z)
    with pytest.raises(RuntimeError):
        abt.lr_linear_fwd(Z, A, B)


def test_allocations_of_a_mode_are_seen_by_it():
    from torch.utils._python_dispatch import TorchDispatchMode
    _, X, A, B = layer(torch.float32)
    seen = []

    class Watch(TorchDispatchMode):
        def __torch_dispatch__(self, func, types, args=(), kwargs=None):
            seen.append(str(func))
            return func(*args, **(kwargs or {}))

    want = abt.lr_linear_fwd(X, A, B)
    with Watch():
        got = abt.lr_linear_fwd(X, A, B)
    assert any("empty" in f for f in seen) and torch.equal(got[0], want[0])


def test_runs_on_the_current_stream_and_in_a_capture():
    dY, X, A, B = layer(torch.bfloat16, 300)
    want = abt.lr_linear_fwd(X, A, B)
    torch.cuda.synchronize()
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        X2 = X * 1                                       # on s: a call on another stream could read it unfinished
        got = abt.lr_linear_fwd(X2, A, B)
    s.synchronize()
    assert torch.equal(got[0], want[0])
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        Y, T = abt.lr_linear_fwd(X, A, B)
        grads = abt.lr_linear_bwd(dY, X, T, A, B)
    first = abt.lr_linear_bwd(dY, X, want[1], A, B)
    for _ in range(3):
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(Y, want[0]) and all(torch.equal(a, b) for a, b in zip(grads, first))
        Y.zero_()
