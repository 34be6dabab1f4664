"""Forwards that do not keep T, of few rows above all: the same results as with T kept, whatever was asked before, and nothing
written but the outputs."""
import pytest

torch = pytest.importorskip("torch")
from paper_2405_01067_amd import binding as abt

pytestmark = pytest.mark.gpu
BF = torch.bfloat16


def layer(M, m, n, r, seed=0):
    g = torch.Generator(device="cuda").manual_seed(seed)
    rn = lambda std, *s: (torch.randn(s, generator=g, device="cuda") * std).to(BF)
    return rn(1, M, n), rn(r ** -0.5, m, r), rn(n ** -0.5, r, n), rn(1e-2, M, m)


def test_a_shape_first_seen_under_a_forced_height():
    X, A, B, _ = layer(199, 2304, 768, 384)
    prev = abt.set_chain_rows(64)
    try:
        abt.lr_linear_fwd(X, A, B, save_T=False)
    finally:
        abt.set_chain_rows(prev)
    assert torch.equal(abt.lr_linear_fwd(X, A, B, save_T=False)[0], abt.lr_linear_fwd(X, A, B)[0])


@pytest.mark.parametrize("dtype", [BF, torch.float32])
def test_a_kept_T_needs_no_workspace(dtype):
    X, A, B, _ = (t.to(dtype) for t in layer(201, 2304, 768, 192))
    small = torch.empty(1, dtype=torch.uint8, device="cuda")
    Y, T = abt.lr_linear_fwd(X, A, B, workspace=small if dtype == BF else None)
    if dtype == torch.float32:                           # one that is named has to hold T there
        with pytest.raises(abt.AbtError):
            abt.lr_linear_fwd(X, A, B, workspace=small)
    taken = lambda: torch.cuda.memory_stats()["allocation.all.allocated"]
    before = taken()
    again = abt.lr_linear_fwd(X, A, B)
    assert taken() == before + 2                         # Y and T
    assert torch.equal(again[0], Y) and torch.equal(again[1], T)


def test_a_forward_leaves_the_workspace_alone():
    # one workspace may serve forwards on several streams: nothing of a bf16 forward is kept there
    M, m, n, r = 203, 2304, 768, 192
    X, A, B, _ = layer(M, m, n, r)
    lib = abt.load()
    assert lib.lr_linear_fwd_workspace_bytes(M, m, n, r, abt.ABT_BF16) == 0
    ws = torch.full((M * r * 4,), 85, dtype=torch.uint8, device="cuda")
    want = abt.lr_linear_fwd(X, A, B)[0]
    assert torch.equal(abt.lr_linear_fwd(X, A, B, save_T=False, workspace=ws)[0], want) and bool((ws == 85).all())
    assert torch.equal(abt.lr_linear_fwd(X, A, B, save_T=False, workspace=ws[:1])[0], want)
    Y = torch.empty_like(want)
    assert lib.lr_linear_fwd(X.data_ptr(), A.data_ptr(), B.data_ptr(), Y.data_ptr(), None, M, m, n, r, abt.ABT_BF16,
                             ws.data_ptr(), ws.numel(), torch.cuda.current_stream().cuda_stream) == 0
    assert bool((ws == 85).all())
    assert float((Y.double() - want.double()).norm() / want.double().norm()) < 2 ** -7       # T and Y rounded once each


# products of M rows below the rule of two launches, of G M rows above it, and shapes on one side with both
@pytest.mark.parametrize("G,M,m,n,r", [(4, 500, 640, 768, 128), (8, 260, 2304, 768, 96), (3, 700, 1024, 960, 96), (2, 40, 64, 64, 32), (5, 300, 768, 768, 352)])
def test_groups_without_T(G, M, m, n, r):
    groups = [dict(zip("XAB", layer(M, m, n, r, seed=g))) for g in range(G)]
    kept = abt.lr_linear_fwd_grouped(groups)
    for (Y, T), (Yk, _) in zip(abt.lr_linear_fwd_grouped(groups, save_T=False), kept):
        assert T is None and torch.equal(Y, Yk)


# the two-product rule of the image and of the matrix (1 x 1), and shapes below it
@pytest.mark.parametrize("N,H,W,C,kh,kw,stride,m,r", [(2, 14, 14, 256, 3, 3, 1, 256, 256), (1, 28, 28, 128, 3, 3, 2, 64, 192), (4, 7, 7, 2048, 1, 1, 1, 512, 128),
                                                      (3, 14, 13, 1024, 1, 1, 2, 64, 384), (2, 6, 5, 64, 3, 3, 1, 64, 32)])
def test_convolution_without_T(N, H, W, C, kh, kw, stride, m, r):
    g = torch.Generator(device="cuda").manual_seed(N + C + r)
    rn = lambda std, *s: (torch.randn(s, generator=g, device="cuda") * std).to(BF)
    act, A, B = rn(1, N, H, W, C), rn(r ** -0.5, m, r), rn((kh * kw * C) ** -0.5, r, kh * kw * C)
    Y, T = abt.lr_conv_fwd(act, A, B, kh, kw, stride=stride)
    bare = abt.lr_conv_fwd(act, A, B, kh, kw, stride=stride, save_T=False)
    assert bare[1] is None and torch.equal(bare[0], Y)
    dY = rn(1e-2, *Y.shape)
    kept, again = (abt.lr_conv_bwd(dY, act, t, A, B, kh, kw, stride=stride)[1] for t in (T, None))
    assert torch.equal(kept, again)


# T again for one group or two of several: the values that the forward of all of them gave
@pytest.mark.parametrize("G,M,m,n,r", [(4, 512, 192, 768, 192), (4, 512, 192, 384, 192), (8, 250, 640, 768, 384), (4, 2500, 64, 3072, 96), (3, 4000, 192, 192, 288)])
def test_some_groups_compute_T_again(G, M, m, n, r):
    groups = [dict(zip(("X", "A", "B", "dY"), layer(M, m, n, r, seed=g))) for g in range(G)]
    for e, (_, T) in zip(groups, abt.lr_linear_fwd_grouped([{k: e[k] for k in "XAB"} for e in groups])):
        e["T"] = T
    kept = abt.lr_linear_bwd_grouped([dict(e, dA=True) for e in groups])
    for without in ([G - 1], [0, 1]):
        again = abt.lr_linear_bwd_grouped([dict(e, T=None if i in without else e["T"], dA=True) for i, e in enumerate(groups)])
        for a, b in zip(again, kept):
            assert torch.equal(a[1], b[1])


@pytest.mark.parametrize("M", [205, 5000])
def test_a_captured_forward_without_T(M):
    # the place for T comes from the graph's own memory: several replays, the program's work in between
    X, A, B, _ = layer(M, 2304, 768, 192)
    want = abt.lr_linear_fwd(X, A, B)[0]
    Y = torch.empty_like(want)
    abt.lr_linear_fwd(X, A, B, save_T=False, Y=Y)
    graph, side = torch.cuda.CUDAGraph(), torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.graph(graph, stream=side):
        abt.lr_linear_fwd(X, A, B, save_T=False, Y=Y)
    for k in range(3):
        Y.zero_()
        if k == 2:
            X.mul_(2)                                    # exact in bf16, and in every product and sum
            want = want * 2
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(Y, want)
