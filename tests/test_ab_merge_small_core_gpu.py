"""Merges whose core is a single pair of column blocks (K = 32) run all Jacobi sweeps in one launch, and sum their Gram matrices in
parts; with a larger layer in the batch the same layer goes through the launches for all sizes.  Both do the same rotations in the same
order, on numbers that differ by the order of fp64 sums: the singular values agree but for their rounding to fp32, 2^-23 at most
where one lies on either side of a boundary.  And decompositions of dense weights around
the sizes where the Cholesky factorisation changes its form, against an fp64 SVD."""
import numpy as np
import pytest
import torch

from paper_2405_01067_amd import binding as abt
from paper_2405_01067_amd import inputs as gen

pytestmark = pytest.mark.gpu


def layer(m, n, k, seed, g=2, gap_at=12):
    lay = gen.merge_layer(m, n, seed=seed, k_in=k, g=g, gap_at=gap_at)
    up = lambda xs: [torch.from_numpy(np.ascontiguousarray(x)).to("cuda:0") for x in xs]
    return {"A_copies": up(lay["A_copies"]), "B_copies": up(lay["B_copies"]), "tau": 0.0}


@pytest.mark.parametrize("m,n,count", [(64, 48, 1), (256, 256, 3), (33, 1000, 2)])
def test_single_pair_core_agrees_with_a_mixed_batch(m, n, count):
    small = [layer(m, n, 32, seed=10 * m + i) for i in range(count)]
    alone = abt.ab_merge_batched(small)
    mixed = abt.ab_merge_batched(small + [layer(128, 96, 64, seed=3)])
    for a, b in zip(alone, mixed):
        assert bool(((a["S"] - b["S"]).abs() <= 2 ** -23 * b["S"]).all()) and a["sweeps"] == b["sweeps"] > 1
        W, V = (o["A"].double() @ o["B"].double() for o in (a, b))
        assert float((W - V).norm() / V.norm()) < 1e-6


def test_single_pair_core_reports_the_sweep_cap():
    lay = layer(200, 100, 32, seed=77)
    prev = abt.set_jacobi_max_sweeps(1)
    try:
        with pytest.raises(abt.AbtError):
            abt.ab_merge_batched([lay])
    finally:
        abt.set_jacobi_max_sweeps(prev)


@pytest.mark.parametrize("m,n", [(128, 128), (160, 160), (544, 600), (700, 576), (100, 96)])
def test_dense_decomposition_around_the_cholesky_forms(m, n):
    # 96, 128: one launch; 160 and more: blocked, 64 x 64 tiles of the trailing matrix with 32-wide remainders
    g = torch.Generator().manual_seed(m + n)
    K = min(m, n) // 32 * 32
    W = torch.randn((m, n), generator=g, dtype=torch.float64)
    W = W[:K] if m <= n else W[:, :K]
    W = (W * torch.logspace(0, -2, W.shape[1], dtype=torch.float64)).float().contiguous()
    keep = K // 2
    out = abt.ab_factorize(W.to("cuda:0"), tau=0.0, k_fixed=keep)
    U, s, V = torch.linalg.svd(W.double(), full_matrices=False)
    assert float(((out["S"].cpu().double()[:keep] - s[:keep]).abs() / s[:keep]).max()) < 1e-5
    got = out["A"].cpu().double()[:, :keep] @ out["B"].cpu().double()[:keep]
    want = (U[:, :keep] * s[:keep]) @ V[:keep]
    # fp32 factors and products; the cut falls into a spectrum without a gap, but the values around it agree
    # to far better than their distance
    assert float((got - want).norm() / want.norm()) < 1e-5


@pytest.mark.parametrize("K", [32, 64, 96, 128, 160, 256, 288, 384, 416, 512, 544, 768])
@pytest.mark.parametrize("zero_tail", [0, 20])
def test_block_iteration_at_the_edges_of_its_forms(K, zero_tail):
    # one form of the kernel up to 32, 128, 256, 384, 512 and 768 columns; the last columns of A (rows of B) zero, as
    # padding of the rank leaves them
    g = torch.Generator().manual_seed(K + zero_tail)
    m, n = K + 40, K + 12
    scale = torch.logspace(0, -2, K, dtype=torch.float64)
    scale[K - zero_tail:] = 0.0
    A = (torch.randn((m, K), generator=g, dtype=torch.float64) * scale).float()
    B = torch.randn((K, n), generator=g, dtype=torch.float64).float()
    B[K - zero_tail:] = 0.0
    W = A.double() @ B.double()
    U, s, V = torch.linalg.svd(W, full_matrices=False)
    keep = (K - zero_tail) // 2
    out = abt.ab_merge([A.to("cuda:0")], [B.to("cuda:0")], tau=0.0, k_fixed=keep)
    # values: fp64 Gram matrices (2^-53 times the square of the condition, below 1e-9 for the kept half), rounded once to fp32
    assert float(((out["S"].cpu().double()[:keep] - s[:keep]).abs() / s[:keep]).max()) < 3e-7
    got = out["A"].cpu().double()[:, :keep] @ out["B"].cpu().double()[:keep]
    want = (U[:, :keep] * s[:keep]) @ V[:keep]
    # fp32 back-projections: sums of K products, (K + 2) 2^-24 at most, some sqrt(K) 2^-24 in the norm; factors rounded to fp32
    assert float((got - want).norm() / want.norm()) < 4e-6


# batches that take four blocks of columns a work-group: one pair of double blocks (all sweeps in one launch), two, sizes up to the limit, and
# sizes mixed, where the work-groups look their layer up in the tables
@pytest.mark.parametrize("zero_tail", [0, 20])
@pytest.mark.parametrize("sizes", [(64,), (64, 64, 64), (128,) * 4, (192,) * 32, (320,) * 20, (384,) * 16, (512,) * 24, (512, 64, 128, 448) * 11,
                                   (512,) * 12, (512, 64, 128, 448) * 6])    # (the last two: two blocks)
def test_four_blocks_a_work_group(sizes, zero_tail):
    made = {}
    for i, K in enumerate(sizes):                        # two different layers of every size
        key = (K, i // len(set(sizes)) % 2)
        if key not in made:
            g = torch.Generator().manual_seed(K + zero_tail + key[1])
            scale = torch.logspace(0, -2, K, dtype=torch.float64)
            scale[K - zero_tail:] = 0.0
            A = (torch.randn((K + 24, K), generator=g, dtype=torch.float64) * scale).float()
            B = torch.randn((K, K + 12), generator=g, dtype=torch.float64).float()
            B[K - zero_tail:] = 0.0
            made[key] = (A.to("cuda:0"), B.to("cuda:0"), (K - zero_tail) // 2)
    keys = [(K, i // len(set(sizes)) % 2) for i, K in enumerate(sizes)]
    outs = abt.ab_merge_batched([{"A_copies": [made[k][0]], "B_copies": [made[k][1]], "tau": 0.0, "k_fixed": made[k][2]} for k in keys])
    first = {}
    for k, out in zip(keys, outs):
        if k in first:                                   # the same layer again: the same bits
            assert all(torch.equal(out[x], first[k][x]) for x in ("A", "B", "S"))
            continue
        first[k] = out
        A, B, keep = made[k]
        U, s, V = torch.linalg.svd((A.cpu().double() @ B.cpu().double()), full_matrices=False)
        # (bounds as above)
        assert float(((out["S"].cpu().double()[:keep] - s[:keep]).abs() / s[:keep]).max()) < 3e-7
        want = (U[:, :keep] * s[:keep]) @ V[:keep]
        got = out["A"].cpu().double()[:, :keep] @ out["B"].cpu().double()[:keep]
        assert float((got - want).norm() / want.norm()) < 4e-6


def planted(m, n, values, seed):
    """Factors (fp32) with these singular values (fp64), their columns mixed, and the product that they make."""
    g = torch.Generator().manual_seed(seed)
    K = values.numel()
    frame = lambda rows: torch.linalg.qr(torch.randn((rows, K), generator=g, dtype=torch.float64).to("cuda:0"))[0]
    U, V, R, root = frame(m), frame(n), frame(K), values.to("cuda:0").sqrt()
    A, B = ((U * root) @ R).float().contiguous(), (R.T @ (root[:, None] * V.T)).float().contiguous()
    return A, B, A.double() @ B.double()


# Two clusters of values three orders apart.  With the Gram matrix of a block pair in fp64 the iteration takes 14 or 15 sweeps of 768 columns (two
# blocks a work-group) and of 512 (four) at any of six seeds; in fp32, where the difference of nearly equal squared norms and what is left of a
# small column's beside a large one's are rounding, 18 to 20 and 16 or 17.
@pytest.mark.parametrize("K,count,sweeps", [(768, 1, 16), (512, 24, 15)])
def test_clusters_far_apart_take_the_sweeps_of_fp64(K, count, sweeps):
    g = torch.Generator().manual_seed(K)
    s = torch.where(torch.arange(K) < K // 2, 1.0, 1e-3).double() * (1 + 1e-5 * torch.rand(K, generator=g, dtype=torch.float64))
    A, B, W = planted(K + 72, K + 40, s, seed=K)
    out = abt.ab_merge_batched([{"A_copies": [A], "B_copies": [B], "tau": 0.0, "k_fixed": K, "k_cap": K}] * count)[-1]
    assert out["sweeps"] <= sweeps
    ref = torch.linalg.svdvals(W)[:K]
    # columns of a cluster that are left with a cosine of c have norms c / 2 off the values; the last sweep leaves some 1e-7 inside a cluster
    assert float(((out["S"].double() - ref).abs() / ref).max()) < 1e-6


# Eight clusters between 1 and 1/2, equal inside or nearly so, through every form of the iteration: one pair of blocks, one pair of double blocks in one
# launch, two blocks a work-group, four.
@pytest.mark.parametrize("gap", [0.0, 1e-6, 1e-5, 1e-4, 1e-3])
@pytest.mark.parametrize("K,count", [(32, 1), (64, 1), (96, 1), (128, 4), (256, 1), (384, 16), (768, 1)])
def test_clustered_values(K, count, gap):
    i = torch.arange(K, dtype=torch.float64)
    s = 2.0 ** -((i // (K // 8)) / 8) * (1 + gap * (i % (K // 8)) / (K // 8))
    A, B, W = planted(K + 72, K + 40, s, seed=K + 1)
    out = abt.ab_merge_batched([{"A_copies": [A], "B_copies": [B], "tau": 0.0, "k_fixed": K, "k_cap": K}] * count)[-1]
    a, b = out["A"].double(), out["B"].double().T
    # The iteration ends with a sweep in which no pair that it came to had a cosine above 3e-4: that is what columns may be left with where values are
    # equal, and up to twice that (the ratio of the values) on the side that is found from the other.
    for x in (a, b):
        x = x / x.norm(dim=0)
        assert float((x.T @ x - torch.eye(K, device="cuda:0", dtype=torch.float64)).abs().max()) < 6e-4
    # U U^T W for the U that was found: as far off as its columns are from orthogonal, in the norm
    assert float((a @ b.T - W).norm() / W.norm()) < 6e-4
    ref = torch.linalg.svdvals(W)[:K]
    assert float(((out["S"].double() - ref).abs() / ref).max()) < 3e-4 / 2


# shapes around the 64 contraction indices of a step and the 16 work-groups of a side, rows that are not multiples of four, one to five copies, more
# columns than the core has and fewer
@pytest.mark.parametrize("m,n,G,k_cap,k_fixed", [(33, 32, 1, 32, 0), (64, 65, 2, 32, 0), (1024, 1025, 3, 20, 0), (1088, 2047, 5, 40, 7), (3072, 130, 4, 32, 32)])
def test_stages_around_a_core_of_32(m, n, G, k_cap, k_fixed):
    layers = [dict(layer(m, n, 32, seed=m + n + i, g=G), k_cap=k_cap, k_fixed=k_fixed, tau=0.01, want_W=True) for i in range(2)]
    for lay, out in zip(layers, abt.ab_merge_batched(layers)):
        A, B = (torch.stack(lay[x]).double().mean(0) for x in ("A_copies", "B_copies"))
        W = (A @ B).cpu()
        U, S, Vt = torch.linalg.svd(W, full_matrices=False)
        want = min(k_fixed or int((S[:32].float() >= 0.01 * S[0].float()).sum()), k_cap, 32)
        k = int(out["k"])
        assert k == want
        # values: fp32 averages of the factors and fp32 output, 2^-24 each, relative to the largest by the products
        kept = min(k_cap, 32)
        assert float((out["S"][:kept].double().cpu() - S[:kept]).abs().max() / S[0]) < 1e-6 and not bool(out["S"][kept:].any())
        T = U[:, :k] * S[:k] @ Vt[:k]
        a, b = out["A"].double().cpu(), out["B"].double().cpu()
        assert float((a @ b - T).norm() / T.norm()) < 6e-6 and not bool(a[:, k:].any()) and not bool(b[k:].any())
        assert float((out["W"].double().cpu() - W).norm() / W.norm()) < 1e-6
        # A'^T A' = B' B'^T = the values
        for q in (a[:, :k].T @ a[:, :k], b[:k] @ b[:k].T):
            assert float((q - torch.diag(S[:k])).norm() / S[:k].norm()) < 1e-4


# the smallest tables go up in launch arguments, larger ones as a copy: a stream that is being captured is refused by both, before anything is launched
@pytest.mark.parametrize("k,count,dense", [(32, 1, False), (32, 64, False), (64, 1, False), (32, 1, True), (64, 1, True)])
def test_a_capture_is_refused(k, count, dense):
    layers = [dict(layer(96, 80, k, seed=i), k_cap=k) for i in range(count)]
    W = torch.randn((96, k), generator=torch.Generator().manual_seed(k)).to("cuda:0")
    merge = lambda: abt.ab_factorize(W, tau=0.0, check_converged=False) if dense else abt.ab_merge_batched(layers, check_converged=False)
    merge()
    x = torch.zeros(16, device="cuda:0")
    stream, graph = torch.cuda.Stream(), torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.stream(stream):
        graph.capture_begin(capture_error_mode="thread_local")
        try:
            x.add_(1.0)
            with pytest.raises(abt.AbtError, match="ABT_EHIP"):
                merge()
        finally:
            graph.capture_end()
    graph.replay()
    graph.replay()
    torch.cuda.synchronize()
    assert bool((x == 2.0).all())
    merge()                                               # and is served again afterwards
