"""The work that a user of this framework has it do, as cases that can be measured.

A case is a dict of plain values; prepare() makes what a training program holds before the call,
run() takes it once through the public entry points of paper_2405_01067_amd.binding, the way
paper_2405_01067_amd.driver calls them (outputs and workspaces allocated per call), work() states
the bytes and operations that cannot be avoided and tolerance() how far another correct
implementation of the same precision may be off.

Kinds of work, all phases of Algorithm 1:
    linear     one training step of a factored linear layer: forward, then backward
    groups     one step of the group-training phase: G groups forward and backward in grouped calls (the
               first half of the groups trains A, the rest B), then the optimiser on the trained factors
    conv       one training step of a factored convolution on a channels-last activation
    merge      the end of a low-rank phase: averaging the group copies, re-decomposition with the rank
               rule, and the product of the new factors
    factorize  the start of a low-rank phase: decomposition of dense weights, and the product of the factors
"""
import torch

from paper_2405_01067_amd import binding as abt
from paper_2405_01067_amd.inputs import VIT_B16_LINEARS, VIT_TOKENS, CFG5_TAU_GAP

_DT = {"bf16": torch.bfloat16, "f32": torch.float32}

# Square 3 x 3 / 1 x 1 convolutions of ResNet-50's blocks: (side, C, m, window)
_CONV_LAYERS = ((56, 64, 64, 3), (28, 128, 128, 3), (14, 256, 256, 3), (7, 512, 512, 3),
                (56, 256, 128, 1), (28, 512, 256, 1), (14, 1024, 256, 1), (7, 2048, 512, 1))


def _linear(name, dtype, M, m, n, r, train="AB", keep_T=True, accumulate=False):
    c = {"kind": "linear", "dtype": dtype, "M": M, "m": m, "n": n, "r": r, "train": train, "keep_T": keep_T,
         "accumulate": accumulate}
    return dict(c, name=name) if name else c


def _conv(name, N, side, C, m, r, window, stride):
    c = {"kind": "conv", "N": N, "H": side, "W": side, "C": C, "m": m, "r": r, "window": window, "stride": stride}
    return dict(c, name=name) if name else c


def _merge(name, layers, m, n, k, G, mode, keep, want_W):
    """m = n = 0: the four linear shapes of ViT-B/16 in turn; keep: values above the planted gap."""
    c = {"kind": "merge", "layers": layers, "m": m, "n": n, "k": k, "G": G, "mode": mode, "keep": keep, "want_W": want_W}
    return dict(c, name=name) if name else c


def _factorize(name, layers, m, n, keep, k_cap):
    c = {"kind": "factorize", "layers": layers, "m": m, "n": n, "keep": keep, "k_cap": k_cap}
    return dict(c, name=name) if name else c


def listed():
    return [
        # the fp32 toy layer (64 samples, a 256 x 256 weight at rank 32): launches and host time
        _linear("f32_toy_step", "f32", 64, 256, 256, 32),
        # the driver's default type on a ViT-B/16 MLP layer, a batch of 16 images
        _linear("f32_fc1_batch16", "f32", 16 * VIT_TOKENS, 3072, 768, 192),
        # one image through the attention's qkv layer: 197 rows, a ragged last row block, latency
        _linear("bf16_qkv_one_image", "bf16", VIT_TOKENS, 2304, 768, 96),
        # the MLP layer at the paper's local batch of 64
        _linear("bf16_fc1_batch64", "bf16", 64 * VIT_TOKENS, 3072, 768, 192),
        # the last, incomplete batch of an epoch (201 images, an odd number of rows) at a low rank: memory
        _linear("bf16_fc2_batch201_r96", "bf16", 201 * VIT_TOKENS, 768, 3072, 96),
        # a batch of 256 at the highest rank the layer kernels take: the largest layer step
        _linear("bf16_fc1_batch256_r384", "bf16", 256 * VIT_TOKENS, 3072, 768, 384),
        # a step of the group-training phase with four groups, optimiser included
        {"name": "bf16_group_step_4x64", "kind": "groups", "G": 4, "M": 64 * VIT_TOKENS, "m": 3072, "n": 768, "r": 192},
        # ResNet-50's 14 x 14 convolution at a batch of 256
        _conv("conv3x3_256_14", 256, 14, 256, 256, 64, 3, 1),
        # a down-sampling convolution (28 x 28 to 14 x 14) at a batch of 256
        _conv("conv3x3_s2_128_28", 256, 28, 128, 128, 64, 3, 2),
        # the merge of one small layer, two copies, with the dense weight for the rebound phase: latency
        _merge("merge_one_small_layer", 1, 256, 256, 32, 2, 0, 20, True),
        # the merge of all 48 linear layers of ViT-B/16, four copies at rank 384
        _merge("merge_vit_b16", 48, 0, 0, 384, 4, 0, 192, False),
        # the decomposition of the dense weights of four blocks of ViT-B/16
        _factorize("factorize_4_blocks", 16, 0, 0, 192, 384),
    ]


def _log(rng, lo, hi):
    """Whole number between lo and hi, spread evenly over the logarithm."""
    return min(hi, max(lo, int(round(lo * (hi / lo) ** rng.random()))))


def draw(rng):
    kind = rng.choice(("linear",) * 8 + ("groups",) * 2 + ("conv",) * 4 + ("merge",) * 3 + ("factorize",))
    if kind == "linear":
        dtype = rng.choice(("bf16", "bf16", "bf16", "f32"))
        if rng.random() < 0.5:
            _, m, n = rng.choice(VIT_B16_LINEARS)
        elif dtype == "bf16":
            m, n = 64 * _log(rng, 1, 30), 64 * _log(rng, 1, 30)
        else:
            m, n = _log(rng, 24, 3072), _log(rng, 24, 3072)      # fp32 takes any size
        r = 32 * rng.randint(1, 12)
        M = _log(rng, 1, 256 * VIT_TOKENS if dtype == "bf16" else 16 * VIT_TOKENS)
        return _linear(None, dtype, M, m, n, r, rng.choice(("AB", "AB", "A", "B")), rng.random() < 0.8, rng.random() < 0.25)
    if kind == "groups":
        G = rng.randint(2, 8)
        _, m, n = rng.choice(VIT_B16_LINEARS)
        return {"kind": "groups", "G": G, "M": _log(rng, VIT_TOKENS, 256 * VIT_TOKENS // G), "m": m, "n": n,
                "r": 32 * rng.randint(1, 12)}
    if kind == "conv":
        side, C, m, window = rng.choice(_CONV_LAYERS)
        side += rng.choice((0, 0, -1, 1))                        # other image sizes give odd sides
        r = 32 * rng.choice((1, 2, 2, 3, 4, 5, 6, 8))
        return _conv(None, _log(rng, 1, 256 if side < 50 else 128), side, C, m, r, window, rng.choice((1, 1, 2)))
    if kind == "merge":
        mode = rng.choice((0, 0, 1))
        G = rng.randint(2, 8 if mode == 0 else 4)
        k = 32 * rng.randint(1, 12 if mode == 0 else 4)
        K = k if mode == 0 else k * G
        layers = _log(rng, 1, 24 if K <= 384 else 8)
        m, n = (0, 0) if rng.random() < 0.5 else (_log(rng, 2 * k, 3072), _log(rng, 2 * k, 3072))
        return _merge(None, layers, m, n, k, G, mode, rng.randint(1, k), layers <= 12)
    side = 32 * _log(rng, 2, 24)
    m, n = (side, _log(rng, side, 3072)) if rng.random() < 0.5 else (_log(rng, side, 3072), side)
    keep = rng.randint(1, side)
    return _factorize(None, _log(rng, 1, 16), m, n, keep, max(32, side // 2))


# --------------------------------------------------------------------------------------- inputs
def _rng(seed):
    return torch.Generator(device="cuda").manual_seed(int(seed))


def _normal(g, shape, std, dtype):
    return torch.randn(shape, generator=g, device="cuda").mul_(std).to(dtype)


def _frame(g, rows, cols):
    """rows x cols (rows >= cols) with orthonormal columns, fp64."""
    x = torch.randn((rows, cols), generator=g, device="cuda", dtype=torch.float64)
    low = torch.linalg.cholesky(x.T @ x)
    return torch.linalg.solve_triangular(low, x.T, upper=False).T.contiguous()


def _planted(g, m, n, count, keep):
    """Thin factors (fp64) of a matrix with singular values i^-0.8 and a drop to a tenth after `keep`."""
    s = torch.arange(1, count + 1, device="cuda", dtype=torch.float64) ** -0.8
    s[keep:] *= 0.1
    root = s.sqrt()
    return _frame(g, m, count) * root, (root[:, None] * _frame(g, n, count).T).contiguous()


def _cut(count, keep):
    """Threshold in the middle (geometric) of the planted gap; 0 keeps everything."""
    if keep >= count:
        return 0.0
    if (count, keep) == (384, 192):
        return CFG5_TAU_GAP
    return float((keep ** -0.8 * 0.1 * (keep + 1) ** -0.8) ** 0.5)


def _layer_shapes(case):
    if case["m"]:
        return [(case["m"], case["n"])] * case["layers"]
    return [VIT_B16_LINEARS[i % 4][1:] for i in range(case["layers"])]


def prepare(case, seed):
    g = _rng(seed)
    kind = case["kind"]
    if kind == "linear":
        # layer inputs follow a normalisation (unit variance), gradients are small, factors well scaled
        dt, M, m, n, r = _DT[case["dtype"]], case["M"], case["m"], case["n"], case["r"]
        st = {"case": case, "X": _normal(g, (M, n), 1.0, dt), "dY": _normal(g, (M, m), 1e-2, dt),
              "A": _normal(g, (m, r), r ** -0.5, dt), "B": _normal(g, (r, n), n ** -0.5, dt), "dA": None, "dB": None}
        if case["accumulate"]:
            if "A" in case["train"]:
                st["dA"] = torch.zeros((m, r), device="cuda")
            if "B" in case["train"]:
                st["dB"] = torch.zeros((r, n), device="cuda")
        return st
    if kind == "groups":
        G, M, m, n, r = case["G"], case["M"], case["m"], case["n"], case["r"]
        bf = torch.bfloat16
        groups, table = [], []
        for i in range(G):
            A, B = _normal(g, (m, r), r ** -0.5, torch.float32), _normal(g, (r, n), n ** -0.5, torch.float32)
            e = {"X": _normal(g, (M, n), 1.0, bf), "A": A.to(bf), "B": B.to(bf), "dY": _normal(g, (M, m), 1e-2, bf)}
            key = "A" if i < (G + 1) // 2 else "B"
            p = A if key == "A" else B
            t = {"param": p, "grad": torch.zeros_like(p), "exp_avg": torch.zeros_like(p), "exp_avg_sq": torch.zeros_like(p),
                 "param_bf16": e[key]}
            e["grad_key"] = "d" + key
            groups.append(e)
            table.append(t)
        return {"case": case, "groups": groups, "table": table, "plan": abt.AdamwPlan(table), "step": 0}
    if kind == "conv":
        N, H, W, C, m, r, w, s = (case[k] for k in ("N", "H", "W", "C", "m", "r", "window", "stride"))
        rows = N * -(-H // s) * -(-W // s)
        bf = torch.bfloat16
        return {"case": case, "act": _normal(g, (N, H, W, C), 1.0, torch.float32).clamp_(min=0).to(bf),
                "dY": _normal(g, (rows, m), 1e-2, bf), "A": _normal(g, (m, r), r ** -0.5, bf),
                "B": _normal(g, (r, w * w * C), (w * w * C) ** -0.5, bf)}
    if kind == "merge":
        k, G = case["k"], case["G"]
        k_cap = k if case["mode"] == 0 else min(k * G, 2 * k)
        shapes = _layer_shapes(case)
        S = torch.empty((len(shapes), k_cap), device="cuda")
        kept = torch.zeros((len(shapes),), dtype=torch.int32, device="cuda")
        layers = []
        for i, (m, n) in enumerate(shapes):
            a, b = _planted(g, m, n, k, case["keep"])
            layers.append({"A_copies": [(a + 1e-3 * torch.randn(a.shape, generator=g, device="cuda")).float() for _ in range(G)],
                           "B_copies": [(b + 1e-3 * torch.randn(b.shape, generator=g, device="cuda")).float() for _ in range(G)],
                           "tau": _cut(k, case["keep"]), "mode": case["mode"], "k_cap": k_cap, "k_fixed": case["keep"],
                           "want_W": case["want_W"], "S_out": S[i], "k_out": kept[i]})
            if case["keep"] in (20, 192):       # a wide gap in a well-resolved spectrum: the rank rule decides
                layers[-1]["k_fixed"] = 0
        return {"case": case, "layers": layers, "S": S, "k": kept}
    layers = []
    for m, n in _layer_shapes(case):
        count = min(m, n)
        a, b = _planted(g, m, n, count, case["keep"])
        layers.append({"W": (a @ b).float(), "tau": _cut(count, case["keep"]), "k_cap": case["k_cap"]})
    return {"case": case, "layers": layers}


# --------------------------------------------------------------------------------------- one pass
def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "linear":
        Y, T = abt.lr_linear_fwd(state["X"], state["A"], state["B"], save_T=case["keep_T"])
        dX, dA, dB = abt.lr_linear_bwd(state["dY"], state["X"], T, state["A"], state["B"], need_dA="A" in case["train"],
                                       need_dB="B" in case["train"], dA=state["dA"], dB=state["dB"],
                                       accumulate=case["accumulate"])
        return Y, T, dX, dA, dB
    if kind == "groups":
        groups, table = state["groups"], state["table"]
        fwd = abt.lr_linear_fwd_grouped([{k: e[k] for k in ("X", "A", "B")} for e in groups])
        bwd = abt.lr_linear_bwd_grouped([dict(dY=e["dY"], X=e["X"], T=y[1], A=e["A"], B=e["B"], dX=True,
                                              **{e["grad_key"]: t["grad"]}) for e, t, y in zip(groups, table, fwd)])
        state["step"] += 1
        abt.ab_adamw_step(state["plan"], step=state["step"], lr=1e-4)
        return [(y, t, b[0]) for (y, t), b in zip(fwd, bwd)], [(t["grad"], t["param"], t["param_bf16"]) for t in table]
    if kind == "conv":
        w, s = case["window"], case["stride"]
        Y, T = abt.lr_conv_fwd(state["act"], state["A"], state["B"], w, w, stride=s)
        return (Y, T) + abt.lr_conv_bwd(state["dY"], state["act"], T, state["A"], state["B"], w, w, stride=s)
    # The factors of a decomposition are determined up to one sign per pair of a column of A and a row
    # of B (and a rotation among equal values); their product, the weight that training goes on with, is not.
    if kind == "merge":
        outs = abt.ab_merge_batched(state["layers"])
        extra = [o["W"] for o in outs if o["W"] is not None]
        return [abt.ab_reconstruct(o["A"], o["B"]) for o in outs], extra, state["S"], state["k"]
    outs = abt.ab_factorize_batched(state["layers"])
    return [abt.ab_reconstruct(o["A"], o["B"]) for o in outs], [(o["S"], o["k"]) for o in outs]


# --------------------------------------------------------------------------------------- what it needs
def _decomposition_work(m, n, K, k_out, in_bytes):
    """Bytes and operations of a truncated SVD of a rank-K product of thin factors: their Gram matrices,
    the K x K core and its SVD with one set of vectors (4 K^3), the new factors, and their product."""
    nbytes = in_bytes + 4 * (k_out * (m + n) + k_out + m * n)
    flops = K * K * (m + n) + 6 * K ** 3 + 2 * K * k_out * (m + n) + 2 * m * n * k_out
    return nbytes, flops


def work(case):
    kind = case["kind"]
    if kind in ("linear", "groups"):
        M, m, n, r = case["M"], case["m"], case["n"], case["r"]
        if kind == "groups":
            G = case["G"]
            ga = (G + 1) // 2
            trained = ga * m * r + (G - ga) * r * n
            act = G * 2 * (2 * M * n + 2 * M * m + M * r + (m + n) * r)
            # optimiser: parameter and two moments read and written, gradient written, bf16 copy written
            return {"bytes": act + trained * (6 * 4 + 4 + 2),
                    "flops": G * 4 * M * r * (m + n) + 2 * M * r * (ga * m + (G - ga) * n) + 12 * trained}
        e = 4 if case["dtype"] == "f32" else 2
        grads = (m * r if "A" in case["train"] else 0) + (r * n if "B" in case["train"] else 0)
        return {"bytes": e * (2 * M * n + 2 * M * m + (M * r if case["keep_T"] else 0) + (m + n) * r)
                + 4 * grads * (2 if case["accumulate"] else 1),
                "flops": 4 * M * r * (m + n) + 2 * M * grads}
    if kind == "conv":
        N, H, W, C, m, r, w, s = (case[k] for k in ("N", "H", "W", "C", "m", "r", "window", "stride"))
        rows, n = N * -(-H // s) * -(-W // s), w * w * C
        return {"bytes": 2 * (2 * N * H * W * C + 2 * rows * m + rows * r + (m + n) * r) + 4 * (m + n) * r,
                "flops": 6 * rows * r * (m + n)}
    nbytes = flops = 0
    for m, n in _layer_shapes(case):
        if kind == "merge":
            k, G = case["k"], case["G"]
            K, cap = (k, k) if case["mode"] == 0 else (k * G, min(k * G, 2 * k))
            b, f = _decomposition_work(m, n, K, cap, 4 * G * k * (m + n))
            if case["want_W"]:
                b, f = b + 4 * m * n, f + 2 * m * n * K
        else:
            b, f = _decomposition_work(m, n, min(m, n), case["k_cap"], 4 * m * n)
        nbytes, flops = nbytes + b, flops + f
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    kind = case["kind"]
    if kind in ("conv", "groups") or case.get("dtype") == "bf16":
        # results rounded to bf16, T and dT rounded to bf16 in between: 2.4e-3 against the same step in fp64
        return {"rel": 1e-2}
    # fp32 products summed over up to 3152 rows: up to 1.4e-6 against fp64; decompositions, K x K stages in
    # fp64 and back-projections in fp32: up to 8e-7 against an fp64 SVD, with the rank the same
    return {"rel": 6e-6}
