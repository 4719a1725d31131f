"""The calls whose speed this library is judged by, as a user's program makes them.

A case is one pass through the public entry points of ``paper_2101_07948_amd``: a sparse
linear layer (``Plan.spmm``), the same layer with K spread over workgroups
(``Plan.spmm_split``), a sparse 3x3 convolution (``Plan.conv3x3``, ``Plan.conv3x3_split``)
or the six chained products of a pruned encoder layer.  ``listed()`` names the fixed ones,
``draw()`` gives more of the same ranges: 64 to 3072 rows and columns, 70 to 98 % zeros in
the three patterns of pruned weights, N from a single column to 16384, every epilogue, with
and without bias, column counts that are and are not multiples of 4, and convolutions of 16
to 256 channels on images of 7 to 56 pixels.

Layer sizes are those of ``inputs.workload`` (BERT-base attention and feed-forward layers,
MobileNet 1x1 convolutions), of the paper-shaped problems M = K = 256 ... 2048, and of the
3x3 convolution benchmark.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2101_07948_amd as sd

DEV = "cuda:0"
PATTERNS = ("uniform", "lognormal", "grouped8")
EPILOGUES = ("none", "relu", "gelu")


def _linear(name, M, K, N, sparsity, pattern="uniform", epi="none", bias=True, relu_input=False,
            split_chunks=0):
    return {"name": name, "op": "split" if split_chunks else "linear", "M": M, "K": K, "N": N,
            "sparsity": sparsity, "pattern": pattern, "epi": epi, "bias": bias,
            "relu_input": relu_input, "split_chunks": split_chunks}


def _conv(name, OC, IC, H, W, NB, sparsity, epi="none", bias=True, split_chunks=0):
    return {"name": name, "op": "conv", "OC": OC, "IC": IC, "H": H, "W": W, "NB": NB,
            "sparsity": sparsity, "epi": epi, "bias": bias, "split_chunks": split_chunks}


def listed():
    return [
        # the smallest layer of the workloads, one short sequence: launch and latency
        _linear("tiny_256", 256, 256, 64, 0.90, bias=False),
        # BERT-base attention projection, 8 sequences of 128 tokens
        _linear("projection_90", 768, 768, 1024, 0.90),
        # BERT-base feed-forward down projection, 32 sequences of 128 tokens: the benchmark's layer
        _linear("ffn_down_90", 768, 3072, 4096, 0.90),
        # the same layer at a serving batch of 8 sequences, through the call meant for few columns
        _linear("ffn_down_90_split", 768, 3072, 1024, 0.90, split_chunks=4),
        # feed-forward up projection with uneven row lengths and the fused GELU
        _linear("ffn_up_94_gelu", 3072, 768, 4096, 0.94, pattern="lognormal", epi="gelu"),
        # MobileNet 1x1 convolution on 16 images of 14 x 14 after a ReLU, ReLU epilogue
        _linear("pointwise_80_relu", 512, 512, 3136, 0.80, epi="relu", relu_input=True),
        # pruneBERT-like up projection, block-correlated columns, offline batch: the largest call
        _linear("ffn_up_97_gelu", 3072, 768, 16384, 0.97, pattern="grouped8", epi="gelu"),
        # the paper's least sparse grade on its largest matrix
        _linear("square_70", 2048, 2048, 512, 0.70, bias=False),
        # odd sizes: a layer and a token count that no tile divides
        _linear("ragged_85_relu", 997, 1531, 1023, 0.85, epi="relu"),
        # 3x3 convolution of the paper's benchmark, 16 images
        _conv("conv_256_14", 256, 256, 14, 14, 16, 0.90),
        # its late, small-image stage, through the call meant for few pixels
        _conv("conv_256_7_split", 256, 256, 7, 7, 16, 0.95, epi="relu", split_chunks=3),
        # one pruned encoder layer: four projections, up projection with GELU, down projection
        {"name": "encoder_97", "op": "encoder", "H": 768, "F": 3072, "N": 4096, "sparsity": 0.97,
         "pattern": "grouped8"},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choices(("linear", "split", "conv", "encoder"), (10, 3, 3, 1))[0]
    sparsity = round(rng.uniform(0.70, 0.98), 3)
    epi = rng.choice(EPILOGUES)
    bias = rng.random() < 0.8
    if kind == "encoder":
        H = 64 * rng.randint(2, 12)
        return {"op": "encoder", "H": H, "F": 4 * H, "N": 4 * _log_int(rng, 16, 1024),
                "sparsity": max(sparsity, 0.95), "pattern": rng.choice(PATTERNS)}
    if kind == "conv":
        side = rng.randint(7, 56)
        ch = 128 if side > 28 else 256
        return _drop_name(_conv("", _log_int(rng, 16, ch), _log_int(rng, 16, ch), side,
                                rng.randint(7, side), 4 * rng.randint(1, 4),
                                max(sparsity, 0.80), epi, bias, rng.choice((0, 0, 2, 4))))
    M, K = _log_int(rng, 64, 3072), 8 * _log_int(rng, 8, 384)
    N = _log_int(rng, 1, 16384)
    if rng.random() < 0.7:
        N = (N + 3) // 4 * 4
    else:
        K = max(1, K - rng.randint(1, 7))
    if kind == "split":
        N = min(N, 2048)
    # no more work than the largest listed case: its outputs and its multiply-adds
    while (M * N > 3072 * 16384 or K * N > 3072 * 16384 or
           (1.0 - sparsity) * M * K * N > 0.03 * 3072 * 768 * 16384):
        N = max(4, N // 8 * 4)
    pattern = rng.choice(PATTERNS if K % 8 == 0 else PATTERNS[:2])
    return _drop_name(_linear("", M, K, N, sparsity, pattern, epi, bias, rng.random() < 0.3,
                              rng.randint(1, 6) if kind == "split" else 0))


def _drop_name(case):
    del case["name"]
    return case


# ---- weights --------------------------------------------------------------------------


def _nnz(M, K, sparsity):
    return int(np.rint((1.0 - sparsity) * M * K))


def _row_counts(rng, M, K, nnz, pattern):
    """Entries per row: equal (grouped8), or proportional to exp(N(0, 0.5^2)) (lognormal)."""
    weights = np.exp(rng.normal(0.0, 0.5, M)) if pattern == "lognormal" else np.ones(M)
    counts = np.zeros(M, dtype=np.int64)
    while counts.sum() < nnz:
        room = counts < K
        share = np.where(room, weights, 0.0)
        add = np.floor(share / share.sum() * (nnz - counts.sum())).astype(np.int64)
        if not add.any():
            free = rng.permutation(np.flatnonzero(room))[:int(nnz - counts.sum())]
            add[free] = 1
        counts = np.minimum(counts + add, K)
    return counts


def _csr(rng, M, K, sparsity, pattern, std):
    """(row_ptr, col_idx, values) of an M x K matrix with exactly _nnz entries."""
    nnz = _nnz(M, K, sparsity)
    if pattern == "uniform":
        pos = np.sort(rng.choice(M * K, size=nnz, replace=False))
        rows, cols = pos // K, pos % K
    else:
        counts = _row_counts(rng, M, K, nnz, pattern)
        if pattern == "grouped8":  # columns in random groups of 8; a row takes whole groups
            group_of = np.empty(K, dtype=np.int64)
            group_of[rng.permutation(K)] = np.arange(K) // 8
            key = rng.random((M, K // 8))[:, group_of] + rng.random((M, K)) * 1e-9
        else:
            key = rng.random((M, K))
        order = np.argsort(key, axis=1)
        take = np.arange(K)[None, :] < counts[:, None]
        mask = np.zeros((M, K), dtype=bool)
        np.put_along_axis(mask, order, take, axis=1)
        rows, cols = np.nonzero(mask)
    row_ptr = np.zeros(M + 1, dtype=np.int32)
    np.cumsum(np.bincount(rows, minlength=M), out=row_ptr[1:])
    values = rng.standard_normal(nnz, dtype=np.float32) * np.float32(std)
    return row_ptr, cols.astype(np.int32), values


def _dense64(csr, M, K):
    """The matrix in double precision on the GPU."""
    row_ptr, cols, values = csr
    W = np.zeros((M, K), dtype=np.float64)
    W[np.repeat(np.arange(M), np.diff(row_ptr)), cols] = values
    return torch.from_numpy(W).to(DEV)


def _host_inputs(case, seed):
    """The layers of a case, (csr, M, K, bias, epilogue) each, made from the seed alone."""
    rng = np.random.default_rng([seed, 20210107948])
    op = case["op"]
    if op == "encoder":
        H, F = case["H"], case["F"]
        shapes = [(H, H)] * 4 + [(F, H), (H, F)]
        epis = ["none"] * 4 + ["gelu", "none"]
    elif op == "conv":
        shapes, epis = [(case["OC"], case["IC"] * 9)], [case["epi"]]
    else:
        shapes, epis = [(case["M"], case["K"])], [case["epi"]]
    layers = []
    for (M, K), epi in zip(shapes, epis):
        # values that keep the activations near one
        std = 1.0 / math.sqrt(max(1.0, (1.0 - case["sparsity"]) * K))
        csr = _csr(rng, M, K, case["sparsity"], case.get("pattern", "uniform"), std)
        bias = rng.normal(0.0, 0.02, M).astype(np.float32) if case.get("bias", True) else None
        layers.append((csr, M, K, bias, epi))
    return layers


def _activations(case, seed):
    """The activations a call starts from, on the GPU."""
    gen = torch.Generator(device=DEV).manual_seed(seed * 1000003 + 17)
    if case["op"] == "conv":
        shape = (case["IC"], case["H"], case["W"], case["NB"])
    elif case["op"] == "encoder":
        shape = (case["H"], case["N"])
    else:
        shape = (case["K"], case["N"])
    X = torch.randn(shape, generator=gen, device=DEV)
    return X.clamp_(min=0.0) if case.get("relu_input") else X


# ---- the measured pass ----------------------------------------------------------------


def prepare(case, seed):
    """Activations, bias and plans, outputs and (for the split calls) the workspace: all
    that a serving program allocates once."""
    X = _activations(case, seed)
    split = case.get("split_chunks", 0)
    layers = []
    for (row_ptr, cols, values), M, K, bias, epi in _host_inputs(case, seed):
        plan = sd.Plan(row_ptr, cols, values, M, K, split_chunks=split)
        shape = (M,) + tuple(X.shape[1:])
        layers.append({"plan": plan, "epi": epi, "C": torch.empty(shape, device=DEV),
                       "bias": None if bias is None else torch.from_numpy(bias).to(DEV)})
    ws = None
    if split:
        n = X.numel() // X.shape[0]
        ws = torch.empty(max(1, layers[0]["plan"].workspace_floats(n)), device=DEV)
    return {"op": case["op"], "split": split, "X": X, "layers": layers, "workspace": ws}


def run(state):
    L = state["layers"][0]
    if state["op"] == "conv":
        if state["split"]:
            return L["plan"].conv3x3_split(state["X"], L["C"], L["bias"], L["epi"],
                                           workspace=state["workspace"])
        return L["plan"].conv3x3(state["X"], L["C"], L["bias"], L["epi"])
    if state["op"] == "split":
        return L["plan"].spmm_split(state["X"], L["C"], L["bias"], L["epi"],
                                    workspace=state["workspace"])
    X = state["X"]
    for L in state["layers"]:
        X = L["plan"].spmm(X, L["C"], L["bias"], L["epi"])
    return X


# ---- what a pass cannot do without ----------------------------------------------------


def work(case):
    """Each weight (value and column) and input read once, each output written once; a
    multiply and an add per weight and column."""
    s = case["sparsity"]
    if case["op"] == "conv":
        n = case["H"] * case["W"] * case["NB"]
        nnz = _nnz(case["OC"], case["IC"] * 9, s)
        return {"bytes": 8 * nnz + 4 * n * (case["IC"] + case["OC"]) + 4 * case["OC"],
                "flops": 2 * nnz * n}
    if case["op"] == "encoder":
        H, F, n = case["H"], case["F"], case["N"]
        shapes = [(H, H)] * 4 + [(F, H), (H, F)]
    else:
        shapes, n = [(case["M"], case["K"])], case["N"]
    nnz = [_nnz(M, K, s) for M, K in shapes]
    return {"bytes": sum(8 * z + 4 * n * (M + K) + 4 * M for z, (M, K) in zip(nnz, shapes)),
            "flops": sum(2 * z * n for z in nnz)}


def tolerance(case):
    """32-bit sums of up to about a thousand terms.  Measured against exact(): at most 4.4e-7
    in the 2-norm and 4.2e-6 at one element over the listed cases and ten drawn ones, the
    six chained products of the encoder layer included; stated at about four times that."""
    return {"rel": 2e-6, "max": 2e-5}


# ---- the same in 64 bits --------------------------------------------------------------


def _epilogue64(Y, epi):
    if epi == "relu":
        return Y.clamp(min=0.0)
    if epi == "gelu":
        return 0.5 * Y * (1.0 + torch.erf(Y / math.sqrt(2.0)))
    return Y


def exact(case, seed):
    X = _activations(case, seed).double()
    if case["op"] == "conv":  # rows of the virtual operand: channel, tap row, tap column
        IC, H, W, NB = X.shape
        P = torch.zeros((IC, H + 2, W + 2, NB), dtype=torch.float64, device=DEV)
        P[:, 1:-1, 1:-1] = X
        taps = [P[:, y:y + H, x:x + W] for y in range(3) for x in range(3)]
        X2 = torch.stack(taps, dim=1).reshape(IC * 9, H * W * NB)
        (csr, M, K, bias, epi), = _host_inputs(case, seed)
        Y = _dense64(csr, M, K) @ X2
        if bias is not None:
            Y += torch.from_numpy(bias).to(DEV).double()[:, None]
        return _epilogue64(Y, epi).reshape(M, H, W, NB)
    for csr, M, K, bias, epi in _host_inputs(case, seed):
        X = _dense64(csr, M, K) @ X
        if bias is not None:
            X += torch.from_numpy(bias).to(DEV).double()[:, None]
        X = _epilogue64(X, epi)
    return X
