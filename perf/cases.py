"""Workloads of the Bi-Mask hot path, for timing through the public calls of `paper_2302_06058_amd`.

Three kinds of work occur in training with N:M masks in both directions:

  layer    one linear / convolution-as-matrix-product layer, the whole step of Alg. 1: forward mask, forward
           product, (when it is due) permutation search, backward mask, backward product.  The search runs once
           in a hundred steps, so most layer cases leave it out.
  weights  the weight side of a search step alone: forward mask, search, backward mask (large matrices, where a
           program refreshes the masks apart from the products).
  network  the same for all layers of a network: masks and searches through the grouped calls, the products layer
           by layer, or (acts = False) the weight side alone.

Sizes are those of this repository's five configurations (`paper_2302_06058_amd/synth.py`).  `prepare` makes what a
training program holds before the step -- weights, activations, gradients, candidates, the layer's mask, operand and
workspace buffers --, `run` issues one step on the current stream; Y and dX of single layers are allocated by the
calls, as activations are.
"""
import math

import torch

import paper_2302_06058_amd as bm
from paper_2302_06058_amd import synth


def listed():
    def layer(name, I, J, T, N=2, M=4, K=0, dtype="bf16", relu=False, pad=0):
        return dict(name=name, op="layer", dtype=dtype, N=N, M=M, I=I, J=J, T=T, K=K, relu=relu, pad=pad)

    return [
        # the smallest step: one fp32 layer with a search over 4 candidates; five calls, bound by latency
        layer("linear-f32-step", 64, 128, 32, K=4, dtype="f32"),
        # the classifier of a ResNet-50 at batch 64: ragged output width, few tokens, weights dominate
        layer("head-train", 1000, 2048, 64, relu=True),
        # stem convolution 7x7 over 112 x 112 positions: 147 inputs padded by one zero column, the most tokens
        layer("stem-train", 64, 148, 802816, pad=1),
        # 3x3 convolution of the first stage: many tokens, narrow weights
        layer("conv3x3-early-train", 64, 576, 200704, relu=True),
        # 3x3 convolution of the third stage: the ordinary convolution
        layer("conv3x3-mid-train", 256, 2304, 12544, relu=True),
        # attention projections of a small vision transformer at 128 images
        layer("qkv-2of4-train", 1152, 384, 25216),
        # its first MLP matrix at the ratio that runs on dense matrix instructions
        layer("fc1-4of8-train", 1536, 384, 25216, N=4, M=8),
        # its second MLP matrix at 1:4: long contraction forward, wide output backward
        layer("fc2-1of4-train", 384, 1536, 25216, N=1),
        # a large transformer MLP matrix, search step: the largest single layer
        layer("mlp-up-step", 11008, 4096, 8192, K=100),
        # masks and search of the other MLP matrix, without products
        dict(name="mlp-down-weights", op="weights", dtype="bf16", N=2, M=4, I=4096, J=11008, K=100),
        # masks and searches of all 54 matrices of a ResNet-50 through the grouped calls
        dict(name="resnet50-weights", op="network", net="resnet50", depth=1, batch=64, N=2, M=4, K=100, acts=False),
        # a whole training pass over the 54 matrices (no search due): grouped masks, every product
        dict(name="resnet50-train", op="network", net="resnet50", depth=1, batch=64, N=2, M=4, K=0, acts=True),
    ]


RATIOS = ((2, 4), (2, 4), (2, 4), (2, 4), (1, 4), (4, 8), (4, 8), (2, 8), (1, 16))


def draw(rng):
    def size(lo, hi, multiple):
        """Spread over the logarithm; two thirds on multiples of 32, the others on the smallest step allowed."""
        v = math.exp(rng.uniform(math.log(lo), math.log(hi)))
        step = multiple if rng.random() < 1 / 3 else max(32, multiple)
        return max(step, round(v / step) * step)

    def tokens(lo, hi, I, J):
        cap = min(hi, 802816 * 212 // (I + J), 8192 * 11008 * 4096 // (I * J))
        return max(1, round(math.exp(rng.uniform(math.log(lo), math.log(max(lo, cap))))))

    kind = rng.choice(("conv", "conv", "conv", "linear", "linear", "mlp", "f32", "head", "weights", "network"))
    N, M = rng.choice(RATIOS)
    c = dict(op="layer", dtype="bf16", N=N, M=M, K=0, relu=False, pad=0)
    if kind == "conv":
        c.update(I=size(32, 2048, M), J=size(64, 4608, M), relu=True)
        c["T"] = tokens(784, 802816, c["I"], c["J"])
        c["K"] = rng.choice((0, 0, 0, 100))
    elif kind == "linear":
        c.update(I=size(192, 2048, M), J=size(192, 2048, M))
        c["T"] = tokens(1024, 32768, c["I"], c["J"])
    elif kind == "mlp":
        c.update(I=size(2048, 11008, M), J=size(2048, 11008, M))
        c["T"] = tokens(1024, 8192, c["I"], c["J"])
        c["K"] = rng.choice((0, 100))
    elif kind == "f32":
        c.update(dtype="f32", I=size(32, 512, M), J=size(32, 512, M), T=round(math.exp(rng.uniform(math.log(8), math.log(512)))))
        c["K"] = rng.randint(1, 16)
    elif kind == "head":
        c.update(I=size(64, 4096, M), J=size(256, 4096, M), T=rng.randint(1, 256))
    elif kind == "weights":
        c = dict(op="weights", dtype="bf16", N=N, M=M, I=size(256, 11008, M), J=size(256, 11008, M), K=rng.randint(16, 100))
        c["J"] = min(c["J"], 11008 * 4096 // c["I"] // M * M)
    else:
        net = rng.choice(("resnet50", "deit")) if M <= 8 else "deit"
        acts = rng.random() < 0.5
        c = dict(op="network", net=net, N=N, M=M, K=rng.choice((0, 100)), acts=acts,
                 depth=1 if net == "resnet50" else rng.randint(1, 12), batch=rng.randint(1, 16))
    return c


def _layers(case):
    """[(I, J, T, std of W, relu, zero columns)] of a case, in the order of the forward pass."""
    if case["op"] != "network":
        J = case["J"]
        std = math.sqrt(2.0 / J) if case.get("relu") or case.get("pad") else 0.02
        return [(case["I"], J, case.get("T", 0), std, bool(case.get("relu")), case.get("pad", 0))]
    M, out = case["M"], []
    if case["net"] == "resnet50":
        for name, I, J, T in synth.resnet50_gemm_shapes(case["batch"]):
            Jp = -(-J // M) * M
            out.append((I, Jp, T, math.sqrt(2.0 / J), name != "stem.conv7x7", Jp - J))
    else:
        for _ in range(case["depth"]):
            for I, J in ((1152, 384), (384, 384), (1536, 384), (384, 1536)):
                out.append((I, J, 197 * case["batch"], 0.02, False, 0))
    return out


def _acts(case):
    return case["op"] == "layer" or (case["op"] == "network" and case["acts"])


def prepare(case, seed):
    dt = torch.float32 if case.get("dtype") == "f32" else torch.bfloat16
    code = bm.F32 if dt == torch.float32 else bm.BF16
    N, M, K, layers, acts = case["N"], case["M"], case["K"], _layers(case), _acts(case)
    dev = torch.device("cuda")
    g = torch.Generator(device=dev)
    g.manual_seed(seed)

    def normal(rows, cols, std):
        return torch.empty((rows, cols), dtype=dt, device=dev).normal_(0.0, std, generator=g)

    def flat(sizes, dtype):
        """One allocation cut into 16-byte aligned pieces (a network keeps the buffers of its layers together)."""
        unit = 16 // torch.empty((), dtype=dtype).element_size()
        starts, at = [], 0
        for n in sizes:
            starts.append(at)
            at += -(-n // unit) * unit
        buf = torch.zeros((max(at, unit),), dtype=dtype, device=dev)
        return buf, [buf[a:a + n] for a, n in zip(starts, sizes)]

    state = dict(case=dict(case), code=code, N=N, M=M, K=K, layers=[])
    bufs = {}

    def kept(name, sizes, dtype):
        bufs[name], pieces = flat(sizes, dtype)
        return pieces

    shapes = [(I, J) for I, J, *_ in layers]
    B = kept("B", [I * bm.mask_words(J) for I, J in shapes], torch.int32)
    Bbar = kept("Bbar", [I * bm.mask_words(J) for I, J in shapes], torch.int32)
    vf = kept("vf", [bm.operand_elems(I, J, N, M) for I, J in shapes], dt)
    vb = kept("vb", [bm.operand_elems(J, I, N, M) for I, J in shapes], dt)
    if N <= 2:
        xf = kept("xf", [bm.operand_index_words(I, J, N, M) for I, J in shapes], torch.int32)
        xb = kept("xb", [bm.operand_index_words(J, I, N, M) for I, J in shapes], torch.int32)
    else:
        xf = xb = [None] * len(shapes)
    P = kept("P", [I for I, _ in shapes], torch.int32)
    if K:
        scores, best = kept("scores", [K] * len(shapes), torch.int32), kept("best", [1] * len(shapes), torch.int32)
    if acts and case["op"] == "network":
        Y = kept("Y", [T * I for I, _, T, *_ in layers], dt)
        dX = kept("dX", [T * J for _, J, T, *_ in layers], dt)

    ws_bwd = 16                                          # one scratch buffer serves the backward products in turn
    for l, (I, J, T, std, relu, pad) in enumerate(layers):
        W = normal(I, J, std)
        e = dict(I=I, J=J, W=W, B_bits=B[l].view(I, -1), Wf_values=vf[l], Wf_index=xf[l],
                 Bbar_bits=Bbar[l].view(I, -1), Wb_values=vb[l], Wb_index=xb[l], best_perm=P[l], X=None, dY=None, Y=None, dX=None)
        if pad:
            W[:, J - pad:] = 0
        if K:
            e["perms"] = torch.rand((K, I), device=dev, generator=g).argsort(dim=1).to(torch.int32)
            e["scores"], e["best"] = scores[l], best[l]
            need = bm.workspace_bytes(bm.WS_PERM_SEARCH, I, J, 0, K, code, N, M)
            e["workspace"] = torch.empty((max(16, need),), dtype=torch.uint8, device=dev)
        else:                                            # the permutation an earlier search found
            P[l].copy_(torch.rand((I,), device=dev, generator=g).argsort())
        if acts:
            e["X"], e["dY"] = normal(T, J, 1.0), normal(T, I, 1e-2)
            if relu:
                e["X"].relu_()
            if pad:
                e["X"][:, J - pad:] = 0
            ws_bwd = max(ws_bwd, bm.workspace_bytes(bm.WS_GEMM_BWD, I, J, T, 0, code, N, M))
            if case["op"] == "network":
                e["Y"], e["dX"] = Y[l].view(T, I), dX[l].view(T, J)
        state["layers"].append(e)
    state["ws_bwd"] = torch.empty((ws_bwd,), dtype=torch.uint8, device=dev)
    state["bufs"] = bufs
    if case["op"] == "network":
        keys = ("W", "B_bits", "Wf_values", "Wf_index", "perms", "scores", "best", "best_perm", "workspace",
                "Bbar_bits", "Wb_values", "Wb_index")
        state["group"] = bm.group_layers([{k: e.get(k) for k in keys} for e in state["layers"]])
    return state


def run(state):
    N, M, K, bufs = state["N"], state["M"], state["K"], state["bufs"]

    def product_fwd(e):
        return bm.bimask_sparse_gemm_fwd(e["X"], e["Wf_values"], e["Wf_index"], e["I"], e["J"], N, M, Y=e["Y"])

    def product_bwd(e):
        return bm.bimask_sparse_gemm_bwd(e["dY"], e["best_perm"], e["Wb_values"], e["Wb_index"], e["I"], e["J"], N, M,
                                         dX=e["dX"], workspace=state["ws_bwd"])

    if state["case"]["op"] == "network":
        group, acts = state["group"], state["case"]["acts"]
        bm.bimask_forward_mask_compress_group(group, state["code"], N, M)
        if acts:
            for e in state["layers"]:
                product_fwd(e)
        if K:
            bm.bimask_perm_search_group(group, N, M, K)
        bm.bimask_backward_mask_compress_group(group, state["code"], N, M)
        if acts:
            for e in reversed(state["layers"]):
                product_bwd(e)
        return bufs

    e = state["layers"][0]
    out = dict(bufs)
    bm.bimask_forward_mask_compress(e["W"], N, M, B_bits=e["B_bits"], values=e["Wf_values"], index=e["Wf_index"])
    if e["X"] is not None:
        out["Y"] = product_fwd(e)
    if K:
        bm.bimask_perm_search(e["B_bits"], e["I"], e["J"], N, M, e["perms"], scores=e["scores"], best=e["best"],
                              best_perm=e["best_perm"], workspace=e["workspace"])
    bm.bimask_backward_mask_compress(e["W"], N, M, e["B_bits"], e["best_perm"], Bbar_bits=e["Bbar_bits"],
                                     values=e["Wb_values"], index=e["Wb_index"])
    if e["dY"] is not None:
        out["dX"] = product_bwd(e)
    return out


def work(case):
    """Inputs read once, outputs written once; multiplications by kept weights only (N of M)."""
    esz = 4 if case.get("dtype") == "f32" else 2
    N, M, K = case["N"], case["M"], case["K"]
    nbytes = flops = 0
    for I, J, T, *_ in _layers(case):
        nbytes += esz * I * J + 2 * 4 * I * bm.mask_words(J)                  # W; B and Bbar
        keep = 0.5 if N <= 2 else 1.0                                         # operand values per weight
        nbytes += 2 * int(keep * esz * I * J) + (2 * I * J // 8 if N <= 2 else 0)
        nbytes += 4 * I + (4 * K * I + 4 * K + 4 if K else 0)                 # permutation; candidates, scores, best
        if _acts(case):
            nbytes += 2 * esz * T * (I + J)                                   # X, dY, Y, dX
            flops += 2 * 2 * T * I * J * N // M
    return dict(bytes=nbytes, flops=flops)


def tolerance(case):
    if not _acts(case):
        return "exact"                                   # masks, scores, permutations, operands: integers and copies
    # Products with fp32 accumulation.  Against the same products in float64 the path measures, over all listed cases,
    # 1.7e-3 / 3.9e-3 (norm / largest) in bf16 -- the rounding of the output -- and 1.4e-7 / 6.4e-7 in fp32 with 128
    # terms (about twice that with 512); stated are about four times these.
    return {"rel": 1.2e-6, "max": 1e-5} if case.get("dtype") == "f32" else {"rel": 6e-3, "max": 1.6e-2}
