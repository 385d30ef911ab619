"""Workloads of the library as its users run it: what they have in hand, one pass, and what the pass cannot do without.

Six paths, each over the range of sizes that it meets (`draw` gives more cases of the same ranges):

  encode       inference: the four pruned linear layers of one encoder layer (QKV, attention output + residual, FFN up +
               GELU, FFN down + residual) through the plan that a server builds once per model
  compact      a layer straight on its compact storage, without a plan: a model that is run once or whose values change
  backward     retraining with a fixed mask: a layer's input gradient and the gradient of its kept weights
  update       one weight update: with the regulariser's gradient and fresh reweighting factors, or masked
  prune_layer  one-shot pruning of an encoder layer's matrices: norms, percentile, compact storage, plan, masked weights,
               and a calibration batch through the new plan
  prune_model  the same decision over all weights of a model at once, and the compact storage of all of them

Shapes are BERT-base and BERT-large's (768 / 3072 and 1024 / 4096) and smaller encoders of the same proportions; rates
are the paper's range, 1.43x to 5x; weights and biases are N(0, 0.02), activations N(0, 1).
"""
import ctypes
import math

import torch

import paper_2009_08065_amd as bsp

_DT = {"f32": torch.float32, "bf16": torch.bfloat16, "f16": torch.float16}
_RATES = (1.4285, 1.5, 2.0, 3.0, 5.0)
_HIDDEN = (256, 384, 512, 640, 768, 896, 1024)


def listed():
    return [
        # one short request at a server: 24 tokens, where launches and latency are all there is
        dict(name="encode_short", path="encode", hidden=768, ffn=3072, tokens=24, R=16, rate=2.0, dtype="bf16"),
        # a ragged batch of medium size, the other 16-bit type, the lowest block height
        dict(name="encode_ragged", path="encode", hidden=768, ffn=3072, tokens=1537, R=8, rate=3.0, dtype="f16"),
        # the benchmark's configuration: 64 sequences of 128 tokens
        dict(name="encode_batch", path="encode", hidden=1024, ffn=4096, tokens=8192, R=16, rate=5.0, dtype="bf16"),
        # the paper's standard operating point (30 % sparsity) in high blocks
        dict(name="encode_dense", path="encode", hidden=1024, ffn=4096, tokens=4099, R=32, rate=1.4285, dtype="bf16"),
        # one sequence through a single-precision attention projection
        dict(name="compact_f32", path="compact", M=768, N=768, tokens=128, R=16, rate=2.0, dtype="f32"),
        # an FFN up-projection in training, its values new in every step
        dict(name="compact_bf16", path="compact", M=3072, N=768, tokens=4096, R=16, rate=3.0, dtype="bf16"),
        # a small ragged batch in retraining
        dict(name="backward_small", path="backward", M=2304, N=768, tokens=509, R=8, rate=2.0, dtype="f16", grad="f32"),
        # a full batch in retraining
        dict(name="backward_batch", path="backward", M=4096, N=1024, tokens=8192, R=16, rate=5.0, dtype="bf16", grad="f32"),
        # a step of reweighted training on one projection
        dict(name="update_mixed", path="update", M=1024, N=1024, R=16, mixed=True, grad="f32"),
        # a step of retraining on the up-projections of six layers in one buffer, gradients in bf16
        dict(name="update_masked", path="update", M=24576, N=1024, R=16, mixed=False, grad="bf16"),
        # one encoder layer pruned at its own rate
        dict(name="prune_layer", path="prune_layer", hidden=768, ffn=3072, R=16, rate=3.0, dtype="bf16", tile=0),
        # a 24-layer model's 302 million weights under one global percentile
        dict(name="prune_model", path="prune_model", hidden=1024, ffn=4096, layers=24, R=16, rate=5.0),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    path = rng.choice(("encode", "encode", "compact", "backward", "update", "prune_layer", "prune_model"))
    R, rate, low = rng.choice((8, 16, 16, 16, 32)), rng.choice(_RATES), rng.choice(("bf16", "bf16", "f16"))
    h = rng.choice(_HIDDEN)
    M, N = rng.choice(((3 * h, h), (h, h), (4 * h, h), (h, 4 * h)))
    if path == "encode":
        return dict(path=path, hidden=h, ffn=4 * h, tokens=_log(rng, 8, 8192), R=R, rate=rate, dtype=low)
    if path == "compact":
        t = rng.choice(("f32", low, low))
        return dict(path=path, M=M, N=N, tokens=_log(rng, 16, 1024 if t == "f32" else 8192), R=R, rate=rate, dtype=t)
    if path == "backward":
        return dict(path=path, M=M, N=N, tokens=_log(rng, 64, 8192), R=R, rate=rate, dtype=low, grad=rng.choice(("f32", low)))
    if path == "update":
        return dict(path=path, M=M * _log(rng, 1, 8), N=N, R=R, mixed=rng.random() < 0.5, grad=rng.choice(("f32", "bf16")))
    if path == "prune_layer":
        return dict(path=path, hidden=h, ffn=4 * h, R=R, rate=rate, dtype=low, tile=rng.choice((0, 0, 32)))
    return dict(path=path, hidden=h, ffn=4 * h, layers=rng.randint(2, 24), R=R, rate=rate)


def _normal(gen, shape, std, dtype):
    x = torch.empty(shape, dtype=torch.float32, device="cuda").normal_(0.0, std, generator=gen)
    return x if dtype == torch.float32 else x.to(dtype)


def _keep_count(groups, rate):
    return int(groups / rate)


def _capacity(M, N, R, rate):
    """Columns that hold the storage (k_align = 32) of any mask of this rate over M x N weights."""
    return min(_keep_count(M // R * N, rate) + 31 * (M // R), M // R * (N + 31))


def _shapes(case):
    h, f = case["hidden"], case["ffn"]
    return [(3 * h, h), (h, h), (f, h), (h, f)]


def _pruned(gen, M, N, R, rate, dtype):
    """A pruned layer's compact storage and bias."""
    W = _normal(gen, (M, N), 0.02, dtype)
    sumsq, _, _ = bsp.bsp_group_norms(W, R, want=("sumsq",))
    keep, _ = bsp.bsp_prune_mask(sumsq, n_keep=_keep_count(sumsq.numel(), rate), scope=bsp.SCOPE_MATRIX)
    return bsp.bsp_pack(W, R, keep, 32), _normal(gen, (M,), 0.02, dtype)


def prepare(case, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    path, R = case["path"], case["R"]
    s = dict(case=case)
    if path == "encode":
        dt, T, h = _DT[case["dtype"]], case["tokens"], case["hidden"]
        s["layers"] = []
        for M, N in _shapes(case):
            packed, bias = _pruned(gen, M, N, R, case["rate"], dt)
            s["layers"].append((packed, bsp.bsp_linear_plan(packed), bias))
        s["x"], s["context"] = _normal(gen, (T, h), 1.0, dt), _normal(gen, (T, h), 1.0, dt)
    elif path == "compact":
        dt = _DT[case["dtype"]]
        s["packed"], s["bias"] = _pruned(gen, case["M"], case["N"], R, case["rate"], dt)
        s["x"] = _normal(gen, (case["tokens"], case["N"]), 1.0, dt)
    elif path == "backward":
        dt = _DT[case["dtype"]]
        p, _ = _pruned(gen, case["M"], case["N"], R, case["rate"], dt)
        s["packed"] = p
        s["x"], s["dy"] = _normal(gen, (case["tokens"], p.N), 1.0, dt), _normal(gen, (case["tokens"], p.M), 0.01, dt)
        # the mask is fixed during retraining: the first step builds the work list, later ones reuse it
        need = bsp.lib().bsp_linear_dvals_workspace_bytes(p.M, p.N, p.R, p.total_cols)
        s["ws"] = torch.empty(max(need, 256), dtype=torch.uint8, device="cuda")
        # and the gradient's buffer is kept too, large enough for any mask of this rate
        s["d"] = torch.zeros(R * _capacity(p.M, p.N, R, case["rate"]), dtype=_DT[case["grad"]], device="cuda")
        bsp.bsp_linear_dvals(s["x"], s["dy"], p, D=s["d"], ws=s["ws"], ws_state=bsp.DVALS_BUILD)
    elif path == "update":
        M, N = case["M"], case["N"]
        s["w"], s["g"] = _normal(gen, (M, N), 0.02, torch.float32), _normal(gen, (M, N), 1e-3, _DT[case["grad"]])
        s["m"] = _normal(gen, (M, N), 1e-3, torch.float32)
        s["v"] = _normal(gen, (M, N), 1e-3, torch.float32).square_()
        if not case["mixed"]:
            sumsq, _, _ = bsp.bsp_group_norms(s["w"], R, want=("sumsq",))
            s["keep"], _ = bsp.bsp_prune_mask(sumsq, n_keep=_keep_count(sumsq.numel(), 2.0), scope=bsp.SCOPE_MATRIX)
    elif path == "prune_layer":
        dt = _DT[case["dtype"]]
        s["w"] = [_normal(gen, shape, 0.02, dt) for shape in _shapes(case)]
        s["x"] = {N: _normal(gen, (128, N), 1.0, dt) for N in (case["hidden"], case["ffn"])}
    else:
        h, f, n = case["hidden"], case["ffn"], case["layers"]
        # matrices of one width stacked along their rows, as a flat parameter buffer holds them
        s["w"] = [_normal(gen, (n * (4 * h + f), h), 0.02, torch.float32), _normal(gen, (n * h, f), 0.02, torch.float32)]
        s["grad"] = [torch.empty_like(w) for w in s["w"]]
        # a pruning run allocates its storage once, for whatever share of the percentile falls to a stack
        n_keep = _keep_count(sum(w.numel() // R for w in s["w"]), case["rate"])
        s["store"] = []
        for w in s["w"]:
            B, N = w.shape[0] // R, w.shape[1]
            cap = min(n_keep, B * N) + 31 * B
            s["store"].append((cap, torch.empty(B, dtype=torch.int32, device="cuda"),
                               torch.empty(B + 1, dtype=torch.int32, device="cuda"),
                               torch.zeros(cap, dtype=torch.int32, device="cuda"),
                               torch.zeros(R * cap, dtype=torch.bfloat16, device="cuda")))
    return s


def _add_layer(x, layer, act=bsp.ACT_NONE, residual=None):
    """One planned layer with its epilogue; a residual the layer kernel does not fuse is a pass of its own."""
    packed, plan, bias = layer
    if residual is None and act == bsp.ACT_NONE:
        return bsp.bsp_linear_planned(x, packed, plan, bias)
    if residual is not None and not (packed.N > 1024 or (packed.N > 512 and packed.M <= 1024)):
        return bsp.bsp_linear_planned(x, packed, plan, bias).add_(residual)
    return bsp.bsp_linear_planned_fused(x, packed, plan, bias, act=act, residual=residual)


def _prune_one(w, x, R, rate, tile):
    sumsq, _, _ = bsp.bsp_group_norms(w, R, want=("sumsq",))
    if tile:
        tiles = bsp.bsp_tile_sumsq(sumsq, tile)
        kept, t = bsp.bsp_prune_mask(tiles, n_keep=_keep_count(tiles.numel(), rate), scope=bsp.SCOPE_MATRIX, want_t_used=True)
        keep = bsp.bsp_expand_tile_mask(kept, tile)
        cnt, ptr = bsp.bsp_pack_count(keep, 32)
    else:
        t = torch.empty(1, dtype=torch.float32, device="cuda")
        keep, _, cnt, ptr = bsp.bsp_prune_mask_count(sumsq, n_keep=_keep_count(sumsq.numel(), rate), scope=bsp.SCOPE_MATRIX,
                                                     k_align=32, t_used=t)
    packed = bsp.bsp_pack(w, R, keep, 32, blk_cnt=cnt, blk_ptr=ptr)
    plan = bsp.bsp_linear_plan(packed)
    bsp.bsp_mask_weights(w, R, keep)
    y = bsp.bsp_linear_planned(x, packed, plan)
    # (the storage's own size differs from mask to mask; what it holds shows in the layer's output)
    return dict(sumsq=sumsq, t=t, keep=keep, cnt=cnt, ptr=ptr, w=w, y=y)


def _pack_into(w, R, keep, store):
    """bsp_pack through the C interface, into buffers that the caller holds."""
    cap, cnt, ptr, col, vals = store
    bsp.bsp_pack_count(keep, 32, blk_cnt=cnt, blk_ptr=ptr)
    at = [ctypes.c_void_p(a.data_ptr()) for a in (w, keep, cnt, ptr, col, vals)]
    stream = ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)
    st = bsp.lib().bsp_pack(at[0], bsp.F32, w.shape[0], w.shape[1], R, at[1], 32, at[2], at[3], cap, at[4], at[5], bsp.BF16, stream)
    if st != 0:
        raise bsp.BspError(st, "bsp_pack")
    return cnt, ptr, col, vals


def run(s):
    case = s["case"]
    path, R = case["path"], case["R"]
    if path == "encode":
        qkv, out, up, down = s["layers"]
        a = _add_layer(s["x"], qkv)
        b = _add_layer(s["context"], out, residual=s["x"])
        c = _add_layer(b, up, act=bsp.ACT_GELU)
        return a, b, c, _add_layer(c, down, residual=b)
    if path == "compact":
        return bsp.bsp_linear(s["x"], s["packed"], s["bias"])
    if path == "backward":
        dx = bsp.bsp_linear_transposed(s["dy"], s["packed"])
        return dx, bsp.bsp_linear_dvals(s["x"], s["dy"], s["packed"], D=s["d"], ws=s["ws"], ws_state=bsp.DVALS_REUSE)
    if path == "update":
        if case["mixed"]:
            _, _, alpha = bsp.bsp_group_norms(s["w"], R, want=("alpha",))
            bsp.bsp_adam_step(s["w"], s["g"], s["m"], s["v"], R, 3e-5, t=100, alpha=alpha, lam=1e-4)
            return alpha, s["w"], s["m"], s["v"]
        bsp.bsp_adam_step(s["w"], s["g"], s["m"], s["v"], R, 3e-5, t=100, keep=s["keep"])
        return s["w"], s["m"], s["v"]
    if path == "prune_layer":
        # the weights stay as they came for the next pass: a pass prunes a copy, as a sweep over rates does
        return [_prune_one(w.clone(), s["x"][w.shape[1]], R, case["rate"], case["tile"]) for w in s["w"]]
    ws, grads = s["w"], s["grad"]
    groups = [w.numel() // R for w in ws]
    sumsq = torch.empty(sum(groups), dtype=torch.float32, device="cuda")
    parts = [a.view(w.shape[0] // R, w.shape[1]) for a, w in zip(sumsq.split(groups), ws)]
    alphas = [bsp.bsp_group_norms_grad(w, R, 1e-4, sumsq=part, grad=g)[2] for w, part, g in zip(ws, parts, s["grad"])]
    keep, t = bsp.bsp_prune_mask(sumsq.view(1, -1), n_keep=_keep_count(sumsq.numel(), case["rate"]), scope=bsp.SCOPE_MATRIX,
                                 want_t_used=True)
    stored = [_pack_into(w, R, k.view(w.shape[0] // R, w.shape[1]), store)
              for w, k, store in zip(ws, keep.view(-1).split(groups), s["store"])]
    return dict(sumsq=sumsq, alpha=alphas, grad=s["grad"], t=t, keep=keep, stored=stored)


def _size(dtype):
    return 4 if dtype == "f32" else 2


def work(case):
    path, R = case["path"], case["R"]
    if path == "encode":
        T, h, e = case["tokens"], case["hidden"], 2
        kept = [M * N / case["rate"] for M, N in _shapes(case)]
        weights = sum(k * (e + 4 / R) for k in kept) + e * sum(M for M, _ in _shapes(case))
        # each layer's input and output once, and the two residuals
        acts = e * T * (sum(M + N for M, N in _shapes(case)) + 2 * h)
        return dict(bytes=weights + acts, flops=2.0 * T * sum(kept))
    if path in ("compact", "backward"):
        M, N, T, e = case["M"], case["N"], case["tokens"], _size(case["dtype"])
        kept = M * N / case["rate"]
        if path == "compact":
            return dict(bytes=e * T * (M + N) + kept * (e + 4 / R) + e * M, flops=2.0 * T * kept)
        return dict(bytes=e * T * (M + 2 * N) + kept * (e + _size(case["grad"]) + 4 / R), flops=4.0 * T * kept)
    if path == "update":
        n = case["M"] * case["N"]
        # weights and both moments read and written, the gradient read; the factors written, or the mask read
        return dict(bytes=n * (24 + _size(case["grad"]) + (4 / R if case["mixed"] else 1 / R)), flops=14.0 * n)
    if path == "prune_layer":
        n, e = sum(M * N for M, N in _shapes(case)), 2
        h, f = case["hidden"], case["ffn"]
        kept = n / case["rate"]
        # read the weights, write them masked, their sums and flags, the storage; the calibration batch
        return dict(bytes=n * (2 * e + 5 / R) + kept * (e + 4 / R) + e * 128 * (3 * h + f + sum(M for M, _ in _shapes(case))),
                    flops=2.0 * n + 2.0 * 128 * kept)
    n = case["layers"] * (4 * case["hidden"] ** 2 + 2 * case["hidden"] * case["ffn"])
    # read the weights once, write gradient, sums, factors and flags, and the storage in bf16
    return dict(bytes=n * (8 + 9 / R) + n / case["rate"] * (2 + 4 / R), flops=3.0 * n)


def tolerance(case):
    # norms, factors, gradients of the regulariser, masks, storage and updates are defined operation by operation
    if case["path"] in ("update", "prune_model"):
        return "exact"
    if case["dtype"] == "f32":
        return dict(rel=1e-5)
    # against sums in 64 bits: bf16 1.7e-3 for one product and 2.4e-3 through an encoder layer, fp16 an eighth of that
    return dict(rel=1e-2 if case["dtype"] == "bf16" else 1.2e-3, max=0.06)
