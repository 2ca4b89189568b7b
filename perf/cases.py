"""The work that users of this library have it do, as a set of measurable cases.

A case is a dict of plain values.  ``kind`` names the entry points a pass goes through:

* ``forward``   moe.layer_forward: serving (decode and prefill) and evaluation, bf16 or fp32, with or without a
                capacity and an always-on shared expert;
* ``train``     moe.layer_forward_train and moe.layer_backward: one micro-batch of a training step; ``relayout``
                adds moe.expert_weights_transpose, which a program pays for whenever the weights have changed since
                the last micro-batch (no gradient accumulation);
* ``fp8``       moe.router_topk, moe.permute_fp8, moe.grouped_gemm_swiglu_fp8, moe.unpermute_combine: the E4M3
                expert FFN with delayed scaling, weights quantised beforehand;
* ``ep_share``  moe.sort_chunks, moe.grouped_gemm_swiglu, moe.sort_chunks: what one GPU of an expert-parallel group
                does between the two exchanges.

The layer shapes are those of moe_inputs.configs, or generic.  Values follow the same recipe: tokens N(0, 1), weights
N(0, 0.02^2), a per-expert logit bias N(0, 1) or Zipf-like for skewed routing.
"""
from __future__ import annotations

import functools
import math

import torch

import paper_2504_14960_amd as moe
from moe_inputs import get_config

WEIGHT_STD = 0.02


def _shape(config: str, **kw) -> dict:
    c = get_config(config)
    case = dict(T=c.T, H=c.H, E=c.E, K=c.K, F=c.F, dtype=c.dtype, renormalize=c.renormalize, bias=c.bias or "none",
                capacity_factor=c.capacity_factor or 0.0, shared_F=c.shared_F)
    case.update(kw)
    return case


def listed():
    return [
        # one sequence being decoded: launches and the weight stream of the two selected experts
        dict(name="decode_1_8x7b", kind="forward", **_shape("mixtral8x7b", T=1)),
        # a batch of sequences being decoded by a fine-grained layer with a shared expert: about every expert is
        # selected, each by a few tokens
        dict(name="decode_64_qwen2", kind="forward", **_shape("qwen2_57b_a14b", T=64)),
        # the fp32 layer of the parity configuration (debugging, reference runs): latency of a small call
        dict(name="tiny_f32", kind="forward", **_shape("tiny")),
        # sizes that are multiples of 8 only, a capacity above one, an odd number of tokens and experts
        dict(name="odd_777", kind="forward",
             **_shape("mixtral8x7b", T=777, H=1000, E=12, K=3, F=1416, bias="normal", capacity_factor=1.25)),
        # a short prompt: some sixty rows per expert
        dict(name="prefill_500_qwen2", kind="forward", **_shape("qwen2_57b_a14b", T=500)),
        # the benchmark's layer: long prompts or a forward-only pass over 2 x 4096 tokens
        dict(name="prefill_8192_8x22b", kind="forward", **_shape("mixtral8x22b")),
        # many tokens on 64 experts with a strongly skewed router, token drop at capacity factor 1
        dict(name="tokendrop_32768", kind="forward", **_shape("tokendrop")),
        # one micro-batch of training at the benchmark's layer (gradient accumulation: weights laid out once)
        dict(name="train_8192_8x22b", kind="train", relayout=False, **_shape("mixtral8x22b")),
        # a smaller micro-batch on the fine-grained layer, token drop, weights updated after every micro-batch
        dict(name="train_2048_g8t8", kind="train", relayout=True, **_shape("mixtral8x22b_g8t8", T=2048)),
        # the FP8 forward at the benchmark's layer
        dict(name="fp8_8192_8x22b", kind="fp8", **_shape("mixtral8x22b")),
        # a batch of sequences being decoded with FP8 weights
        dict(name="fp8_decode_32_8x7b", kind="fp8", **_shape("mixtral8x7b", T=32)),
        # one GPU's share of an 8-rank expert-parallel group of the fine-grained layer, 4096 tokens per rank
        dict(name="ep8_share_g8t8", kind="ep_share", ranks=8, **_shape("mixtral8x22b_g8t8", T=4096, capacity_factor=0.0)),
    ]


def _log_int(rng, lo, hi) -> int:
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _cost(case) -> float:
    w = work(case)
    return max(w["flops"] / 1e15, w["bytes"] / 4e12)


@functools.lru_cache(maxsize=None)
def _largest_listed() -> float:
    return max(_cost(c) for c in listed())


def draw(rng):
    """One more case of the same ranges: kinds in turn, tokens and sizes over their logarithm, odd ones among them."""
    while True:
        kind = rng.choice(["decode", "decode", "prefill", "prefill", "f32", "odd", "train", "fp8", "fp8", "ep_share"])
        E, K = rng.choice([(4, 1), (8, 2), (8, 1), (12, 3), (16, 2), (16, 4), (32, 4), (60, 4), (64, 6), (64, 8), (128, 8)])
        H = 128 * rng.randint(8, 56)                               # 1024 .. 7168
        F = 128 * _log_int(rng, 6, 128 if E <= 16 else 24)         # 768 .. 16384 (few experts) or 3072 (many)
        case = dict(kind="forward", H=H, E=E, K=K, F=F, dtype="bf16", renormalize=rng.random() < 0.5,
                    bias=rng.choice(["none", "normal", "zipf1.2"]), capacity_factor=0.0, shared_F=0)
        if rng.random() < 0.3:
            case["capacity_factor"] = rng.choice([1.0, 1.25, 2.0])
        if kind == "decode":
            case["T"] = _log_int(rng, 1, 256)
            if rng.random() < 0.25:
                case["shared_F"] = 64 * rng.randint(16, 320)
        elif kind == "prefill":
            case["T"] = _log_int(rng, 256, 32768)
            if rng.random() < 0.25:
                case["shared_F"] = 64 * rng.randint(16, 320)
            if rng.random() < 0.5:                                  # multiples of 64 that are not multiples of 128
                case["H"], case["F"] = H - 64, F - 64
        elif kind == "f32":
            if E > 16:
                continue
            case.update(dtype="f32", T=_log_int(rng, 16, 4096), H=4 * rng.randint(16, 256), F=4 * rng.randint(16, 512))
        elif kind == "odd":
            if E > 16:
                continue
            case.update(T=_log_int(rng, 1, 2048), H=8 * rng.randint(32, 256), F=8 * rng.randint(32, 256))
        elif kind == "train":
            case.update(kind="train", T=_log_int(rng, 256, 8192), relayout=rng.random() < 0.5)
        elif kind == "fp8":
            case.update(kind="fp8", T=_log_int(rng, 1, 16384))
        else:
            case.update(kind="ep_share", ranks=rng.choice([2, 4]) if E % 8 else rng.choice([2, 4, 8]),
                        T=_log_int(rng, 64, 8192), capacity_factor=0.0)
            if E // case["ranks"] < 1:
                continue
        if E * case["H"] * case["F"] * 6 > 6e9:                     # the experts' bf16 weights: at most 6 GB
            continue
        if _cost(case) <= _largest_listed():
            return case


# ---------------------------------------------------------------------------------------------------------------
# sizes

def _capacity(case) -> int:
    return moe.capacity_from_factor(case["capacity_factor"], case["T"], case["K"], case["E"])


def _bias_values(kind: str, E: int, gen: torch.Generator, device: str):
    """Per-expert logit bias [E] fp32, or None."""
    if kind == "none":
        return None
    if kind == "normal":
        return torch.randn(E, generator=gen, device=device)
    rank = torch.randperm(E, generator=gen, device=device) + 1
    return -1.2 * torch.log(rank.float())


@functools.lru_cache(maxsize=None)
def _routing(T, H, E, K, bias, capacity):
    """Kept rows and experts with rows that a pass over such tokens has on average (a seeded simulation)."""
    gen = torch.Generator().manual_seed(1)
    tries = max(1, min(64, 4096 // T))
    rows = touched = 0
    for _ in range(tries):
        logits = torch.randn(T, E, generator=gen) * (WEIGHT_STD * math.sqrt(H))
        b = _bias_values(bias, E, gen, "cpu")
        if b is not None:
            logits += b
        n = torch.bincount(logits.topk(K, dim=1).indices.flatten(), minlength=E)
        if capacity > 0:
            n = n.clamp(max=capacity)
        rows += int(n.sum())
        touched += int((n > 0).sum())
    return rows / tries, touched / tries


def work(case):
    """Bytes and operations a pass cannot do without."""
    T, H, E, K, F = (case[k] for k in "THEKF")
    s = 4 if case["dtype"] == "f32" else 2
    if case["kind"] == "ep_share":
        experts = E // case["ranks"]
        rows = T * K                                               # ranks * T tokens, K / ranks of them here
        return {"bytes": 2 * rows * H * s + 3 * experts * H * F * s, "flops": 6 * rows * H * F}
    rows, touched = _routing(T, H, E, K, case["bias"], _capacity(case))
    weights = 3 * touched * H * F
    router = 2 * T * H * E
    if case["kind"] == "train":
        # tokens, output, its gradient, the tokens' gradient; weights read, their gradients written
        return {"bytes": 4 * T * H * 2 + weights * 2 + 3 * E * H * F * 2 + E * H * (2 + 4),
                "flops": 18 * rows * H * F + 3 * router}
    if case["kind"] == "fp8":
        return {"bytes": 2 * T * H * 2 + weights + E * H * 2, "flops": 6 * rows * H * F + router}
    shared = 3 * H * case["shared_F"]
    return {"bytes": 2 * T * H * s + (weights + shared + E * H) * s,
            "flops": 6 * rows * H * F + 2 * T * shared + router}


def tolerance(case):
    """Relative 2-norms, each about four times what was measured on small copies of the cases.

    fp32: 4e-7 against the same formulas in 64 bits (H = 128, F = 256); the sums of the largest layers drawn are eight
    times longer, which makes that about 1.2e-6.
    bf16 forward: 3e-4 to 5e-4 between the MFMA kernels and the plain fp32-FMA kernel (the same roundings, the sums in
    another order), 1.7e-3 against 64 bits with h and y_perm rounded; one token of 8192 whose last selected expert and
    the next lie within the logits' own rounding adds at most about 4e-3.
    Gradients: 3.6e-3 against 64 bits with every intermediate but dh rounded to bf16.
    FP8: 1.6e-3 against 64 bits on the same codes (some codes of h land on the neighbouring value).
    """
    if case["dtype"] == "f32":
        return {"rel": 5e-6}
    return {"rel": {"forward": 6e-3, "ep_share": 6e-3, "fp8": 6e-3, "train": 1.5e-2}[case["kind"]]}


# ---------------------------------------------------------------------------------------------------------------
# inputs

def _normal(shape, std, dtype, gen):
    return torch.empty(shape, dtype=dtype, device="cuda").normal_(0.0, std, generator=gen)


def _bytes(n):
    return torch.empty(max(int(n), 256), dtype=torch.uint8, device="cuda")


def _fp8_weights(shape, gen):
    """E4M3 codes of N(0, 0.02^2) weights and the scale they were quantised with."""
    w = _normal(shape, WEIGHT_STD, torch.bfloat16, gen)
    scale = moe.fp8_delayed_scale([5.5 * WEIGHT_STD])
    codes = torch.empty(shape, dtype=torch.uint8, device="cuda")
    moe.fp8_quantize(w, scale, codes)
    return codes, scale


def prepare(case, seed):
    gen = torch.Generator(device="cuda").manual_seed(int(seed))
    dtype = torch.float32 if case["dtype"] == "f32" else torch.bfloat16
    T, H, E, K, F = (case[k] for k in "THEKF")
    st = dict(case=case, capacity=_capacity(case))
    if case["kind"] == "ep_share":
        _prepare_ep_share(st, case, gen, dtype)
        return st
    st["x"] = _normal((T, H), 1.0, dtype, gen)
    st["w_router"] = _normal((E, H), WEIGHT_STD, dtype, gen)
    st["bias"] = _bias_values(case["bias"], E, gen, "cuda")
    st["y"] = torch.empty_like(st["x"])
    if case["kind"] == "fp8":
        _prepare_fp8(st, case, gen)
        return st
    st["w_gate"] = _normal((E, F, H), WEIGHT_STD, dtype, gen)
    st["w_up"] = _normal((E, F, H), WEIGHT_STD, dtype, gen)
    st["w_down"] = _normal((E, H, F), WEIGHT_STD, dtype, gen)
    Fs = case["shared_F"] if case["kind"] == "forward" else 0
    st["shared"] = (None, None, None)
    if Fs:
        st["shared"] = (_normal((Fs, H), WEIGHT_STD, dtype, gen), _normal((Fs, H), WEIGHT_STD, dtype, gen),
                        _normal((H, Fs), WEIGHT_STD, dtype, gen))
    st["ws"] = _bytes(moe.layer_workspace_bytes(T, H, E, K, F, Fs, st["capacity"],
                                                moe.MOE_F32 if dtype == torch.float32 else moe.MOE_BF16))
    if case["kind"] == "train":
        bf = dict(dtype=torch.bfloat16, device="cuda")
        st["dy"] = _normal((T, H), 1.0, torch.bfloat16, gen)
        st["gu"] = torch.empty((moe.max_rows(T, K, E, st["capacity"]), 2 * F), **bf)
        st["wgu_t"], st["wd_t"] = torch.empty((E, H, 2 * F), **bf), torch.empty((E, F, H), **bf)
        moe.expert_weights_transpose(st["w_gate"], st["w_up"], st["w_down"], st["wgu_t"], st["wd_t"])
        st["dx"] = torch.empty_like(st["x"])
        st["dw_router"] = torch.empty((E, H), dtype=torch.float32, device="cuda")
        st["dbias"] = torch.empty((E,), dtype=torch.float32, device="cuda")
        st["dw_gate"], st["dw_up"] = torch.empty_like(st["w_gate"]), torch.empty_like(st["w_up"])
        st["dw_down"] = torch.empty_like(st["w_down"])
        st["bws"] = _bytes(moe.layer_backward_workspace_bytes(T, H, E, K, F, st["capacity"]))
    return st


def _prepare_fp8(st, case, gen):
    T, H, E, K, F = (case[k] for k in "THEKF")
    i32 = dict(dtype=torch.int32, device="cuda")
    rows = moe.max_rows(T, K, E, st["capacity"])
    st["w_gate"], s_gate = _fp8_weights((E, F, H), gen)
    st["w_up"], s_up = _fp8_weights((E, F, H), gen)
    st["w_down"], s_down = _fp8_weights((E, H, F), gen)
    # scales from the amax values of earlier steps: tokens reach about 5.5; g and u have the variance 0.02^2 H, and
    # the largest silu(g) u of a batch lies near 20 of it
    st["s_x"] = moe.fp8_delayed_scale([5.5, 5.25, 5.75])
    st["s_h"] = moe.fp8_delayed_scale([20.0 * WEIGHT_STD ** 2 * H])
    st["dq"] = (1.0 / (st["s_x"] * s_gate), 1.0 / (st["s_x"] * s_up), 1.0 / (st["s_h"] * s_down))
    st["logits"] = torch.empty((T, E), dtype=torch.float32, device="cuda")
    st["idx"] = torch.empty((T, K), **i32)
    st["gate"] = torch.empty((T, K), dtype=torch.float32, device="cuda")
    st["counts"], st["offsets"] = torch.empty((E,), **i32), torch.empty((E + 1,), **i32)
    st["roa"], st["aor"] = torch.empty((T * K,), **i32), torch.empty((rows,), **i32)
    st["x_perm"] = torch.empty((rows, H), dtype=torch.uint8, device="cuda")
    st["h"] = torch.empty((rows, F), dtype=torch.uint8, device="cuda")
    st["y_perm"] = torch.empty((rows, H), dtype=torch.bfloat16, device="cuda")
    st["amax"] = torch.zeros((2,), dtype=torch.float32, device="cuda")
    st["ws"] = _bytes(moe.permute_workspace_bytes(T, K, E))


def _prepare_ep_share(st, case, gen, dtype):
    """The most ordinary rank: T tokens on each of `ranks` ranks send it T*K rows in all, in uneven chunks."""
    T, H, E, K, F, S = (case[k] for k in ("T", "H", "E", "K", "F", "ranks"))
    experts = E // S
    n = S * experts
    share = torch.softmax(0.3 * torch.randn(n, generator=gen, device="cuda"), 0).cpu().double()
    ends = torch.round(torch.cumsum(share, 0) / share.sum() * (T * K)).to(torch.int32)
    rows = torch.diff(ends, prepend=torch.zeros(1, dtype=torch.int32))
    st["chunk_rows"] = rows.cuda()
    order = torch.arange(n, dtype=torch.int32).reshape(S, experts)
    st["by_expert"] = order.t().contiguous().flatten().cuda()
    st["by_source"] = torch.arange(n, dtype=torch.int32).reshape(experts, S).t().contiguous().flatten().cuda()
    st["x"] = _normal((T * K, H), 1.0, dtype, gen)
    st["w_gate"] = _normal((experts, F, H), WEIGHT_STD, dtype, gen)
    st["w_up"] = _normal((experts, F, H), WEIGHT_STD, dtype, gen)
    st["w_down"] = _normal((experts, H, F), WEIGHT_STD, dtype, gen)
    for name in ("grouped", "y_perm", "back"):
        st[name] = torch.empty_like(st["x"])
    st["h"] = torch.empty((T * K, F), dtype=dtype, device="cuda")
    st["rows_by_expert"], st["rows_by_source"] = torch.empty_like(st["chunk_rows"]), torch.empty_like(st["chunk_rows"])
    st["offsets"] = torch.empty((experts + 1,), dtype=torch.int32, device="cuda")
    st["ws"] = _bytes(moe.sort_chunks_workspace_bytes(n))


# ---------------------------------------------------------------------------------------------------------------
# one pass

def run(st):
    return _RUN[st["case"]["kind"]](st)


def _run_forward(st):
    c = st["case"]
    moe.layer_forward(st["x"], st["w_router"], st["bias"], st["w_gate"], st["w_up"], st["w_down"], *st["shared"],
                      c["K"], c["renormalize"], st["capacity"], st["y"], st["ws"])
    return st["y"]


def _run_train(st):
    c = st["case"]
    if c["relayout"]:
        moe.expert_weights_transpose(st["w_gate"], st["w_up"], st["w_down"], st["wgu_t"], st["wd_t"])
    moe.layer_forward_train(st["x"], st["w_router"], st["bias"], st["w_gate"], st["w_up"], st["w_down"], c["K"],
                            c["renormalize"], st["capacity"], st["y"], st["gu"], st["ws"])
    moe.layer_backward(st["x"], st["w_router"], st["w_gate"], st["w_up"], st["wgu_t"], st["wd_t"], st["dy"], c["K"],
                       c["renormalize"], st["capacity"], st["ws"], st["gu"], st["dx"], st["dw_router"], st["dbias"],
                       st["dw_gate"], st["dw_up"], st["dw_down"], st["bws"])
    return {k: st[k] for k in ("y", "dx", "dw_router", "dbias", "dw_gate", "dw_up", "dw_down")}


def _run_fp8(st):
    c = st["case"]
    amax = st["amax"]
    amax.zero_()
    moe.router_topk(st["x"], st["w_router"], st["bias"], st["logits"], c["K"], c["renormalize"], st["idx"], st["gate"])
    moe.permute_fp8(st["x"], st["idx"], c["E"], st["capacity"], st["s_x"], st["x_perm"], st["counts"], st["offsets"],
                    st["roa"], st["aor"], amax[:1], st["ws"])
    moe.grouped_gemm_swiglu_fp8(st["x_perm"], st["offsets"], st["w_gate"], st["w_up"], st["w_down"], st["dq"][0],
                                st["dq"][1], st["s_h"], st["dq"][2], st["h"], amax[1:], st["y_perm"])
    moe.unpermute_combine(st["y_perm"], st["roa"], st["gate"], None, st["y"])
    return {"y": st["y"], "amax": amax}


def _run_ep_share(st):
    S = st["case"]["ranks"]
    moe.sort_chunks(st["x"], st["chunk_rows"], st["by_expert"], S, st["grouped"], st["rows_by_expert"], st["offsets"],
                    st["ws"])
    moe.grouped_gemm_swiglu(st["grouped"], st["offsets"], st["w_gate"], st["w_up"], st["w_down"], st["h"], st["y_perm"])
    moe.sort_chunks(st["y_perm"], st["rows_by_expert"], st["by_source"], 0, st["back"], st["rows_by_source"], None,
                    st["ws"])
    return {"back": st["back"], "rows_by_source": st["rows_by_source"], "offsets": st["offsets"]}


_RUN = dict(forward=_run_forward, train=_run_train, fp8=_run_fp8, ep_share=_run_ep_share)
