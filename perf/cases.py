"""The calls whose speed is tracked, over the range in which the library is used.

Three kinds of call, all through the package's entry points with torch tensors on the GPU:

  product    the fused RMSNorm -> MatMul family (plain, without gain, gated, GLU, SwiGLU)
  softmax    softmax(X) . W
  attention  group-query attention at one query position

``listed()`` names twelve of them, from the smallest call to the largest; ``draw(rng)`` gives further ones of the same
ranges.  Inputs follow the recipe of ``prism_inputs``: X ~ N(0, 1), g ~ U(0.5, 1.5), W ~ N(0, 1/K); for the softmax
X ~ N(0, 3^2) and W ~ N(0, 1); for attention Q, K, V ~ N(0, 1).
"""
import math

import torch

import paper_2604_15272_amd as prism

EPS = 1e-6

DTYPES = {"f32": torch.float32, "bf16": torch.bfloat16, "f16": torch.float16}

# Family members: (weight matrices, whether the call takes a gain tensor).
PRODUCTS = {"plain": (1, True), "plain_nogain": (1, False), "gated": (2, True), "glu": (2, True), "glu_nogain": (2, False),
            "swiglu": (2, False)}


def _product(name, op, dtype, M, K, N):
    return {"name": name, "kind": "product", "op": op, "dtype": dtype, "M": M, "K": K, "N": N}


def listed():
    return [
        # The smallest call: one small projection in full precision, nothing but launch latency.
        _product("f32_small", "plain", "f32", 8, 256, 512),
        # One decoding step of sixteen sequences: normalised hidden states onto a square projection.
        _product("decode", "plain", "bf16", 16, 4096, 4096),
        # The same step's feed-forward block, eight sequences: two wide weight matrices and the SiLU gate.
        _product("decode_gated", "gated", "bf16", 8, 4096, 14336),
        # The paper's RMSNorm-MLP in its own precision and one of its sizes: no gain, no activation.
        _product("decode_glu_half", "glu_nogain", "f16", 8, 1024, 4096),
        # Decoding onto a vocabulary whose size is no multiple of anything (entries added to a round table).
        _product("decode_odd_width", "plain", "bf16", 8, 4096, 32003),
        # A short prompt of ragged length.
        _product("short_prompt", "plain", "bf16", 200, 4096, 4096),
        # Prompts: the query/key/value projection and the gated feed-forward block; the second is the largest call.
        _product("prompt_qkv", "plain", "bf16", 2048, 4096, 6144),
        _product("prompt_gated", "gated", "bf16", 4096, 4096, 14336),
        # A feed-forward block in full precision, as a reference run or an evaluation takes it.
        _product("f32_gated", "gated", "f32", 512, 1024, 4096),
        # The paper's running example at its size.
        {"name": "softmax", "kind": "softmax", "dtype": "f16", "M": 4096, "K": 4096, "N": 128},
        # Attention of one decoding step: the paper's QK-Attention, and a serving batch with a ragged context.
        {"name": "attention", "kind": "attention", "dtype": "f16", "B": 2, "G": 8, "H": 2048, "D": 128, "qk_norm": True,
         "scale": 1.0},
        {"name": "attention_batch", "kind": "attention", "dtype": "bf16", "B": 32, "G": 8, "H": 5001, "D": 128,
         "qk_norm": False, "scale": 128 ** -0.5},
    ]


def _log_int(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi + 1)))))))


def _choose(rng, weighted):
    r = rng.random() * sum(w for _, w in weighted)
    for v, w in weighted:
        r -= w
        if r < 0:
            return v
    return weighted[-1][0]


# Multiply-adds of one call, at most: the largest listed call of the storage type, and of sizes that are no multiple of 8.
_MOST = {"bf16": 4096 * 4096 * 14336 * 2, "f16": 4096 * 4096 * 14336 * 2, "f32": 512 * 1024 * 4096 * 2}
_MOST_ODD = 512 * 1024 * 4096 * 2


def draw(rng):
    kind = _choose(rng, [("product", 6), ("softmax", 2), ("attention", 2)])
    if kind == "product":
        op = _choose(rng, [("plain", 4), ("plain_nogain", 1), ("gated", 3), ("glu", 1), ("glu_nogain", 1), ("swiglu", 1)])
        dtype = _choose(rng, [("bf16", 5), ("f16", 3), ("f32", 2)])
        step = _choose(rng, [(64, 7), (8, 2), (1, 1)])  # hidden sizes are round; some are not
        M = _log_int(rng, 1, 4096)
        K = max(step, _log_int(rng, 256, 8192) // step * step)
        N = max(step, _log_int(rng, 256, 16384) // step * step)
        most = _MOST[dtype] if K % 8 == 0 and N % 8 == 0 else min(_MOST[dtype], _MOST_ODD)
        M = max(1, min(M, most // (K * N * PRODUCTS[op][0])))
        return {"kind": kind, "op": op, "dtype": dtype, "M": M, "K": K, "N": N}
    if kind == "softmax":
        dtype = _choose(rng, [("f16", 5), ("bf16", 3), ("f32", 2)])
        step = _choose(rng, [(32, 6), (8, 3), (1, 1)])
        K = _log_int(rng, 256, 16384) // step * step
        N = _log_int(rng, 64, 1024) // step * step
        most = 4096 * 4096 * (512 if dtype != "f32" and step > 1 else 128)
        M = max(1, min(_log_int(rng, 8, 4096), most // (K * N)))
        return {"kind": kind, "dtype": dtype, "M": M, "K": K, "N": N}
    D = _choose(rng, [(128, 3), (64, 1)])
    B = _log_int(rng, 1, 64)
    return {"kind": kind, "dtype": _choose(rng, [("f16", 5), ("bf16", 4), ("f32", 1)]), "B": B,
            "G": _choose(rng, [(1, 1), (4, 2), (8, 3), (16, 1)]), "H": min(_log_int(rng, 100, 16384), 160000 // B), "D": D,
            "qk_norm": rng.random() < 0.5, "scale": _choose(rng, [(1.0, 1), (D ** -0.5, 2)])}


def prepare(case, seed):
    """Inputs and weights of the call on the GPU, and the buffer that its result goes to."""
    gen = torch.Generator(device="cuda").manual_seed(seed)
    dtype = DTYPES[case["dtype"]]

    def normal(*shape, std=1.0):
        return torch.empty(shape, dtype=torch.float32, device="cuda").normal_(0.0, std, generator=gen).to(dtype)

    state = {"case": case}
    if case["kind"] == "attention":
        B, G, H, D = case["B"], case["G"], case["H"], case["D"]
        state.update(Q=normal(B, G, D), K=normal(B, H, D), V=normal(B, H, D),
                     O=torch.empty((B, G, D), dtype=dtype, device="cuda"))
        return state
    M, K, N = case["M"], case["K"], case["N"]
    state["Y"] = torch.empty((M, N), dtype=dtype, device="cuda")
    if case["kind"] == "softmax":
        state.update(X=normal(M, K, std=3.0), W=normal(K, N))
        return state
    matrices, gain = PRODUCTS[case["op"]]
    state["X"] = normal(M, K)
    state["g"] = torch.empty(K, dtype=torch.float32, device="cuda").uniform_(0.5, 1.5, generator=gen).to(dtype) if gain else None
    state["W"] = [normal(K, N, std=K ** -0.5) for _ in range(matrices)]
    return state


def run(state):
    case = state["case"]
    if case["kind"] == "attention":
        return prism.prism_gqa_decode_attention(state["Q"], state["K"], state["V"], state["O"], scale=case["scale"],
                                                qk_norm=case["qk_norm"], eps=EPS)
    X, Y, W = state["X"], state["Y"], state["W"]
    if case["kind"] == "softmax":
        return prism.prism_softmax_matmul(X, W, Y)
    op = case["op"]
    if op == "swiglu":
        return prism.prism_swiglu(X, W[0], W[1], Y)
    if op == "gated":
        return prism.prism_rmsnorm_gated_mlp(X, state["g"], W[0], W[1], Y, eps=EPS)
    if op in ("glu", "glu_nogain"):
        return prism.prism_rmsnorm_glu(X, state["g"], W[0], W[1], Y, eps=EPS)
    return prism.prism_rmsnorm_matmul(X, state["g"], W[0], Y, eps=EPS)


def exact(case, seed):
    """What run() returns for these inputs, evaluated in 64 bits by torch."""
    state = prepare(case, seed)
    wide = {k: v.double() for k, v in state.items() if isinstance(v, torch.Tensor)}

    def normalised(x):
        return x * torch.rsqrt(x.square().mean(-1, keepdim=True) + EPS)

    if case["kind"] == "attention":
        Q = normalised(wide["Q"]) if case["qk_norm"] else wide["Q"]
        return torch.softmax(torch.bmm(Q, wide["K"].transpose(1, 2).contiguous()) * case["scale"], -1) @ wide["V"]
    X = wide["X"]
    if case["kind"] == "softmax":
        return torch.softmax(X, -1) @ wide["W"]
    op = case["op"]
    if op != "swiglu":
        X = normalised(X)
    if state["g"] is not None:
        X = X * wide["g"]
    A = [X @ w.double() for w in state["W"]]
    if op in ("gated", "swiglu"):
        A[0] = A[0] * torch.sigmoid(A[0])
    return A[0] * A[1] if len(A) > 1 else A[0]


def work(case):
    """Every input read once, every output written once; two operations per multiply-add of the products."""
    size = 4 if case["dtype"] == "f32" else 2
    if case["kind"] == "attention":
        B, G, H, D = case["B"], case["G"], case["H"], case["D"]
        return {"bytes": size * (2 * B * G * D + 2 * B * H * D), "flops": 4 * B * G * H * D}
    M, K, N = case["M"], case["K"], case["N"]
    if case["kind"] == "softmax":
        return {"bytes": size * (M * K + K * N + M * N), "flops": 2 * M * K * N}
    matrices, gain = PRODUCTS[case["op"]]
    return {"bytes": size * (M * K + (K if gain else 0) + matrices * K * N + M * N), "flops": 2 * M * K * N * matrices}


# Four times the largest errors seen against a 64-bit evaluation over the listed calls and 60 drawn ones: bf16 2.9e-3
# (largest 4.0e-2, a two-matrix output of a long prompt), f16 3.6e-4 (2.3e-3), f32 1.5e-6 (1.2e-5); scores of fp32
# attention that are not scaled down carry an error proportional to their size on top.
_TOLERANCE = {"bf16": {"rel": 1.2e-2, "max": 0.16}, "f16": {"rel": 1.5e-3, "max": 1e-2}, "f32": {"rel": 6e-6, "max": 6e-5}}
_TOLERANCE_F32_ATTENTION = {"rel": 2e-5, "max": 2e-4}


def tolerance(case):
    if case["kind"] == "attention" and case["dtype"] == "f32":
        return _TOLERANCE_F32_ATTENTION
    return _TOLERANCE[case["dtype"]]
