"""Products of 32-bit precision from 16-bit parts (the kernels for any shape)."""
import pytest
import torch

pytestmark = pytest.mark.gpu

DTYPES = {"f32": torch.float32, "bf16": torch.bfloat16, "f16": torch.float16}
# Of 32-bit products and sums: the project's bar for fp32; 16-bit storage rounds the output alone: with p significant
# bits by at most 2^-p of it (half a unit of the last place of 1.00..), p = 8 and 11.
TOL = {"f32": 1e-5, "bf16": 1e-5 + 2.0 ** -8, "f16": 1e-5 + 2.0 ** -11}


def _code(P, dtype):
    return {"f32": P.PRISM_F32, "bf16": P.PRISM_BF16, "f16": P.PRISM_F16}[dtype]


def _check(Y, ref, dtype):
    err = (Y.double() - ref).abs() / (ref.abs() + 1.0)
    assert float(err.max()) <= TOL[dtype], float(err.max())


# One, two, .. stages of 32 (128 rows) or 64 (64 rows) K values, and a last one that is not full: fewer than the ring holds, the first
# trip of the loop, the last ones.
@pytest.mark.parametrize("dtype", ["f32", "bf16", "f16"])
@pytest.mark.parametrize("rows,M,N", [(128, 1999, 2047), (64, 1023, 2046)])
def test_number_of_stages(dtype, rows, M, N):
    import paper_2604_15272_amd as P
    gen = torch.Generator(device="cuda").manual_seed(41)
    rand = lambda *s: torch.empty(s, device="cuda").normal_(generator=gen)
    seen = set()
    for K in (31, 33, 63, 65, 97, 127, 129, 161, 193, 225, 255, 257, 289, 321, 353, 385, 417, 449, 513, 577, 641, 643):
        if P.prism_plan(0, M, K, N, _code(P, dtype))["tile_m"] != rows:
            continue
        seen.add(K)
        X, g, W = rand(M, K).to(DTYPES[dtype]), (rand(K).abs() + 0.5).to(DTYPES[dtype]), (rand(K, N) * K ** -0.5).to(DTYPES[dtype])
        Y = torch.full((M, N), float("nan"), dtype=DTYPES[dtype], device="cuda")
        P.prism_rmsnorm_matmul(X, g, W, Y, eps=1e-6)
        Xd = X.double()
        _check(Y, (Xd * torch.rsqrt(Xd.square().mean(-1, keepdim=True) + 1e-6) * g.double()) @ W.double(), dtype)
    assert len(seen) >= 8 or P.prism_diag_cu_count() != 256


@pytest.mark.parametrize("M,K,N", [(1999, 290, 1023), (1021, 1201, 1023), (1999, 60, 1023)])
def test_values_without_parts(M, K, N):
    """Values that round to infinity in bf16 have finite products with small weights; an infinity stays in its row."""
    import paper_2604_15272_amd as P
    gen = torch.Generator().manual_seed(42)
    X, W1, W2 = torch.randn(M, K, generator=gen), torch.randn(K, N, generator=gen) * K ** -0.5, torch.randn(K, N, generator=gen) * K ** -0.5
    X[5, 3], X[M - 1, 3], W1[3], W2[3] = 3.402e38, -3.4e38, W1[3] * 1e-37, W2[3] * 1e-37
    W1[7, N - 2] = 3.4e38
    X[:, 7] = 1e-38 * torch.randn(M, generator=gen)
    Y = torch.empty(M, N, device="cuda")
    P.prism_swiglu(X.cuda(), W1.cuda(), W2.cuda(), Y)
    Xd, a, b = X.double(), W1.double(), W2.double()
    ref = torch.nn.functional.silu(Xd @ a) * (Xd @ b)
    assert bool(torch.isfinite(ref).all())
    _check(Y.cpu(), ref, "f32")
    X[9, K - 1] = float("inf")
    P.prism_swiglu(X.cuda(), W1.cuda(), W2.cuda(), Y)
    keep = torch.arange(M) != 9
    _check(Y.cpu()[keep], ref[keep], "f32")
    # (silu(-inf) is NaN in the kernels, as in the formula x / (1 + exp(-x)); +inf times the other branch's sign is an infinity)
    assert not bool(torch.isfinite(Y[9]).any())


# Rows of very different size, gains included: the error of an output is relative to the products it sums.
@pytest.mark.parametrize("M,K,N", [(1999, 290, 2047), (1023, 501, 2046), (130, 4096, 4096)])
def test_error_against_64_bits(M, K, N):
    import paper_2604_15272_amd as P
    gen = torch.Generator(device="cuda").manual_seed(43)
    rand = lambda *s: torch.empty(s, device="cuda").normal_(generator=gen)
    X = rand(M, K) * torch.exp2(torch.randint(-20, 20, (M, 1), device="cuda", generator=gen).float())
    W = rand(K, N) * torch.exp2(torch.randint(-20, 20, (1, N), device="cuda", generator=gen).float())
    g = torch.exp2(rand(K) * 4)
    Y = torch.empty(M, N, device="cuda")
    P.prism_rmsnorm_matmul(X, g, W, Y, eps=0.0)
    Xd = X.double() * g.double()
    r = torch.rsqrt(X.double().square().mean(-1, keepdim=True))
    ref, size = (Xd @ W.double()) * r, (Xd.abs() @ W.double().abs()) * r
    # Every product is off by at most 2^-23 (the fp32 rounding of x * g and what the parts leave out), every addition by 2^-24 of a
    # partial sum; their number is K / 4 to 6 K / 16, and independent roundings add up as the square root.
    bound = size * (2.0 ** -23 + 2.0 ** -24 * 4 * K ** 0.5)
    assert bool(((Y.double() - ref).abs() <= bound).all())


# 16-bit storage: x * g beyond the format's range (and a third of it near the f16 limit), small rows whose second part would leave f16's
# exponents unscaled, and a column of large weights; one case per form of the kernels.
@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("M,K,N", [(5, 301, 131), (12, 2601, 41), (20, 4128, 35), (40, 700, 1001), (15, 333, 4099), (18, 69, 4255), (132, 71, 3555), (200, 161, 515), (7600, 81, 33), (1999, 290, 2047), (1023, 501, 2046), (1999, 60, 1023)])
def test_16_bit_storage_at_the_ends_of_its_range(dtype, M, K, N):
    import paper_2604_15272_amd as P
    gen = torch.Generator(device="cuda").manual_seed(44)
    rand = lambda *s: torch.empty(s, device="cuda").normal_(generator=gen)
    X, g, W = rand(M, K), rand(K).abs() + 0.5, rand(K, N) * K ** -0.5
    X[0] *= 2e-3
    X[1, 2], g[2] = 3e4, 8.0
    W[:, 5] *= 300.0
    X, g, W = (t.to(DTYPES[dtype]) for t in (X, g, W))
    Y = torch.full((M, N), float("nan"), dtype=DTYPES[dtype], device="cuda")
    P.prism_rmsnorm_matmul(X, g, W, Y, eps=0.0)
    Xd = X.double()
    _check(Y, (Xd * torch.rsqrt(Xd.square().mean(-1, keepdim=True)) * g.double()) @ W.double(), dtype)
    X[2, K - 1] = float("inf")
    P.prism_rmsnorm_matmul(X, g, W, Y, eps=0.0)
    assert bool(Y[2].isnan().all()) and bool(Y[0].isfinite().all())


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("M,K,N", [(9, 301, 67), (20, 3001, 515), (700, 1001, 1283), (300, 161, 131)])
def test_softmax_of_any_shape_in_parts(dtype, M, K, N):
    import paper_2604_15272_amd as P
    gen = torch.Generator(device="cuda").manual_seed(45)
    rand = lambda *s: torch.empty(s, device="cuda").normal_(generator=gen)
    X, W = rand(M, K) * 3, rand(K, N)
    X[0] = 0.0                      # equal weights: 1 / K each
    X[1, : K // 2] = -float("inf")  # a mask
    W[:, 3] = 100.0
    X, W = X.to(DTYPES[dtype]), W.to(DTYPES[dtype])
    Y = torch.full((M, N), float("nan"), dtype=DTYPES[dtype], device="cuda")
    P.prism_softmax_matmul(X, W, Y)
    assert P.prism_plan(P.PRISM_OP_SOFTMAX_MATMUL, M, K, N, _code(P, dtype))["path"] == P.PRISM_PATH_SIMPLE
    _check(Y, torch.softmax(X.double(), -1) @ W.double(), dtype)


# Whole blocks of 32 keys, a rest, fewer keys than a block or than wavefronts; one head, more than sixteen; beyond 16 MB of keys and values.
@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("B,G,H,D", [(2, 8, 1, 64), (2, 1, 31, 64), (3, 16, 32, 64), (2, 5, 33, 64), (2, 8, 257, 64), (1, 17, 600, 64), (2, 8, 1000, 64), (2, 20, 300, 128), (2, 17, 5, 128), (33, 4, 2051, 64)])
@pytest.mark.parametrize("qk_norm", [False, True])
def test_attention_in_parts(dtype, B, G, H, D, qk_norm):
    import paper_2604_15272_amd as P
    gen = torch.Generator(device="cuda").manual_seed(46 + H)
    rand = lambda *s: torch.empty(s, device="cuda").normal_(generator=gen).to(DTYPES[dtype])
    Q, K, V = rand(B, G, D), rand(B, H, D), rand(B, H, D)
    O = torch.full_like(Q, float("nan"))
    P.prism_gqa_decode_attention(Q, K, V, O, scale=0.5, qk_norm=qk_norm)
    assert P.prism_attention_plan(B, G, H, D, _code(P, dtype))["path"] == P.PRISM_PATH_SIMPLE
    Qd = Q.double()
    if qk_norm:
        Qd = Qd * torch.rsqrt(Qd.square().mean(-1, keepdim=True) + 1e-6)
    # Scores are sums of D products of size one: their fp32 error, 2^-24 sqrt(D) of about sqrt(D) at most, is the output's relative error.
    _check(O, torch.softmax(torch.bmm(Qd, K.double().transpose(1, 2).contiguous()) * 0.5, -1) @ V.double(), dtype)


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
def test_attention_in_parts_infinities_of_v(dtype):
    import paper_2604_15272_amd as P
    gen = torch.Generator(device="cuda").manual_seed(47)
    rand = lambda *s: torch.empty(s, device="cuda").normal_(generator=gen).to(DTYPES[dtype])
    Q, K, V = rand(2, 8, 64), rand(2, 100, 64), rand(2, 100, 64)
    V[0, 5, 7], V[0, 6, 9], V[1, 99, 0] = float("inf"), -float("inf"), float("nan")
    O = torch.empty_like(Q)
    P.prism_gqa_decode_attention(Q, K, V, O, scale=0.125)
    ref = torch.softmax(torch.bmm(Q.double(), K.double().transpose(1, 2).contiguous()) * 0.125, -1)
    assert bool((O[0, :, 7] == float("inf")).all()) and bool((O[0, :, 9] == -float("inf")).all()) and bool(O[1, :, 0].isnan().all())
    keep = torch.ones(2, 64, dtype=torch.bool, device="cuda")
    keep[0, 7] = keep[0, 9] = keep[1, 0] = False
    Vd = torch.where(V.double().isfinite(), V.double(), torch.zeros((), dtype=torch.float64, device="cuda"))
    for b in range(2):
        _check(O[b][:, keep[b]], (ref[b] @ Vd[b])[:, keep[b]], dtype)


# An infinity in one element of a key is a score of its sign times that of the head's value there: -inf has weight 0, +inf makes the head a NaN.
@pytest.mark.parametrize("dtype", ["f32", "bf16", "f16"])
@pytest.mark.parametrize("G,H,D", [(8, 100, 64), (8, 9, 64), (4, 70000, 64), (20, 300, 128)])
@pytest.mark.parametrize("scale,qk_norm", [(0.125, False), (0.3, False), (-0.5, True)])
def test_attention_infinities_of_k(dtype, G, H, D, scale, qk_norm):
    import paper_2604_15272_amd as P
    gen = torch.Generator(device="cuda").manual_seed(48)
    rand = lambda *s: torch.empty(s, device="cuda").normal_(generator=gen).to(DTYPES[dtype])
    Q, K, V = rand(2, G, D), rand(2, H, D), rand(2, H, D)
    K[0, 5, 7], K[0, H - 1, 9], K[1, 3, 0] = float("inf"), -float("inf"), -float("inf")
    Q[0, 0, 7], Q[0, 0, 9], Q[0, 1, 7], Q[0, 1, 9] = -1.0, 0.5, 1.0, -0.5
    O = torch.empty_like(Q)
    P.prism_gqa_decode_attention(Q, K, V, O, scale=scale, qk_norm=qk_norm)
    Qd = Q.double()
    if qk_norm:
        Qd = Qd * torch.rsqrt(Qd.square().mean(-1, keepdim=True) + 1e-6)
    ref = torch.softmax(torch.bmm(Qd, K.double().transpose(1, 2).contiguous()) * scale, -1) @ V.double()
    assert torch.equal(O.isnan(), ref.isnan()) and 0 < int(ref.isnan().sum()) < ref.numel()
    _check(O.nan_to_num(), ref.nan_to_num(), dtype)


def test_attention_scores_that_only_the_factor_keeps_finite():
    """bf16 Q and K whose products pass fp32's limit by themselves, and do not with the factor."""
    import paper_2604_15272_amd as P
    gen = torch.Generator(device="cuda").manual_seed(49)
    rand = lambda *s: torch.empty(s, device="cuda").normal_(generator=gen)
    Q, K, V = (rand(2, 8, 64) * 1e25).bfloat16(), (rand(2, 300, 64) * 1e15).bfloat16(), rand(2, 300, 64).bfloat16()
    O = torch.empty_like(Q)
    P.prism_gqa_decode_attention(Q, K, V, O, scale=3e-41)
    # (the scale is a fp32 number with few bits: the one that the call sees)
    s = float(torch.tensor(3e-41, dtype=torch.float32))
    _check(O, torch.softmax(torch.bmm(Q.double(), K.double().transpose(1, 2).contiguous()) * s, -1) @ V.double(), "bf16")


# Products whose sums are not finite in parts: infinities and NaNs in W, an infinity in X (no normalisation: it stays one), values that only round to
# infinity; in the first and last columns, where a group of columns is moved in from the right edge.
@pytest.mark.parametrize("dtype", ["f32", "bf16", "f16"])
@pytest.mark.parametrize("M,K,N", [(5, 301, 131), (20, 301, 131), (40, 700, 1001), (15, 333, 4099), (200, 161, 515), (1999, 290, 2047), (1023, 501, 2046),
                                   (1999, 60, 1023), (70, 17, 643)])
@pytest.mark.parametrize("gated", [False, True])
def test_sums_that_are_not_finite(dtype, M, K, N, gated):
    import paper_2604_15272_amd as P
    inf = float("inf")
    gen = torch.Generator(device="cuda").manual_seed(50)
    rand = lambda *s: torch.empty(s, device="cuda").normal_(generator=gen)
    X, W, W2 = rand(M, K), rand(K, N) * K ** -0.5, rand(K, N) * K ** -0.5
    W[2, 0], W[3, N - 1], W[4, N - 2], W2[5, N // 2] = inf, -inf, float("nan"), inf
    X, W, W2 = X.to(DTYPES[dtype]), W.to(DTYPES[dtype]), W2.to(DTYPES[dtype])
    ones = torch.ones(K, device="cuda", dtype=DTYPES[dtype])
    Y = torch.empty((M, N), dtype=DTYPES[dtype], device="cuda")

    def check(ref):
        assert torch.equal(Y.isnan(), ref.isnan()) and torch.equal(Y.isposinf(), ref.isposinf()) and torch.equal(Y.isneginf(), ref.isneginf())
        keep = ref.isfinite()
        _check(torch.where(keep, Y, 0), torch.where(keep, ref, 0), dtype)

    Xd = X.double()
    Xn = Xd * torch.rsqrt(Xd.square().mean(-1, keepdim=True) + 1e-6)
    if gated:
        P.prism_rmsnorm_glu(X, ones, W, W2, Y, eps=1e-6)
        check((Xn @ W.double()) * (Xn @ W2.double()))
        X[M - 1, 7] = inf
        P.prism_swiglu(X, W, W2, Y)
        Xd = X.double()
        check(torch.nn.functional.silu(Xd @ W.double()) * (Xd @ W2.double()))
    else:
        P.prism_rmsnorm_matmul(X, ones, W, Y, eps=1e-6)
        check(Xn @ W.double())


# A NaN that reaches every output: a second pass at most, not a serial loop for each of them (tens of milliseconds here).
@pytest.mark.parametrize("dtype,M,K,N", [("bf16", 8, 4096, 32003), ("f32", 1000, 4096, 2000), ("f16", 500, 4001, 2001)])
def test_a_nan_in_the_gain_takes_bounded_time(dtype, M, K, N):
    import paper_2604_15272_amd as P
    X, g, W = (torch.ones(s, device="cuda", dtype=DTYPES[dtype]) for s in ((M, K), (K,), (K, N)))
    Y = torch.empty((M, N), dtype=DTYPES[dtype], device="cuda")
    times = []
    for value in (1.0, float("nan")):
        g[K // 2] = value
        e = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
        P.prism_rmsnorm_matmul(X, g, W, Y)
        e[0].record()
        for _ in range(5):
            P.prism_rmsnorm_matmul(X, g, W, Y)
        e[1].record()
        torch.cuda.synchronize()
        times.append(e[0].elapsed_time(e[1]) / 5)
    print(f"{dtype} {M} x {K} x {N}: {times[0] * 1e3:.1f} us, with a NaN {times[1] * 1e3:.1f} us")
    assert bool(Y.isnan().all()) and times[1] < 25 * times[0], times


# Rows of NaNs are NaNs whatever their products: nothing is gone through again for them.
@pytest.mark.parametrize("dtype,M,K,N", [("bf16", 8, 4096, 32003), ("f32", 1000, 4096, 2000)])
def test_rows_of_nans_take_no_longer(dtype, M, K, N):
    import paper_2604_15272_amd as P
    X, g, W = (torch.ones(s, device="cuda", dtype=DTYPES[dtype]) for s in ((M, K), (K,), (K, N)))
    Y = torch.empty((M, N), dtype=DTYPES[dtype], device="cuda")
    times = []
    for value in (1.0, float("nan")):
        X[2, K // 2] = value
        e = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
        for _ in range(20):
            P.prism_rmsnorm_matmul(X, g, W, Y)
        e[0].record()
        for _ in range(20):
            P.prism_rmsnorm_matmul(X, g, W, Y)
        e[1].record()
        torch.cuda.synchronize()
        times.append(e[0].elapsed_time(e[1]) / 20)
    keep = torch.arange(M, device="cuda") != 2
    assert bool(Y[2].isnan().all()) and bool(Y[keep].isfinite().all()) and times[1] < 2 * times[0], times


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("B,G,H,D", [(2, 8, 16384, 64), (2, 33, 3001, 128), (2, 5, 33, 64), (1, 3, 7, 64)])
def test_attention_a_nan_or_infinities_in_v_take_bounded_time(dtype, B, G, H, D):
    """One more pass over the keys at most (a serial loop over H x D for each output: tens of milliseconds)."""
    import paper_2604_15272_amd as P
    gen = torch.Generator(device="cuda").manual_seed(51)
    rand = lambda *s: torch.empty(s, device="cuda").normal_(generator=gen).to(DTYPES[dtype])
    Q, K, V = rand(B, G, D), rand(B, H, D), rand(B, H, D)
    O = torch.empty_like(Q)
    times = []
    for step in range(2):
        if step == 1:
            V[0, H // 2], V[0, H - 1, 5] = float("nan"), float("inf")
            V[B - 1, H - 1], V[B - 1, 0, :7] = float("inf"), -float("inf")
        e = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
        for _ in range(5):
            P.prism_gqa_decode_attention(Q, K, V, O, scale=0.125)
        e[0].record()
        for _ in range(5):
            P.prism_gqa_decode_attention(Q, K, V, O, scale=0.125)
        e[1].record()
        torch.cuda.synchronize()
        times.append(e[0].elapsed_time(e[1]) / 5)
    print(f"{dtype} {B} x {G} x {H} x {D}: {times[0] * 1e3:.1f} us, then {times[1] * 1e3:.1f} us")
    w = torch.softmax(torch.bmm(Q.double(), K.double().transpose(1, 2).contiguous()) * 0.125, -1)
    # (weights that are 0 in fp32 and not in 64 bits would differ; there are none with these scores)
    ref = w @ V.double()
    assert torch.equal(O.isnan(), ref.isnan()) and torch.equal(O.isposinf(), ref.isposinf()) and torch.equal(O.isneginf(), ref.isneginf())
    assert times[1] < 25 * times[0], times


# The largest weight meets zeros of W or V, what is left are small weights: their own error counts.  f16 weights have 2^-22 of themselves (two parts, the
# exponential's own rounding) from 2^-29 of the largest on, and 2^-51 of the largest below.
@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("M,K,N", [(9, 16383, 67), (3, 501, 131), (300, 161, 131), (700, 1001, 1283)])
def test_softmax_of_small_weights(dtype, M, K, N):
    import paper_2604_15272_amd as P
    gen = torch.Generator(device="cuda").manual_seed(52)
    X = -torch.linspace(5.0, 27.0, M, device="cuda")[:, None].expand(M, K).contiguous()
    W = torch.empty(K, N, device="cuda").uniform_(2e4, 6e4, generator=gen)
    X[:, 3], W[3] = 0.0, 0.0
    X, W = X.to(DTYPES[dtype]), W.to(DTYPES[dtype])
    Y = torch.empty((M, N), dtype=DTYPES[dtype], device="cuda")
    P.prism_softmax_matmul(X, W, Y)
    w = torch.softmax(X.double(), -1)
    ref = w @ W.double()
    bits = 8 if dtype == "bf16" else 11
    bound = ref * 2.0 ** -bits + (w * 2.0 ** -21 + (2.0 ** -51 if dtype == "f16" else 0.0)) @ W.double() + 2.0 ** -25
    assert bool(((Y.double() - ref).abs() <= bound).all()), float(((Y.double() - ref).abs() / bound).max())


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("B,G,H,D", [(2, 8, 16000, 64), (2, 20, 300, 128), (3, 4, 33, 64)])
def test_attention_of_small_probabilities(dtype, B, G, H, D):
    import paper_2604_15272_amd as P
    gen = torch.Generator(device="cuda").manual_seed(53)
    Q, K = torch.zeros(B, G, D, device="cuda"), torch.zeros(B, H, D, device="cuda")
    V = torch.empty(B, H, D, device="cuda").uniform_(2e4, 6e4, generator=gen)
    Q[:, :, 0], K[:, :, 0] = torch.linspace(5.0, 27.0, G, device="cuda"), -1.0
    K[:, H // 2], V[:, H // 2] = 0.0, 0.0
    Q, K, V = (t.to(DTYPES[dtype]) for t in (Q, K, V))
    O = torch.empty_like(Q)
    P.prism_gqa_decode_attention(Q, K, V, O, scale=1.0)
    w = torch.softmax(torch.bmm(Q.double(), K.double().transpose(1, 2).contiguous()), -1)
    ref = w @ V.double()
    bits = 8 if dtype == "bf16" else 11
    bound = ref * 2.0 ** -bits + (w * 2.0 ** -21 + (2.0 ** -51 if dtype == "f16" else 0.0)) @ V.double() + 2.0 ** -25
    assert bool(((O.double() - ref).abs() <= bound).all()), float(((O.double() - ref).abs() / bound).max())


# f16: rows and gains whose products leave the range in which two parts carry them, and rows of zeros; relative to the products that an output sums, whose
# own roundings are those of fp32 (as in test_error_against_64_bits), and of the stored output.
@pytest.mark.parametrize("M,K,N", [(5, 301, 131), (12, 2601, 41), (20, 4128, 35), (40, 700, 1001), (15, 333, 4099), (18, 69, 4255), (132, 71, 3555), (200, 161, 515), (7600, 81, 33), (1999, 290, 2047), (1023, 501, 2046), (1999, 60, 1023)])
@pytest.mark.parametrize("gain", [1.0, 1e-4])
def test_f16_products_of_small_values(M, K, N, gain):
    import paper_2604_15272_amd as P
    gen = torch.Generator(device="cuda").manual_seed(54)
    rand = lambda *s: torch.empty(s, device="cuda").normal_(generator=gen)
    X = (rand(M, K) * 10.0 ** torch.linspace(-7, 0, M, device="cuda")[:, None]).half()
    g, W = ((rand(K).abs() + 0.5) * gain).half(), rand(K, N).half()
    X[M // 2] = 0.0
    # Outputs of a size that f16 stores to 2^-11: a power of two undoes the gain's.
    W *= 2.0 ** -round(float(torch.log2(torch.tensor(gain))) + 0.5 * float(torch.log2(torch.tensor(float(K)))))
    Y = torch.empty((M, N), dtype=torch.float16, device="cuda")
    P.prism_rmsnorm_matmul(X, g, W, Y, eps=0.0)
    keep = (X != 0).any(1)
    Xd = X.double()[keep]
    r = torch.rsqrt(Xd.square().mean(-1, keepdim=True))
    Xd = Xd * g.double()
    ref, size = (Xd @ W.double()) * r, (Xd.abs() @ W.double().abs()) * r
    bound = ref.abs() * 2.0 ** -11 + 2.0 ** -25 + size * (2.0 ** -23 + 2.0 ** -24 * 4 * K ** 0.5)
    assert bool(((Y.double()[keep] - ref).abs() <= bound).all()), float(((Y.double()[keep] - ref).abs() / bound).max())
    assert bool(Y[~keep].isnan().all()) and int(keep.sum()) >= M // 2


# ... but one lane's share of an ordinary row can be small (the end of a ragged K has it hold a single value): no second pass for that.
@pytest.mark.parametrize("M,K,N,gated,lanes", [(124, 169, 2437, True, slice(168, 169)), (397, 209, 759, False, slice(208, 209)), (8, 265, 8001, False, slice(264, 265)),
                                               (1999, 290, 2047, False, slice(20, 290, 32)), (1023, 501, 1023, True, slice(8, 501, 64))])
def test_f16_small_values_beside_ordinary_ones_take_no_longer(M, K, N, gated, lanes):
    import paper_2604_15272_amd as P
    gen = torch.Generator(device="cuda").manual_seed(55)
    rand = lambda *s: torch.empty(s, device="cuda").normal_(generator=gen)
    X, g, W = rand(M, K).half(), torch.ones(K, device="cuda", dtype=torch.float16), (rand(K, N) * K ** -0.5).half()
    X[X.abs() < 0.01] = 0.01
    Y = torch.empty((M, N), dtype=torch.float16, device="cuda")
    call = (lambda: P.prism_rmsnorm_glu(X, g, W, W, Y)) if gated else (lambda: P.prism_rmsnorm_matmul(X, g, W, Y))
    times = []
    for step in range(2):
        if step == 1:
            for i in range(4 if lanes.step else 1):   # the four neighbouring values of a thread
                X[:, lanes.start + i::lanes.step or K] = 1e-5
        e = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
        for _ in range(20):
            call()
        e[0].record()
        for _ in range(20):
            call()
        e[1].record()
        torch.cuda.synchronize()
        times.append(e[0].elapsed_time(e[1]) / 20)
    print(f"f16 {M} x {K} x {N}: {times[0] * 1e3:.1f} us, then {times[1] * 1e3:.1f} us")
    assert times[1] < 1.5 * times[0], times


# 16-bit calls of a shallow K as a default user's are dispatched: every form of the kernel for any shape that they take, rows and columns past a tile.
# 0: one matrix, 1: two, 2: softmax.
@pytest.mark.parametrize("op,dtype,M,K,N,form", [
    (0, "bf16", 136, 96, 1800, (16, 16, 256)), (0, "f16", 1, 64, 24, (16, 16, 512)), (0, "bf16", 1, 64, 8264, (16, 64, 512)), (0, "f16", 34, 64, 8840, (16, 128, 512)),
    (0, "f16", 454, 96, 1072, (32, 64, 512)), (0, "bf16", 81, 64, 5392, (32, 64, 512)), (0, "bf16", 8, 1024, 1024, (16, 16, 512)), (0, "f16", 512, 512, 40, (16, 16, 512)),
    (1, "f16", 1, 64, 6168, (16, 16, 256)), (1, "f16", 8, 1024, 4096, (16, 16, 512)), (1, "f16", 35, 64, 9440, (16, 64, 256)), (1, "bf16", 1, 64, 8296, (16, 64, 512)),
    (1, "bf16", 75, 64, 11656, (16, 128, 256)), (1, "bf16", 39, 64, 8408, (16, 128, 512)), (1, "f16", 20, 64, 10616, (32, 16, 256)), (1, "f16", 18, 64, 2352, (32, 16, 512)),
    (1, "bf16", 69, 64, 10680, (16, 128, 256)), (1, "bf16", 305, 64, 1592, (32, 64, 512)), (2, "bf16", 1, 32, 8, (16, 16, 512)), (2, "f16", 51, 256, 672, (16, 16, 512)),
    (2, "bf16", 1, 40, 4128, (16, 64, 512)), (2, "f16", 19, 32, 9528, (16, 128, 512)), (2, "bf16", 2296, 32, 136, (32, 64, 512)), (2, "f16", 2179, 40, 168, (32, 64, 512))])
def test_shallow_16_bit_calls_as_dispatched(op, dtype, M, K, N, form):
    import paper_2604_15272_amd as P
    P.prism_set_override(0, 0, 0)
    plan = P.prism_plan(op, M, K, N, _code(P, dtype))
    assert (plan["path"] == P.PRISM_PATH_SIMPLE and (plan["tile_m"], plan["tile_n"], plan["block"]) == form) or P.prism_diag_cu_count() != 256, plan
    gen = torch.Generator(device="cuda").manual_seed(61)
    rand = lambda *s: torch.empty(s, device="cuda").normal_(generator=gen)
    X, g = (rand(M, K) * (3.0 if op == 2 else 1.0)).to(DTYPES[dtype]), (rand(K).abs() + 0.5).to(DTYPES[dtype])
    W, W2 = ((rand(K, N) * (1.0 if op == 2 else K ** -0.5)).to(DTYPES[dtype]) for _ in range(2))
    Y = torch.full((M, N), float("nan"), dtype=DTYPES[dtype], device="cuda")
    Xd = X.double()
    if op == 2:
        P.prism_softmax_matmul(X, W, Y)
        _check(Y, torch.softmax(Xd, -1) @ W.double(), dtype)
        return
    Xn = Xd * torch.rsqrt(Xd.square().mean(-1, keepdim=True) + 1e-6) * g.double()
    if op == 1:
        P.prism_rmsnorm_gated_mlp(X, g, W, W2, Y, eps=1e-6)
        _check(Y, torch.nn.functional.silu(Xn @ W.double()) * (Xn @ W2.double()), dtype)
    else:
        P.prism_rmsnorm_matmul(X, g, W, Y, eps=1e-6)
        _check(Y, Xn @ W.double(), dtype)
