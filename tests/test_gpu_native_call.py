"""The native route of ordinary calls from Python: the same results as the general route, the same refusals."""
import pytest
import torch


@pytest.fixture(scope="module")
def P():
    import paper_2604_15272_amd as P
    return P


def _tensors(device, dtype=torch.bfloat16, M=5, K=256, N=192):
    gen = torch.Generator().manual_seed(5)
    t = {n: torch.randn(*s, generator=gen).to(dtype).to(device)
         for n, s in (("X", (M, K)), ("g", (K,)), ("W1", (K, N)), ("W2", (K, N)))}
    t["Y"] = torch.zeros(M, N, dtype=dtype, device=device)
    return t


def _calls(P):
    return {
        "matmul": lambda t, **kw: P.prism_rmsnorm_matmul(t["X"], t["g"], t["W1"], t["Y"], eps=1e-5, **kw),
        "nogain": lambda t, **kw: P.prism_rmsnorm_matmul(t["X"], None, t["W1"], t["Y"], eps=1e-5, **kw),
        "static": lambda t, **kw: P.prism_rmsnorm_matmul_static(t["X"], t["g"], t["W1"], t["Y"], eps=1e-5, **kw),
        "gated": lambda t, **kw: P.prism_rmsnorm_gated_mlp(t["X"], t["g"], t["W1"], t["W2"], t["Y"], eps=1e-5, **kw),
        "glu": lambda t, **kw: P.prism_rmsnorm_glu(t["X"], t["g"], t["W1"], t["W2"], t["Y"], eps=1e-5, **kw),
        "swiglu": lambda t, **kw: P.prism_swiglu(t["X"], t["W1"], t["W2"], t["Y"], **kw),
        "softmax": lambda t, **kw: P.prism_softmax_matmul(t["X"], t["W1"], t["Y"], **kw),
    }


NAMES = ["matmul", "nogain", "static", "gated", "glu", "swiglu", "softmax"]


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16, torch.float16])
@pytest.mark.parametrize("name", NAMES)
def test_both_routes_give_the_same_bits(P, name, dtype):
    t = _tensors("cuda", dtype)
    call = _calls(P)[name]
    M, K = t["X"].shape
    N = t["W1"].shape[1]
    side = torch.cuda.Stream()
    expect = call(t, M=M, K=K, N=N).clone()  # sizes given: the general route
    for stream in (None, torch.cuda.current_stream(), torch.cuda.current_stream().cuda_stream):
        t["Y"].zero_()
        assert call(t, stream=stream) is t["Y"]
        assert torch.equal(t["Y"], expect)
    torch.cuda.synchronize()
    t["Y"].zero_()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):  # the current stream, whichever it is
        call(t)
        after = t["Y"].clone()
    side.synchronize()
    assert torch.equal(after, expect)
    t["W1"] = torch.nn.Parameter(t["W1"])
    t["Y"].zero_()
    call(t)
    assert torch.equal(t["Y"], expect)


@pytest.mark.gpu
def test_attention_and_missing_workspace(P):
    gen = torch.Generator(device="cuda").manual_seed(6)
    Q, K, V = (torch.randn(*s, generator=gen, device="cuda").half() for s in ((2, 8, 128), (2, 2000, 128), (2, 2000, 128)))
    O = torch.zeros_like(Q)
    P.prism_gqa_decode_attention(Q, K, V, O, scale=0.1, qk_norm=True, dtype=P.PRISM_F16)  # a type given: the general route
    expect = O.clone()
    from paper_2604_15272_amd import binding
    torch.cuda.synchronize()
    kept = binding._workspaces.pop(torch.cuda.current_device())
    P.prism_set_workspace(0, 0)
    O.zero_()
    P.prism_gqa_decode_attention(Q, K, V, O, scale=0.1, qk_norm=True)  # finds none and registers one
    assert torch.equal(O, expect)
    torch.cuda.synchronize()
    P.prism_set_workspace(kept.data_ptr(), kept.numel())
    binding._workspaces[torch.cuda.current_device()] = kept


@pytest.mark.gpu
@pytest.mark.parametrize("name", NAMES)
def test_refusals_on_the_gpu(P, name):
    call = _calls(P)[name]
    t = _tensors("cuda")
    t["W1"] = t["W1"].t().contiguous().t()
    with pytest.raises(ValueError, match="contiguous"):
        call(t)
    t = _tensors("cuda", torch.float64)
    with pytest.raises(TypeError, match="unsupported tensor dtype"):
        call(t)
    t = _tensors("cuda")
    t["X"] = t["X"][None]
    with pytest.raises(ValueError, match="unpack"):
        call(t)
    t = _tensors("cuda")
    t["X"] = torch.empty(5 * 256 + 1, dtype=torch.bfloat16, device="cuda")[1:].view(5, 256)
    with pytest.raises(P.PrismError, match="invalid argument"):
        call(t)


@pytest.mark.parametrize("name", NAMES)
def test_calls_that_are_not_the_native_routes_keep_their_errors(P, name):
    call = _calls(P)[name]
    t = _tensors("cpu", torch.float64)
    with pytest.raises(TypeError, match="unsupported tensor dtype"):
        call(t)
    t["X"] = t["X"][0]
    with pytest.raises(ValueError, match="unpack"):
        call(t)
