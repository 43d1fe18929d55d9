"""The native route of ordinary calls from Python: the same results as the general route, the same refusals."""
import importlib.util
import os
import subprocess
import sys
import sysconfig

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


def test_the_package_works_without_the_native_module(repo_root):
    """The module only shortens calls: where it was not built the general route takes them."""
    code = ("import sys; sys.modules['paper_2604_15272_amd._marshal'] = None\n"
            "import paper_2604_15272_amd as P; from paper_2604_15272_amd import binding\n"
            "assert binding._native is None and P.prism_version() >= 200")
    res = subprocess.run([sys.executable, "-c", code], cwd=repo_root, capture_output=True, text=True)
    assert res.returncode == 0, res.stderr[-2000:]


def test_the_library_is_built_without_pythons_headers(repo_root, monkeypatch, tmp_path):
    spec = importlib.util.spec_from_file_location("_prism_build_for_test",
                                                  os.path.join(repo_root, "paper_2604_15272_amd", "build.py"))
    build = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(build)
    assert os.path.basename(build.MARSHAL).startswith("_marshal.cpython-")  # found by the interpreter it is for, no other
    monkeypatch.setattr(sysconfig, "get_paths", lambda: {"include": str(tmp_path)})
    assert build.build_marshal() is None
    calls = []
    monkeypatch.setattr(build, "build_marshal", lambda: calls.append("marshal"))
    monkeypatch.setattr(build, "LIB", str(tmp_path / "libprism.so"))

    def compiler(cmd, **kw):
        calls.append(os.path.basename(cmd[0]))
        open(cmd[cmd.index("-o") + 1], "w").close()
        return subprocess.CompletedProcess(cmd, 0, "", "")

    monkeypatch.setattr(build.subprocess, "run", compiler)
    assert build.build_library() == build.LIB and calls == [os.path.basename(build.hipcc_path())]


@pytest.mark.gpu
def test_the_native_route_is_the_one_that_runs(P):
    from paper_2604_15272_amd import binding
    assert binding._native is not None
    t = _tensors("cuda")
    assert binding._native.product(*binding._SOFTMAX, t["X"], None, t["W1"], None, t["Y"], 0.0) == 0
