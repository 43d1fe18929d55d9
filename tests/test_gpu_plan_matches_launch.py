"""What prism_plan and prism_attention_plan report is what is launched: calls are recorded in a HIP graph and the grid and
block of the kernel in it are compared with the plan."""
import ctypes

import pytest

pytestmark = pytest.mark.gpu


class _Dim3(ctypes.Structure):
    _fields_ = [("x", ctypes.c_uint32), ("y", ctypes.c_uint32), ("z", ctypes.c_uint32)]


class _KernelNodeParams(ctypes.Structure):
    _fields_ = [("block", _Dim3), ("extra", ctypes.c_void_p), ("func", ctypes.c_void_p), ("grid", _Dim3),
                ("params", ctypes.c_void_p), ("lds", ctypes.c_uint32)]


def _hip():
    """The HIP runtime that is already in the process (PyTorch's copy)."""
    import torch
    torch.cuda.init()
    with open("/proc/self/maps") as f:
        paths = {line.split()[-1] for line in f if "libamdhip64" in line}
    assert len(paths) == 1, paths
    return ctypes.CDLL(paths.pop())


def _recorded(call):
    """(grid, block) of the one kernel that ``call(stream handle)`` launches."""
    import torch
    hip, stream = _hip(), torch.cuda.Stream()
    handle, graph, count = ctypes.c_void_p(stream.cuda_stream), ctypes.c_void_p(), ctypes.c_size_t(0)
    torch.cuda.synchronize()
    assert hip.hipStreamBeginCapture(handle, 2) == 0
    try:
        call(stream)
    finally:
        assert hip.hipStreamEndCapture(handle, ctypes.byref(graph)) == 0
    assert hip.hipGraphGetNodes(graph, None, ctypes.byref(count)) == 0 and count.value == 1
    node, kind, p = ctypes.c_void_p(), ctypes.c_int(-1), _KernelNodeParams()
    assert hip.hipGraphGetNodes(graph, ctypes.byref(node), ctypes.byref(count)) == 0
    assert hip.hipGraphNodeGetType(node, ctypes.byref(kind)) == 0 and kind.value == 0  # a kernel
    assert hip.hipGraphKernelNodeGetParams(node, ctypes.byref(p)) == 0
    assert hip.hipGraphDestroy(graph) == 0
    return (p.grid.x, p.grid.y, p.grid.z), (p.block.x, p.block.y, p.block.z)


@pytest.fixture(scope="module")
def P():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_2604_15272_amd as P
    P.prism_set_override(0, 0, 0)
    P.ensure_workspace(1 << 26)
    return P


def _compare(plan, recorded):
    grid, block = recorded
    assert grid == (plan["grid_x"], plan["grid_y"], max(1, plan["grid_z"])) and block == (plan["block"], 1, 1), (plan, recorded)


# fp32 and any shape: both kernels, narrow and wide, few rows and many; 16-bit: decode with and without K-slices, several row
# groups, prefill; softmax: fp32, 16 rows, K-slices.
@pytest.mark.parametrize("op,dtype,M,K,N", [
    (0, "f32", 8, 256, 512), (0, "f32", 1000, 512, 3000), (1, "f32", 512, 1024, 4096), (0, "bf16", 8, 1023, 9001),
    (1, "f16", 1021, 1201, 1023), (0, "f32", 3, 37, 3), (0, "bf16", 1999, 290, 2047), (0, "f16", 700, 13, 5001),
    (0, "bf16", 16, 4096, 4096), (1, "bf16", 8, 4096, 14336), (1, "f16", 8, 1024, 4096), (0, "bf16", 8, 64, 64),
    (0, "bf16", 200, 4096, 4096), (0, "bf16", 33, 520, 5128), (1, "bf16", 40, 512, 1024), (0, "bf16", 2048, 1024, 6144),
    (1, "bf16", 1000, 512, 4096), (2, "f32", 100, 1000, 200), (2, "f16", 4096, 512, 128), (2, "f16", 16, 8192, 128),
    (2, "bf16", 2000, 17, 900)])
def test_products_and_softmax(P, op, dtype, M, K, N):
    import torch
    dt = {"f32": torch.float32, "bf16": torch.bfloat16, "f16": torch.float16}[dtype]
    code = {"f32": P.PRISM_F32, "bf16": P.PRISM_BF16, "f16": P.PRISM_F16}[dtype]
    X, W, Y = (torch.zeros(s, dtype=dt, device="cuda") for s in ((M, K), (K, N), (M, N)))
    call = {0: lambda s: P.prism_rmsnorm_matmul(X, None, W, Y, stream=s),
            1: lambda s: P.prism_rmsnorm_glu(X, None, W, W, Y, stream=s),
            2: lambda s: P.prism_softmax_matmul(X, W, Y, stream=s)}[op]
    _compare(P.prism_plan(op, M, K, N, code), _recorded(call))


# Kernels by name, of calls that the dispatcher gives to another one.
@pytest.mark.parametrize("path,split,variant,op,dtype,M,K,N", [
    (2, 0, 0, 1, "f16", 8, 1024, 4096), (2, 0, 0, 1, "bf16", 40, 512, 1024), (2, 0, 108, 1, "bf16", 8, 512, 1024), (2, 3, 64, 0, "f16", 100, 512, 520),
    (2, 0, 0, 0, "bf16", 8, 512, 1024), (3, 0, 0, 1, "f16", 192, 512, 384), (1, 0, 0, 0, "bf16", 16, 4096, 4096), (1, 0, 0, 1, "f16", 2048, 512, 1024),
    (4, 0, 16, 2, "f16", 48, 1024, 128), (4, 2, 32, 2, "bf16", 48, 1024, 128), (1, 0, 0, 2, "f16", 4096, 512, 128)])
def test_kernels_by_name(P, path, split, variant, op, dtype, M, K, N):
    P.prism_set_override(path, split, variant)
    try:
        code = {"bf16": P.PRISM_BF16, "f16": P.PRISM_F16}[dtype]
        assert P.prism_plan(op, M, K, N, code)["path"] == path
        test_products_and_softmax(P, op, dtype, M, K, N)
    finally:
        P.prism_set_override(0, 0, 0)


@pytest.mark.parametrize("dtype,B,G,H,D", [("f16", 2, 8, 2048, 128), ("bf16", 3, 5, 100, 128), ("f32", 2, 8, 2048, 128),
                                           ("f16", 2, 8, 2000, 64), ("bf16", 3, 33, 700, 128), ("f32", 3, 33, 20, 64),
                                           ("f32", 2, 7, 300, 80)])
def test_attention(P, dtype, B, G, H, D):
    import torch
    dt = {"f32": torch.float32, "bf16": torch.bfloat16, "f16": torch.float16}[dtype]
    code = {"f32": P.PRISM_F32, "bf16": P.PRISM_BF16, "f16": P.PRISM_F16}[dtype]
    Q, K, O = (torch.zeros(s, dtype=dt, device="cuda") for s in ((B, G, D), (B, H, D), (B, G, D)))
    plan = P.prism_attention_plan(B, G, H, D, code)
    recorded = _recorded(lambda s: P.prism_gqa_decode_attention(Q, K, K, O, stream=s))
    _compare(plan, recorded)
    if plan["path"] == P.PRISM_PATH_SIMPLE:
        assert plan["grid_x"] == (G + plan["tile_m"] - 1) // plan["tile_m"]
