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
