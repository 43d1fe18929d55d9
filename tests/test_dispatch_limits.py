"""Limits between kernels and forms, on 256 compute units, with the times that put them there."""
import pytest


@pytest.fixture()
def P():
    import paper_2604_15272_amd as P
    P.prism_diag_set_cu_count(256)
    yield P
    P.prism_diag_set_cu_count(0)


def test_f16_softmax_of_very_shallow_k_and_many_outputs_on_the_rows_kernel(P):
    path = lambda dtype, M, K, N: P.prism_plan(P.PRISM_OP_SOFTMAX_MATMUL, M, K, N, dtype)["path"]
    for M, N in ((3745, 2072), (2633, 7368), (6067, 2936), (4676, 5504)):   # us: 41.5 / 62.0 on the kernel for any shape, 96 / 145, 91 / 134, 125 / 191
        assert path(P.PRISM_F16, M, 32, N) == P.PRISM_PATH_ROWS
    assert path(P.PRISM_F16, 480, 32, 4496) == P.PRISM_PATH_SIMPLE    # 23.0 / 19.6
    assert path(P.PRISM_BF16, 7263, 32, 4240) == P.PRISM_PATH_SIMPLE  # 168 / 139


def test_few_workgroups_of_two_narrow_matrices(P):
    for M, K, N in ((1, 1536, 8), (8, 1536, 24), (8, 1792, 24)):   # us from HBM: 5.1 / 7.3 on the decode kernel, 6.9 / 7.9, 7.8 / 8.2
        assert P.prism_plan(1, M, K, N, P.PRISM_BF16)["path"] == P.PRISM_PATH_SIMPLE
    assert P.prism_plan(1, 8, 1792, 1024, P.PRISM_BF16)["path"] == P.PRISM_PATH_DECODE   # 13.6 / 10.1


def test_form_for_rows_of_x_at_even_elements(P):
    form = lambda gated, dtype, M, K, N: (lambda p: (p["tile_m"], p["tile_n"]))(P.prism_plan(gated, M, K, N, dtype))
    bf16, f16 = P.PRISM_BF16, P.PRISM_F16
    for c in ((0, bf16, 61, 4650, 5271), (1, bf16, 62, 6800, 6621), (0, f16, 127, 6644, 2853), (0, f16, 23, 7518, 11117)):   # us: 28 / 36, 57 / 73, 39 / 50, 38 / 54
        assert form(*c) == (32, 64), c
    for c in ((0, f16, 82, 4609, 4357), (0, bf16, 297, 788, 858)):   # in 16 x 128 42.0, 46.5 in 32 x 64; 7.0 / 8.4
        assert form(*c) == (16, 128), c
