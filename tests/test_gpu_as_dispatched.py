"""Calls that the dispatcher gives to whichever kernel it estimates to be the fastest, by default settings, against the oracle: the sizes at which the
tests of the single kernels ask for them by name, and sizes near the limits between the forms of the kernels for any shape."""
import pytest

import prism_inputs as pi
from gpu_util import assert_parity, run_gpu, run_gpu_softmax, run_oracle, run_oracle_softmax

pytestmark = pytest.mark.gpu

# Two matrices or one, M, K, N (ALIGNED: M, K, N, seed)
F32 = [(False, 1682, 43, 19), (False, 1649, 65, 19), (False, 23, 47, 18), (False, 3061, 131, 209), (False, 3, 43, 4255), (False, 2100, 1263, 18),
       (False, 737, 137, 2005), (False, 2052, 135, 69), (False, 3279, 43, 262), (False, 1106, 41, 1861), (True, 1652, 41, 18), (True, 1654, 67, 19),
       (True, 3, 41, 18), (True, 4148, 137, 65), (True, 3, 43, 4255), (True, 4199, 287, 71), (True, 2296, 275, 18), (True, 4887, 129, 135),
       (True, 2075, 133, 75), (True, 4082, 47, 195), (True, 1950, 41, 1047)]
ANY_SHAPE_16 = [(False, 1720, 43, 19), (False, 1713, 65, 18), (False, 23, 45, 18), (False, 4088, 153, 130), (False, 3, 43, 4307), (False, 4093, 159, 258),
                (False, 1409, 137, 129), (False, 2123, 145, 18), (False, 8710, 133, 167), (False, 2116, 271, 66), (False, 4124, 41, 235),
                (False, 4708, 45, 385), (True, 1705, 41, 22), (True, 1734, 75, 18), (True, 23, 45, 19), (True, 4237, 129, 82), (True, 3, 45, 4355),
                (True, 3244, 137, 197), (True, 1390, 131, 129), (True, 4117, 129, 67), (True, 33, 125, 1429), (True, 4999, 133, 130), (True, 2307, 193, 67),
                (True, 2389, 43, 389), (True, 623, 41, 3353)]
# K and N multiples of 8: the kernels made for 16-bit storage, or the one for any shape
ALIGNED = [(1, 512, 128, 429), (7, 1024, 1000, 8102), (7, 4096, 1024, 1331), (8, 1000, 264, 572), (13, 64, 8, 321), (16, 8, 16, 332), (16, 4104, 4104, 4420),
           (5, 264, 5128, 478), (16, 520, 5128, 478), (40, 264, 5128, 478), (33, 520, 5128, 478), (8, 136, 33288, 478), (1, 512, 2048, 471),
           (16, 8192, 1024, 486), (16, 1024, 4096, 486), (3, 2048, 7168, 473), (33, 2048, 136, 475), (200, 4104, 520, 475), (8, 256, 512, 908),
           (8, 1024, 1024, 908), (13, 2056, 1160, 913), (30, 200, 264, 930), (300, 712, 648, 1200), (100, 1024, 1024, 475)]
SOFTMAX = [(1, 8, 8), (16, 512, 128), (33, 1000, 264), (100, 4096, 128), (7, 72, 16), (257, 2056, 136), (64, 8200, 128), (16, 256, 4096)]


@pytest.fixture(scope="module")
def P():
    import paper_2604_15272_amd as P
    P.prism_set_override(0, 0, 0)
    P.prism_set_stream_balance(0, 0)
    return P


@pytest.mark.parametrize("dtype,gated,M,K,N,seed", [(pi.F32, *s, 310 + s[2]) for s in F32] + [(d, *s, 310 + s[2]) for d in (pi.BF16, pi.F16) for s in ANY_SHAPE_16] +
                         [(d, g, *s) for d in (pi.BF16, pi.F16) for g in (False, True) for s in ALIGNED])
def test_products(P, dtype, gated, M, K, N, seed):
    stored = pi.draw(dtype, M, K, N, gated, seed)
    assert_parity(run_gpu(stored, dtype, gated, 1e-6), run_oracle(stored, dtype, gated, 1e-6), dtype, f"M={M} K={K} N={N} gated={gated}")


@pytest.mark.parametrize("dtype", [pi.BF16, pi.F16])
@pytest.mark.parametrize("M,K,N", SOFTMAX)
def test_softmax(P, dtype, M, K, N):
    stored = pi.draw_softmax(dtype, M, K, N, 1000 + M + K, 3.0)
    assert_parity(run_gpu_softmax(stored, dtype), run_oracle_softmax(stored, dtype), dtype, f"softmax M={M} K={K} N={N}")
