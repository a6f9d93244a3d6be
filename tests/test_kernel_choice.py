"""Which kernel the estimates pick, at shapes timed on both sides (no GPU needed: the library's own functions are asked)."""
import ctypes

import pytest

import paper_2509_22418_amd as pp

SWIGLU, SWIGLU_BWD, ROPE = 2, 3, 4

# (epilogue, M, hidden units / columns / d, K, small tiles): us, 256 x 256 / 128 x 192 tiles
FUSED = [(SWIGLU, 3055, 3072, 768, True),           # 43.9 / 36.4
         (SWIGLU, 200, 3072, 768, True),            # 19.4 / 13.7
         (SWIGLU, 1625, 4936, 1088, True),          # 69.4 / 54.9
         (SWIGLU, 1437, 2400, 2432, True),          # 62.0 / 52.4
         (SWIGLU, 8192, 3072, 768, False),          # 82.9 / 115
         (SWIGLU, 3470, 6128, 2368, False),         # 196 / 207
         (SWIGLU_BWD, 8192, 3072, 768, True),       # 69.4 / 65.3
         (SWIGLU_BWD, 2000, 2048, 512, True),       # 23.8 / 14.6
         (SWIGLU_BWD, 6674, 2776, 1472, True),      # 89.6 / 77.8
         (SWIGLU_BWD, 8192, 2048, 768, False),      # 38.0 / 41.3
         (SWIGLU_BWD, 3847, 8096, 448, False),      # 68.2 / 76.5
         (SWIGLU_BWD, 4894, 2800, 320, False),      # 28.9 / 31.8
         (ROPE, 8192, 768, 768, True),              # 50.4 / 36.1
         (ROPE, 16384, 768, 768, True),             # 74.3 / 68.2
         (ROPE, 1000, 3072, 3072, False),           # 70.2 / 76.7
         (ROPE, 753, 3840, 3840, False),            # 87.0 / 93.4
         (ROPE, 2967, 1536, 1536, False)]           # 44.0 / 62.1


@pytest.mark.parametrize("epi,M,n,K,small", FUSED)
def test_fused_gemms_run_on_the_faster_tiles(epi, M, n, K, small):
    f = pp.load_library()["_ZN2pp18gemm_fused_on_ringEiiii"]
    f.restype = ctypes.c_bool
    pp.pp_set_option(None, "gemm_small_tiles", 1)
    assert f(epi, M, n, K) == small
    pp.pp_set_option(None, "gemm_small_tiles", 0)
    off = f(epi, M, n, K)
    pp.pp_set_option(None, "gemm_small_tiles", 1)
    assert not off


# (M, N, K, rows in whole groups of four, fragments a step ahead): us, plain loop / a step ahead
F32 = [(1024, 512, 2048, True, True),           # 32.1 / 26.3
       (1024, 1536, 512, True, True),           # 19.7 / 18.7
       (128, 64, 256, True, True),              # 4.3 / 4.0
       (128, 64, 64, True, False),              # 3.8 / 4.2
       (1024, 2048, 512, True, False),          # 23.2 / 24.2
       (1170, 1000, 320, True, False),          # 14.6 / 15.1
       (49, 254, 263, False, False),            # 7.5 / 8.1
       (1748, 146, 285, False, False),          # 12.0 / 12.7
       (308, 30, 271, False, False)]            # 7.1 / 7.6


@pytest.mark.parametrize("M,N,K,vec,ahead", F32)
def test_fp32_gemm_runs_the_faster_loop(M, N, K, vec, ahead):
    f = pp.load_library()["_ZN2pp20gemm_f32_reads_aheadElib"]
    f.restype, f.argtypes = ctypes.c_bool, [ctypes.c_long, ctypes.c_int, ctypes.c_bool]
    assert f(-(-M // 32) * -(-N // 32), K, vec) == ahead
