"""The smaller-tile NT GEMM around the length of its ring: every tile with 1 .. 9 K steps (fewer than, as many as and more than the stages, odd and
even counts) and on both sides of a tile's edge, against fp64 on the same bf16 inputs."""
import pytest
import torch

import paper_2509_22418_amd as pp

TILES = ["32 x 64", "64 x 64", "64 x 96", "64 x 128", "64 x 192", "128 x 128", "128 x 192", "128 x 256"]
SHAPES = [
    # M, N, residual, tile at 1 .. 9 steps (asserted)
    (33, 200, True, [0] * 9),
    (1003, 772, False, [3] + [1] * 8),
    (8333, 129, True, [1] * 9),
    (2100, 512, True, [0, 0] + [3] * 6 + [2]),
    (9303, 265, False, [2] * 9),
    (1024, 2044, False, [1, 1] + [3] * 7),
    (6201, 198, False, [1] + [3] * 8),
    (3055, 769, True, [4] * 9),
    (2047, 2041, True, [5] * 9),
    (8191, 761, True, [6] * 9),
    (3000, 2300, False, [7] * 9),
]
# From K = 2048 on the tiles from 64 x 128 also touch B ahead of their steps (up to four words per thread, the rest of B not at all)
LONG = [(1003, 520, 2048, False, 1), (500, 1000, 2112, True, 1), (2100, 512, 2048, True, 2), (1024, 1020, 2112, False, 1), (3055, 769, 2112, True, 4), (2047, 768, 4096, False, 2), (8191, 761, 2048, True, 6),
        (4095, 2041, 2048, False, 7), (33, 2047, 2112, True, 0), (300, 24, 32000, False, 0), (5441, 197, 2112, True, 3), (5443, 200, 2048, False, 3), (3359, 583, 2112, False, 5), (2047, 2041, 2048, True, 5)]


def tile(M, N, K):
    return pp.load_library()["_ZN2pp14gemm_ring_tileEiii"](M, N, K)


def test_every_tile_and_length_is_among_the_cases():
    for M, N, _, tiles in SHAPES:
        assert [tile(M, N, 64 * s) for s in range(1, 10)] == tiles
        assert -(-M // 256) * -(-N // 256) <= 128          # or the big tiles run
    for M, N, K, _, t in LONG:
        assert tile(M, N, K) == t and -(-M // 256) * -(-N // 256) <= 128
    for s in range(9):
        assert {tiles[s] for _, _, _, tiles in SHAPES} == set(range(8))
    assert {t for _, _, _, _, t in LONG} == set(range(8))


@pytest.mark.gpu
@pytest.mark.parametrize("steps", [1, 2, 3, 4, 5, 6, 7, 8, 9])
@pytest.mark.parametrize("M,N,res,tiles", SHAPES)
def test_matches_fp64(M, N, res, tiles, steps):
    check(M, N, 64 * steps, res)


@pytest.mark.gpu
@pytest.mark.parametrize("M,N,K,res,t", LONG)
def test_long_contraction(M, N, K, res, t):
    check(M, N, K, res)


def check(M, N, K, res):
    print(f"case gemm ring steps {M}x{N}x{K} res={res}", flush=True)
    pp.pp_set_option(None, "gemm_variant", 1)
    pp.pp_set_option(None, "gemm_small_tiles", 1)
    g = torch.Generator(device="cuda").manual_seed(1)
    A, B = (torch.randn((n, K), device="cuda", generator=g).bfloat16() for n in (M, N))
    R = torch.randn((M, N), device="cuda", generator=g).bfloat16() if res else None
    C = torch.full((M, N), 7.0, device="cuda").bfloat16()
    pp.pp_op_gemm_nt(torch.cuda.current_stream().cuda_stream, pp.PP_BF16, A.data_ptr(), K, B.data_ptr(), K, C.data_ptr(), N, M, N, K, R.data_ptr() if res else None)
    torch.cuda.synchronize()
    ref = A.double() @ B.double().T + (R.double() if res else 0.0)
    bound = A.double().abs() @ B.double().abs().T + (R.double().abs() if res else 0.0)
    # one bf16 rounding of the result, fp32 sums of K products
    assert bool(((C.double() - ref).abs() <= 2.0 ** -8 * ref.abs() + (K + 2) * 2.0 ** -24 * bound).all())
