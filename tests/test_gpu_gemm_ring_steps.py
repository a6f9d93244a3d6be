"""The smaller-tile NT GEMM around the length of its ring: every tile with 1 .. 9 K steps (fewer than, as many as and more than the stages, odd and
even counts) and on both sides of a tile's edge, against fp64 on the same bf16 inputs."""
import pytest
import torch

import paper_2509_22418_amd as pp

pytestmark = pytest.mark.gpu

SHAPES = [
    # M, N, residual (tile that the dispatch picks at most of these lengths)
    (33, 200, True),          # 32 x 64
    (1003, 772, False),       # 32 x 64, 64 x 64
    (2100, 512, True),        # 64 x 96
    (1024, 2044, False),      # 64 x 128
    (3055, 769, True),        # 128 x 128
    (8191, 761, True),        # 128 x 192, two and three stages
    (3000, 2300, False),      # 128 x 256
]


@pytest.mark.parametrize("steps", [1, 2, 3, 4, 5, 6, 7, 8, 9])
@pytest.mark.parametrize("M,N,res", SHAPES)
def test_matches_fp64(M, N, res, steps):
    check(M, N, 64 * steps, res)


@pytest.mark.parametrize("M,N,K,res", [(1003, 520, 2048, False), (500, 1000, 2112, True), (2100, 512, 2048, True), (1024, 1020, 2112, False), (3055, 769, 2112, True), (2047, 768, 4096, False),
                                       (8191, 761, 2048, True), (4095, 2041, 2048, False), (33, 2047, 2112, True), (300, 24, 32000, False)])
def test_long_contraction(M, N, K, res):
    """From K = 2048 on the kernel also touches B ahead of its steps (up to four words per thread, the rest of B not at all)."""
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
