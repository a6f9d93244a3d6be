"""The smaller-tile NT GEMM at the edges of its five tiles: one row or column past a tile, one K step and fewer steps than the ring has
stages, column counts that 16-byte stores do not take, residual; against fp64 on the same bf16 inputs."""
import pytest
import torch

import paper_2509_22418_amd as pp

pytestmark = pytest.mark.gpu

CASES = [
    # M, N, K, residual (tile that the dispatch picks)
    (1, 8, 64, False), (65, 63, 128, True), (1003, 768, 192, False),        # 64 x 64
    (3055, 772, 256, True), (3054, 761, 320, False),                         # 64 x 96
    (2048, 2040, 64, True), (2047, 1921, 320, False),                        # 128 x 128
    (8192, 768, 64, True), (8191, 761, 448, False),                          # 128 x 192
    (4096, 2048, 128, False), (4095, 2047, 256, True),                       # 256 x 128
]


@pytest.mark.parametrize("M,N,K,res", CASES)
def test_matches_fp64(M, N, K, res):
    print(f"case gemm ring {M}x{N}x{K} res={res}", flush=True)
    pp.pp_set_option(None, "gemm_variant", 1)
    pp.pp_set_option(None, "gemm_small_tiles", 1)
    g = torch.Generator(device="cuda").manual_seed(1)
    A = torch.randn((M, K + 8), device="cuda", generator=g).bfloat16()
    B = torch.randn((N, K + 16), device="cuda", generator=g).bfloat16()
    ldc = N + 3 if N % 8 else N
    R = torch.randn((M, ldc), device="cuda", generator=g).bfloat16() if res else None
    C = torch.full((M, ldc), 7.0, device="cuda").bfloat16()
    pp.pp_op_gemm_nt(torch.cuda.current_stream().cuda_stream, pp.PP_BF16, A.data_ptr(), K + 8, B.data_ptr(), K + 16, C.data_ptr(), ldc, M, N, K,
                     R.data_ptr() if res else None, 0, 1, None, 0)
    torch.cuda.synchronize()
    ref = A[:, :K].double() @ B[:, :K].double().T + (R[:, :N].double() if res else 0.0)
    bound = A[:, :K].double().abs() @ B[:, :K].double().abs().T + (R[:, :N].double().abs() if res else 0.0)
    # one bf16 rounding of the result, fp32 sums of K products
    assert bool(((C[:, :N].double() - ref).abs() <= 2.0 ** -8 * ref.abs() + (K + 2) * 2.0 ** -24 * bound).all())
    assert bool((C[:, N:] == 7.0).all())          # nothing past the last column
