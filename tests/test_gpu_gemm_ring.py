"""The smaller-tile NT GEMM at the edges of its tiles: one row or column past a tile, one K step and fewer steps than the ring has
stages, column counts that 16-byte stores do not take, residual; against fp64 on the same bf16 inputs."""
import pytest
import torch

import paper_2509_22418_amd as pp

pytestmark = pytest.mark.gpu

CASES = [
    # M, N, K, residual (tile that the dispatch picks)
    (1, 8, 64, False), (65, 63, 128, True),                                  # 32 x 64
    (1003, 768, 192, False),                                                 # 64 x 64
    (3055, 772, 256, True), (3054, 761, 320, False),                         # 64 x 192
    (2048, 2040, 64, True), (2047, 1921, 320, False),                        # 128 x 128
    (8192, 768, 64, True), (8191, 761, 448, False),                          # 128 x 192
    (4096, 2048, 128, False), (4095, 2047, 256, True),                       # 128 x 256
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


def time_us(f):
    f()
    torch.cuda.synchronize()
    best = float("inf")
    for _ in range(5):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        for _ in range(50):
            f()
        b.record()
        torch.cuda.synchronize()
        best = min(best, a.elapsed_time(b) / 50 * 1e3)
    return best


@pytest.mark.parametrize("M,N,K,res,pad", [(1003, 772, 192, False, 0), (3055, 772, 256, True, 0), (2048, 2044, 320, True, 4), (8192, 764, 128, False, 0), (4096, 2044, 64, True, 0), (2000, 768, 64, False, 4)])
def test_columns_in_multiples_of_four(M, N, K, res, pad):
    """N or the leading dimension a multiple of 4 but not of 8: the same values as in rows of odd length, which are stored one column at a
    time, nothing written between the rows, and a time of at most 1.5 times that of the next multiple of 8."""
    print(f"case gemm ring by four {M}x{N}x{K} res={res} pad={pad}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(1)
    A, B, R = (torch.randn((n, k), device="cuda", generator=g).bfloat16() for n, k in ((M, K), (N + 8, K), (M, N + 8)))
    st, outs, us = torch.cuda.current_stream().cuda_stream, [], []
    for n, ldc in ((N, N + pad), (N, N + 3), ((N + 7) // 8 * 8, (N + pad + 7) // 8 * 8)):
        C = torch.full((M, ldc), 7.0, device="cuda").bfloat16()
        r = torch.zeros((M, ldc), device="cuda").bfloat16()
        r[:, :n] = R[:, :n]
        call = lambda: pp.pp_op_gemm_nt(st, pp.PP_BF16, A.data_ptr(), K, B.data_ptr(), K, C.data_ptr(), ldc, M, n, K, r.data_ptr() if res else None)  # noqa: E731
        us.append(time_us(call))
        assert bool((C[:, n:] == 7.0).all())
        outs.append(C[:, :N])
    assert torch.equal(outs[0], outs[1])
    assert us[0] <= 1.5 * us[2], us
