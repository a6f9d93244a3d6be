"""The fp32-multiply NT GEMM around its number of K steps (64 each): short and long ranges, remainders, rows that are not 16-byte aligned, split ranges and
few or many tiles give the plain kernel's bits."""
import pytest
import torch

import paper_2509_22418_amd as pp

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,N", [(1, 1), (33, 70), (128, 64), (1000, 520), (1100, 2100)])
@pytest.mark.parametrize("K", [255, 256, 257, 320, 384, 449, 512, 1023])
def test_same_bits_as_the_plain_kernel(M, N, K):
    check(M, N, K, (K + 3) // 4 * 4, 1)


@pytest.mark.parametrize("M,N,K,ld,splits", [(65, 130, 512, 513, 1), (65, 130, 1024, 1024, 2), (200, 72, 1280, 1281, 4), (200, 72, 2048, 2049, 4), (31, 33, 260, 262, 1), (31, 33, 511, 514, 1)])
def test_unaligned_rows_and_split_ranges(M, N, K, ld, splits):
    check(M, N, K, ld, splits)


def check(M, N, K, ld, splits):
    print(f"case gemm f32 steps {M}x{N}x{K} ld={ld} splits={splits}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(1)
    A, B = (torch.randn((n, ld), device="cuda", generator=g) for n in (M, N))
    R = torch.randn((M, N), device="cuda", generator=g) if splits == 1 else None
    out = []
    for path in (0, 1):
        C = torch.full((M, N), 7.0, device="cuda")
        scratch = torch.empty(M * N * splits, device="cuda")
        pp.pp_op_gemm_nt(torch.cuda.current_stream().cuda_stream, pp.PP_F32, A.data_ptr(), ld, B.data_ptr(), ld, C.data_ptr(), N, M, N, K,
                         R.data_ptr() if R is not None else None, int(splits > 1), splits, scratch.data_ptr() if splits > 1 else None, path)
        torch.cuda.synchronize()
        out.append(C)
    assert torch.equal(out[0], out[1])
