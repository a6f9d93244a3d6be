"""Weight gradients over token counts that are not a multiple of the token-major kernel's K step, and column blocks that are not
whole tiles: a bf16 step against the same step on the plain kernels."""
import ctypes

import numpy as np
import pytest
import torch

import pp_inputs as gen
import paper_2509_22418_amd as pp
from harness import cosine

pytestmark = pytest.mark.gpu

# (batch, seq): one token, one row short of / past a K step of 64, and counts that several K ranges cut unevenly
TOKENS = [(1, 1), (1, 63), (1, 65), (3, 171), (2, 641)]


@pytest.mark.parametrize("B,S", TOKENS)
@pytest.mark.parametrize("mname", ["all", "slices"])
def test_ragged_token_counts_match_the_plain_kernels(B, S, mname):
    """mask "slices": 24 hidden units (gate and up blocks of 24 columns in one tile) and one head.  Both paths multiply the same
    bf16 operands and sum in fp32, but round the activations between layers from differently ordered sums: two layers of bf16
    roundings (2^-9 each) on gradients of a common scale stay within 2 % of it."""
    print(f"case dw ragged B={B} S={S} {mname}", flush=True)
    cfg = gen.make_config("tiny", n_layers=2, d_model=128, n_heads=2, d_ff=256, vocab=576, batch=B, seq=S, dtype="bf16")
    weights = gen.make_weights(cfg, seed=31)
    mask = gen.all_mask(cfg) if mname == "all" else dict(ffn_lo=8, ffn_hi=32, head_lo=1, head_hi=2, train_wo=1, train_norms=0, train_embed=0, train_lm_head=1)
    tok, tgt = gen.make_tokens(cfg, seed=31)
    if B * S == 1:
        tgt[:] = 7
    g, calls = [], []
    for plain in (0, 1):
        m = pp.LocalStepModel(cfg, mask)
        m.load_weights(weights)
        m.set_mask()
        m.set_option("force_plain", plain)
        m.step(*m.upload_tokens(tok, tgt), None)
        g.append(m.get_state("g").astype(np.float64))
        calls.append(m.launch_counts())
        m.close()
    assert calls[0]["plain_calls"] == 0, calls[0]
    assert np.all(np.isfinite(g[0]))
    assert cosine(g[0], g[1]) >= 0.9995
    assert np.linalg.norm(g[0] - g[1]) <= 0.02 * np.linalg.norm(g[1])


@pytest.mark.parametrize("M,N,splits", [(1024, 2048, 8), (1024, 2048, 4), (1160, 2056, 16), (1160, 2056, 6)])
def test_more_ranges_than_fill_the_gpu_are_joined(M, N, splits):
    """128 tiles: eight ranges are run as four, four as four.  170 tiles: sixteen are run as four, six as six.  fp32 sums of at most K products and `splits` partial
    sums: (K + splits) half-ulp roundings of sum |a b| bound the error, and no partial is left out or added twice."""
    K = 64 * splits * 2
    g = torch.Generator(device="cuda").manual_seed(9)
    A = torch.randn(K, M, device="cuda", generator=g).bfloat16()
    B = torch.randn(K, N, device="cuda", generator=g).bfloat16()
    C = torch.full((M, N), float("nan"), device="cuda")
    scratch = torch.full((M * N * splits,), float("nan"), device="cuda")
    pp.pp_op_gemm_tn(torch.cuda.current_stream().cuda_stream, A.data_ptr(), M, M, 0, B.data_ptr(), N, C.data_ptr(), N, M, N, K, splits, scratch.data_ptr())
    torch.cuda.synchronize()
    ref = A.double().T.contiguous() @ B.double()
    bound = A.double().abs().T.contiguous() @ B.double().abs()
    assert bool(((C.double() - ref).abs() <= (K + splits) * 2.0 ** -24 * bound).all())


@pytest.mark.parametrize("splits", [2, 4])
def test_joined_ranges_are_summed_apart(splits):
    """512 tiles: all ranges joined to one, which writes C itself.  The first range of 128 rows sums to 2^30 (spacing 128), each later one to 128
    by sixteens: added one by one they would be lost, as sums of their own they are exact.  Rows of C are longer than N."""
    M, N, K, ldc = 2048, 4096, 128 * splits, 4104
    col = torch.ones(K, 1, device="cuda")
    col[:128] = 0.0
    col[5] = 2.0 ** 15
    A, B = (col.expand(K, n).bfloat16().contiguous() for n in (M, N))
    C = torch.full((M, ldc), 7.0, device="cuda")
    scratch = torch.empty((M * N * splits,), device="cuda")
    pp.pp_op_gemm_tn(torch.cuda.current_stream().cuda_stream, A.data_ptr(), M, M, 0, B.data_ptr(), N, C.data_ptr(), ldc, M, N, K, splits, scratch.data_ptr())
    torch.cuda.synchronize()
    assert bool((C[:, :N] == 2.0 ** 30 + 128.0 * (splits - 1)).all())
    assert bool((C[:, N:] == 7.0).all())


@pytest.mark.parametrize("K", [1, 63, 65, 130, 200])
def test_infinities_in_the_last_row_reach_no_padding(K):
    """The last K step of a ragged count is filled up with copies of the last row and then with zeros.  An infinity in that row gives
    infinities of the right sign where its own products do, and no NaN: neither panel is zeroed without the other.  (The kernel's C++
    entry: the C one takes whole steps only.)"""
    print(f"case dw last row K={K}", flush=True)
    M, N = 136, 72
    tn = ctypes.CDLL(pp.lib_path())["_ZN2pp14k_gemm_tn_mfmaEP12ihipStream_tPKviilS3_iPfiiiiiS4_i"]
    P, I = ctypes.c_void_p, ctypes.c_int
    tn.argtypes = [P, P, I, I, ctypes.c_long, P, I, P, I, I, I, I, I, P, I]
    g = torch.Generator(device="cuda").manual_seed(K)
    A, B = (torch.randn((K, n), device="cuda", generator=g).bfloat16() for n in (M, N))
    A[-1, 3] = float("inf")
    B[-1, 70] = float("-inf")
    C = torch.zeros((M, N), device="cuda")
    assert tn(torch.cuda.current_stream().cuda_stream, A.data_ptr(), M, M, 0, B.data_ptr(), N, C.data_ptr(), N, M, N, K, (K + 63) // 64 * 64, None, 1 << 30) == 0
    torch.cuda.synchronize()
    ref, bound = A.double().T.contiguous() @ B.double(), A.double().abs().T.contiguous() @ B.double().abs()
    fin = torch.isfinite(ref)
    assert int((~fin).sum()) == M + N - 1 and not bool(torch.isnan(ref).any())
    assert torch.equal(C.double()[~fin], ref[~fin])
    assert bool(((C.double() - ref).abs()[fin] <= K * 2.0 ** -24 * bound[fin]).all())
