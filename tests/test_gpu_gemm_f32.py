"""fp32-multiply MFMA GEMM (fp32 models, and bf16 shapes that the bf16 MFMA kernels refuse) against fp64 products of the same
stored values, at the edges of its two tiles: remainders in M, N and K, unaligned leading dimensions, split K, residual."""
import numpy as np
import pytest
import torch

import pp_inputs as gen
import paper_2509_22418_amd as pp

pytestmark = pytest.mark.gpu


def rnd(shape, seed):
    return gen.normal(gen.stream_key(seed, gen.STREAM_MISC, 3), int(np.prod(shape))).reshape(shape)


CASES = [
    # M, N, K, lda - K, residual, splits
    (1, 1, 1, 0, False, 1),
    (33, 31, 5, 0, True, 1),                 # one tile and a row, odd K: single-element loads
    (64, 96, 128, 4, False, 1),              # whole 32 x 32 tiles, one K step
    (70, 45, 257, 3, True, 1),               # K one past two steps, unaligned rows
    (32, 64, 384, 0, False, 3),              # split K
    (48, 40, 60, 0, False, 4),               # split K with 15 elements per range: no vector loads
    (2052, 2049, 36, 0, True, 1),            # 64 x 64 tiles (1089 of them), remainders in all three
    (2048, 2048, 96, 1, False, 1),
]


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("M,N,K,pad,res,splits", CASES)
def test_gemm_nt_f32_matches_fp64(M, N, K, pad, res, splits, dtype):
    print(f"case gemm f32 {M}x{N}x{K} pad={pad} res={res} splits={splits} {dtype}", flush=True)
    bf16 = dtype == "bf16"
    if bf16 and K // splits % 64 == 0 and (K + pad) % 8 == 0:
        pytest.skip("taken by the bf16 kernels")
    td = torch.bfloat16 if bf16 else torch.float32
    A = torch.from_numpy(rnd((M, K + pad), 1)).to(td).cuda()
    B = torch.from_numpy(rnd((N, K + pad), 2)).to(td).cuda()
    R = torch.from_numpy(rnd((M, N), 3)).to(td).cuda() if res else None
    ref = A[:, :K].double() @ B[:, :K].double().T + (R.double() if res else 0.0)
    f32out = not bf16 or splits > 1
    out = []
    for path in (0, 1):
        C = torch.full((M, N), float("nan"), dtype=torch.float32 if f32out else td, device="cuda")
        scratch = torch.empty(M * N * splits, dtype=torch.float32, device="cuda")
        pp.pp_op_gemm_nt(torch.cuda.current_stream().cuda_stream, pp.PP_BF16 if bf16 else pp.PP_F32, A.data_ptr(), K + pad, B.data_ptr(), K + pad, C.data_ptr(), N, M, N, K,
                         R.data_ptr() if res else None, int(splits > 1), splits, scratch.data_ptr(), path)
        torch.cuda.synchronize()
        out.append(C)
    C = out[0]
    assert torch.equal(out[0], out[1])          # the same fmaf chain per element as the plain kernel
    # K products and a residual summed in fp32: at most (K + 1) half-ulp roundings of partial sums bounded by sum |a b| + |r|
    bound = A[:, :K].double().abs() @ B[:, :K].double().abs().T + (R.double().abs() if res else 0.0)
    tol = (K + 2) * 2.0 ** -24 * bound + (0.0 if f32out else 2.0 ** -8 * ref.abs())
    assert bool(((C.double() - ref).abs() <= tol).all())


STEPS = [
    (1, 1, {}), (3, 19, dict(d_model=72, n_heads=3, d_ff=200, vocab=264)), (2, 150, dict(d_model=96, n_heads=6, d_ff=136, vocab=520)),
    (2, 512, {}),                                                             # 1024 tokens: four K ranges, summed in order
    (2, 257, dict(n_layers=1, d_model=264, n_heads=3, vocab=8200)),           # lm_head: 645 tiles of 64 x 64; two K ranges of 257 tokens elsewhere
    (1, 37, dict(d_model=48, n_heads=8, d_ff=72, vocab=104)),                 # head dim 6: column blocks of 12 at an offset of 6, no vector loads
]


@pytest.mark.parametrize("B,S,over", STEPS)
@pytest.mark.parametrize("mname", ["all", "heads"])
def test_f32_step_weight_gradients_match_the_plain_kernels(B, S, over, mname):
    """Token-major weight gradients (column blocks, ragged token counts) and projections of an fp32 model add in the order of the
    plain kernels: the same step on those gives the same bits."""
    cfg = gen.make_config("tiny", **dict(dict(batch=B, seq=S), **over))
    weights = gen.make_weights(cfg, seed=5)
    mask = gen.all_mask(cfg) if mname == "all" else dict(gen.ffn_slice_mask(cfg, 0, 1), ffn_lo=8, ffn_hi=24, head_lo=1, head_hi=3, train_wo=1)
    tok, tgt = gen.make_tokens(cfg, seed=5)
    if B * S == 1:
        tgt[:] = 7
    g, loss = [], []
    for plain in (0, 1):
        m = pp.LocalStepModel(cfg, mask)
        m.load_weights(weights)
        m.set_mask()
        m.set_option("force_plain", plain)
        loss.append(float(m.step(*m.upload_tokens(tok, tgt), None).item()))
        g.append(m.get_state("g").astype(np.float64))
        m.close()
    assert loss[0] == loss[1]
    assert np.array_equal(g[0], g[1])


def test_f32_weight_gradients_through_transposed_copies_have_the_same_bits():
    """Option dw_tn = 0 sends an fp32 model's weight gradients through transposed copies (which appear in the workspace: two runs alike leave it
    alike) with the same ranges and order of sums."""
    cfg = gen.make_config("tiny", batch=2, seq=257)
    m = pp.LocalStepModel(cfg, gen.all_mask(cfg))
    m.load_weights(gen.make_weights(cfg, seed=5))
    m.set_mask()
    tok = m.upload_tokens(*gen.make_tokens(cfg, seed=5))
    g, ws = [], []
    for dw_tn in (1, 1, 0):
        m.set_option("dw_tn", dw_tn)
        m.step(*tok, None)
        g.append(m.get_state("g"))
        ws.append(m.ws.clone())
    m.close()
    assert np.array_equal(g[0], g[1]) and np.array_equal(g[0], g[2])
    assert torch.equal(ws[0], ws[1]) and not torch.equal(ws[0], ws[2])
