"""The SwiGLU and rotary GEMMs on small tiles give the bits of the big-tile kernels: whole steps of models whose token counts, widths and hidden units end in the
middle of a tile, with the smaller-tile kernels on and off."""
import ctypes

import pytest
import torch

import pp_inputs as gen
import paper_2509_22418_amd as pp

pytestmark = pytest.mark.gpu

# (d_model, heads, d_ff, batch, seq): rotated tiles of 768 and 1536 columns (heads of 64 and 128), hidden units that end 8 past a tile of 96 or 192, token counts on
# both sides of a tile of 128, and widths whose rotation stays on the big tiles
CASES = [(768, 12, 1544, 1, 127), (768, 6, 200, 3, 43), (768, 12, 96, 1, 1), (1536, 12, 392, 1, 385), (256, 4, 1024, 2, 300), (192, 3, 104, 1, 65)]


@pytest.mark.parametrize("mname", ["all", "slice"])
@pytest.mark.parametrize("d,h,ff,B,S", CASES)
def test_same_bits_as_big_tiles(d, h, ff, B, S, mname):
    print(f"case fused tiles d={d} h={h} ff={ff} B={B} S={S} {mname}", flush=True)
    cfg = gen.make_config("tiny", n_layers=2, d_model=d, n_heads=h, d_ff=ff, vocab=256, batch=B, seq=S, dtype="bf16")
    mask = gen.all_mask(cfg) if mname == "all" else dict(ffn_lo=8, ffn_hi=ff // 2 // 8 * 8, head_lo=0, head_hi=0)
    tok, tgt = gen.make_tokens(cfg, seed=5)
    if S == 1:
        tgt[:] = 7
    weights, out = gen.make_weights(cfg, seed=5), []
    on_small = pp.load_library()["_ZN2pp18gemm_fused_on_ringEiiii"]
    on_small.restype = ctypes.c_bool
    pp.pp_set_option(None, "gemm_small_tiles", 1)
    n = ff if mname == "all" else mask["ffn_hi"] - mask["ffn_lo"]
    assert on_small(2, B * S, ff, d) and on_small(3, B * S, n, d) and on_small(4, B * S, d, d)          # SwiGLU, its backward, rotary: the second pass is on small tiles
    for small in (0, 1):
        pp.pp_set_option(None, "gemm_variant", 1)
        pp.pp_set_option(None, "gemm_small_tiles", small)
        m = pp.LocalStepModel(cfg, mask)
        m.load_weights(weights)
        m.set_mask()
        loss = m.step(*m.upload_tokens(tok, tgt), None)
        torch.cuda.synchronize()
        out.append((loss.clone(), torch.from_numpy(m.get_state("g").copy())))
        m.close()
    pp.pp_set_option(None, "gemm_small_tiles", 1)
    assert torch.equal(out[0][0], out[1][0])
    assert torch.equal(out[0][1], out[1][1]) and bool(torch.isfinite(out[0][1]).all())
