"""K ranges of a bf16 step's weight gradients: several numbers of them against the same step on the plain kernels, and the order in which their sums are added."""
import numpy as np
import pytest

import pp_inputs as gen
import paper_2509_22418_amd as pp
from harness import cosine, segment_slices

import torch  # noqa: F401

pytestmark = pytest.mark.gpu

# (d_model, heads, d_ff, batch, seq): 1280 x 640 gradients (50 tiles) over 4096 tokens in 16 ranges; 768 and 1537 tokens in 2 and 4; 3001 in 8; 255 in one
CASES = [(640, 10, 1280, 8, 512), (128, 2, 512, 3, 256), (128, 2, 512, 1, 1537), (256, 4, 768, 1, 3001), (128, 2, 256, 1, 255)]


@pytest.mark.parametrize("d,h,ff,B,S", CASES)
def test_matches_the_plain_kernels(d, h, ff, B, S):
    """Both paths multiply the same bf16 operands and sum in fp32, but round the activations between layers from differently ordered sums: one layer of bf16
    roundings (2^-9 each) on gradients of a common scale stays within 2 % of it."""
    print(f"case dw ranges d={d} ff={ff} B={B} S={S}", flush=True)
    cfg = gen.make_config("tiny", n_layers=1, d_model=d, n_heads=h, d_ff=ff, vocab=512, batch=B, seq=S, dtype="bf16")
    weights, mask = gen.make_weights(cfg, seed=31), gen.all_mask(cfg)
    tok, tgt = gen.make_tokens(cfg, seed=31)
    g = []
    for plain in (0, 1):
        m = pp.LocalStepModel(cfg, mask)
        m.load_weights(weights)
        m.set_mask()
        m.set_option("force_plain", plain)
        m.step(*m.upload_tokens(tok, tgt), None)
        g.append(m.get_state("g").astype(np.float64))
        m.close()
    assert np.all(np.isfinite(g[0]))
    assert cosine(g[0], g[1]) >= 0.9995
    assert np.linalg.norm(g[0] - g[1]) <= 0.02 * np.linalg.norm(g[1])


@pytest.mark.parametrize("d,B,S", [(1280, 8, 448), (704, 8, 384), (768, 16, 384)])
def test_range_sums_are_added_one_after_the_other(d, B, S):
    """B = 2^k copies of one sequence, as long as a K range of the d x d gradient (100 tiles in 8 ranges, 36 in 8 with tiles cut at the edges and in 16): the
    mean over B times the targets scales every gradient by 2^-k exactly, so every range's sum is that of the sequence alone / B, and the gradient is B of them added one after the
    other to 0 in fp32 (pairs added first would give the exact multiple)."""
    print(f"case dw order d={d} B={B} S={S}", flush=True)
    rng = np.random.default_rng(7)
    tok, tgt = (rng.integers(0, 512, (1, S)).astype(np.int32) for _ in range(2))
    g = []
    for n in (1, B):
        cfg = gen.make_config("tiny", n_layers=1, d_model=d, n_heads=d // 64, d_ff=256, vocab=512, batch=n, seq=S, dtype="bf16")
        m = pp.LocalStepModel(cfg, gen.all_mask(cfg))
        m.load_weights(gen.make_weights(cfg, seed=31))
        m.set_mask()
        m.step(*m.upload_tokens(np.repeat(tok, n, 0), np.repeat(tgt, n, 0)), None)
        at = next((o, c) for name, o, c in segment_slices(cfg, gen.all_mask(cfg)) if "wo" in name)
        g.append(m.get_state("g")[at[0]:at[0] + at[1]].astype(np.float32))
        m.close()
    want = np.zeros_like(g[0])
    for _ in range(B):
        want += g[0] / np.float32(B)
    assert float(np.abs(want).max()) > 0.0 and not np.array_equal(want, g[0])
    assert np.array_equal(g[1], want)
