"""The number of K ranges of a bf16 step's weight gradients: fewer ranges than a power of two (summed in pieces of the former length), more of them, and one, against
the same step on the plain kernels."""
import numpy as np
import pytest

import pp_inputs as gen
import paper_2509_22418_amd as pp
from harness import cosine

import torch  # noqa: F401

pytestmark = pytest.mark.gpu

# (d_model, heads, d_ff, batch, seq): 1280 x 640 gradients (50 tiles) over 4096 tokens in 8 ranges of two pieces each; 768 and 1537 tokens in 3 and 5 ranges; 3001 in
# 10 short ones; 255 in one
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
