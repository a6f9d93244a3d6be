"""The gradient of the final norm's output, a contraction over the vocabulary, in several K ranges (few tokens, long vocabulary) and in one: a bf16 step against the
same step on the plain kernels."""
import numpy as np
import pytest

import pp_inputs as gen
import paper_2509_22418_amd as pp
from harness import cosine

pytestmark = pytest.mark.gpu


# (batch, seq, vocab, d_model): 500 and 257 K steps (257 is prime: one range), 320, and a vocabulary below the line; a token count past a tile
@pytest.mark.parametrize("B,S,V,d", [(1, 300, 32000, 256), (3, 171, 16448, 128), (2, 64, 20480, 192), (1, 257, 16384, 64), (2, 100, 8192, 128)])
def test_matches_the_plain_kernels(B, S, V, d):
    """Both paths multiply the same bf16 operands and sum in fp32, but round the activations between layers from differently ordered sums: one layer of bf16
    roundings (2^-9 each) on gradients of a common scale stays within 2 % of it."""
    print(f"case vocab ranges B={B} S={S} V={V} d={d}", flush=True)
    cfg = gen.make_config("tiny", n_layers=1, d_model=d, n_heads=d // 64, d_ff=256, vocab=V, batch=B, seq=S, dtype="bf16")
    weights, mask = gen.make_weights(cfg, seed=3), gen.all_mask(cfg)
    tok, tgt = gen.make_tokens(cfg, seed=3)
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
