"""Long contractions of a bf16 step, over the vocabulary (the gradient of the final norm's output) and over gate and up (the gradient of the FFN norm's output): against
the same step on the plain kernels, and one order of sums for a row whatever else is in the batch."""
import numpy as np
import pytest

import pp_inputs as gen
import paper_2509_22418_amd as pp
from harness import cosine

pytestmark = pytest.mark.gpu


# (batch, seq, vocab, d_model): 500, 257 (a prime), 320, 256 and 128 K steps; a token count past a tile
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


# (seq, vocab, d_model, d_ff, copies): contractions over 32000 and over 2 x 8192; a few big tiles with one copy, 38 and 75 with all
@pytest.mark.parametrize("S,V,d,ff,n", [(300, 32000, 256, 256, 32), (300, 512, 256, 8192, 64)])
def test_a_row_has_the_same_bits_in_any_batch(S, V, d, ff, n):
    """One sequence of distinct tokens, alone and n = 2^k times over: the mean over n times the targets scales every gradient of an activation by 2^-k exactly, and
    the embedding gradient adds n equal bf16 rows exactly (fp32), so it has the same bits where every product sums a row in one order on any grid."""
    print(f"case rows in any batch S={S} V={V} d={d} ff={ff} n={n}", flush=True)
    rng = np.random.default_rng(7)
    tok, tgt = rng.permutation(V)[:S].astype(np.int32)[None], rng.integers(0, V, (1, S)).astype(np.int32)
    g = []
    for B in (1, n):
        cfg = gen.make_config("tiny", n_layers=1, d_model=d, n_heads=d // 64, d_ff=ff, vocab=V, batch=B, seq=S, dtype="bf16")
        m = pp.LocalStepModel(cfg, gen.all_mask(cfg))
        m.load_weights(gen.make_weights(cfg, seed=3))
        m.set_mask()
        m.step(*m.upload_tokens(np.repeat(tok, B, 0), np.repeat(tgt, B, 0)), None)
        g.append(m.get_state("g")[:V * d].reshape(V, d)[tok[0]])          # the embedding comes first
        m.close()
    assert np.all(np.isfinite(g[0])) and float(np.abs(g[0]).max()) > 0.0
    assert np.array_equal(g[0], g[1])
