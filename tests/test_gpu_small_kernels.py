"""Norm-gain and embedding gradients at the edges of their kernels: widths around a 512-column piece, token counts around a rank
block of 64 and a scan chunk of 4096, one token that takes every position, and tokens outside the vocabulary; a step whose only trainable tensors
are the gains and the embedding, against the same sums in fp64 of the tensors the step left behind."""
import numpy as np
import pytest

import pp_inputs as gen
import paper_2509_22418_amd as pp

pytestmark = pytest.mark.gpu

# d_model, heads, vocab, B, S, tokens
CASES = [(64, 1, 64, 1, 1, "zipf"), (520, 4, 72, 3, 43, "zipf"), (512, 4, 72, 1, 65, "one"), (1032, 6, 4104, 9, 457, "zipf"), (256, 2, 520, 2, 2048, "one"), (128, 2, 64, 4, 1024, "outside")]


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("d,h,V,B,S,kind", CASES)
def test_gain_and_embedding_gradients(d, h, V, B, S, kind, dtype):
    print(f"case small kernels d={d} V={V} B={B} S={S} {kind} {dtype}", flush=True)
    cfg = gen.make_config("tiny", n_layers=1, d_model=d, n_heads=h, d_ff=64, vocab=V, batch=B, seq=S, dtype=dtype)
    mask = dict(ffn_lo=0, ffn_hi=0, head_lo=0, head_hi=0, train_wo=0, train_norms=1, train_embed=1, train_lm_head=0)
    tok, tgt = gen.make_tokens(cfg, seed=6)
    if kind == "one":
        tok[:] = V - 1
    if kind == "outside":
        tok[0, :9] = V + 5          # the forward clamps them, the embedding gradient leaves them out
        tok[1, :3] = -1
    tgt[:, -1] = 1
    m = pp.LocalStepModel(cfg, mask)
    m.load_weights(gen.make_weights(cfg, seed=6))
    m.set_mask()
    m.step(*m.upload_tokens(tok, tgt), None)
    g = m.get_state("g").astype(np.float64)
    T, store = B * S, np.uint16 if dtype == "bf16" else np.float32
    tap = lambda n: (lambda r: (gen.bf16_bits_to_f32(r) if dtype == "bf16" else r).astype(np.float64))(m.get_raw("dbg." + n, (T, d), store))  # noqa: E731
    dx, dn, x = tap("dx"), tap("dn"), tap("x.0")
    m.close()
    # embedding: row sums of dL/dx, at most T fp32 additions
    ref = np.zeros((V, d))
    ok = (tok.reshape(-1) >= 0) & (tok.reshape(-1) < V)
    np.add.at(ref, tok.reshape(-1)[ok], dx[ok])
    mag = np.zeros((V, d))
    np.add.at(mag, tok.reshape(-1)[ok], np.abs(dx[ok]))
    assert np.all(np.abs(g[:V * d].reshape(V, d) - ref) <= T * 2.0 ** -24 * mag)
    # gain of the attention norm: dn still holds its output gradient; the fp32 1 / rms adds a few ulp per term
    rstd = 1.0 / np.sqrt((x * x).mean(1, keepdims=True) + cfg["rms_eps"])
    terms = dn * x * rstd
    assert np.all(np.abs(g[V * d:V * d + d] - terms.sum(0)) <= (T + 16 + d) * 2.0 ** -24 * np.abs(terms).sum(0))
