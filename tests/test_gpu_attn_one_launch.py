"""Attention backward of few sequences (dQ and dK/dV in one grid) at the edges of its blocks: the bits of the same sequences in a batch that fills the chip (two
kernels), and close to float64."""
import math

import pytest
import torch

import paper_2509_22418_amd as pp

pytestmark = pytest.mark.gpu


def run(qkv, do, B, S, h, dh):
    d, st = h * dh, torch.cuda.current_stream().cuda_stream
    o, dqkv = torch.empty(B * S, d, device="cuda", dtype=torch.bfloat16), torch.full((B * S, 3 * d), 7.0, device="cuda").bfloat16()
    lse, rows = torch.empty(B * h * S, device="cuda"), torch.full((B * h * S,), 7.0, device="cuda")
    pp.pp_op_attention_fwd(st, pp.PP_BF16, qkv.data_ptr(), o.data_ptr(), lse.data_ptr(), None, B, S, h, dh)
    pp.pp_op_attention_bwd(st, pp.PP_BF16, qkv.data_ptr(), o.data_ptr(), lse.data_ptr(), do.data_ptr(), dqkv.data_ptr(), rows.data_ptr(), None, B, S, h, dh)
    torch.cuda.synchronize()
    return o, dqkv, rows


@pytest.mark.parametrize("dh", [64, 128])
@pytest.mark.parametrize("S", [1, 63, 64, 127, 128, 129, 255, 256, 257, 385, 641, 777])
def test_same_bits_as_in_a_full_grid(S, dh):
    print(f"case attention one launch S={S} dh={dh}", flush=True)
    h, nb_kv, nb_dq = 3, (S + 127) // 128, (S + 255) // 256
    full = 800 // (h * (nb_kv + nb_dq)) + 1          # more than 768 workgroups: two kernels
    g = torch.Generator(device="cuda").manual_seed(1)
    qkv = torch.randn((full * S, 3 * h * dh), device="cuda", generator=g).bfloat16()
    do = torch.randn((full * S, h * dh), device="cuda", generator=g).bfloat16()
    _, want, want_rows = run(qkv, do, full, S, h, dh)
    for B in (1, 2):
        o, got, rows = run(qkv, do, B, S, h, dh)
        assert torch.equal(got, want[:B * S])
        assert torch.equal(rows, want_rows[:B * h * S])
    d = h * dh
    x = qkv[:S].double().reshape(S, 3, h, dh).permute(1, 2, 0, 3).contiguous().requires_grad_(True)
    sc = torch.matmul(x[0], x[1].transpose(1, 2).contiguous()) / math.sqrt(dh)
    sc = sc.masked_fill(torch.ones(S, S, dtype=torch.bool, device="cuda").triu(1), -math.inf)
    y = torch.matmul(torch.softmax(sc, -1), x[2])
    y.backward(do[:S].double().reshape(S, h, dh).transpose(0, 1).contiguous())
    ref = x.grad.permute(2, 0, 1, 3).reshape(S, 3 * d)
    # bf16 inputs and outputs, probabilities and score gradients rounded to bf16 (2^-9 each) on the way
    assert float((got[:S].double() - ref).norm() / ref.norm()) <= 1e-2
    assert o.shape == (2 * S, d)
