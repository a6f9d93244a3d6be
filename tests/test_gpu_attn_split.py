"""bf16 attention at the edges of its work split: single blocks, dQ's KV tiles dealt to two groups of waves (an odd tile count,
one row past a block, groups without a visible tile), and paired blocks once the grid fills the chip; against fp64."""
import math

import pytest
import torch

import paper_2509_22418_amd as pp

pytestmark = pytest.mark.gpu

# (B, S, h, dh): split, then single blocks, then paired
CASES = [(1, 129, 1, 64), (2, 191, 3, 128), (1, 321, 2, 64), (3, 777, 4, 64), (2, 640, 1, 128), (8, 257, 22, 64), (8, 257, 11, 128), (4, 1025, 13, 64), (4, 260, 64, 64), (8, 257, 64, 128), (8, 140, 64, 64)]


@pytest.mark.parametrize("B,S,h,dh", CASES)
def test_matches_fp64(B, S, h, dh):
    print(f"case attention split B={B} S={S} h={h} dh={dh}", flush=True)
    d, st = h * dh, torch.cuda.current_stream().cuda_stream
    g = torch.Generator(device="cuda").manual_seed(2)
    qkv = torch.randn((B * S, 3 * d), device="cuda", generator=g).bfloat16()
    dO = torch.randn((B * S, d), device="cuda", generator=g).bfloat16()
    o = torch.zeros((B * S, d), device="cuda").bfloat16()
    dqkv = torch.zeros((B * S, 3 * d), device="cuda").bfloat16()
    lse, rows = (torch.zeros(B * h * S, device="cuda") for _ in range(2))
    pp.pp_op_attention_fwd(st, pp.PP_BF16, qkv.data_ptr(), o.data_ptr(), lse.data_ptr(), None, B, S, h, dh, 0)
    pp.pp_op_attention_bwd(st, pp.PP_BF16, qkv.data_ptr(), o.data_ptr(), lse.data_ptr(), dO.data_ptr(), dqkv.data_ptr(), rows.data_ptr(), None, B, S, h, dh, 0)
    torch.cuda.synchronize()
    mask = torch.ones((S, S), dtype=torch.bool, device="cuda").triu(1)
    for b in range(B):
        x = qkv.double().reshape(B, S, 3, h, dh)[b].permute(1, 2, 0, 3).contiguous().requires_grad_(True)
        sc = (torch.matmul(x[0], x[1].transpose(1, 2).contiguous()) / math.sqrt(dh)).masked_fill(mask, -math.inf)
        y = torch.matmul(torch.softmax(sc, -1), x[2])
        y.backward(dO.double().reshape(B, S, h, dh)[b].transpose(0, 1))
        assert float((lse.reshape(B, h, S)[b].double() - torch.logsumexp(sc.detach(), -1)).abs().max()) <= 2e-3
        got = o.double().reshape(B, S, h, dh)[b].transpose(0, 1)
        # probabilities and the output are rounded to bf16 once each: 2 * 2^-9 of values of order one, with room for a row's sum
        assert float((got - y.detach()).abs().max()) <= 2e-2
        for i, name in enumerate(("dq", "dk", "dv")):
            a, r = dqkv.double().reshape(B, S, 3, h, dh)[b, :, i].transpose(0, 1), x.grad[i]
            assert float((a - r).norm() / r.norm()) <= 1e-2, name
            assert float((a - r).abs().max()) <= 0.03 * float(r.abs().max()), name
