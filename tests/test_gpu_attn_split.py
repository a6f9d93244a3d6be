"""bf16 attention at the edges of its work split: single blocks (an odd tile count, one row past a block) and paired blocks once
equal workgroups fill the chip; against fp64, and one sequence and head alone against the same inside a full launch."""
import math

import pytest
import torch

import paper_2509_22418_amd as pp

pytestmark = pytest.mark.gpu

# (B, S, h, dh): few blocks, then a partly filled chip, then paired forward and dK/dV
CASES = [(1, 129, 1, 64), (2, 191, 3, 128), (1, 321, 2, 64), (3, 777, 4, 64), (2, 640, 1, 128), (8, 257, 22, 64), (8, 257, 11, 128), (4, 1025, 13, 64), (4, 260, 64, 64), (8, 257, 64, 128), (8, 140, 64, 64)]


def inputs(B, S, h, dh):
    g = torch.Generator(device="cuda").manual_seed(2)
    qkv = torch.randn((B * S, 3 * h * dh), device="cuda", generator=g).bfloat16()
    return qkv, torch.randn((B * S, h * dh), device="cuda", generator=g).bfloat16()


def run(qkv, dO, B, S, h, dh):
    st, o, dqkv = torch.cuda.current_stream().cuda_stream, torch.zeros_like(dO), torch.zeros_like(qkv)
    lse, rows = (torch.zeros(B * h * S, device="cuda") for _ in range(2))
    pp.pp_op_attention_fwd(st, pp.PP_BF16, qkv.data_ptr(), o.data_ptr(), lse.data_ptr(), None, B, S, h, dh, 0)
    pp.pp_op_attention_bwd(st, pp.PP_BF16, qkv.data_ptr(), o.data_ptr(), lse.data_ptr(), dO.data_ptr(), dqkv.data_ptr(), rows.data_ptr(), None, B, S, h, dh, 0)
    torch.cuda.synchronize()
    return o, lse, dqkv, rows


# (B, S, h, dh): the launch that the one sequence and head is taken from; alone it is a few blocks of 128 positions
@pytest.mark.parametrize("B,S,h,dh", [(8, 777, 16, 64), (8, 130, 32, 64), (8, 1100, 10, 128), (8, 300, 32, 128)])
def test_bits_do_not_depend_on_the_rest_of_the_batch(B, S, h, dh):
    print(f"case attention alone B={B} S={S} h={h} dh={dh}", flush=True)
    qkv, dO = inputs(B, S, h, dh)
    o, lse, dqkv, rows = run(qkv, dO, B, S, h, dh)
    for b, j in ((0, 0), (B - 1, h - 1), (B // 2, 1)):
        heads = lambda t, n: t.reshape(B, S, n, h, dh)[b, :, :, j].reshape(S, n * dh).contiguous()  # noqa: E731
        stats = lambda t: t.reshape(B, h, S)[b, j]  # noqa: E731
        alone = run(heads(qkv, 3), heads(dO, 1), 1, S, 1, dh)
        for got, ref, name in zip(alone, (heads(o, 1), stats(lse), heads(dqkv, 3), stats(rows)), ("o", "lse", "dqkv", "rowsum")):
            assert torch.equal(got, ref), name


@pytest.mark.parametrize("B,S,h,dh", CASES)
def test_matches_fp64(B, S, h, dh):
    print(f"case attention split B={B} S={S} h={h} dh={dh}", flush=True)
    qkv, dO = inputs(B, S, h, dh)
    o, lse, dqkv, _ = run(qkv, dO, B, S, h, dh)
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
