"""Both sides of the lines between the vector kernels and the fp32-multiply MFMA attention, and the one-grid backward on both sides of its line: the same bits as the
plain kernels, at the edges of blocks of 32 rows, chunks of 128 keys and the LDS limit."""
import pytest
import torch

import paper_2509_22418_amd as pp

pytestmark = pytest.mark.gpu

# (B, S, h, dh): rows just below and at the forward's line, lengths at the edges of its LDS limit, and long rows of few pairs
CASES = [(1, 287, 16, 16), (1, 288, 16, 16), (1, 215, 16, 64), (1, 216, 16, 64), (4, 1152, 1, 32), (3, 1153, 1, 64), (3, 1184, 1, 128), (4, 1184, 1, 16), (3, 1185, 1, 32), (111, 31, 1, 32), (105, 33, 1, 64),
         # backward: pairs x S^2 on both sides of its lines, and more than 400 blocks of 32 rows at head dim 128
         (1, 100, 1, 16), (1, 99, 1, 16), (1, 215, 1, 32), (1, 214, 1, 32), (2, 198, 1, 64), (2, 197, 1, 64), (1, 332, 1, 128), (1, 331, 1, 128), (3, 129, 27, 128), (2, 161, 41, 128)]


@pytest.mark.parametrize("B,S,h,dh", CASES)
def test_same_bits_as_the_plain_kernels(B, S, h, dh):
    print(f"case attention f32 lines B={B} S={S} h={h} dh={dh}", flush=True)
    g, st, d = torch.Generator(device="cuda").manual_seed(3), torch.cuda.current_stream().cuda_stream, h * dh
    qkv, do = torch.randn((B * S, 3 * d), device="cuda", generator=g), torch.randn((B * S, d), device="cuda", generator=g)
    out = []
    for path in (0, 1):
        o, dqkv = torch.full((B * S, d), 7.0, device="cuda"), torch.full((B * S, 3 * d), 7.0, device="cuda")
        lse, rows = (torch.full((B * h * S,), 7.0, device="cuda") for _ in range(2))
        pp.pp_op_attention_fwd(st, pp.PP_F32, qkv.data_ptr(), o.data_ptr(), lse.data_ptr(), None, B, S, h, dh, path)
        pp.pp_op_attention_bwd(st, pp.PP_F32, qkv.data_ptr(), o.data_ptr(), lse.data_ptr(), do.data_ptr(), dqkv.data_ptr(), rows.data_ptr(), None, B, S, h, dh, path)
        torch.cuda.synchronize()
        out.append((o, lse, dqkv, rows))
    assert all(torch.equal(a, b) for a, b in zip(*out))
