"""Both sides of the lines between the vector kernels and the fp32-multiply MFMA attention: which of the two runs, and the same bits as the plain kernels either way, at the
edges of blocks of 32 rows, chunks of 128 keys and the LDS limit."""
import ctypes

import pytest
import torch

import paper_2509_22418_amd as pp

pytestmark = pytest.mark.gpu

# (pairs, S, dh, forward, backward on the MFMA kernels): one pair below and at each line, at lengths around a block, a chunk and the LDS limit, and the shortest rows taken
CASES = [(140, 33, 16, 0, 1), (141, 33, 16, 1, 1), (25, 33, 16, 0, 0), (26, 33, 16, 0, 1), (36, 129, 16, 0, 1), (37, 129, 16, 1, 1), (3, 1184, 16, 0, 1), (4, 1184, 16, 1, 1), (2048, 7, 16, 0, 0), (2048, 8, 16, 1, 1),
         (150, 33, 32, 0, 1), (151, 33, 32, 1, 1), (40, 33, 32, 0, 0), (41, 33, 32, 0, 1), (33, 129, 32, 0, 1), (34, 129, 32, 1, 1), (2, 129, 32, 0, 0), (3, 129, 32, 0, 1), (2, 1184, 32, 0, 1), (3, 1184, 32, 1, 1),
         (3, 1185, 32, 0, 1), (2048, 7, 32, 0, 0), (2048, 8, 32, 1, 1),
         (124, 33, 64, 0, 1), (125, 33, 64, 1, 1), (48, 33, 64, 0, 0), (49, 33, 64, 0, 1), (24, 129, 64, 0, 1), (25, 129, 64, 1, 1), (6, 129, 64, 0, 0), (7, 129, 64, 0, 1), (1, 385, 64, 0, 0), (2, 385, 64, 0, 1),
         (1, 1184, 64, 0, 1), (2, 1184, 64, 1, 1), (2048, 7, 64, 0, 0), (2048, 8, 64, 1, 0), (2048, 11, 64, 1, 0), (2048, 12, 64, 1, 1),
         (101, 33, 128, 0, 1), (102, 33, 128, 1, 1), (46, 33, 128, 0, 0), (47, 33, 128, 0, 1), (19, 129, 128, 0, 1), (20, 129, 128, 1, 1), (7, 129, 128, 0, 0), (8, 129, 128, 0, 1), (1, 385, 128, 0, 0), (2, 385, 128, 0, 1),
         (1, 1184, 128, 0, 1), (2, 1184, 128, 1, 1), (3, 1184, 128, 1, 1), (2048, 7, 128, 0, 0), (2048, 17, 128, 1, 0), (2048, 18, 128, 1, 1), (82, 161, 128, 1, 1)]

# (pairs, S, dh, direction, on the MFMA kernel): 1.2 times and more apart (fp32, us, vector / MFMA)
CLEAR = [(4, 1150, 16, 0, 1),          # 67 / 48
         (12, 256, 32, 0, 1),          # 22 / 18
         (4, 850, 64, 0, 1),           # 80 / 50
         (16, 200, 64, 0, 1),          # 23 / 19
         (12, 256, 128, 0, 1),         # 63 / 31
         (2, 1150, 128, 0, 1),         # 128 / 99
         (1, 1150, 128, 0, 0),         # 77 / 98
         (1, 850, 64, 0, 0),           # 0.71 of the MFMA kernel
         (32768, 4, 64, 0, 0),         # 191 / 381
         (1, 420, 128, 1, 0),          # 53 / 73
         (2, 200, 64, 1, 0),           # 22.5 / 27.4
         (128, 24, 128, 1, 1)]         # 33 / 23


def split(pairs):
    return next((pairs // h, h) for h in (16, 12, 10, 8, 7, 6, 5, 4, 3, 2, 1) if pairs % h == 0)          # batch, heads


def tensors(B, S, h, dh, dtype):
    td, dt = (torch.bfloat16, pp.PP_BF16) if dtype == "bf16" else (torch.float32, pp.PP_F32)
    off = 4 if dtype == "bf16" and dh >= 64 else 0          # 8 bytes off a 16-byte boundary: not taken by the bf16 kernels
    g = torch.Generator(device="cuda").manual_seed(3)
    return dt, *(torch.randn(B * S * n * h * dh + off, device="cuda", generator=g).to(td)[off:] for n in (3, 1))


def runs_on_mfma(dt, qkv, do, B, S, h, dh):
    """(forward, backward): whether the C++ entries take the shape (they launch nothing where they do not)."""
    lib, P, I = pp.load_library(), ctypes.c_void_p, ctypes.c_int
    fwd = lib["_ZN2pp14k_attn_fwd_f32EP12ihipStream_tiPKvPvPfiiii"]
    bwd = lib["_ZN2pp14k_attn_bwd_f32EP12ihipStream_tiPKvS3_PKfS3_PvPfiiii"]
    fwd.argtypes, bwd.argtypes = [P, I, P, P, P, I, I, I, I], [P, I, P, P, P, P, P, P, I, I, I, I]
    st, o, dqkv, (lse, rows) = torch.cuda.current_stream().cuda_stream, torch.empty_like(do), torch.empty_like(qkv), torch.zeros((2, B * h * S), device="cuda")
    got = (fwd(st, dt, qkv.data_ptr(), o.data_ptr(), lse.data_ptr(), B, S, h, dh),
           bwd(st, dt, qkv.data_ptr(), o.data_ptr(), lse.data_ptr(), do.data_ptr(), dqkv.data_ptr(), rows.data_ptr(), B, S, h, dh))
    torch.cuda.synchronize()
    return tuple(int(rc == 0) for rc in got)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("pairs,S,dh,fwd,bwd", CASES)
def test_same_bits_as_the_plain_kernels(pairs, S, dh, fwd, bwd, dtype):
    print(f"case attention f32 lines pairs={pairs} S={S} dh={dh} {dtype}", flush=True)
    B, h = split(pairs)
    dt, qkv, do = tensors(B, S, h, dh, dtype)
    assert runs_on_mfma(dt, qkv, do, B, S, h, dh) == (fwd, bwd)
    st, out = torch.cuda.current_stream().cuda_stream, []
    for path in (0, 1):
        o, dqkv = torch.zeros_like(do), torch.zeros_like(qkv)
        lse, rows = (torch.full((B * h * S,), 7.0, device="cuda") for _ in range(2))
        pp.pp_op_attention_fwd(st, dt, qkv.data_ptr(), o.data_ptr(), lse.data_ptr(), None, B, S, h, dh, path)
        pp.pp_op_attention_bwd(st, dt, qkv.data_ptr(), o.data_ptr(), lse.data_ptr(), do.data_ptr(), dqkv.data_ptr(), rows.data_ptr(), None, B, S, h, dh, path)
        torch.cuda.synchronize()
        out.append((o, lse, dqkv, rows))
    assert all(torch.equal(a, b) for a, b in zip(*out))


@pytest.mark.parametrize("pairs,S,dh,direction,mfma", CLEAR)
def test_the_clearly_faster_kernel_runs(pairs, S, dh, direction, mfma):
    print(f"case attention f32 choice pairs={pairs} S={S} dh={dh} direction={direction}", flush=True)
    B, h = split(pairs)
    dt, qkv, do = tensors(B, S, h, dh, "f32")
    assert runs_on_mfma(dt, qkv, do, B, S, h, dh)[direction] == mfma
