"""fp32-multiply MFMA attention (fp32 models, bf16 head dims 16 and 32, bf16 tensors that are not 16-byte aligned) against the plain kernels: the same sums in the same
order, so the same bits, at the edges of its 32-query blocks, 128-key chunks and LDS limit, and with values that are not finite."""
import pytest
import torch

import paper_2509_22418_amd as pp
from test_gpu_attn_f32_lines import runs_on_mfma

pytestmark = pytest.mark.gpu

# (B, S, h, dh), enough rows each that both directions take these kernels (asserted): the shortest rows taken, one short of / past a block, past a chunk, and
# around the last length whose scores fit LDS (1184; the forward of 1185 is the plain kernel's); single positions, which stay with the plain kernels in any number
CASES = [(4096, 8, 1, 16), (24, 31, 12, 32), (2, 33, 64, 64), (8, 128, 2, 128), (3, 161, 12, 16), (5, 257, 2, 128), (3, 1152, 1, 32), (2, 1153, 1, 64), (2, 1184, 1, 128), (4, 1184, 1, 16),
         (1, 1185, 1, 32), (131072, 1, 1, 16)]


def run(qkv, dO, B, S, h, dh, dt, path):
    st, d = torch.cuda.current_stream().cuda_stream, h * dh
    o = torch.zeros((B * S, d), dtype=qkv.dtype, device="cuda")
    lse, rows = (torch.zeros(B * h * S, dtype=torch.float32, device="cuda") for _ in range(2))
    dqkv = torch.zeros((B * S, 3 * d), dtype=qkv.dtype, device="cuda")
    pp.pp_op_attention_fwd(st, dt, qkv.data_ptr(), o.data_ptr(), lse.data_ptr(), None, B, S, h, dh, path)
    pp.pp_op_attention_bwd(st, dt, qkv.data_ptr(), o.data_ptr(), lse.data_ptr(), dO.data_ptr(), dqkv.data_ptr(), rows.data_ptr(), None, B, S, h, dh, path)
    torch.cuda.synchronize()
    return o, lse, dqkv, rows


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("B,S,h,dh", CASES)
def test_same_bits_as_the_plain_kernels(B, S, h, dh, dtype):
    print(f"case attention f32 B={B} S={S} h={h} dh={dh} {dtype}", flush=True)
    td, dt = (torch.bfloat16, pp.PP_BF16) if dtype == "bf16" else (torch.float32, pp.PP_F32)
    g = torch.Generator(device="cuda").manual_seed(3)
    off = 4 if dtype == "bf16" and dh >= 64 else 0          # 8 bytes off a 16-byte boundary: not taken by the bf16 kernels
    qkv, dO = (torch.randn(n + off, device="cuda", generator=g).to(td)[off:] for n in (B * S * 3 * h * dh, B * S * h * dh))
    assert runs_on_mfma(dt, qkv, dO, B, S, h, dh) == (int(1 < S <= 1184), int(S > 1))
    for a, b in zip(run(qkv, dO, B, S, h, dh, dt, 0), run(qkv, dO, B, S, h, dh, dt, 1)):
        assert torch.equal(a, b)


@pytest.mark.parametrize("value", [float("inf"), float("nan")])
def test_values_that_are_not_finite_stay_behind_the_mask(value):
    """One position whose q, k, v and dO are not finite: earlier queries do not see it, later keys are not reached by it, and every
    output equals the plain kernels' (NaN where they have NaN)."""
    B, S, h, dh, at = 1, 150, 32, 32, 70
    g = torch.Generator(device="cuda").manual_seed(4)
    qkv = torch.randn((S, 3 * h * dh), device="cuda", generator=g)
    dO = torch.randn((S, h * dh), device="cuda", generator=g)
    qkv[at, 5::7] = value
    dO[at, 3] = value
    assert runs_on_mfma(pp.PP_F32, qkv, dO, B, S, h, dh) == (1, 1)
    got, ref = run(qkv, dO, B, S, h, dh, pp.PP_F32, 0), run(qkv, dO, B, S, h, dh, pp.PP_F32, 1)
    assert bool(torch.isfinite(ref[0][:at]).all()) and not bool(torch.isfinite(ref[0][at:]).all())
    for a, b in zip(got, ref):
        assert torch.equal(torch.isnan(a), torch.isnan(b))
        assert torch.equal(torch.nan_to_num(a, nan=7.0), torch.nan_to_num(b, nan=7.0))


# (B, S, h, dh, bf16): short rows and few rows, where a workgroup per row is the faster split
@pytest.mark.parametrize("B,S,h,dh,dtype", [(4, 33, 4, 16, "f32"), (1, 48, 1, 16, "f32"), (8, 16, 12, 16, "f32"), (1, 33, 1, 128, "f32"), (1, 40, 2, 16, "bf16"), (1, 100, 4, 32, "f32")])
def test_few_short_rows_are_not_slower_than_on_the_plain_kernels(B, S, h, dh, dtype):
    print(f"case attention few rows B={B} S={S} h={h} dh={dh} {dtype}", flush=True)
    td, dt = (torch.bfloat16, pp.PP_BF16) if dtype == "bf16" else (torch.float32, pp.PP_F32)
    qkv, dO = torch.randn((B * S, 3 * h * dh), device="cuda").to(td), torch.randn((B * S, h * dh), device="cuda").to(td)
    o, dqkv = torch.empty_like(dO), torch.empty_like(qkv)
    lse, rows = (torch.empty(B * h * S, device="cuda") for _ in range(2))
    st = torch.cuda.current_stream().cuda_stream
    fwd = lambda path: pp.pp_op_attention_fwd(st, dt, qkv.data_ptr(), o.data_ptr(), lse.data_ptr(), None, B, S, h, dh, path)  # noqa: E731
    bwd = lambda path: pp.pp_op_attention_bwd(st, dt, qkv.data_ptr(), o.data_ptr(), lse.data_ptr(), dO.data_ptr(), dqkv.data_ptr(), rows.data_ptr(), None, B, S, h, dh, path)  # noqa: E731
    for call in (fwd, bwd):
        best = [float("inf")] * 2
        for _ in range(8):
            for path in (0, 1):
                a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
                a.record()
                for _ in range(50):
                    call(path)
                b.record()
                torch.cuda.synchronize()
                best[path] = min(best[path], a.elapsed_time(b))
        assert best[0] <= 1.2 * best[1], best
