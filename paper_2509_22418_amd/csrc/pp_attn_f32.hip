// Causal attention in fp32 multiplies on the matrix cores, for fp32 models and for what the bf16 kernels do not take (head dims 16 and 32,
// tensors on 8-byte but not 16-byte boundaries): head dims 16, 32, 64 and 128, any sequence length (forward: up to the scores of 32 queries in LDS, MAX_S).
//
// Same bits as the plain kernels.  v_mfma_f32_32x32x2 / 16x16x4 add their products one after the other with one rounding each,
// so an accumulator fed in index order is the plain kernel's fmaf chain: scores run over the head dim, P V / dS K over the keys and
// P^T dO / dS^T Q over the queries in ascending order, never split over waves; the softmax sum is formed in the plain kernel's
// order (128 interleaved partial sums, two 64-lane butterflies); masked entries enter a chain as exact zeros.  A masked zero
// times an infinity would be NaN where the plain kernel skips the product: where a 32-entry piece of a chain touches the
// diagonal and its operand holds a non-finite value, the piece is added element by element instead.
//
// Work split: one workgroup per 32 queries (forward, dQ) or 32 keys (dK, dV) of a head.  Its four waves share the score tiles
// (32 x 32 each, operands straight from global memory: 32 MFMAs of 64 cycles at head dim 64 against 16 loads), leave them in LDS, and then
// own 16 columns of the output each (16x16x4 MFMAs: 8 cycles per chain step, two row blocks in flight).  Bound by the
// chain of dependent phases and keys of one block (matrix pipe busy 0.12 to 0.25, waves waiting 0.50 to 0.56 in the call below: profiles/op_kernels_pmc.txt).
// 4 x 256 tokens, 8 heads of 64, fp32 (us, vector kernels / these): forward 246 / 20.9, dQ 561 / 21.6, dK and dV 577 / 25.5.
#include "pp_kernels.h"
#include "pp_dev.h"

#include <type_traits>

namespace pp {

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

namespace {

__device__ __forceinline__ float4 load_row4(const float* p) { return *reinterpret_cast<const float4*>(p); }
__device__ __forceinline__ float4 load_row4(const bf16_t* p) {
  const uint2 w = *reinterpret_cast<const uint2*>(p);
  return make_float4(__uint_as_float(w.x << 16), __uint_as_float(w.x & 0xffff0000u), __uint_as_float(w.y << 16), __uint_as_float(w.y & 0xffff0000u));
}
// 32x32x2 operand: elements 2 t + lane / 32 of the lane's row
template <int DH, class T> __device__ __forceinline__ void row_frag(float (&f)[DH / 2], const T* row, int lh) {
#pragma unroll
  for (int u = 0; u < DH / 4; ++u) {
    const float4 v = load_row4(row + 4 * u);
    f[2 * u] = lh ? v.y : v.x;
    f[2 * u + 1] = lh ? v.w : v.z;
  }
}
template <int DH> __device__ __forceinline__ f32x16 dot_tile(const float (&a)[DH / 2], const float (&b)[DH / 2]) {
  f32x16 acc;
#pragma unroll
  for (int r = 0; r < 16; ++r) acc[r] = 0.f;
#pragma unroll
  for (int t = 0; t < DH / 2; ++t) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a[t], b[t], acc, 0, 0, 0);
  return acc;
}

// acc[hb] (rows 16 hb .. + 15 of the block's 32, 16 columns) += W[row][0 .. n) X[x0 .. x0 + n)[columns], ascending; n a multiple of 32.
// w: LDS, row pitch `pitch`; entry e of row r is masked (its W is 0) iff mask(r, e).  xrow(e) -> pointer to the lane's column of row e.
template <class XR, class MK>
__device__ __forceinline__ void chain(f32x4 (&acc)[2], const float* w, int pitch, int n, int lane, XR&& xrow, MK&& mask, int diag_lo, int diag_hi) {
  const int l16 = lane & 15, lg = lane >> 4;
  for (int e0 = 0; e0 < n; e0 += 32) {
    float x[8];
    bool bad = false;
#pragma unroll
    for (int u = 0; u < 8; ++u) { x[u] = to_f32(*xrow(e0 + 4 * u + lg)); bad |= !(fabsf(x[u]) < INFINITY); }
    const bool diag = e0 < diag_hi && e0 + 32 > diag_lo;          // some entry of the piece is masked for some row
    if (diag && __builtin_amdgcn_ballot_w64(bad) != 0) {
#pragma unroll
      for (int u = 0; u < 8; ++u)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          const float xv = __shfl(x[u], g * 16 + l16, 64);
          const int e = e0 + 4 * u + g;
#pragma unroll
          for (int hb = 0; hb < 2; ++hb)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
              const int row = 16 * hb + 4 * lg + r;
              if (!mask(row, e)) acc[hb][r] = fmaf(w[row * pitch + e], xv, acc[hb][r]);
            }
        }
      continue;
    }
    float a[2][8];
#pragma unroll
    for (int hb = 0; hb < 2; ++hb)
#pragma unroll
      for (int u = 0; u < 8; ++u) a[hb][u] = w[(16 * hb + l16) * pitch + e0 + 4 * u + lg];
#pragma unroll
    for (int u = 0; u < 8; ++u)
#pragma unroll
      for (int hb = 0; hb < 2; ++hb) acc[hb] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[hb][u], x[u], acc[hb], 0, 0, 0);
  }
}

constexpr int CHUNK = 128;          // keys (queries) whose scores are in LDS at a time in the backward kernels
constexpr int BPITCH = CHUNK + 1;   // odd: the rows of a chain's reads start on different banks

}  // namespace

// ------------------------------------------------------------------------------------------ forward
template <int DH, class T>
__global__ __launch_bounds__(256) void attn_fwd_f32_kernel(const T* __restrict__ qkv, T* __restrict__ o, float* __restrict__ lse, int S, int h, int n_pairs, int pitch) {
  extern __shared__ float sc[];          // [32][pitch] scores, then 32 sums
  float* sums = sc + 32 * pitch;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, l32 = lane & 31, lh = lane >> 5;
  const int pair = blockIdx.x % n_pairs, qb = (S + 31) / 32 - 1 - blockIdx.x / n_pairs;          // longest rows first
  const int head = pair % h, b = pair / h, q0 = qb * 32, nk = min(S, q0 + 32), npad = (nk + 31) & ~31;
  const int d = h * DH;
  const size_t ld = (size_t)3 * d;
  const T* base = qkv + (size_t)b * S * ld + (size_t)head * DH;
  const float scale = 1.0f / sqrtf((float)DH);
  {
    float qf[DH / 2];
    row_frag<DH>(qf, base + (size_t)min(q0 + l32, S - 1) * ld, lh);
    for (int k0 = wave * 32; k0 < npad; k0 += 128) {
      float kf[DH / 2];
      row_frag<DH>(kf, base + (size_t)min(k0 + l32, S - 1) * ld + d, lh);
      const f32x16 s = dot_tile<DH>(qf, kf);
#pragma unroll
      for (int r = 0; r < 16; ++r) sc[(8 * (r >> 2) + 4 * lh + (r & 3)) * pitch + k0 + l32] = s[r] * scale;
    }
  }
  __syncthreads();
  {          // eight rows per wave, together; the 128 threads of the plain kernel's row are a lane's two partial sums
    float* rows = sc + wave * 8 * pitch;
    const int i0 = q0 + wave * 8;
    float mx[8], s0[8], s1[8];
#pragma unroll
    for (int r = 0; r < 8; ++r) { mx[r] = -INFINITY; s0[r] = 0.f; s1[r] = 0.f; }
    for (int j = lane; j < npad; j += 64)
#pragma unroll
      for (int r = 0; r < 8; ++r) mx[r] = j <= i0 + r ? fmaxf(mx[r], rows[r * pitch + j]) : mx[r];
#pragma unroll
    for (int r = 0; r < 8; ++r) mx[r] = wave_max(mx[r]);
    for (int j = lane; j < npad; j += 128) {
      const bool two = j + 64 < npad;
#pragma unroll
      for (int r = 0; r < 8; ++r) {
        const float e0 = expf(rows[r * pitch + j] - mx[r]), e1 = two ? expf(rows[r * pitch + j + 64] - mx[r]) : 0.f;
        const bool v0 = j <= i0 + r, v1 = two && j + 64 <= i0 + r;
        rows[r * pitch + j] = v0 ? e0 : 0.f;
        if (two) rows[r * pitch + j + 64] = v1 ? e1 : 0.f;
        s0[r] = v0 ? s0[r] + e0 : s0[r];
        s1[r] = v1 ? s1[r] + e1 : s1[r];
      }
    }
#pragma unroll
    for (int r = 0; r < 8; ++r) {
      const float sum = (0.f + wave_sum(s0[r])) + wave_sum(s1[r]);
      if (lane == 0) {
        sums[wave * 8 + r] = sum;
        if (i0 + r < S) lse[((size_t)b * h + head) * S + i0 + r] = mx[r] + logf(sum);
      }
    }
  }
  __syncthreads();
  const int l16 = lane & 15, lg = lane >> 4;
  for (int cb = wave; cb < DH / 16; cb += 4) {
    const T* vcol = base + 2 * d + cb * 16 + l16;
    f32x4 acc[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
    chain(acc, sc, pitch, npad, lane, [&](int j) { return vcol + (size_t)min(j, S - 1) * ld; }, [&](int r, int j) { return j > q0 + r; }, q0, npad);
#pragma unroll
    for (int hb = 0; hb < 2; ++hb)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int row = 16 * hb + 4 * lg + r;
        if (q0 + row < S) o[((size_t)b * S + q0 + row) * d + (size_t)head * DH + cb * 16 + l16] = from_f32<T>(acc[hb][r] / sums[row]);
      }
  }
}

// ------------------------------------------------------------------------------------------ backward: dQ
template <int DH, class T>
__device__ __forceinline__ void attn_bwd_dq_f32(float* ds, float* Ls, float* Ds, const T* __restrict__ qkv, const float* __restrict__ lse, const float* __restrict__ Dbuf,
                                                const T* __restrict__ dO, T* __restrict__ dqkv, int S, int h, int pair, int rank) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, l32 = lane & 31, lh = lane >> 5, l16 = lane & 15, lg = lane >> 4;
  const int qb = (S + 31) / 32 - 1 - rank;
  const int head = pair % h, b = pair / h, q0 = qb * 32, nk = min(S, q0 + 32);
  const int d = h * DH;
  const size_t ld = (size_t)3 * d;
  const T* base = qkv + (size_t)b * S * ld + (size_t)head * DH;
  const float scale = 1.0f / sqrtf((float)DH);
  if (threadIdx.x < 32) {
    const size_t stat = ((size_t)b * h + head) * S + min(q0 + (int)threadIdx.x, S - 1);
    Ls[threadIdx.x] = lse[stat]; Ds[threadIdx.x] = Dbuf[stat];
  }
  float qf[DH / 2], of[DH / 2];
  row_frag<DH>(qf, base + (size_t)min(q0 + l32, S - 1) * ld, lh);
  row_frag<DH>(of, dO + ((size_t)b * S + min(q0 + l32, S - 1)) * d + (size_t)head * DH, lh);
  constexpr int NCB = (DH / 16 + 3) / 4;
  f32x4 acc[NCB][2];
#pragma unroll
  for (int c = 0; c < NCB; ++c)
#pragma unroll
    for (int hb = 0; hb < 2; ++hb) acc[c][hb] = f32x4{0.f, 0.f, 0.f, 0.f};
  __syncthreads();
  for (int c0 = 0; c0 < nk; c0 += CHUNK) {
    const int n = min(CHUNK, (nk - c0 + 31) & ~31), k0 = c0 + wave * 32;
    if (wave * 32 < n) {
      float xf[DH / 2];
      row_frag<DH>(xf, base + (size_t)min(k0 + l32, S - 1) * ld + d, lh);
      const f32x16 s = dot_tile<DH>(qf, xf);
      row_frag<DH>(xf, base + (size_t)min(k0 + l32, S - 1) * ld + 2 * d, lh);
      const f32x16 dp = dot_tile<DH>(of, xf);
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int row = 8 * (r >> 2) + 4 * lh + (r & 3);
        const float L = Ls[row], Di = Ds[row];
        const float p = expf(s[r] * scale - L);
        ds[row * BPITCH + wave * 32 + l32] = k0 + l32 > q0 + row ? 0.f : p * (dp[r] - Di);
      }
    }
    __syncthreads();
#pragma unroll
    for (int c = 0; c < NCB; ++c) {
      const int cb = wave + 4 * c;
      if (cb * 16 >= DH) continue;
      const T* kcol = base + d + cb * 16 + l16;
      chain(acc[c], ds, BPITCH, n, lane, [&](int j) { return kcol + (size_t)min(c0 + j, S - 1) * ld; }, [&](int r, int j) { return c0 + j > q0 + r; }, q0 - c0, n);
    }
    __syncthreads();
  }
#pragma unroll
  for (int c = 0; c < NCB; ++c) {
    const int cb = wave + 4 * c;
    if (cb * 16 >= DH) continue;
#pragma unroll
    for (int hb = 0; hb < 2; ++hb)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int row = q0 + 16 * hb + 4 * lg + r;
        if (row < S) dqkv[((size_t)b * S + row) * ld + (size_t)head * DH + cb * 16 + l16] = from_f32<T>(acc[c][hb][r] * scale);
      }
  }
}

// ------------------------------------------------------------------------------------------ backward: dK, dV
template <int DH, class T>
__device__ __forceinline__ void attn_bwd_dkv_f32(float* Pt, float* DSt, const T* __restrict__ qkv, const float* __restrict__ lse, const float* __restrict__ Dbuf,
                                                 const T* __restrict__ dO, T* __restrict__ dqkv, int S, int h, int pair, int kb) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, l32 = lane & 31, lh = lane >> 5, l16 = lane & 15, lg = lane >> 4;
  const int head = pair % h, b = pair / h, k0 = kb * 32;
  const int d = h * DH;
  const size_t ld = (size_t)3 * d;
  const T* base = qkv + (size_t)b * S * ld + (size_t)head * DH;
  const T* dob = dO + (size_t)b * S * d + (size_t)head * DH;
  const float scale = 1.0f / sqrtf((float)DH);
  float kf[DH / 2], vf[DH / 2];
  row_frag<DH>(kf, base + (size_t)min(k0 + l32, S - 1) * ld + d, lh);
  row_frag<DH>(vf, base + (size_t)min(k0 + l32, S - 1) * ld + 2 * d, lh);
  // 16-column units of dV (0 .. DH / 16 - 1) and dK (the rest), dealt to the waves
  constexpr int NU = (DH / 8 + 3) / 4;
  f32x4 acc[NU][2];
#pragma unroll
  for (int c = 0; c < NU; ++c)
#pragma unroll
    for (int hb = 0; hb < 2; ++hb) acc[c][hb] = f32x4{0.f, 0.f, 0.f, 0.f};
  for (int c0 = k0; c0 < S; c0 += CHUNK) {
    const int n = min(CHUNK, (S - c0 + 31) & ~31), i0 = c0 + wave * 32;
    if (wave * 32 < n) {
      const int ic = min(i0 + l32, S - 1);
      const size_t stat = ((size_t)b * h + head) * S + ic;
      const float L = lse[stat], Di = Dbuf[stat];
      float xf[DH / 2];
      row_frag<DH>(xf, base + (size_t)ic * ld, lh);
      const f32x16 s = dot_tile<DH>(kf, xf);          // rows: keys, the lane's column: its query
      row_frag<DH>(xf, dob + (size_t)ic * d, lh);
      const f32x16 dp = dot_tile<DH>(vf, xf);
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int row = 8 * (r >> 2) + 4 * lh + (r & 3);
        const bool off = i0 + l32 < k0 + row || i0 + l32 >= S;
        const float p = expf(s[r] * scale - L);
        Pt[row * BPITCH + wave * 32 + l32] = off ? 0.f : p;
        DSt[row * BPITCH + wave * 32 + l32] = off ? 0.f : p * (dp[r] - Di);
      }
    }
    __syncthreads();
    // as four functions: the loop, inlined into a kernel of this size, is not unrolled in full, and its accumulators are then addressed by index (s_set_gpr_idx)
    auto unit = [&](auto C) {
      constexpr int c = decltype(C)::value;
      const int u = wave + 4 * c;
      if (u * 8 >= DH) return;
      const bool isv = u < DH / 16;
      const int cb = isv ? u : u - DH / 16;
      const T* col = (isv ? dob : base) + cb * 16 + l16;
      const size_t xld = isv ? (size_t)d : ld;
      // masked: queries before the row's key (first 32 of the first chunk) and the padding of the last piece
      chain(acc[c], isv ? Pt : DSt, BPITCH, n, lane, [&](int i) { return col + (size_t)min(c0 + i, S - 1) * xld; },
            [&](int r, int i) { return c0 + i < k0 + r || c0 + i >= S; }, c0 == k0 || c0 + n > S ? 0 : n, n);
    };
    unit(std::integral_constant<int, 0>{});
    if constexpr (NU > 1) unit(std::integral_constant<int, 1>{});
    if constexpr (NU > 2) { unit(std::integral_constant<int, 2>{}); unit(std::integral_constant<int, 3>{}); }
    static_assert(NU == 1 || NU == 2 || NU == 4, "units per wave");
    __syncthreads();
  }
#pragma unroll
  for (int c = 0; c < NU; ++c) {
    const int u = wave + 4 * c;
    if (u * 8 >= DH) continue;
    const bool isv = u < DH / 16;
    const int cb = isv ? u : u - DH / 16;
#pragma unroll
    for (int hb = 0; hb < 2; ++hb)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int row = k0 + 16 * hb + 4 * lg + r;
        if (row < S) dqkv[((size_t)b * S + row) * ld + (isv ? 2 * d : d) + (size_t)head * DH + cb * 16 + l16] = from_f32<T>(isv ? acc[c][hb][r] : acc[c][hb][r] * scale);
      }
  }
}

// ------------------------------------------------------------------------------------------ backward: both in one grid, heaviest blocks first (early keys see the most
// queries, late queries the most keys).  They share nothing but D, and together they leave fewer units idle behind the longest blocks.  us, two launches / one: 4 x 256, 8 heads of
// 64 47.5 / 36.9, 1 x 256, 8 heads of 64 46.7 / 27.9, 2 x 1000, 4 heads of 64 140 / 103, 8 x 320, 12 heads of 64 123 / 119, 4 x 128, 16 heads of 32 21 / 15; fp32, head dim 128: 45 pairs of 378 222 /
// 208, 25 of 928 0.93 of the two, 120 of 198 (840 blocks of 32 rows) 216 / 218.  Widened bf16 at head dim 128 (tensors on 8-byte boundaries): dQ alone has the registers for two workgroups per
// unit, which the common kernel has not: 36 pairs of 373 (432 blocks) 133 / 130, 100 of 101 (400) 72.1 / 72.1, 222 of 35 (444) 61.5 / 67.9, 81 of 404 (1053) 306 / 339.
constexpr unsigned kOneGrid128 = 400;          // blocks of 32 rows
template <int DH, class T, bool DQ, bool DKV>
__global__ __launch_bounds__(256, DH <= 32 ? 3 : 1) void attn_bwd_f32_kernel(const T* __restrict__ qkv, const float* __restrict__ lse, const float* __restrict__ Dbuf,
                                                           const T* __restrict__ dO, T* __restrict__ dqkv, int S, int h, int n_pairs) {
  __shared__ float x0[32 * BPITCH], x1[DKV ? 32 * BPITCH : 64];          // dK/dV: P and dS, [key][query of the chunk]; dQ: dS, statistics of 32 rows
  constexpr int KINDS = DQ + DKV;
  const int rank = blockIdx.x / (KINDS * n_pairs), x = blockIdx.x - rank * KINDS * n_pairs;
  if (DKV && x < n_pairs) attn_bwd_dkv_f32<DH>(x0, x1, qkv, lse, Dbuf, dO, dqkv, S, h, x, rank);
  else if (DQ) attn_bwd_dq_f32<DH>(x0, x1, x1 + 32, qkv, lse, Dbuf, dO, dqkv, S, h, DKV ? x - n_pairs : x, rank);
}
template <int DH, class T>
static void bwd_f32(hipStream_t st, const void* qkv, const float* lse, const float* Dbuf, const void* dO, void* dqkv, int B, int S, int h) {
  const unsigned blocks = (unsigned)B * h * ((S + 31) / 32);
  if (DH < 128 || sizeof(T) == 4 || blocks <= kOneGrid128) {
    attn_bwd_f32_kernel<DH, T, true, true><<<2 * blocks, 256, 0, st>>>((const T*)qkv, lse, Dbuf, (const T*)dO, (T*)dqkv, S, h, B * h);
  } else if constexpr (DH == 128 && sizeof(T) == 2) {
    attn_bwd_f32_kernel<DH, T, true, false><<<blocks, 256, 0, st>>>((const T*)qkv, lse, Dbuf, (const T*)dO, (T*)dqkv, S, h, B * h);
    attn_bwd_f32_kernel<DH, T, false, true><<<blocks, 256, 0, st>>>((const T*)qkv, lse, Dbuf, (const T*)dO, (T*)dqkv, S, h, B * h);
  }
}

// ------------------------------------------------------------------------------------------ host side
static bool shapes_ok(int dtype, const void* a, const void* b, int S, int h, int dh) {
  const uintptr_t al = dtype == 0 ? 15 : 7;          // rows are read four elements at a time
  return S >= 1 && h >= 1 && (dh == 16 || dh == 32 || dh == 64 || dh == 128) && (((uintptr_t)a | (uintptr_t)b) & al) == 0;
}
constexpr int MAX_S = 1184;                               // positions, a multiple of 32 (rows are padded to one)
constexpr int MAX_LDS = (32 * (MAX_S + 1) + 32) * 4;      // forward: 32 rows of scores and their sums, 148 KB of the compute unit's 160
template <int DH, class T>
static int fwd_f32(hipStream_t st, const void* qkv, void* o, float* lse, int B, int S, int h, int pitch) {
  static const bool ok = hipFuncSetAttribute(reinterpret_cast<const void*>(attn_fwd_f32_kernel<DH, T>), hipFuncAttributeMaxDynamicSharedMemorySize, MAX_LDS) == hipSuccess;
  const int bytes = (32 * pitch + 32) * 4;
  if (!ok) return 1;
  attn_fwd_f32_kernel<DH, T><<<dim3((unsigned)B * h * ((S + 31) / 32)), 256, bytes, st>>>((const T*)qkv, (T*)o, lse, S, h, B * h, pitch);
  return 0;
}
#define PP_F32_ATTN(dtype, dh, CALL)                                                                        \
  do {                                                                                                      \
    if ((dtype) == 0) { using T = float; if (dh == 16) { constexpr int DH = 16; CALL; } else if (dh == 32) { constexpr int DH = 32; CALL; } \
                        else if (dh == 64) { constexpr int DH = 64; CALL; } else { constexpr int DH = 128; CALL; } }                        \
    else { using T = bf16_t; if (dh == 16) { constexpr int DH = 16; CALL; } else if (dh == 32) { constexpr int DH = 32; CALL; }            \
           else if (dh == 64) { constexpr int DH = 64; CALL; } else { constexpr int DH = 128; CALL; } }                                     \
  } while (0)

// Few rows, short rows: the vector kernels run a workgroup per row, all at once up to about 3000 of them; then they last as long as one row, and beyond that their time grows with rows x
// length.  Here a workgroup of 32 rows is a chain of dependent phases over the keys, 128 at a time, whatever the number of rows (pairs = B h).  So the lines are pairs x S x (S + b) >= c x (S rounded up to
// 128 + d), where both took the same time; for the backward of head dims 16 and 32, whose vector chain is short, pairs x (S + b)^3.  Rows of fewer than 8 to 18 positions stay with the vector kernels
// whatever their number: most of a block of 32 would be padding.  From 820 shapes per head dim (pairs 1 .. 32768, S 1 .. 1184, fp32 and bf16), 98 % of which run on the faster kernel or within 3 % of it; the
// nearest and the far ends (fp32, us, vector / these):
//   forward   dh 16: 64 x 64 8.8 / 9.5, 3 x 850 31 / 38, 16 x 256 19.7 / 16.3, 4 x 1150 67 / 48      dh 32: 48 x 80 9.9 / 10.9, 12 x 256 22 / 18, 4 x 850 51 / 41      dh 64: 16 x 160 16.6 / 18.5, 2 x 850
//             46 / 49, 32768 x 4 191 / 381, 16 x 200 23 / 19, 12 x 256 34 / 21, 4 x 850 80 / 50      dh 128: 16 x 160 26.7 / 27.2, 1 x 1150 77 / 98, 16 x 200 37 / 28, 12 x 256 63 / 31, 2 x 1150 128 / 99
//   backward  dh 16: 20 x 34 7.9 / 8.9, 1 x 128 11.0 / 9.1      dh 32: 18 x 53 10.4 / 11.0, 3 x 160 17.0 / 15.8      dh 64: 2 x 200 22.5 / 27.4, 1 x 420 38 / 43, 32 x 48 15.2 / 16.6      dh 128: 8 x 100
//             28.7 / 29.9, 2 x 256 42 / 47, 1 x 420 53 / 73, 128 x 24 33 / 23
static bool fwd_pays(long pairs, int S, int dh) {
  const int b = dh == 16 ? 256 : dh == 32 ? 96 : 64, d = dh == 16 ? 256 : 128, c = dh == 16 ? 3500 : dh == 32 ? 2500 : dh == 64 ? 1560 : 1275;
  return S >= 8 && pairs * S * (S + b) >= (long)c * ((S + 127) / 128 * 128 + d);
}
static bool bwd_pays(long pairs, int S, int dh) {
  if (dh <= 32) {
    const double l = S + dh, line = dh == 16 ? 144 : 224;
    return S >= 8 && (double)pairs * l * l * l >= line * line * line;
  }
  const int d = dh == 64 ? 256 : 128, c = dh == 64 ? 269 : 388;
  return S >= (dh == 64 ? 12 : 18) && pairs * S * (S + 32) >= (long)c * ((S + 127l) / 128 * 128 + d);
}
// The scores of 32 queries against the whole sequence sit in LDS: sequences of more than MAX_S positions return 1.
int k_attn_fwd_f32(hipStream_t st, int dtype, const void* qkv, void* o, float* lse, int B, int S, int h, int dh) {
  if (S > MAX_S || !shapes_ok(dtype, qkv, o, S, h, dh) || !fwd_pays((long)B * h, S, dh)) return 1;
  const int pitch = ((S + 31) & ~31) + 1;
  int rc = 1;
  PP_F32_ATTN(dtype, dh, (rc = fwd_f32<DH, T>(st, qkv, o, lse, B, S, h, pitch)));
  return rc;
}
int k_attn_bwd_f32(hipStream_t st, int dtype, const void* qkv, const void* o, const float* lse, const void* dO, void* dqkv, float* Dbuf, int B, int S, int h, int dh) {
  if (!shapes_ok(dtype, qkv, dO, S, h, dh) || !bwd_pays((long)B * h, S, dh)) return 1;
  k_attn_D(st, dtype, o, dO, Dbuf, B, S, h, dh);
  PP_F32_ATTN(dtype, dh, (bwd_f32<DH, T>(st, qkv, lse, Dbuf, dO, dqkv, B, S, h)));
  return 0;
}

}  // namespace pp
