// fp32-multiply MFMA GEMM for gfx950 (fp32 operands, fp32 accumulate), any M, N, K and alignment:
//   NT:  C[M x N] = A[M x K] B[N x K]^T (+ R)      both operands K-contiguous (projections, input gradients)
//   TN:  C[M x N] = A^T B, A [K x M'], B [K x N]    both operands token-major (weight gradients; no transposed copies)
// It carries every contraction of an fp32 model, and the bf16 contractions whose K or alignment the bf16 MFMA kernels do
// not take (operands are widened to fp32 while they are staged; the products are then exact).
//
// Order of summation: v_mfma_f32_32x32x2_f32 and v_mfma_f32_16x16x4_f32 add their 2 / 4 products one after the other, each
// with one rounding (compared bit for bit with fmaf chains, denormal results included), so an accumulator that is fed k = 0, 1, 2, ...
// holds exactly the fmaf chain of the plain kernel: this kernel returns the plain kernel's bits.  That is why lane group i of an
// MFMA is given k = 2 j + i (4 j + i) and why no wave splits K.
//
// What bounds it: the matrix pipe (64 FLOP per clock and SIMD = 157 TFLOP/s on the chip, twice the vector-FMA rate).
// Against that the operand feed is cheap (a 64 x 64 tile needs 16 bytes of global loads and 32 bytes of LDS reads per clock
// and compute unit), so small tiles cost little and the tile is chosen to fill the chip:
//   * 64 x 64 tile, four waves of 32 x 32 (32x32x2 MFMAs: 32 cycles per k), K steps of 32, when there are enough of them;
//   * 32 x 32 tile, four waves of 16 x 16 (16x16x4 MFMAs: 8 cycles per k), K steps of 64, otherwise: four times the
//     workgroups and a quarter of the serial chain, which is what a launch of few tiles lasts as long as.
// Staging goes through registers (two sets, loads run two K steps ahead) by buffer loads: a piece past the last row, column
// or k is given an offset outside the buffer and reads as zero without a branch, so edges and remainders need no case of their own.
// Not taken: rows so long that a tile's offsets pass 31 bits (offsets_fit: about 8.3 M elements), and TN column blocks that are not
// multiples of 4.  An NT panel row is cut into groups of 8 (16) k; the 16-byte chunk i of a group holds the k
// that lane group i needs (k = i mod 2, resp. mod 4), so one 16-byte read feeds four MFMAs.  Chunks are permuted by row so that 16
// rows of one chunk lie on different banks; all the same a third of the kernel's LDS-active cycles are counted as conflicts (LDS active 0.31 to 0.50, matrix pipe
// busy 0.53 with 32 x 32 tiles without DEEP and 0.64 with it, 0.81 with 64 x 64: profiles/op_kernels_pmc.txt).  TN panels are stored [k][m] as they lie
// in memory, with bit 5 (bit 4) of m flipped for every second k (pair of k), and are read 4 bytes per lane.
#include "pp_kernels.h"
#include "pp_dev.h"

namespace pp {

typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
constexpr uint32_t OOB = 0x80000000u;          // past every buffer below: reads as zero
__device__ __forceinline__ __amdgpu_buffer_rsrc_t buf_of(const void* p) { return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, 0x7fffffff, 0x00020000); }

// four consecutive elements at byte offset off (+ uniform soff), widened; VEC: all four exist or none (off == OOB); otherwise the
// first `valid` exist
template <class T, bool VEC> __device__ __forceinline__ float4 load4(__amdgpu_buffer_rsrc_t r, uint32_t off, uint32_t soff, int valid) {
  if constexpr (VEC) {
    if constexpr (sizeof(T) == 4) return __builtin_bit_cast(float4, __builtin_amdgcn_raw_buffer_load_b128(r, valid > 0 ? off : OOB, soff, 0));
    else {
      const u32x2 w = __builtin_bit_cast(u32x2, __builtin_amdgcn_raw_buffer_load_b64(r, valid > 0 ? off : OOB, soff, 0));
      return make_float4(__uint_as_float(w[0] << 16), __uint_as_float(w[0] & 0xffff0000u), __uint_as_float(w[1] << 16), __uint_as_float(w[1] & 0xffff0000u));
    }
  } else {
    float v[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const uint32_t o = valid > e ? off + e * sizeof(T) : OOB;
      if constexpr (sizeof(T) == 4) v[e] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(r, o, soff, 0));
      else v[e] = bf16_to_f32(__builtin_amdgcn_raw_buffer_load_b16(r, o, soff, 0));
    }
    return make_float4(v[0], v[1], v[2], v[3]);
  }
}

struct F32GemmArgs {
  int lda, ldb, ldc, M, N, K, kchunk;
  int m_blk; long a_blk_stride;          // TN only: column m of the product is column (m / m_blk) * a_blk_stride + m % m_blk of A
  int epi;
};

// VEC: groups of four elements are aligned and exist as a whole
// DEEP: fragments one step ahead (see step below)
template <class T, class TO, bool TN, bool SMALL, bool VEC, bool DEEP>
__global__ __launch_bounds__(256) void gemm_f32_mfma_kernel(const T* __restrict__ A, const T* __restrict__ B, TO* C, const T* R, const F32GemmArgs g) {
  constexpr int BM = SMALL ? 32 : 64, BK = SMALL ? 64 : 32;
  constexpr int CPR = BK / 4;                              // NT: 16-byte chunks per panel row
  constexpr int NV = BM * BK / 4 / 256;                    // float4 pieces per thread and operand
  constexpr int PANEL = BM * BK;                           // floats
  __shared__ __align__(16) float lds[2 * 2 * PANEL];       // two stages of A panel, B panel
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int lr = SMALL ? lane & 15 : lane & 31, lg = SMALL ? lane >> 4 : lane >> 5;          // row within a wave's block, k group of the MFMA
  const int m0 = blockIdx.y * BM, n0 = blockIdx.x * BM, z = blockIdx.z;
  const int kb = z * g.kchunk, ke = min(g.K, kb + g.kchunk), nk = (ke - kb + BK - 1) / BK;
  // float offset of chunk c of row r in an NT panel
  auto at = [](int r, int c) {
    if constexpr (SMALL) return (r * CPR + (c ^ (((r & 1) << 1) | ((r >> 1) & 1) | (r & 12)))) * 4;
    else return (r * CPR + (c ^ ((r >> 1) & 7))) * 4;
  };
  // column of element m of row k in a TN panel
  auto tcol = [](int k, int m) { return SMALL ? m ^ (((k >> 1) & 1) << 4) : m ^ ((k & 1) << 5); };

  // ---- staging: piece i of this thread is 4 elements of one panel row (NT: 4 k of a row; TN: 4 columns of one k)
  // Offsets are relative to the tile's first row (NT; the step enters as a uniform offset) or to the step's first k (TN; the base
  // pointer moves), so that they fit 31 bits whatever M and N are; the launchers check the rows' lengths (offsets_fit).
  uint32_t oa[NV], ob[NV];
  int va[NV], vb[NV], kk[NV], row[NV];          // elements that exist (TN: columns; NT: 4 or 0).  kk = k of the piece within a step
#pragma unroll
  for (int i = 0; i < NV; ++i) {
    const int q = tid + 256 * i;
    if constexpr (TN) {
      const int c4 = (q % (BM / 4)) * 4;
      kk[i] = q / (BM / 4); row[i] = c4;
      const int m = m0 + c4, mc = min(m, g.M - 1);
      va[i] = g.M - m; vb[i] = g.N - (n0 + c4);
      oa[i] = (uint32_t)(kk[i] * g.lda + (int)((long)(mc / g.m_blk) * g.a_blk_stride) + mc % g.m_blk) * sizeof(T);
      ob[i] = (uint32_t)(kk[i] * g.ldb + n0 + c4) * sizeof(T);
    } else {
      row[i] = q / CPR; kk[i] = 4 * (q % CPR);
      va[i] = m0 + row[i] < g.M ? 4 : 0; vb[i] = n0 + row[i] < g.N ? 4 : 0;
      oa[i] = (uint32_t)(row[i] * g.lda + kk[i]) * sizeof(T);
      ob[i] = (uint32_t)(row[i] * g.ldb + kk[i]) * sizeof(T);
    }
  }
  const T* const baseA = TN ? A + (size_t)kb * g.lda : A + (size_t)m0 * g.lda + kb;
  const T* const baseB = TN ? B + (size_t)kb * g.ldb : B + (size_t)n0 * g.ldb + kb;
  auto load = [&](float4 (&ra)[NV], float4 (&rb)[NV], int s) {          // K step s (past the end: zeros, nothing read)
    const auto bufA = buf_of(TN ? baseA + (size_t)s * BK * g.lda : baseA), bufB = buf_of(TN ? baseB + (size_t)s * BK * g.ldb : baseB);
    const uint32_t soff = TN ? 0u : (uint32_t)(s * BK) * (uint32_t)sizeof(T);
#pragma unroll
    for (int i = 0; i < NV; ++i) {
      const int left = ke - kb - s * BK - kk[i];          // k from this piece on that exist
      const int na = TN ? (left > 0 ? va[i] : 0) : min(va[i], left), nb = TN ? (left > 0 ? vb[i] : 0) : min(vb[i], left);
      ra[i] = load4<T, VEC>(bufA, oa[i], soff, na);
      rb[i] = load4<T, VEC>(bufB, ob[i], soff, nb);
    }
  };
  auto put_piece = [&](float* s, int i, const float4& v) {
    if constexpr (TN) *reinterpret_cast<float4*>(s + kk[i] * BM + tcol(kk[i], row[i])) = v;
    else if constexpr (SMALL) {          // k = 16 grp + 4 j + e: element j of chunk 4 grp + e
      const int c = 4 * (kk[i] >> 4), j = (kk[i] >> 2) & 3;
      s[at(row[i], c) + j] = v.x; s[at(row[i], c + 1) + j] = v.y; s[at(row[i], c + 2) + j] = v.z; s[at(row[i], c + 3) + j] = v.w;
    } else {                             // k = 8 grp + 4 j + e: element 2 j + e / 2 of chunk 2 grp + e % 2
      const int c = 2 * (kk[i] >> 3), j = 2 * ((kk[i] >> 2) & 1);
      *reinterpret_cast<float2*>(s + at(row[i], c) + j) = make_float2(v.x, v.z);
      *reinterpret_cast<float2*>(s + at(row[i], c + 1) + j) = make_float2(v.y, v.w);
    }
  };
  auto store = [&](const float4 (&ra)[NV], const float4 (&rb)[NV], int stage) {
    float* s = lds + stage * 2 * PANEL;
#pragma unroll
    for (int i = 0; i < NV; ++i) { put_piece(s, i, ra[i]); put_piece(s + PANEL, i, rb[i]); }
  };
  // ---- a wave's block of the tile: 32 x 32 or 16 x 16
  constexpr int WB = BM / 2, NR = SMALL ? 4 : 16;
  typedef float facc __attribute__((ext_vector_type(NR)));
  const int wm = (wave >> 1) * WB, wn = (wave & 1) * WB;
  facc acc;
#pragma unroll
  for (int r = 0; r < NR; ++r) acc[r] = 0.f;
  auto mfma = [&](float x, float y) {
    if constexpr (SMALL) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(x, y, acc, 0, 0, 0);
    else acc = __builtin_amdgcn_mfma_f32_32x32x2f32(x, y, acc, 0, 0, 0);
  };
  float4 a0[NV], b0[NV], a1[NV], b1[NV];
  if constexpr (DEEP) {
    static_assert(!DEEP || !TN, "fragments of K-contiguous panels");
    // ---- a step is 16 MFMAs, k ascending; its fragments are in registers when it starts
    constexpr int G = SMALL ? 4 : 2;          // k per MFMA
    float fa[2][16], fb[2][16];
    auto read = [&](int set, int stage, int j) {          // operands of MFMAs 4 j .. 4 j + 3
      const float* sa = lds + stage * 2 * PANEL;
      *reinterpret_cast<float4*>(fa[set] + 4 * j) = *reinterpret_cast<const float4*>(sa + at(wm + lr, j * G + lg));
      *reinterpret_cast<float4*>(fb[set] + 4 * j) = *reinterpret_cast<const float4*>(sa + PANEL + at(wn + lr, j * G + lg));
    };
    auto meet = [&]() {          // this wave's LDS accesses are done, then everybody's; loads stay in flight
      __builtin_amdgcn_s_waitcnt(0xC07F);
      __builtin_amdgcn_s_barrier();
      __builtin_amdgcn_sched_barrier(0);
    };
    // Step s, with everything else that happens meanwhile spread behind its MFMAs: the fragments of step s + 1, step s + 2 from
    // registers into the slot that step s was read from, the requests of step s + 4 into those registers.  One barrier per step.
    // (With the step's own fragments read in front of its MFMAs and the panels stored behind them the matrix pipe was busy 0.53 of the time with
    // 32 x 32 tiles, two workgroups per unit: 1024 x 512, K = 2048 31 us.)
    auto step = [&](int set, float4 (&ra)[NV], float4 (&rb)[NV], int s) {
#pragma unroll
      for (int j = 0; j < 16; ++j) {
        mfma(fa[set][j], fb[set][j]);
        __builtin_amdgcn_sched_barrier(0);
        if (j < 4) read(1 - set, 1 - set, j);
        if (j >= 4 && j < 4 + 4 * NV && (j & 3) == 0) {
          const int i = j / 4 - 1;
          float* d = lds + set * 2 * PANEL;
          put_piece(d, i, ra[i]); put_piece(d + PANEL, i, rb[i]);
        }
        if (j == 4 + 4 * NV - 3) load(ra, rb, s + 4);
        __builtin_amdgcn_sched_barrier(0);
      }
      meet();
    };
    load(a0, b0, 0);
    load(a1, b1, 1);
    store(a0, b0, 0);
    if (nk > 1) {
      load(a0, b0, 2);
      store(a1, b1, 1);
      load(a1, b1, 3);
    }
    meet();
#pragma unroll
    for (int j = 0; j < 4; ++j) read(0, 0, j);
    if (nk > 1) meet();
    int s = 0;
    for (; s + 2 < nk; s += 2) {
      step(0, a0, b0, s);
      step(1, a1, b1, s + 1);
    }
    if (s + 1 < nk) {
      step(0, a0, b0, s);
#pragma unroll
      for (int j = 0; j < 16; ++j) mfma(fa[1][j], fb[1][j]);
    } else {
#pragma unroll
      for (int j = 0; j < 16; ++j) mfma(fa[0][j], fb[0][j]);
    }
  } else {
    auto compute = [&](int stage) {
      const float* sa = lds + stage * 2 * PANEL;
      const float* sb = sa + PANEL;
      constexpr int G = SMALL ? 4 : 2;          // k per MFMA
      if constexpr (TN) {
#pragma unroll
        for (int h = 0; h < BK / G; h += 16) {
          float fa[16], fb[16];
#pragma unroll
          for (int j = 0; j < 16; ++j) {
            const int k = (h + j) * G + lg;
            fa[j] = sa[k * BM + tcol(k, wm + lr)];
            fb[j] = sb[k * BM + tcol(k, wn + lr)];
          }
#pragma unroll
          for (int j = 0; j < 16; ++j) mfma(fa[j], fb[j]);
        }
      } else {
        const int ra = wm + lr, rb = wn + lr;
#pragma unroll
        for (int h = 0; h < CPR / G; h += 4) {
          float4 fa[4], fb[4];
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            fa[i] = *reinterpret_cast<const float4*>(sa + at(ra, (h + i) * G + lg));
            fb[i] = *reinterpret_cast<const float4*>(sb + at(rb, (h + i) * G + lg));
          }
#pragma unroll
          for (int i = 0; i < 4; ++i) { mfma(fa[i].x, fb[i].x); mfma(fa[i].y, fb[i].y); mfma(fa[i].z, fb[i].z); mfma(fa[i].w, fb[i].w); }
        }
      }
    };
    // ---- main loop: step s is multiplied from stage s & 1 while step s + 1 goes from registers to the other stage and step
    // s + 2 is requested; one barrier per step
    load(a0, b0, 0);
    load(a1, b1, 1);
    store(a0, b0, 0);
    __syncthreads();
    for (int s = 0; s + 1 < nk; s += 2) {
      load(a0, b0, s + 2);
      __builtin_amdgcn_sched_barrier(0);          // the requests leave before the MFMAs, not after them
      compute(0);
      __builtin_amdgcn_sched_barrier(0);
      store(a1, b1, 1);
      __syncthreads();
      load(a1, b1, s + 3);
      __builtin_amdgcn_sched_barrier(0);
      compute(1);
      __builtin_amdgcn_sched_barrier(0);
      store(a0, b0, 0);
      __syncthreads();
    }
    if (nk & 1) compute(0);
  }

  // ---- epilogue: 32 x 32: element r of a lane is row 8 (r / 4) + 4 (lane / 32) + r % 4, column lane % 32; 16 x 16: row 4 (lane / 16) + r
  C += (size_t)z * (size_t)g.M * (size_t)g.ldc;          // split-K partials are dense [z][M][ldc]
#pragma unroll
  for (int r = 0; r < NR; ++r) {
    const int orow = m0 + wm + (SMALL ? 4 * lg + r : 8 * (r >> 2) + 4 * lg + (r & 3)), col = n0 + wn + lr;
    if (orow < g.M && col < g.N) {
      const size_t o = (size_t)orow * g.ldc + col;
      float v = acc[r];
      if (g.epi == EPI_ADD_RES) v += to_f32(R[o]);
      C[o] = from_f32<TO>(v);
    }
  }
}

// Tile rule, from both tiles timed on M = 1024 / 2048, fp32 (us, 64 x 64 tile / 32 x 32 tile): 128 tiles of 64 x 64 with K = 512 14.9 / 9.7,
// with K = 2048 48 / 31; 384 tiles 24.8 / 22.1; 512 tiles 25.3 / 27.3; 1024 tiles 43 / 50.  Two 64 x 64 workgroups per compute unit are
// enough to hide each other's barriers; below that the shorter chain and the fourfold workgroups win.
// (1024 x 512 x 2048 on the vector-FMA kernel: 212 us; 4096 x 4096 x 1024: 286 us = 120 TFLOP/s.)
constexpr long kLargeTiles = 512;

// Up to kDeepTiles 32 x 32 tiles of fp32 K-contiguous operands the fragments are read a step ahead (DEEP, 132 registers a wave): with one or two workgroups per
// unit nothing else covers the reads and stores of a step.  us without / with: 1024 x 512 (512 tiles), K = 2048 32.1 / 26.3, K = 8000 101 / 80.5; 1024 x 1536 (1536), K = 512
// 19.7 / 18.7; from there on the workgroups that the registers cost are worth more: 1024 x 2048 (2048) 23.2 / 24.2, and so they are with 64 x 64 tiles
// (1024 x 4096, K = 512 39.7 / 49.1, 168 registers).  Short ranges lose to the longer code (128 x 64, K = 64 3.8 / 4.2; K = 256 4.3 / 4.0): 448 it takes on more than 600 tiles (1170 x 1000,
// K = 320 14.6 / 15.1, while 1024 x 1536, K = 512 gains) and where rows are loaded element by element (VEC = false: 49 x 254, K = 263 7.5 / 8.1, 1748 x 146, K = 285 12.0 / 12.7, 176 x 152, K = 429
// 9.3 / 9.6, from 448 on 0.92 to 0.95 of the plain loop's time), else 256.  Token-major panels, read four bytes at a time, gain nothing (512 x 512 over 1024 in ranges of 256: 9.9 / 10.6), and
// widened bf16 operands would be waited for right behind their requests (1000 x 520, K = 1000 21.7 / 23.2).
constexpr long kDeepTiles = 1536;
bool gemm_f32_reads_ahead(long tiles, int range, bool vec) { return tiles <= kDeepTiles && range >= (vec && tiles <= 600 ? 256 : 448); }

template <class T, class TO, bool TN, bool VEC>
static void launch_f32(hipStream_t st, const void* A, const void* B, void* C, const void* R, const F32GemmArgs& g, int splits) {
  const long t64 = (long)((g.M + 63) / 64) * ((g.N + 63) / 64) * splits;
  constexpr bool kDeep = sizeof(T) == 4 && !TN;
  const dim3 grid32((g.N + 31) / 32, (g.M + 31) / 32, splits);
  if (t64 >= kLargeTiles)
    gemm_f32_mfma_kernel<T, TO, TN, false, VEC, false><<<dim3((g.N + 63) / 64, (g.M + 63) / 64, splits), 256, 0, st>>>((const T*)A, (const T*)B, (TO*)C, (const T*)R, g);
  else if (kDeep && gemm_f32_reads_ahead((long)grid32.x * grid32.y * grid32.z, g.kchunk, VEC))
    gemm_f32_mfma_kernel<T, TO, TN, true, VEC, kDeep><<<grid32, 256, 0, st>>>((const T*)A, (const T*)B, (TO*)C, (const T*)R, g);
  else
    gemm_f32_mfma_kernel<T, TO, TN, true, VEC, false><<<grid32, 256, 0, st>>>((const T*)A, (const T*)B, (TO*)C, (const T*)R, g);
}
template <class T, class TO, bool TN>
static void launch_f32(hipStream_t st, const void* A, const void* B, void* C, const void* R, const F32GemmArgs& g, int splits, bool vec) {
  if (vec) launch_f32<T, TO, TN, true>(st, A, B, C, R, g, splits);
  else launch_f32<T, TO, TN, false>(st, A, B, C, R, g, splits);
}

// Offsets within a tile's 64 rows (NT: plus all of K) are 31-bit: longer rows stay on the vector kernel (TN: are refused).
static bool offsets_fit(int lda, int ldb, int K) { return (64ull * (size_t)(lda > ldb ? lda : ldb) + (size_t)K) * 4 < 0x7f000000ull; }
// rows of groups of four elements that can be read at once
static bool vec4_ok(int dtype, const void* p, int ld) { return ld % 4 == 0 && ((uintptr_t)p & (dtype == 0 ? 15 : 7)) == 0; }

void k_gemm_nt_f32(hipStream_t st, int dtype, const void* A, int lda, const void* B, int ldb, void* C, int ldc, int M, int N, int K, int epi, const void* R,
                   int out_f32, int splits, float* partial) {
  if (M == 0 || N == 0) return;
  if (!offsets_fit(lda, ldb, K)) {
    if (splits > 1) k_gemm_nt_plain_splitk(st, dtype, A, lda, B, ldb, partial, M, N, K, splits);
    else k_gemm_nt_plain(st, dtype, A, lda, B, ldb, C, ldc, M, N, K, epi, R, out_f32);
    return;
  }
  const F32GemmArgs g{lda, ldb, splits > 1 ? N : ldc, M, N, K, K / splits, M, 0, epi};
  const bool vec = vec4_ok(dtype, A, lda) && vec4_ok(dtype, B, ldb) && g.kchunk % 4 == 0;
  void* out = splits > 1 ? (void*)partial : C;
  if (dtype == 0) launch_f32<float, float, false>(st, A, B, out, R, g, splits, vec);
  else if (out_f32 || splits > 1) launch_f32<bf16_t, float, false>(st, A, B, out, R, g, splits, vec);
  else launch_f32<bf16_t, bf16_t, false>(st, A, B, out, R, g, splits, vec);
}

// returns 1 (nothing launched) if a group of four columns of A could straddle two column blocks, or rows are too long for the offsets
int k_gemm_tn_f32(hipStream_t st, const float* A, int lda, int m_blk, long a_blk_stride, const float* B, int ldb, float* C, int ldc, int M, int N, int K,
                  int splits, float* partial) {
  if ((M > m_blk && (m_blk % 4 || a_blk_stride % 4)) || !offsets_fit(lda, ldb, 0)) return 1;
  if (M == 0 || N == 0) return 0;
  const F32GemmArgs g{lda, ldb, splits > 1 ? N : ldc, M, N, K, K / splits, m_blk, a_blk_stride, EPI_STORE};
  const bool vec = vec4_ok(0, A, lda) && vec4_ok(0, B, ldb) && M % 4 == 0 && N % 4 == 0;
  launch_f32<float, float, true>(st, A, B, splits > 1 ? partial : C, nullptr, g, splits, vec);
  return 0;
}

}  // namespace pp
