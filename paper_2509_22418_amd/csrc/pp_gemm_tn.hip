// bf16 MFMA GEMM for gfx950 with the contraction index as the ROW index of both operands ("TN"):
//     C[M x N] (fp32) = A^T B,   A: [K x M] row-major (lda),  B: [K x N] row-major (ldb).
// This is the weight-gradient form of the local step (Appendix "Partial Backward": dW_n = dH_n X^T, dV_n = G A_n^T in the
// paper's features x tokens convention): K runs over tokens, and both operands are activations stored token-major, i.e.
// exactly as the forward and backward passes leave them.  No transposed copies are made: tiles go from global memory to
// LDS as they are ([k][m], rows of 256 bytes), and the MFMA operand fragments -- 8 consecutive k for one m -- are
// gathered by the LDS transpose read (ds_read_b64_tr_b16), two per fragment.
//
// Transpose read, 16-bit elements: within each group of 16 lanes, lane i receives element i % 4 of the four 8-byte
// pieces addressed by lanes i/4, i/4 + 4, i/4 + 8, i/4 + 12.  If lane j points at T[k0 + j/4][m0 + 4 (j % 4)], lane i
// therefore gets T[k0 .. k0+3][m0 + i]: four consecutive k of one column.
//
// Tiling: 128 x 128 output tile per workgroup of 256 threads (4 waves, 2 x 2, each 64 x 64 = 2 x 2 blocks of
// v_mfma_f32_32x32x16_bf16, 64 accumulator registers); K advances in steps of 64 rows; two LDS stages of 16 KB per
// operand (64 KB per workgroup, two workgroups per compute unit), the next step's tiles in flight while the current one
// is multiplied, one barrier per step.  (A ring of four 32-row stages was slower on every shape when each
// transpose read still waited for all loads in flight, see read_frags; it has not been timed since.)  Tiles are filled
// by direct-to-LDS loads (one wave load = 4 rows); the 16-byte chunk c of row r is stored at chunk c ^ ((r & 3) << 2), applied on the source side, so
// that the 4 rows x 2 x 32 bytes touched by one phase of a transpose read fall into 8 different 32-byte bank groups.
// Few output tiles and a long K: the K range is split over blockIdx.y; partial products are summed in fixed order by
// the caller (k_splitk_reduce), so the result is reproducible run to run.
#include "pp_kernels.h"
#include "pp_dev.h"

#include <type_traits>

namespace pp {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef short s16x4 __attribute__((ext_vector_type(4)));

constexpr int TN_BM = 128, TN_BN = 128, TN_BK = 64;
constexpr int TN_OPERAND_BYTES = TN_BK * 256;                 // 64 rows of 128 elements
constexpr int TN_STAGE_BYTES = 2 * TN_OPERAND_BYTES;          // A tile, then B tile
constexpr int TN_LDS_BYTES = 2 * TN_STAGE_BYTES;

#define PP_TN_GPTR(p) ((const __attribute__((address_space(1))) void*)(p))
#define PP_TN_LPTR(p) ((__attribute__((address_space(3))) void*)(p))

// A's columns may come in blocks: column m of the product is column (m / m_blk) * a_blk_stride + m % m_blk of A
// (gate and up gradients of a hidden-unit slice sit d_ff columns apart; the Q, K, V parts of a head range d_model apart).
// Blocks are multiples of 8 columns, so a 16-byte chunk never straddles two of them; every lane finds its own chunk's block once.
// K need not be a multiple of 64: in the last step the rows past the end are loaded from the last row (in bounds) and then
// overwritten with zeros in both panels, so neither their values nor infinities among them reach a product.  (A token count that
// is not a multiple of 64 used to send every weight gradient through element-wise transposes and fp32 multiplies: 4 layers of
// 768 x 3072 on 3055 tokens spent 12.8 ms there.)
// PIECES: the range is summed in pieces of sub_steps steps (a kernel of its own: with the counting and the second set of sums in every launch
// 240 x 528 over 256 rows took 6.5 us instead of 6.1).
template <bool PIECES>
__global__ __launch_bounds__(256, 2) void gemm_tn_mfma_kernel(const bf16_t* __restrict__ A, int lda, int m_blk, long a_blk_stride,
                                                               const bf16_t* __restrict__ B, int ldb, float* __restrict__ C, int ldc,
                                                               int M, int N, int K, int Ksplit, int sub_steps, int tiles_m, int tiles_n) {
  extern __shared__ __align__(16) unsigned char tn_lds[];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 1, wn = wave & 1;
  // Workgroup id -> (K range z, tile).  The hardware deals workgroups to the 8 XCDs round-robin by id; XCD k = id % 8 is
  // given a contiguous range of the (z, tile) list (z slowest), so that with 8 or more K ranges an XCD reads only its own
  // rows of A and B (they then sit in that XCD's L2 for all the tiles that share them), and with fewer it works on
  // neighbouring tiles (groups of 8 M-tiles by all N-tiles) that share panels.
  const int tiles = tiles_m * tiles_n, nb = tiles * (int)gridDim.y;
  int pid = blockIdx.y * tiles + blockIdx.x;
  if ((nb & 7) == 0) pid = (pid & 7) * (nb >> 3) + (pid >> 3);
  const int z = pid / tiles, t = pid - z * tiles;
  constexpr int GROUP = 8;
  const int per_group = GROUP * tiles_n;
  const int group = t / per_group, first_m = group * GROUP;
  const int gsz = min(tiles_m - first_m, GROUP);
  const int in_group = t - group * per_group;
  const int tm = first_m + in_group % gsz, tn = in_group / gsz;
  const int m0 = tm * TN_BM, n0 = tn * TN_BN;
  const size_t kbase = (size_t)z * Ksplit;
  const int kz = min(Ksplit, K - (int)kbase);          // rows of this range (>= 1)
  const int ns = (kz + TN_BK - 1) / TN_BK, last = kz - (ns - 1) * TN_BK;          // rows of the last step

  // ---- direct-to-LDS fill: wave w moves wave-loads 4w .. 4w+3 of each operand tile; wave-load q = rows 4q .. 4q+3,
  // lane l -> row 4q + l/16, chunk position l%16, which receives source chunk (l%16) ^ ((row & 3) << 2).
  const int frow = lane >> 4;                                          // row within a wave-load (== row & 3)
  const int fchunk = (lane & 15) ^ (frow << 2);                        // source chunk of this lane
  const int a_valid = min(M, m0 + TN_BM) - m0, b_valid = min(N, n0 + TN_BN) - n0;          // columns of the tile that exist (multiples of 8)
  const int a_col = min(fchunk * 8, a_valid - 8), b_col = min(fchunk * 8, b_valid - 8);    // clamped: padded columns repeat the last chunk
  const int am = m0 + a_col;
  const long acol = M > m_blk ? (long)(am / m_blk) * a_blk_stride + am % m_blk : am;
  const bf16_t* gA = A + (kbase + (size_t)(wave * 16 + frow)) * lda + acol;
  const bf16_t* gB = B + (kbase + (size_t)(wave * 16 + frow)) * ldb + n0 + b_col;
  auto issue = [&](int s, int stage) {          // K-step s into LDS stage `stage`: 8 loads per wave
    unsigned char* dst = tn_lds + stage * TN_STAGE_BYTES + wave * 4 * 1024;
    if (s < ns - 1 || last == TN_BK) {
      const size_t ka = (size_t)s * TN_BK * lda, kb = (size_t)s * TN_BK * ldb;
#pragma unroll
      for (int i = 0; i < 4; ++i) __builtin_amdgcn_global_load_lds(PP_TN_GPTR(gA + ka + (size_t)(4 * i) * lda), PP_TN_LPTR(dst + i * 1024), 16, 0, 0);
#pragma unroll
      for (int i = 0; i < 4; ++i)
        __builtin_amdgcn_global_load_lds(PP_TN_GPTR(gB + kb + (size_t)(4 * i) * ldb), PP_TN_LPTR(dst + TN_OPERAND_BYTES + i * 1024), 16, 0, 0);
    } else {          // a short last step: rows past the end repeat the last one
      const int r0 = wave * 16 + frow;          // row of gA / gB within a step
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const long dr = (long)s * TN_BK + min(r0 + 4 * i, last - 1) - r0;
        __builtin_amdgcn_global_load_lds(PP_TN_GPTR(gA + dr * lda), PP_TN_LPTR(dst + i * 1024), 16, 0, 0);
        __builtin_amdgcn_global_load_lds(PP_TN_GPTR(gB + dr * ldb), PP_TN_LPTR(dst + TN_OPERAND_BYTES + i * 1024), 16, 0, 0);
      }
    }
  };

  // ---- fragment addresses.  Lane l: j = l % 16 (position in its group of 16), grp = l / 16: column half grp & 1 of a
  // 32-column block, k half grp >> 1 of a 16-row MFMA step.  It points at row (j / 4) of a 4-row band, 8-byte piece
  // j % 4 of the 32-byte column segment: chunk (col / 8) ^ ((j / 4) << 2), byte 8 * (j & 1) within the chunk.
  const int j = lane & 15, grp = lane >> 4;
  auto frag_off = [&](int w_half, int blk) {          // byte offset inside an operand tile, for K-row 0 of the step
    const int col = w_half * 64 + blk * 32 + (grp & 1) * 16 + 4 * (j & 3);
    const int chunk = (col >> 3) ^ ((j >> 2) << 2);
    return ((grp >> 1) * 8 + (j >> 2)) * 256 + chunk * 16 + (j & 1) * 8;
  };
  const int offA0 = frag_off(wm, 0), offA1 = frag_off(wm, 1);
  const int offB0 = TN_OPERAND_BYTES + frag_off(wn, 0), offB1 = TN_OPERAND_BYTES + frag_off(wn, 1);
  // One K16 slice's four fragments: 8 consecutive k (rows 16 kk + 8 (grp >> 1) ..) of one column each, two transpose reads per
  // fragment.  In assembly because of the builtin's waits: while direct-to-LDS loads are pending the compiler waits for all of
  // them (vmcnt(0)) in front of every transpose read, i.e. for the NEXT step's tiles right after they were requested; nothing of
  // a step's load latency was hidden inside a workgroup.  The reads are waited for inside the block, so its outputs are ready.
  // (K = 16384, before / after: 2048 x 2048 unsplit, one workgroup per unit, 252 / 201 us; 6144 x 2048 563 / 476; 32000 x 768 over
  // 3072 rows 186 / 172; shapes with two workgroups per unit that hid each other's loads stay as they were.  Turning the tiles in
  // registers on their way into LDS instead, so that plain 16-byte reads serve as fragments, was slower: 77 against 61 us at
  // 512 x 2048 in 16 ranges.)
  bf16x8 fa[2], fb[2];
  auto read_frags = [&](uint32_t st, auto KK) {          // st = byte offset of the stage in LDS
    constexpr int k0 = decltype(KK)::value * 16 * 256;
    s16x4 r[8];
    asm volatile(
        "ds_read_b64_tr_b16 %0, %8 offset:%12\n\tds_read_b64_tr_b16 %1, %8 offset:%13\n\t"
        "ds_read_b64_tr_b16 %2, %9 offset:%12\n\tds_read_b64_tr_b16 %3, %9 offset:%13\n\t"
        "ds_read_b64_tr_b16 %4, %10 offset:%12\n\tds_read_b64_tr_b16 %5, %10 offset:%13\n\t"
        "ds_read_b64_tr_b16 %6, %11 offset:%12\n\tds_read_b64_tr_b16 %7, %11 offset:%13\n\t"
        "s_waitcnt lgkmcnt(0)"
        : "=&v"(r[0]), "=&v"(r[1]), "=&v"(r[2]), "=&v"(r[3]), "=&v"(r[4]), "=&v"(r[5]), "=&v"(r[6]), "=&v"(r[7])
        : "v"(st + offA0), "v"(st + offA1), "v"(st + offB0), "v"(st + offB1), "n"(k0), "n"(k0 + 4 * 256)
        : "memory");
    auto join = [](s16x4 lo, s16x4 hi) { return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7)); };
    fa[0] = join(r[0], r[1]); fa[1] = join(r[2], r[3]);
    fb[0] = join(r[4], r[5]); fb[1] = join(r[6], r[7]);
  };

  // acc: running sum of a piece; tot (PIECES): sum of the finished ones, so that a range that covers several of the caller's
  // ranges keeps their shorter fp32 chains
  f32x16 acc[2][2], tot[2][2];
  int left = sub_steps;          // steps of this piece to come
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int r = 0; r < 16; ++r) { acc[a][b][r] = 0.f; tot[a][b][r] = 0.f; }

  auto mm = [&]() {
    acc[0][0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[0], fb[0], acc[0][0], 0, 0, 0);
    acc[0][1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[0], fb[1], acc[0][1], 0, 0, 0);
    acc[1][0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[1], fb[0], acc[1][0], 0, 0, 0);
    acc[1][1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[1], fb[1], acc[1][1], 0, 0, 0);
  };
  const uint32_t lds0 = (uint32_t)(uintptr_t)PP_TN_LPTR(tn_lds);
  issue(0, 0);
  for (int s = 0; s < ns; ++s) {
    // this wave's loads of step s have landed; after the barrier everybody's have, and nobody reads the other stage any more
    __builtin_amdgcn_s_waitcnt(0x0070);
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
    if (s + 1 < ns) issue(s + 1, (s + 1) & 1);
    else if (last < TN_BK) {          // rows past the end of K: zeros in both panels (nothing is in flight any more)
      unsigned char* z0 = tn_lds + (s & 1) * TN_STAGE_BYTES + last * 256;
      const int n16 = (TN_BK - last) * 16;
      for (int i = tid; i < 2 * n16; i += 256)
        *reinterpret_cast<uint4*>(z0 + (i < n16 ? i : i - n16) * 16 + (i < n16 ? 0 : TN_OPERAND_BYTES)) = make_uint4(0, 0, 0, 0);
      __builtin_amdgcn_s_waitcnt(0xC07F);          // lgkmcnt(0)
      __builtin_amdgcn_s_barrier();
      __builtin_amdgcn_sched_barrier(0);
    }
    const uint32_t stage = lds0 + (s & 1) * TN_STAGE_BYTES;
    __builtin_amdgcn_sched_barrier(0);
    read_frags(stage, std::integral_constant<int, 0>{}); mm();
    read_frags(stage, std::integral_constant<int, 1>{}); mm();
    read_frags(stage, std::integral_constant<int, 2>{}); mm();
    read_frags(stage, std::integral_constant<int, 3>{}); mm();
    if (PIECES && (--left == 0 || s + 1 == ns)) {
      left = sub_steps;
#pragma unroll
      for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
          for (int r = 0; r < 16; ++r) { tot[a][b][r] += acc[a][b][r]; acc[a][b][r] = 0.f; }
    }
  }

  // ---- epilogue: element r of block (a, b) is row m0 + 64 wm + 32 a + 8 (r / 4) + 4 (lane / 32) + r % 4,
  //      column n0 + 64 wn + 32 b + lane % 32; 32 lanes store 128 consecutive bytes of one row
  float* Cz = C + (size_t)z * (size_t)M * (size_t)ldc;
  const int l32 = lane & 31, lh = lane >> 5;
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      const int col = n0 + wn * 64 + b * 32 + l32;
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int row = m0 + wm * 64 + a * 32 + 8 * (r >> 2) + 4 * lh + (r & 3);
        if (row < M && col < N) Cz[(size_t)row * ldc + col] = PIECES ? tot[a][b][r] : acc[a][b][r];
      }
    }
}

// C[M x N] fp32 (ldc) = A^T B over K rows in ranges of `kchunk` (a multiple of 64; the last may be shorter), each summed in pieces of
// `sub` rows (a multiple of 64, >= kchunk: one piece) that are added in order; more than one range:
// `partial` receives [ranges][M][N] (C is not written; the caller sums the partials in fixed order).  Returns 0 if launched, 1 if
// the shapes are not taken (nothing launched).
int k_gemm_tn_mfma(hipStream_t st, const void* A, int lda, int m_blk, long a_blk_stride, const void* B, int ldb, float* C, int ldc,
                   int M, int N, int K, int kchunk, float* partial, int sub) {
  if (M < 8 || N < 8 || (M & 7) || (N & 7) || (lda & 7) || (ldb & 7) || K < 1 || kchunk < 64 || (kchunk & 63) || sub < 64 || (sub & 63)) return 1;
  if (m_blk < 1 || (m_blk & 7) || (a_blk_stride & 7)) return 1;
  if (((uintptr_t)A | (uintptr_t)B | (uintptr_t)C | (uintptr_t)partial) & 15) return 1;
  const int splits = (int)(((long)K + kchunk - 1) / kchunk);
  if (splits > 1 && !partial) return 1;
  static const bool ok = hipFuncSetAttribute(reinterpret_cast<const void*>(gemm_tn_mfma_kernel<false>), hipFuncAttributeMaxDynamicSharedMemorySize, TN_LDS_BYTES) == hipSuccess &&
                         hipFuncSetAttribute(reinterpret_cast<const void*>(gemm_tn_mfma_kernel<true>), hipFuncAttributeMaxDynamicSharedMemorySize, TN_LDS_BYTES) == hipSuccess;
  if (!ok) return 1;
  const int tiles_m = (M + TN_BM - 1) / TN_BM, tiles_n = (N + TN_BN - 1) / TN_BN;
  dim3 grid(tiles_m * tiles_n, splits);
  float* out = splits > 1 ? partial : C;
  auto kern = sub < kchunk && sub < K ? gemm_tn_mfma_kernel<true> : gemm_tn_mfma_kernel<false>;
  kern<<<grid, 256, TN_LDS_BYTES, st>>>((const bf16_t*)A, lda, m_blk, a_blk_stride, (const bf16_t*)B, ldb, out, splits > 1 ? N : ldc, M, N, K, kchunk, sub / 64, tiles_m, tiles_n);
  return 0;
}

}  // namespace pp
