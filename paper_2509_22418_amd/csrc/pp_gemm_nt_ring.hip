// bf16 MFMA GEMM for gfx950, shapes with few 256 x 256 tiles:  C[M x N] = A[M x K] * B[N x K]^T (+ R), both operands K-contiguous.
//
// The 256 x 256-tile kernel (one workgroup per compute unit, 160 KB of LDS) needs well over 256 tiles to fill the chip; the
// 125M-shape decoder (d_model 768, 8192 tokens) has projections with 96.  One kernel template cuts the output into smaller tiles:
// panels of BM and BN rows x 64 K-elements go straight to LDS (global_load_lds, rows of 128 bytes, chunk c of row r at
// c ^ ((r >> 1) & 7): conflict-free fragment reads), NS such stages form a ring.  All of a tile's fragments of a stage are in
// registers at the stage's one barrier, which therefore also frees its slot: stage s + NS is requested right behind it, so NS - 1 stages are
// in flight while one is multiplied.  v_mfma_f32_16x16x32_bf16 with the B panel as row operand; the accumulators are turned
// around through LDS into 16-byte row pieces, the residual is added in fp32 and the sum rounded once.
// What bounds it: a K step of a BM x BN tile is (BM + BN) * 128 bytes to load and BM * BN / 32 cycles of matrix pipe: 64 B per clock and
// compute unit (all that a unit's load path moves) at 128 x 128, 53 at 128 x 192.  Over whole launches (profiles/op_kernels_pmc.txt) the four larger
// tiles load 16 to 19 B per clock with the matrix pipe busy 0.28 to 0.46 and the waves waiting 0.31 to 0.40 of their cycles: latency behind the barriers,
// and a fifth to a third of a one-round launch in which units start up or drain.
#include "pp_kernels.h"
#include "pp_dev.h"

#include <type_traits>

namespace pp {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

#define PP_R_GPTR(p) ((const __attribute__((address_space(1))) void*)(p))
#define PP_R_LPTR(p) ((__attribute__((address_space(3))) void*)(p))

template <int N> __device__ __forceinline__ void wait_vm_lgkm0() {          // vmcnt(N) lgkmcnt(0)
  static_assert(N < 64, "vmcnt has 6 bits");
  __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | 0x0070);
}

template <int EPI, int BM, int BN, int WM, int WN, int NS>
__global__ __launch_bounds__(64 * WM * WN) void gemm_nt_ring_kernel(const bf16_t* __restrict__ A, int lda, const bf16_t* __restrict__ B, int ldb,
                                                                    bf16_t* C, int ldc, int M, int N, int K, const bf16_t* R, int tiles_m, int tiles_n, int vec) {
  constexpr int NW = WM * WN, TM = BM / WM, TN = BN / WN, MI = TM / 16, NJ = TN / 16;
  constexpr int STAGE = (BM + BN) * 128, LPW = (BM + BN) / 8 / NW;          // bytes of a stage; wave-loads (8 rows) per wave
  constexpr int PITCH = TN * 4 + 16;                                         // epilogue patch: bytes per row
  static_assert((BM + BN) / 8 % NW == 0 && TM % 16 == 0 && TN % 16 == 0 && MI % 2 == 0 && NW * 32 * PITCH <= NS * STAGE, "tile geometry");
  extern __shared__ __align__(16) unsigned char r_lds[];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / WN, wn = wave % WN;
  // XCD k = id % 8 owns a contiguous range of the tile list, ordered in groups of 8 M-tiles by all N-tiles
  const int nb = tiles_m * tiles_n;
  int pid = blockIdx.x;
  if ((nb & 7) == 0) pid = (pid & 7) * (nb >> 3) + (pid >> 3);
  constexpr int GROUP = 8;
  const int per_group = GROUP * tiles_n;
  const int group = pid / per_group, first_m = group * GROUP;
  const int gsz = min(tiles_m - first_m, GROUP);
  const int in_group = pid - group * per_group;
  const int m0 = (first_m + in_group % gsz) * BM, n0 = (in_group / gsz) * BN;
  const int ns = K / 64;

  // ---- fill: wave-load q of a stage is rows 8 q .. 8 q + 7 of the stacked A and B panels; wave w has q = w, w + NW, ...
  const bf16_t* g[LPW];
#pragma unroll
  for (int i = 0; i < LPW; ++i) {
    const int row = (wave + NW * i) * 8 + (lane >> 3), c = (lane & 7) ^ ((row >> 1) & 7);
    g[i] = row < BM ? A + (size_t)min(m0 + row, M - 1) * lda + c * 8 : B + (size_t)min(n0 + row - BM, N - 1) * ldb + c * 8;
  }
  auto issue = [&](int s, int slot) {
    unsigned char* dst = r_lds + slot * STAGE + wave * 1024;
#pragma unroll
    for (int i = 0; i < LPW; ++i) __builtin_amdgcn_global_load_lds(PP_R_GPTR(g[i] + (size_t)s * 64), PP_R_LPTR(dst + i * NW * 1024), 16, 0, 0);
  };

  // ---- fragments: lane l reads, for row l % 16 of a 16-row block, the 8 k 8 (l / 16) .. of K32 slice kk
  const int l16 = lane & 15, lq = lane >> 4, sw = (l16 >> 1) & 7;
  const int fa0 = (wm * TM + l16) * 128, fb0 = (BM + wn * TN + l16) * 128;
  bf16x8 fa[2][MI], fb[2][NJ];
  auto read = [&](int buf, int slot, int kk) {
    const unsigned char* p = r_lds + slot * STAGE + (((4 * kk + lq) ^ sw) << 4);
#pragma unroll
    for (int i = 0; i < MI; ++i) fa[buf][i] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4*>(p + fa0 + i * 2048));
#pragma unroll
    for (int j = 0; j < NJ; ++j) fb[buf][j] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4*>(p + fb0 + j * 2048));
  };
  f32x4 acc[MI][NJ];
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int j = 0; j < NJ; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  auto mm = [&](int buf) {
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
      for (int j = 0; j < NJ; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fb[buf][j], fa[buf][i], acc[i][j], 0, 0, 0);
  };
#pragma unroll
  for (int s = 0; s < NS; ++s)
    if (s < ns) issue(s, s);
  if (ns >= NS) wait_vm_lgkm0<(NS - 1) * LPW>(); else wait_vm_lgkm0<0>();
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_sched_barrier(0);
  read(0, 0, 0);
  int slot = 0;
  for (int s = 0; s < ns; ++s) {
    const int nxt = slot + 1 == NS ? 0 : slot + 1;
    read(1, slot, 1);
    mm(0);
    __builtin_amdgcn_sched_barrier(0);
    // this wave's rows of stage s + 1 have landed and its fragments of stage s are in registers; behind the barrier that holds for all
    if (s + NS <= ns) wait_vm_lgkm0<(NS - 2) * LPW>(); else wait_vm_lgkm0<0>();
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
    if (s + NS < ns) issue(s + NS, slot);
    if (s + 1 < ns) read(0, nxt, 0);
    mm(1);
    __builtin_amdgcn_sched_barrier(0);
    slot = nxt;
  }

  // ---- epilogue: nothing is in flight and nobody reads the stages any more (the last barrier).  Element r of block (i, j) is row
  // 16 i + l % 16, column 16 j + 4 (l / 16) + r of the wave's TM x TN part; it is turned around in a private patch.
  // 32 rows at a time
  unsigned char* patch = r_lds + wave * 32 * PITCH;
  constexpr int PR = TN / 8, NP = 32 * PR / 64;          // 8-column pieces per row, pieces per lane and pass
  static_assert(32 * PR % 64 == 0, "pieces");
#pragma unroll
  for (int p = 0; p < MI / 2; ++p) {
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < NJ; ++j)
        *reinterpret_cast<float4*>(patch + (i * 16 + l16) * PITCH + j * 64 + lq * 16) = make_float4(acc[2 * p + i][j][0], acc[2 * p + i][j][1], acc[2 * p + i][j][2], acc[2 * p + i][j][3]);
    auto store = [&](auto V) {          // V consecutive columns exist as a whole and are aligned
      constexpr int VEC = decltype(V)::value;
#pragma unroll
      for (int it = 0; it < NP; ++it) {
        const int idx = it * 64 + lane, row = idx / PR, c = idx % PR;
        const float4 v0 = *reinterpret_cast<const float4*>(patch + row * PITCH + c * 32);
        const float4 v1 = *reinterpret_cast<const float4*>(patch + row * PITCH + c * 32 + 16);
        const int grow = m0 + wm * TM + p * 32 + row, gcol = n0 + wn * TN + c * 8;
        if (grow >= M || gcol >= N) continue;
        float v[8] = {v0.x, v0.y, v0.z, v0.w, v1.x, v1.y, v1.z, v1.w};
        const size_t off = (size_t)grow * ldc + gcol;
        if constexpr (VEC == 8) {
          if constexpr (EPI == EPI_ADD_RES) {
            float r[8];
            load8(R + off, r);
#pragma unroll
            for (int e = 0; e < 8; ++e) v[e] += r[e];
          }
          store8(C + off, v);
        } else {
#pragma unroll
          for (int e = 0; e < 8; e += VEC) {
            if (gcol + e >= N) continue;
            if constexpr (VEC == 4) {
              if constexpr (EPI == EPI_ADD_RES) {
                const uint2 r = *reinterpret_cast<const uint2*>(R + off + e);
                v[e] += __uint_as_float(r.x << 16); v[e + 1] += __uint_as_float(r.x & 0xffff0000u);
                v[e + 2] += __uint_as_float(r.y << 16); v[e + 3] += __uint_as_float(r.y & 0xffff0000u);
              }
              *reinterpret_cast<uint2*>(C + off + e) = make_uint2(f32x2_to_bf16x2(v[e], v[e + 1]), f32x2_to_bf16x2(v[e + 2], v[e + 3]));
            } else {
              if constexpr (EPI == EPI_ADD_RES) v[e] += to_f32(R[off + e]);
              C[off + e] = from_f32<bf16_t>(v[e]);
            }
          }
        }
      }
    };
    if (vec == 8) store(std::integral_constant<int, 8>{});
    else if (vec == 4) store(std::integral_constant<int, 4>{});
    else store(std::integral_constant<int, 1>{});
  }
}

template <int EPI, int BM, int BN, int WM, int WN, int NS>
static int launch_ring(hipStream_t st, const void* A, int lda, const void* B, int ldb, void* C, int ldc, int M, int N, int K, const void* R) {
  constexpr int LDS = NS * (BM + BN) * 128;
  auto kern = gemm_nt_ring_kernel<EPI, BM, BN, WM, WN, NS>;
  static const bool ok = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, LDS) == hipSuccess;
  if (!ok) return 1;
  const int tiles_m = (M + BM - 1) / BM, tiles_n = (N + BN - 1) / BN;
  // columns per store: with 2-byte stores only, 4096 x 2044, K = 64 took 18.2 us against 10.1 of the 8-byte stores of 128 x 128 tiles
  const uintptr_t al = (uintptr_t)C | (uintptr_t)R;
  const int vec = ((N | ldc) & 7) == 0 && (al & 15) == 0 ? 8 : ((N | ldc) & 3) == 0 && (al & 7) == 0 ? 4 : 1;
  kern<<<dim3(tiles_m * tiles_n), 64 * WM * WN, LDS, st>>>((const bf16_t*)A, lda, (const bf16_t*)B, ldb, (bf16_t*)C, ldc, M, N, K, (const bf16_t*)R, tiles_m, tiles_n, vec);
  return 0;
}
// The tiles, with what one K step of 64 was measured to take (ns) when 1, 2, .. workgroups share a compute unit, and the cost of a
// workgroup outside its main loop (launch, first loads, epilogue).  The times come from M = 1003 .. 8192, N = 640 .. 8192, K = 768 .. 32000; the
// model picks the fastest of the five or one within 5 % of it on all of them.
struct RingTile { int bm, bn, per_cu, step[3], over; };
static const RingTile kTiles[] = {
    {64, 64, 3, {330, 440, 560}, 1400},          // 4 waves of 32 x 32, three stages: 48 KB, three workgroups per unit
    {64, 96, 2, {360, 480, 0}, 1600},            // 4 waves of 32 x 48, three stages: 60 KB, two
    {128, 128, 1, {530, 0, 0}, 1600},            // 8 waves of 64 x 32, four stages: 128 KB
    {128, 192, 1, {700, 0, 0}, 1600},            // 8 waves of 64 x 48, three stages: 120 KB (four stages: 2-5 % slower)
    {256, 128, 1, {840, 0, 0}, 1600},            // 8 waves of 64 x 64, three stages: 144 KB
};
// Which tile: a launch lasts as long as the compute units with the most workgroups, so the tile that divides M x N into full
// rounds of 256 units usually wins over the one with the best rate.  us before (128 x 128 tiles, 4 waves of 64 x 64, two stages) / now: 8192 x 768,
// K = 768 21.9 / 16.6, K = 3072 51 / 41, K = 32000 539 / 413 (128 x 192); 3055 x 768, K = 3072 35.9 / 27.0 (64 x 96); 1003 x 768, K = 768 10.4 / 6.3
// (64 x 64); 2048 x 2048, K = 2048 27.7 / 23.3 (128 x 128); 4096 x 2048, K = 2048 41.1 / 36.3 (256 x 128).
static int ring_tile(int M, int N, int K) {
  int best = 0;
  long t_best = -1;
  for (int v = 0; v < 5; ++v) {
    const RingTile& t = kTiles[v];
    const long per_unit = ((long)((M + t.bm - 1) / t.bm) * ((N + t.bn - 1) / t.bn) + 255) / 256;
    const long full = per_unit / t.per_cu, rest = per_unit % t.per_cu, steps = K / 64;
    const long cost = full * (steps * t.step[t.per_cu - 1] + t.over * 13 / 10) + (rest ? steps * t.step[rest - 1] + t.over : 0);
    if (t_best < 0 || cost < t_best) { t_best = cost; best = v; }
  }
  return best;
}

template <int EPI>
static int dispatch_ring(hipStream_t st, const void* A, int lda, const void* B, int ldb, void* C, int ldc, int M, int N, int K, const void* R) {
  switch (ring_tile(M, N, K)) {
    case 0: return launch_ring<EPI, 64, 64, 2, 2, 3>(st, A, lda, B, ldb, C, ldc, M, N, K, R);
    case 1: return launch_ring<EPI, 64, 96, 2, 2, 3>(st, A, lda, B, ldb, C, ldc, M, N, K, R);
    case 2: return launch_ring<EPI, 128, 128, 2, 4, 4>(st, A, lda, B, ldb, C, ldc, M, N, K, R);
    case 3: return launch_ring<EPI, 128, 192, 2, 4, 3>(st, A, lda, B, ldb, C, ldc, M, N, K, R);
    default: return launch_ring<EPI, 256, 128, 4, 2, 3>(st, A, lda, B, ldb, C, ldc, M, N, K, R);
  }
}

// bf16 output, epi = EPI_STORE or EPI_ADD_RES (R with leading dimension ldc).  Returns 0 if launched, 1 if the shape is not
// taken (K % 64, operand rows not 16-byte aligned).
int k_gemm_nt_ring(hipStream_t st, const void* A, int lda, const void* B, int ldb, void* C, int ldc, int M, int N, int K, int epi, const void* R) {
  if (M < 1 || N < 1 || K < 64 || K % 64 || (lda & 7) || (ldb & 7) || (((uintptr_t)A | (uintptr_t)B) & 15)) return 1;
  if (epi == EPI_ADD_RES) return R ? dispatch_ring<EPI_ADD_RES>(st, A, lda, B, ldb, C, ldc, M, N, K, R) : 1;
  return epi == EPI_STORE ? dispatch_ring<EPI_STORE>(st, A, lda, B, ldb, C, ldc, M, N, K, nullptr) : 1;
}

}  // namespace pp
