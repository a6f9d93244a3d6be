// bf16 MFMA GEMM for gfx950, shapes with few 256 x 256 tiles:  C[M x N] = A[M x K] * B[N x K]^T (+ R), both operands K-contiguous.
//
// The 256 x 256-tile kernel (one workgroup per compute unit, 160 KB of LDS) needs well over 256 tiles to fill the chip; the
// 125M-shape decoder (d_model 768, 8192 tokens) has projections with 96.  One kernel template cuts the output into smaller tiles:
// panels of BM and BN rows x 64 K-elements go straight to LDS (global_load_lds, rows of 128 bytes, chunk c of row r at
// c ^ ((r >> 1) & 7): conflict-free fragment reads), NS such stages form a ring.  A stage's slot is filled again (with stage s + NS) as soon as its last fragments
// are in registers.  v_mfma_f32_16x16x32_bf16 with the B panel as row operand; the accumulators are turned
// around through LDS into 16-byte row pieces, the residual is added in fp32 and the sum rounded once.
// What bounds it: a K step of a BM x BN tile is (BM + BN) * 128 bytes to load and BM * BN / 32 cycles of matrix pipe: 64 B per clock and
// compute unit (all that a unit's load path moves) at 128 x 128, 53 at 128 x 192.  Measured at 128 x 192, K = 8192, one workgroup per unit: MFMAs alone 367 ns a step,
// with the fragment reads 480, with the loads 508, with both 635, before they were interleaved one by one (below): the parts added up instead of overlapping.
// Now 8192 x 768, K = 32000 runs at 1.11 PFLOP/s (was 0.99), a 64 x 64 tile's step takes 180 ns (was 285).
#include "pp_kernels.h"
#include "pp_dev.h"

#include <algorithm>
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

// Where a K step's fragments come from (WHOLE):
//   true: all fragments of step s + 1 are read while step s is multiplied (two whole sets of registers).  One wait and one barrier per step with the
//     whole step's MFMAs between a read and its use: what a tile needs whose MFMAs alone are shorter than two trips to LDS (64 x 64: 8 per wave).
//   false: half a step (32 of K) ahead, half the registers, so that 64 x 48 and 64 x 64 per wave fit without spilling.
// In both forms every fragment read and every load stands behind an MFMA of its own.  With a step's loads issued in one go the waves sat in the
// memory pipeline's queue (16 cycles a load, 40 loads a step at 128 x 192) ahead of their own MFMAs, and the compiler waited for the reads of the NEXT half
// step in front of the current one's MFMAs.  us, before / now: 8192 x 768, K = 32000 408 / 361; 2048 x 2048, K = 2048 21.9 / 17.0 (128 x 128); 3055 x 768, K = 3072 25.6 /
// 21.0 (64 x 96 / 128 x 128); 1003 x 768, K = 768 6.2 / 5.3 (64 x 64); 500 x 2048, K = 8192 40.6 / 27.0 (64 x 64, three / four stages).
struct RingFused {          // operands of the fused epilogues (ring_fused below)
  int half;                 // SWIGLU: d_ff; SWIGLU_BWD: columns from a gate to its up; ROPE: half a head
  int rot;                  // ROPE: leading columns that are rotated (q and k)
  int seq;                  // ROPE: sequence length
  bf16_t* act;              // SWIGLU: silu(gate) * up [M x d_ff]
  const float *cosb, *sinb; // ROPE: [seq x half]
};
template <int EPI, int BM, int BN, int WM, int WN, int NS, bool WHOLE, bool TOUCH>
__global__ __launch_bounds__(64 * WM * WN, WHOLE ? 1 : NS == 2 ? 4 : 2) void gemm_nt_ring_kernel(const bf16_t* __restrict__ A, int lda, const bf16_t* __restrict__ B, int ldb,
                                                                         bf16_t* C, int ldc, int M, int N, int K, const bf16_t* R, int tiles_m, int tiles_n, int vec, int touch, RingFused fu) {
  constexpr int NW = WM * WN, TM = BM / WM, TN = BN / WN, MI = TM / 16, NJ = TN / 16, FR = MI + NJ;
  constexpr int STAGE = (BM + BN) * 128, LPW = (BM + BN) / 8 / NW;          // bytes of a stage; wave-loads (8 rows) per wave
  constexpr int PITCH = TN * 4 + 16;                                         // epilogue patch: bytes per row
  static_assert((BM + BN) / 8 % NW == 0 && TM % 16 == 0 && TN % 16 == 0 && MI % 2 == 0 && NW * 32 * PITCH <= NS * STAGE && NS >= 2, "tile geometry");
  extern __shared__ __align__(16) unsigned char r_lds[];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / WN, wn = wave % WN;
  // XCD k = id % 8 owns a contiguous range of the tile list, ordered in groups of 8 M-tiles by all N-tiles
  const int nb = tiles_m * tiles_n, xcd = blockIdx.x & 7;
  const int pid = xcd * (nb >> 3) + min(xcd, nb & 7) + (blockIdx.x >> 3);          // the first nb % 8 XCDs have one tile more
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
    int brow = min(n0 + row - BM, N - 1);
    if constexpr (EPI == EPI_SWIGLU || EPI == EPI_ROPE) {
      // A wave's TN columns are TN / 2 first members and their partners: gate and up of the same hidden units, or the two halves of rotary pairs
      const int br = row - BM, w = br / TN, q = br % TN, pr = n0 / 2 + w * (TN / 2) + q % (TN / 2), second = q / (TN / 2);
      if constexpr (EPI == EPI_SWIGLU) brow = second * N + min(pr, N - 1);
      else if (n0 < fu.rot) brow = pr / fu.half * 2 * fu.half + pr % fu.half + second * fu.half;
    }
    g[i] = row < BM ? A + (size_t)min(m0 + row, M - 1) * lda + c * 8 : B + (size_t)brow * ldb + c * 8;
  }
  auto load1 = [&](int i, int s, int slot) {          // wave-load i of stage s
    __builtin_amdgcn_global_load_lds(PP_R_GPTR(g[i] + (size_t)s * 64), PP_R_LPTR(r_lds + slot * STAGE + wave * 1024 + i * NW * 1024), 16, 0, 0);
  };

  // ---- fragments: lane l reads, for row l % 16 of a 16-row block, the 8 k 8 (l / 16) .. of K32 slice kk; x counts NJ blocks of B, then MI of A
  constexpr int SETS = WHOLE ? 4 : 2;          // sets of one K32 slice each
  const int l16 = lane & 15, lq = lane >> 4, sw = (l16 >> 1) & 7;
  const int fa0 = (wm * TM + l16) * 128, fb0 = (BM + wn * TN + l16) * 128;
  bf16x8 fa[SETS][MI], fb[SETS][NJ];
  auto read1 = [&](int set, const unsigned char* st, int kk, int x) {
    const unsigned char* p = st + (((4 * kk + lq) ^ sw) << 4);
    if (x < NJ) fb[set][x] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4*>(p + fb0 + x * 2048));
    else fa[set][x - NJ] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4*>(p + fa0 + (x - NJ) * 2048));
  };
  f32x4 acc[MI][NJ];
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int j = 0; j < NJ; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  // NM MFMAs (of slices SET, SET + 1, ..) with the NI items of `item` behind them, as early as one per MFMA allows
  auto run = [&](auto SET_, auto NM_, auto NI_, auto item) {
    constexpr int SET = decltype(SET_)::value, NM = decltype(NM_)::value, NI = decltype(NI_)::value, DEN = NI < NM ? NI : NM;
#pragma unroll
    for (int x = 0; x < NM; ++x) {
      const int set = SET + x / (MI * NJ), y = x % (MI * NJ);
      acc[y / NJ][y % NJ] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fb[set][y % NJ], fa[set][y / NJ], acc[y / NJ][y % NJ], 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
      if (x < DEN) {
#pragma unroll
        for (int it = x * NI / DEN; it < (x + 1) * NI / DEN; ++it) item(it);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  };
  auto meet = [&](auto PENDING_) {          // all but this wave's newest loads have landed, its fragment reads too; then everybody's have
    wait_vm_lgkm0<decltype(PENDING_)::value>();
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
  };
  // Stage s + NS is requested into the slot of stage s once that is in everybody's registers: WHOLE, all of it behind the barrier that opens step s; else
  // its first LB loads behind the barrier in the middle of step s, the other LA in the first half of step s + 1.
  constexpr int LB = WHOLE ? LPW : LPW - LPW / 2, LA = LPW - LB;
  typedef std::integral_constant<int, 0> I0;
  typedef std::integral_constant<int, 1> I1;
  typedef std::integral_constant<int, (NS - 2) * LPW> Steady;
#pragma unroll
  for (int s = 0; s < NS; ++s)
    if (s < ns) {
#pragma unroll
      for (int i = 0; i < (s == NS - 1 ? LB : LPW); ++i) load1(i, s, s);
    }
  // B in the order it lies in memory: the first `touch` * (threads of the grid) of its 128-byte pieces, one word each, on their way into the caches while the
  // first stages arrive.  A step asks for 128 bytes of every row of B at once, K elements apart, and where B comes from HBM (a weight that the pass uses
  // once) those lie in few channels: 3055 x 768 with a B out of cache took 27.5 us at K = 3072 and 51.8 at K = 6144, with the words 22.7 and 41.2.
  uint32_t word[4] = {0, 0, 0, 0};
  if constexpr (TOUCH) {
    const uint32_t per_row = K / 64, last = (uint32_t)N * per_row - 1;
#pragma unroll
    for (int q = 0; q < 4; ++q)
      if (q < touch) {
        const uint32_t id = min((q * gridDim.x + blockIdx.x) * (64u * NW) + tid, last), row = id / per_row;
        word[q] = *reinterpret_cast<const uint32_t*>(B + (size_t)row * ldb + (id - row * per_row) * 64);
      }
    __builtin_amdgcn_sched_barrier(0);
  }
  if (ns >= NS) meet(std::integral_constant<int, (NS - 2) * LPW + LB>{});
  else if (NS > 3 && ns == 3) meet(std::integral_constant<int, 2 * LPW>{});
  else if (ns == 2) meet(std::integral_constant<int, LPW>{});
  else meet(I0{});
#pragma unroll
  for (int x = 0; x < (WHOLE ? 2 : 1) * FR; ++x) read1(x / FR, r_lds, x / FR, x % FR);
  int slot = 0, prev = NS - 1, s = 0;
  if constexpr (WHOLE) {
    // the step of fragment sets BUF, BUF + 1; RD: the other two sets take stage s + 1
    auto step = [&](auto BUF_, auto RD_, auto LD_) {
      constexpr int BUF = decltype(BUF_)::value, NR = decltype(RD_)::value * 2 * FR, LD = decltype(LD_)::value;
      const int nxt = slot + 1 == NS ? 0 : slot + 1;
      const unsigned char* st = r_lds + nxt * STAGE;
      run(BUF_, std::integral_constant<int, 2 * MI * NJ>{}, std::integral_constant<int, NR + LD * LPW>{},
          [&](int it) { if (it < NR) read1(2 - BUF + it / FR, st, it / FR, it % FR); else load1(it - NR, s + NS, slot); });
      slot = nxt; ++s;
    };
    typedef std::integral_constant<int, 2> I2;
    while (s + 1 + NS < ns) {
      meet(Steady{}); step(I0{}, I1{}, I1{});
      meet(Steady{}); step(I2{}, I1{}, I1{});
    }
    auto tail = [&](auto BUF_) {          // at most NS + 1 steps
      const bool ld = s + NS < ns;
      if (s + NS <= ns) meet(Steady{});
      else if (NS >= 4 && s + NS - 1 <= ns) meet(std::integral_constant<int, (NS >= 4 ? NS - 3 : 0) * LPW>{});
      else meet(I0{});
      if (ld) step(BUF_, I1{}, I1{});
      else if (s + 1 < ns) step(BUF_, I1{}, I0{});
      else step(BUF_, I0{}, I0{});
    };
    for (;;) {
      tail(I0{});
      if (s == ns) break;
      tail(I2{});
      if (s == ns) break;
    }
  } else {
    auto half = [&](auto BUF_, auto RD_, auto LD_, int rslot, int ls, int lslot) {          // slice BUF of step s; RD: the other set takes the slice behind it
      constexpr int BUF = decltype(BUF_)::value, NR = decltype(RD_)::value * FR, NLD = decltype(LD_)::value ? (BUF ? LB : LA) : 0;
      const unsigned char* st = r_lds + rslot * STAGE;
      __builtin_amdgcn_s_waitcnt(0xC07F);          // lgkmcnt(0): this slice's fragments (the only reads in flight)
      __builtin_amdgcn_sched_barrier(0);
      run(BUF_, std::integral_constant<int, MI * NJ>{}, std::integral_constant<int, NR + NLD>{},
          [&](int it) { if (it < NR) read1(1 - BUF, st, 1 - BUF, it); else load1((BUF ? 0 : LB) + it - NR, ls, lslot); });
    };
    auto step = [&](auto RD_, auto LDA_, auto LDB_, auto PENDING_) {          // RD: there is a step s + 1
      const int nxt = slot + 1 == NS ? 0 : slot + 1;
      half(I0{}, I1{}, LDA_, slot, s + NS - 1, prev);
      meet(PENDING_);
      half(I1{}, RD_, LDB_, nxt, s + NS, slot);
      prev = slot; slot = nxt; ++s;
    };
    while (s < ns - NS) step(I1{}, I1{}, I1{}, Steady{});
    if (ns >= NS) step(I1{}, I1{}, I0{}, Steady{});          // s = ns - NS: the other loads of the last stage
    if (NS > 3 && s + 3 == ns) step(I1{}, I0{}, I0{}, std::integral_constant<int, LPW>{});
    while (s < ns - 1) step(I1{}, I0{}, I0{}, I0{});
    step(I0{}, I0{}, I0{}, I0{});
  }

  if constexpr (TOUCH) asm volatile("" ::"v"(word[0]), "v"(word[1]), "v"(word[2]), "v"(word[3]));          // loaded for their lines only

  // ---- epilogue: nothing is in flight and nobody reads the stages any more (the last barrier).  Element r of block (i, j) is row
  // 16 i + l % 16, column 16 j + 4 (l / 16) + r of the wave's TM x TN part; it is turned around in a private patch.
  // 32 rows at a time
  unsigned char* patch = r_lds + wave * 32 * PITCH;
  constexpr int PR = TN / 8, NP = 32 * PR / 64;          // 8-column pieces per row, pieces per lane and pass
  static_assert(32 * PR % 64 == 0, "pieces");
#pragma unroll
  for (int p = 0; p < MI / 2; ++p) {
    [[maybe_unused]] uint4 gate[NP], up[NP];          // SWIGLU_BWD: requested ahead of the patch's round trip, from clamped addresses
    if constexpr (EPI == EPI_SWIGLU_BWD) {
#pragma unroll
      for (int it = 0; it < NP; ++it) {
        const int idx = it * 64 + lane;
        const bf16_t* r = R + (size_t)min(m0 + wm * TM + p * 32 + idx / PR, M - 1) * ldc + min(n0 + wn * TN + idx % PR * 8, N - 8);
        gate[it] = *reinterpret_cast<const uint4*>(r);
        up[it] = *reinterpret_cast<const uint4*>(r + fu.half);
      }
    }
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < NJ; ++j)
        *reinterpret_cast<float4*>(patch + (i * 16 + l16) * PITCH + j * 64 + lq * 16) = make_float4(acc[2 * p + i][j][0], acc[2 * p + i][j][1], acc[2 * p + i][j][2], acc[2 * p + i][j][3]);
    if constexpr (EPI == EPI_SWIGLU || EPI == EPI_ROPE) {
      if (EPI == EPI_SWIGLU || n0 < fu.rot) {          // pairs: 8 first members and their partners TN / 2 columns further on
        constexpr int HP = TN / 16;
#pragma unroll
        for (int it = 0; it < (32 * HP + 63) / 64; ++it) {
          const int idx = it * 64 + lane, row = idx / HP, c = idx % HP;
          const int grow = m0 + wm * TM + p * 32 + row, pr = n0 / 2 + wn * (TN / 2) + c * 8;
          if (idx >= 32 * HP || grow >= M) continue;
          float x[8], y[8];
          load8(reinterpret_cast<const float*>(patch + row * PITCH + c * 32), x);
          load8(reinterpret_cast<const float*>(patch + row * PITCH + TN * 2 + c * 32), y);
          bf16_t* out = C + (size_t)grow * ldc;
          if constexpr (EPI == EPI_SWIGLU) {
            if (pr >= N) continue;
            store8(out + pr, x);
            store8(out + N + pr, y);
            float a[8];          // from the rounded values, as a pass over the stored matrix would form it
#pragma unroll
            for (int e = 0; e < 8; ++e) a[e] = silu_mul(bf16_to_f32(f32_to_bf16(x[e])), bf16_to_f32(f32_to_bf16(y[e])));
            store8(fu.act + (size_t)grow * N + pr, a);
          } else {
            const int head = pr / fu.half, i = pr - head * fu.half;
            const size_t at = (size_t)(grow % fu.seq) * fu.half + i;
            float cs[8], sn[8], a[8], b[8];
            load8(fu.cosb + at, cs);
            load8(fu.sinb + at, sn);
#pragma unroll
            for (int e = 0; e < 8; ++e) { a[e] = fmaf(x[e], cs[e], -(y[e] * sn[e])); b[e] = fmaf(y[e], cs[e], x[e] * sn[e]); }          // as the big-tile kernel rounds them
            store8(out + head * 2 * fu.half + i, a);
            store8(out + head * 2 * fu.half + i + fu.half, b);
          }
        }
        continue;
      }
    }
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
        if constexpr (VEC == 8 && EPI == EPI_SWIGLU_BWD) {          // the product is dL/da: dg and du go to the places of gate and up
          float dg[8], du[8];
          const uint32_t gw[4] = {gate[it].x, gate[it].y, gate[it].z, gate[it].w}, uw[4] = {up[it].x, up[it].y, up[it].z, up[it].w};
#pragma unroll
          for (int e = 0; e < 8; ++e) {
            const float gg = (e & 1) ? __uint_as_float(gw[e >> 1] & 0xffff0000u) : __uint_as_float(gw[e >> 1] << 16);
            const float uu = (e & 1) ? __uint_as_float(uw[e >> 1] & 0xffff0000u) : __uint_as_float(uw[e >> 1] << 16);
            const float sg = sigmoid_fast(gg);
            du[e] = v[e] * gg * sg;
            dg[e] = v[e] * uu * sg * (1.0f + gg * (1.0f - sg));
          }
          store8(C + off, dg);
          store8(C + off + fu.half, du);
        } else if constexpr (VEC == 8) {
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
    if constexpr (EPI == EPI_SWIGLU || EPI == EPI_SWIGLU_BWD || EPI == EPI_ROPE) store(std::integral_constant<int, 8>{});          // whole aligned groups of 8 only
    else if (vec == 8) store(std::integral_constant<int, 8>{});
    else if (vec == 4) store(std::integral_constant<int, 4>{});
    else store(std::integral_constant<int, 1>{});
  }
}

template <int EPI, int BM, int BN, int WM, int WN, int NS, bool WHOLE, bool TOUCH = false>
static int launch_ring(hipStream_t st, const void* A, int lda, const void* B, int ldb, void* C, int ldc, int M, int N, int K, const void* R) {
  constexpr int LDS = NS * (BM + BN) * 128;
  auto kern = gemm_nt_ring_kernel<EPI, BM, BN, WM, WN, NS, WHOLE, TOUCH>;
  static const bool ok = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, LDS) == hipSuccess;
  if (!ok) return 1;
  const int tiles_m = (M + BM - 1) / BM, tiles_n = (N + BN - 1) / BN;
  // columns per store: with 2-byte stores only, 4096 x 2044, K = 64 took 18.2 us against 10.1 of the 8-byte stores of 128 x 128 tiles
  const uintptr_t al = (uintptr_t)C | (uintptr_t)R;
  const int vec = ((N | ldc) & 7) == 0 && (al & 15) == 0 ? 8 : ((N | ldc) & 3) == 0 && (al & 7) == 0 ? 4 : 1;
  const long threads = (long)tiles_m * tiles_n * 64 * WM * WN, pieces = (long)N * (K / 64);
  const int touch = TOUCH ? (int)std::min(4l, (pieces + threads - 1) / threads) : 0;          // words of B per thread
  kern<<<dim3(tiles_m * tiles_n), 64 * WM * WN, LDS, st>>>((const bf16_t*)A, lda, (const bf16_t*)B, ldb, (bf16_t*)C, ldc, M, N, K, (const bf16_t*)R, tiles_m, tiles_n, vec, touch, RingFused{});
  return 0;
}
// The tiles, with what was measured of each (ns): one K step of 64 when 1, 2, .. workgroups share a compute unit and every unit has one; the part of
// that by which it is shorter on a nearly idle chip (%); a workgroup outside its main loop (first loads, epilogue) in a last round of fewer workgroups per unit
// and in a full one.  Fitted to 170 shapes, M = 32 .. 16384, N = 64 .. 16384, K = 64 .. 32000, with A in cache and B (the weight) out of it; over those the tile that
// the model picks takes 2 % longer than the best one on average.
struct RingTile { int bm, bn, per_cu, step[3], idle, over, over_full; };
static constexpr RingTile kTiles[] = {
    {32, 64, 3, {205, 271, 414}, 26, 1668, 1243},         // 2 waves of 32 x 32, four stages: 48 KB, three workgroups per unit
    {64, 64, 2, {216, 371, 0}, 19, 1724, 1483},           // 4 waves of 32 x 32, four stages: 64 KB, two
    {64, 96, 2, {286, 456, 0}, 25, 1737, 1956},           // 4 waves of 32 x 48, four stages: 80 KB, two
    {64, 128, 1, {316, 0, 0}, 20, 0, 1604},               // 8 waves of 32 x 32, four stages: 96 KB
    {64, 192, 1, {426, 0, 0}, 35, 0, 1849},               // 8 waves of 32 x 48, four stages: 128 KB
    {128, 128, 1, {493, 0, 0}, 42, 0, 1952},              // 8 waves of 64 x 32, four stages: 128 KB
    {128, 192, 1, {682, 0, 0}, 55, 0, 2446},              // 8 waves of 64 x 48, three stages: 120 KB
    {128, 256, 1, {874, 0, 0}, 56, 0, 2732},              // 8 waves of 64 x 64, three stages: 144 KB
};
// Which tile: a launch lasts as long as the compute units with the most workgroups, so the tile that divides M x N into full
// rounds of 256 units usually wins over the one with the best rate.  Unrolled over the table, so that nothing is divided at run time (this runs for
// every call; as a loop over the table it took 0.2 of the 4 us that a call takes on the host).
template <int V = 0>
static int ring_tile(unsigned M, unsigned N, unsigned steps, int best = 0, long best_cost = 0x7fffffffffffffffl) {
  if constexpr (V < (int)(sizeof(kTiles) / sizeof(kTiles[0]))) {
    constexpr RingTile t = kTiles[V];
    const unsigned tiles = (M + t.bm - 1) / t.bm * ((N + t.bn - 1) / t.bn), per_unit = (tiles + 255) / 256;
    const unsigned full = per_unit / t.per_cu, rest = per_unit % t.per_cu;
    const long step = (long)steps * (tiles >= 256 ? 25600 : 25600 - t.idle * (256 - tiles));          // in 1 / 25600
    const long cost = (long)full * (step * t.step[t.per_cu - 1] / 25600 + t.over_full) + (rest ? step * t.step[rest - 1] / 25600 + t.over : 0);
    return cost < best_cost ? ring_tile<V + 1>(M, N, steps, V, cost) : ring_tile<V + 1>(M, N, steps, best, best_cost);
  }
  return best;
}

int gemm_ring_tile(int M, int N, int K) { return ring_tile(M, N, K / 64); }

// B is touched ahead from K = 2048 on, by the tiles of one workgroup per unit: below that it costs what it saves (3055 x 768, K = 768: 8.3 us without, 8.5 with; its
// code alone 0.5 of the 4.3 us of a K of 64), and the tiles of several workgroups per unit, which are at different K already, lose as often as they gain (3055 x 768 in
// 64 x 96 tiles, K = 3072: 24.7 / 27.8).
template <int EPI, int BM, int BN, int NS>
static int launch_half(hipStream_t st, const void* A, int lda, const void* B, int ldb, void* C, int ldc, int M, int N, int K, const void* R) {
  if (K >= 2048 && (long)N * (K / 64) < (1l << 31)) return launch_ring<EPI, BM, BN, 2, 4, NS, false, true>(st, A, lda, B, ldb, C, ldc, M, N, K, R);
  return launch_ring<EPI, BM, BN, 2, 4, NS, false>(st, A, lda, B, ldb, C, ldc, M, N, K, R);
}

template <int EPI>
static int dispatch_ring(hipStream_t st, const void* A, int lda, const void* B, int ldb, void* C, int ldc, int M, int N, int K, const void* R) {
  switch (ring_tile(M, N, K / 64)) {
    case 0: return launch_ring<EPI, 32, 64, 1, 2, 4, true>(st, A, lda, B, ldb, C, ldc, M, N, K, R);
    case 1: return launch_ring<EPI, 64, 64, 2, 2, 4, true>(st, A, lda, B, ldb, C, ldc, M, N, K, R);
    case 2: return launch_ring<EPI, 64, 96, 2, 2, 4, true>(st, A, lda, B, ldb, C, ldc, M, N, K, R);
    case 3: return launch_half<EPI, 64, 128, 4>(st, A, lda, B, ldb, C, ldc, M, N, K, R);
    case 4: return launch_half<EPI, 64, 192, 4>(st, A, lda, B, ldb, C, ldc, M, N, K, R);
    case 5: return launch_half<EPI, 128, 128, 4>(st, A, lda, B, ldb, C, ldc, M, N, K, R);
    case 6: return launch_half<EPI, 128, 192, 3>(st, A, lda, B, ldb, C, ldc, M, N, K, R);
    default: return launch_half<EPI, 128, 256, 3>(st, A, lda, B, ldb, C, ldc, M, N, K, R);
  }
}

// The SwiGLU and rotary GEMMs on 128 x 192 tiles, two stages, two workgroups per unit (80 KB, 128 registers a wave): the bytes of one's epilogue move behind the other's
// MFMAs.  The same bits as the big-tile kernel's.
template <int EPI>
static int launch_fused(hipStream_t st, const void* A, int lda, const void* B, int ldb, void* C, int ldc, int M, int N, int K, const void* R, int tiles_n, const RingFused& fu) {
  constexpr int LDS = 2 * (128 + 192) * 128;
  auto kern = gemm_nt_ring_kernel<EPI, 128, 192, 2, 4, 2, false, false>;
  static const bool ok = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, LDS) == hipSuccess;
  if (!ok) return 1;
  const int tiles_m = (M + 127) / 128;
  kern<<<dim3(tiles_m * tiles_n), 512, LDS, st>>>((const bf16_t*)A, lda, (const bf16_t*)B, ldb, (bf16_t*)C, ldc, M, N, K, (const bf16_t*)R, tiles_m, tiles_n, 8, 0, fu);
  return 0;
}
int k_gemm_swiglu_fwd_ring(hipStream_t st, const void* X, int ldx, const void* Wgu, int ldw, void* gu, void* a, int M, int F, int K) {
  return launch_fused<EPI_SWIGLU>(st, X, ldx, Wgu, ldw, gu, 2 * F, M, F, K, nullptr, (F + 95) / 96, RingFused{F, 0, 0, (bf16_t*)a, nullptr, nullptr});
}
int k_gemm_swiglu_bwd_ring(hipStream_t st, const void* G, int ldg, const void* Wd_rows, int ldw, const void* gu_c0, void* dgu_c0, int ld2f, int half, int M, int N, int K) {
  return launch_fused<EPI_SWIGLU_BWD>(st, G, ldg, Wd_rows, ldw, dgu_c0, ld2f, M, N, K, gu_c0, (N + 191) / 192, RingFused{half, 0, 0, nullptr, nullptr, nullptr});
}
int k_gemm_qkv_rope_ring(hipStream_t st, const void* X, int ldx, const void* Wqkv, int ldw, void* qkv, int M, int d, int dh, int K, int S, const float* rope_cos, const float* rope_sin) {
  if (d % 192) return 1;          // a tile is all rotated pairs or none, and no row block is cut
  return launch_fused<EPI_ROPE>(st, X, ldx, Wqkv, ldw, qkv, 3 * d, M, 3 * d, K, nullptr, 3 * d / 192, RingFused{dh / 2, 2 * d, S, nullptr, rope_cos, rope_sin});
}

// bf16 output, epi = EPI_STORE or EPI_ADD_RES (R with leading dimension ldc).  Returns 0 if launched, 1 if the shape is not
// taken (K % 64, operand rows not 16-byte aligned).
int k_gemm_nt_ring(hipStream_t st, const void* A, int lda, const void* B, int ldb, void* C, int ldc, int M, int N, int K, int epi, const void* R) {
  if (M < 1 || N < 1 || K < 64 || K % 64 || (lda & 7) || (ldb & 7) || (((uintptr_t)A | (uintptr_t)B) & 15)) return 1;
  if (epi == EPI_ADD_RES) return R ? dispatch_ring<EPI_ADD_RES>(st, A, lda, B, ldb, C, ldc, M, N, K, R) : 1;
  return epi == EPI_STORE ? dispatch_ring<EPI_STORE>(st, A, lda, B, ldb, C, ldc, M, N, K, nullptr) : 1;
}

}  // namespace pp
