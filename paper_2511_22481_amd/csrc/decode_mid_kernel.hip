// gfx950 kernel for sparse MLA decode, 64 head rows to a work group, bf16 or fp8 cache.
// (Paper section 3.2.1: softmax(q K_M^T * scale) V_M with M = sinks + recents.)
//
// Eight waves in two roles, one of each on every SIMD:
//   waves 0 .. 3  S^T and the softmax: wave (th, hg) has the query of 32 heads in registers (144) and computes the logits
//                 of one half of a tile's tokens; the weights go to LDS in the operand order of PV;
//   waves 4 .. 7  the direct global->LDS loads and PV: output columns 128 w .. of all 64 heads (128 accumulators).
// A lone wave per SIMD issues a vector instruction every 4.7 cycles whatever the matrix pipe does, and waits out the
// latency of each dependent one; two waves that do not depend on each other within a step fill those gaps, so the
// matrix instructions are builtins and only their place relative to the softmax is pinned.  A step (one barrier):
//   S^T of tile it + 2 and, behind its matrix instructions, the weights of tile it + 1 | PV of tile it, V of tile it + 1 to
//   registers, tile it + 4 requested.
// Four stages of 36,864 bytes (32 bf16 or 64 fp8 tokens): two are read in a step, two in flight.
// Softmax reference (fixed per segment, second run if a logit leaves its range), masking and partial rows are those of
// decode_kernel, and for a bf16 cache so are the weights (bf16).
//
// fp8 cache: its bytes go to the 8-bit matrix instruction as they are.
//   Query   in two e4m3 terms, q = 2^e (hi + lo / 16), row maximum scaled into [128, 256): a bf16 significand is two e4m3
//           ones long, so elements not below 2^-14 of the row's maximum are exact.  The 1/16 is the block scale of the
//           second product (it keeps lo out of the subnormals).
//   Logits  raw product times the token's scale in fp32.
//   Weights 2^(logit - reference - kk) x token scale, rounded to e4m3, with one power-of-two exponent kk per head and 32
//           tokens, which is the block scale of PV: V is read raw.  Byte 0 of lane (column n, g)'s scale word applies to
//           contraction indices 32 g .. + 31.  kk comes from the largest logit and a bound on the scales: all weights are
//           below 2^8, and the one of the largest logit is above 2^6 if its token's scale is within a factor of two of the
//           bound.  Each halving of that scale costs the other weights one of the 14 binades [2^-6, 2^8) in which e4m3
//           rounds by at most 2^-4; with a scale 2^-10 of the bound the largest lies above 2^-3.
//   Sums    the rows are normalised by the sum of the rounded weights (each over its token's scale), lse uses the exact one.
//           A token scale far below its half's largest is raised to 2^-10 of it for the weight, or the weight would vanish
//           from the rounded sum while its softmax weight counts in full.
// The 8-bit matrix instruction aligns the products of 64 dims to the largest before it adds, so what lies 2^-15 .. 2^-18
// below that is lost; each 64 dims by themselves.
//
// Cycles per tile in the long loop (counters, 60 and 64 tiles' difference): bf16 1,743, its matrix instructions 1,088, LDS
// operands 816 (288 of them bank conflicts) beside the 36 KB that the direct loads write; fp8 2,220, 1,664 and 800 (32); the
// vector instructions of the softmax waves take most of the rest.  (fp8 with one wave per SIMD and all of it in one
// hand-written stream: 3,140.)  Wave priorities change nothing.
// Where a step goes (cycle counter in both roles): bf16 1,030 cycles of work in the softmax waves, in the others 630 until the
// requests are issued, 780 of PV, 60 in the wait for a tile and 250 at the barrier; fp8 2,020, 570, 1,330, 60 and the rest at the
// barrier.  Start and end of a segment: 21 K cycles bf16, 26 K fp8.  The order as it is beats what that suggests.  us against it: requests between the products of PV 1 to 4 % more, by two of the
// four waves behind them 2 to 8 %; half of PV's products, or all from registers, left for the next step's start (where both
// roles wait for LDS) 3 to 7 %; V read two tiles ahead, for a stage freed earlier and three tiles in flight, 2 to 4 %.
// us per decode, before -> now: fp8, 128 rows: 32 sequences of 8320 tokens 75 -> 67, 93 mixed 127 -> 116 (94 where the
// planner leaves sequences whole), 64 of 32768 477 -> 413, 500 of up to 200 tokens 82 -> 73; bf16, 128 rows (two groups,
// one decode_kernel before): 64 of 2176 58 -> 53.5, two queries each 92 -> 81; 32 of 4096 55 -> 51; 64 rows: 128 of 2176
// 88 -> 66.  The same with input sets in turn, 1.2 GB together (58.7 -> 52.3, 56.6 -> 50.6, 84 -> 64).
// A shorter start and end of a segment since (split_q, the query's read, LAST in step, write_rows), one box: fp8, 32 of 8320 tokens 65.5 -> 62.3,
// 93 mixed 93.5 -> 92.5, ring step of 40 sequences 38.4 -> 34.5; bf16, 64 of 2176 51.7 -> 50.5, two queries each 88.7 -> 87.2, 32 of 4096 49.9 -> 48.8.
// Two groups to a block where every row has just been written by another kernel, which leaves them in the last-level cache:
// 32 of 4096 read 230 MB instead of 162, the second group's tiles are no longer in L2 when it asks for them; 57 -> 66 us,
// 64 of 2176 59 -> 71, 128 of 4096 148 -> 207 (32 of 2176 42 -> 41, 256 rows 91 -> 85).  Reading the rows without `nt` ends that
// (main kernel 57 -> 49 us) and costs everything else 3 to 15 % (64 rows, 256 of 2176: 108 -> 124 us); `nt` for one of the groups, or
// the second group started 1 us later, does no better.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>
#include <utility>

#include "decode_common.h"

namespace omniattn {

namespace {

constexpr int kHB = kHeadBlockMid;  // 64
constexpr int kStagesM = 4;
constexpr int kStageM = 36864;
constexpr int kTailBaseM = 32768;
constexpr int kWavesM = 8;               // 4 for S^T and the softmax, 4 for the loads and PV
constexpr int kRoleWaves = 4;
constexpr int kPRowM = 64;               // a head's weights of one tile
constexpr int kPBytesM = kHB * kPRowM;
constexpr int kStatM = 2 * kHB;          // (token half, head)
constexpr int kScaleM = kTileFp8 * 4;
// stages | weights of two tiles | largest logits of tile 0 and of all | sums, rounded sums, references; in the loop (fp8)
// the waves' weight scales and their reciprocals | tile table | fp8: block exponents of two tiles (bytes) | token scales
constexpr int kOffPM = kStagesM * kStageM;
constexpr int kOffMaxM = kOffPM + 2 * kPBytesM;
constexpr int kOffStatM = kOffMaxM + kStatM * 4;
constexpr int kOffTilesM = kOffStatM + kRoleWaves * 2 * kScaleM;
constexpr int kOffKKM = kOffTilesM + kMaxSegTiles * 4;
constexpr int kOffScalesM = kOffKKM + 2 * kStatM;
constexpr int kLdsMidBf16 = kOffKKM;
constexpr int kLdsMidFp8 = kOffScalesM + kStagesM * kScaleM;
static_assert(3 * kStatM * 4 <= kRoleWaves * 2 * kScaleM && kLdsMidFp8 <= 160 * 1024, "LDS of one compute unit");

constexpr float kRefSlackM = 64.f;  // see the kernel for blocks of 128 rows: fixed softmax reference with retry

// LDS layout of a stage: the value part of the rows, then their rope parts; 16-byte chunks XORed with a
// function of the row, as in the other kernels.
template <bool FP8>
struct LayM;
template <>
struct LayM<false> {
  static constexpr int kTok = kTile, kMain = 1024, kTail = 128, kRow = 1152, kDma = 9;
  __host__ __device__ static constexpr int sw_main(int r) { return ((r & 3) << 2) | ((r >> 2) & 3); }
  __host__ __device__ static constexpr int sw_tail(int r) { return (r >> 1) & 7; }
};
template <>
struct LayM<true> {
  static constexpr int kTok = kTileFp8, kMain = 512, kTail = 64, kRow = 576, kDma = 10;
  __host__ __device__ static constexpr int sw_main(int r) { return ((r & 3) << 1) | ((r >> 2) & 1) | (((r >> 3) & 1) << 3); }
  __host__ __device__ static constexpr int sw_tail(int r) { return (r >> 2) & 3; }
};
// weights: chunks of 16 bytes of a head's row, so that four rows of 64 bytes and the next four differ in bank
__device__ __forceinline__ uint32_t p_chunk(int head, int c) { return head * kPRowM + ((c ^ ((head >> 2) & 3)) << 4); }

__device__ __forceinline__ float half_max(float x) {  // with lane ^ 32
  float a = x, b = x;
  swap32(a, b);
  return fmaxf(a, b);
}
__device__ __forceinline__ float half_sum(float x) {
  float a = x, b = x;
  swap32(a, b);
  return a + b;
}
__device__ __forceinline__ float row_max(float x) {  // with lane ^ 16
  float a = x, b = x;
  swap16(a, b);
  return fmaxf(a, b);
}
__device__ __forceinline__ float row_sum(float x) {
  float a = x, b = x;
  swap16(a, b);
  return a + b;
}

// A segment and what both roles derive from it.
template <bool FP8>
struct SegM {
  using Y = LayM<FP8>;
  int b, tile_lo, n_tiles, slot, L, h0, L0, sink_end, S, W, Wu;
  TileLayout tl;
  __device__ __forceinline__ int pos(int it) const { return tl.logical(tile_lo + it) * Y::kTok; }
  __device__ __forceinline__ bool full(int pos0) const {
    return (pos0 + Y::kTok <= sink_end) || (pos0 >= L - W && pos0 + Y::kTok <= L0);
  }
};

}  // namespace

template <bool FP8>
__global__ __launch_bounds__(kWavesM * 64, 2) void decode_mid_kernel(DecodeParams p) {
  using Y = LayM<FP8>;
  using QY = LayM<false>;
  constexpr int kT = Y::kTok, kDma = Y::kDma;
  extern __shared__ __attribute__((aligned(16))) uint8_t lds_raw[];
  const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint8_t*)lds_raw;
  const uint32_t lds_p = lds0 + kOffPM, lds_max = lds0 + kOffMaxM, lds_stat = lds0 + kOffStatM;
  const uint32_t lds_tiles = lds0 + kOffTilesM, lds_kk = lds0 + kOffKKM, lds_scales = lds0 + kOffScalesM;
  const int tid = threadIdx.x;
  // Per-lane values are derived anew in each phase of a segment from a lane id that went through an
  // opaque move: computed once they would all stay alive across the loops, which have no registers for them.
  auto fresh_lane = [&]() {
    int l = tid & 63;
    asm volatile("" : "+v"(l));
    return l;
  };
  const int wave8 = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wave = wave8 & (kRoleWaves - 1);  // within the role

  // A unit's rows are p.head_block (64 or 128): one work group or two, on one XCD, as both read the same tiles.
  const int groups = p.head_block / kHB;
  const int per_xcd = (p.n_units + p.xcds - 1) / p.xcds * groups;
  const int group = ((int)blockIdx.x % p.xcds) * per_xcd + (int)blockIdx.x / p.xcds;
  const int unit = groups == 2 ? group >> 1 : group, half = groups == 2 ? group & 1 : 0;
  if (unit >= p.n_units) return;
  auto uniform4 = [](u32x4 v) {
    return u32x4{(uint32_t)__builtin_amdgcn_readfirstlane(v.x), (uint32_t)__builtin_amdgcn_readfirstlane(v.y),
                 (uint32_t)__builtin_amdgcn_readfirstlane(v.z), (uint32_t)__builtin_amdgcn_readfirstlane(v.w)};
  };
  const u32x4* hdr = (const u32x4*)(p.units + unit);
  const u32x4 hdr0 = hdr[0], hdr1 = hdr[1], hdr2 = hdr[2];
  const int seg_lo = __builtin_amdgcn_readfirstlane(hdr0.x), seg_hi = __builtin_amdgcn_readfirstlane(hdr0.y);

  auto stage_base = [&](int it) -> uint32_t { return lds0 + ((uint32_t)it & (kStagesM - 1)) * kStageM; };
  auto tile_entry = [&](int it) { return *LDS_PTR(uint32_t, lds_tiles + it * 4); };
  auto stat = [&](int k, int th, int h) { return *LDS_PTR(float, lds_stat + (k * kStatM + th * kHB + h) * 4); };

  // Reads segment si, writes its tile table (unit of the cache that holds the tile, bit 0 = every position kept) and
  // requests the block's 64 query rows, which pass through stages 2 and 3 (8 rows, kQLoads requests to a wave).
  // Returns false for a block that the last head does not reach (a second half).
  constexpr int kQLoads = 9;
  auto begin_segment = [&](int si, SegM<FP8>& sg) -> bool {
    u32x4 a = hdr1, c = hdr2;
    if (si != seg_lo) {
      const u32x4* sp = (const u32x4*)(p.segs + si);
      a = sp[0];
      c = sp[1];
    }
    a = uniform4(a);
    c = uniform4(c);
    sg.b = a.x;
    sg.h0 = (int)a.y * p.head_block + half * kHB;
    if (sg.h0 >= p.H) return false;
    sg.tile_lo = a.z;
    sg.n_tiles = (int)a.w - (int)a.z;
    sg.slot = c.x;
    sg.L = c.z;
    sg.S = p.S;
    sg.W = p.W;
    sg.Wu = p.Wu;
    sg.tl = tile_layout(sg.L, p.S, p.Wu, kT);
    sg.L0 = sg.L - (p.T - 1);
    sg.sink_end = p.S < sg.L0 ? p.S : sg.L0;
    const int n = sg.n_tiles;
    if (n == 0) return true;
    const int lane = fresh_lane(), tid_s = wave8 * 64 + lane;
    // The page-table entries go straight to the tile table and the query's rows right behind them, so that both round
    // trips run together; then each thread turns its own entries into the table's.  (Q landed 7,900 -> 5,200 cycles after
    // the kernel's start, the first S^T 14,800 -> 10,400, fp8 22,700 -> 17,700, with tiles 1 .. 3 requested behind the barriers.)
    constexpr int kTabPerThread = kMaxSegTiles / (kWavesM * 64);
    const uint8_t* pt_row = (const uint8_t*)(p.page_table + (size_t)sg.b * p.max_pages);
#pragma unroll
    for (int u = 0; u < kTabPerThread; ++u) {
      const int t = tid_s + u * kWavesM * 64;
      if (u * kWavesM * 64 + wave8 * 64 < n)
        load_lds4(lds_tiles + (u * kWavesM * 64 + wave8 * 64) * 4, pt_row, (uint32_t)(sg.pos(t < n ? t : n - 1) >> 7) << 2);
    }
    const uint8_t* qbase = (const uint8_t*)p.q + (size_t)sg.b * p.H * QY::kRow;
    auto q_head = [&](int r) -> uint32_t { return sg.h0 + r < p.H ? sg.h0 + r : p.H - 1; };
    const uint32_t lds_q = lds0 + (2 + (wave8 >> 2)) * kStageM;
    const int r0 = 8 * (wave8 & 3);  // the wave's rows within the stage's 32
#pragma unroll
    for (int k = 0; k < 8; ++k)
      load_lds16<false>(lds_q + (r0 + k) * QY::kMain, qbase, q_head(8 * wave8 + k) * QY::kRow + ((lane ^ QY::sw_main(r0 + k)) << 4));
    const int r = r0 + (lane >> 3);
    load_lds16<false>(lds_q + kTailBaseM + r0 * QY::kTail, qbase,
                      q_head(8 * wave8 + (lane >> 3)) * QY::kRow + QY::kMain + (((lane & 7) ^ QY::sw_tail(r)) << 4));
    wait_vm<kQLoads>();
#pragma unroll
    for (int u = 0; u < kTabPerThread; ++u) {
      const int t = tid_s + u * kWavesM * 64;
      if (t < n) {
        const int pos0 = sg.pos(t);
        const uint32_t page = *LDS_PTR(uint32_t, lds_tiles + t * 4);
        *LDS_PTR(uint32_t, lds_tiles + t * 4) = (page * (kPage / kT) + ((pos0 / kT) & (kPage / kT - 1))) << 1 | (uint32_t)sg.full(pos0);
      }
    }
    __syncthreads();
    return true;
  };
  // fp8: the query rows that the wave has fetched, in two e4m3 terms.  In place: 16 bytes that held 8 dims hold their high, then
  // their low terms.  Eight lanes to a row.  Bound by vector instructions, two waves to a SIMD: 5,200 -> 3,100 cycles with seven of
  // them for two elements instead of eleven (split_q4) and a maximum that costs half of one.  (Once for each row: in the four
  // waves of S^T, each for its 32 rows, it took 9 K cycles more per segment.)
  auto split_q = [&]() {
    const int lane = fresh_lane(), part = lane & 7, r = 8 * (wave8 & 3) + (lane >> 3);
    const uint32_t base = lds0 + (2 + (wave8 >> 2)) * kStageM;
    auto chunk = [&](int i) -> uint32_t {
      return i < 8 ? base + r * QY::kMain + (((8 * i + part) ^ QY::sw_main(r)) << 4)
                   : base + kTailBaseM + r * QY::kTail + ((part ^ QY::sw_tail(r)) << 4);
    };
    u32x4 raw[9];
    float mx = 0.f;
#pragma unroll
    for (int i = 0; i < 9; ++i) raw[i] = *LDS_PTR(u32x4, chunk(i));
#pragma unroll
    for (int i = 0; i < 9; ++i)
#pragma unroll
      for (int k = 0; k < 4; k += 2) mx = bf16_max4(mx, raw[i][k], raw[i][k + 1]);
    int m = __builtin_bit_cast(uint32_t, mx) >> 16;
#define OA_DPP_MAX(ctrl)                                                        \
  {                                                                             \
    const int o = __builtin_amdgcn_update_dpp(0, m, (ctrl), 0xf, 0xf, true);    \
    m = m > o ? m : o;                                                          \
  }
    OA_DPP_MAX(0xb1) OA_DPP_MAX(0x4e) OA_DPP_MAX(0x141)  // lanes ^ 1, ^ 2, and the mirror of the eight
#undef OA_DPP_MAX
    const int ex = split_q_exponent(m);
    const float scale = __builtin_amdgcn_ldexpf(1.0f, ex), inv = __builtin_amdgcn_ldexpf(1.0f, -ex);
    if (part == 0) *LDS_PTR(float, lds_max + (8 * wave8 + (lane >> 3)) * 4) = split_q_factor(p.scale_log2, ex);
    if (p.scale_log2 < 0.f)
#pragma unroll
      for (int i = 0; i < 9; ++i) raw[i] ^= 0x80008000u;
#pragma unroll
    for (int i = 0; i < 9; ++i) {
      const u32x2 a = split_q4(raw[i][0], raw[i][1], scale, inv), b = split_q4(raw[i][2], raw[i][3], scale, inv);
      *LDS_PTR(u32x4, chunk(i)) = u32x4{a[0], b[0], a[1], b[1]};
    }
  };
  // (every wave looks at all 64 heads, so all take the same way)
  auto out_of_range = [&]() {
    const int lane = fresh_lane();
    const float m2 = fmaxf(*LDS_PTR(float, lds_max + lane * 4), *LDS_PTR(float, lds_max + (kHB + lane) * 4));
    return __any(m2 > kRefSlackM || (m2 < -kRefSlackM && m2 != -INFINITY));
  };

  if (wave8 < kRoleWaves) {
    // =============================== S^T and softmax ===============================
    const int th = wave & 1, hg = wave >> 1;
    for (int si = seg_lo; si < seg_hi; ++si) {
      SegM<FP8> sg;
      if (!begin_segment(si, sg)) continue;
      const int n = sg.n_tiles;
      if (n > 0) {
        const int lane = fresh_lane();
        const int n16 = lane & 15, q4 = lane >> 4, n32 = lane & 31, g = lane >> 5;
        wait_vm<0>();
        if constexpr (FP8) split_q();
        __syncthreads();  // 1: Q has arrived
        // B operand of S^T.  bf16: heads 32 hg + 16 a .., lane (head n16, q4) holds dims 32 ks + 8 q4 .. + 7.
        // fp8: lane (head n32 of group hg, g) holds dims 64 ks + 32 g .. + 31, as two e4m3 terms.
        constexpr int kKS = FP8 ? kQK / 64 : kQK / 32;
        bf16x8 qf[FP8 ? 1 : 2][FP8 ? 1 : kKS];
        i32x8 qh[FP8 ? kKS : 1], ql[FP8 ? kKS : 1];
        float c = p.scale_log2;  // logits are raw products times c, in the log2 domain
        // Chunk c of row r lies at r * 1024 + ((c ^ sw_main(r)) << 4), and the swizzle touches only the low four bits of c: an address
        // per value of those bits, the rest are immediate offsets.  (An address for each of the 36 reads took 340 vector
        // instructions and 1,000 cycles more.)
        const uint32_t lq = lds0 + (2 + hg) * kStageM;
        auto q_read = [&](uint32_t at, int imm) { return *LDS_PTR(u32x4, at + imm); };
        if constexpr (!FP8) {
          // (the swizzles of rows r and r + 16 are alike)
          uint32_t am[4], at[2];
#pragma unroll
          for (int k = 0; k < 4; ++k) am[k] = lq + n16 * QY::kMain + (((4 * k + q4) ^ QY::sw_main(n16)) << 4);
#pragma unroll
          for (int k = 0; k < 2; ++k) at[k] = lq + kTailBaseM + n16 * QY::kTail + (((4 * k + q4) ^ QY::sw_tail(n16)) << 4);
#pragma unroll
          for (int a = 0; a < 2; ++a)
#pragma unroll
            for (int ks = 0; ks < kKS; ++ks)
              qf[a][ks] = __builtin_bit_cast(bf16x8, ks < 16 ? q_read(am[ks & 3], (ks >> 2) * 256 + a * 16 * QY::kMain)
                                                             : q_read(at[ks & 1], a * 16 * QY::kTail));
        } else {
          uint32_t am[8], at[4];
#pragma unroll
          for (int k = 0; k < 8; ++k) am[k] = lq + n32 * QY::kMain + (((8 * (k >> 2) + 4 * g + (k & 3)) ^ QY::sw_main(n32)) << 4);
#pragma unroll
          for (int k = 0; k < 4; ++k) at[k] = lq + kTailBaseM + n32 * QY::kTail + (((4 * g + k) ^ QY::sw_tail(n32)) << 4);
#pragma unroll
          for (int ks = 0; ks < kKS; ++ks)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
              const u32x4 r = ks < 8 ? q_read(am[4 * (ks & 1) + j], (ks >> 1) * 256) : q_read(at[j], 0);
              qh[ks][2 * j] = r[0];
              qh[ks][2 * j + 1] = r[1];
              ql[ks][2 * j] = r[2];
              ql[ks][2 * j + 1] = r[3];
            }
          c = *LDS_PTR(float, lds_max + (32 * hg + n32) * 4);
        }
        __syncthreads();  // 2: Q has been read, its stages may be filled

        // What a lane computes.  bf16: tokens 16 th + 4 q4 + i (i < 4) of heads 32 hg + 16 a + n16 (a = 0, 1), element
        // 4 a + i.  fp8: tokens 32 th + 8 (i / 4) + 4 g + i % 4 (i < 16) of head 32 hg + n32.
        constexpr int kE = FP8 ? 16 : 8, kA = FP8 ? 1 : 2;
        const int head0 = 32 * hg + (FP8 ? n32 : n16);  // (bf16, a = 1: + 16)
        const int row_s = (FP8 ? 32 : 16) * th + (FP8 ? n32 : n16);
        const int c0 = FP8 ? 2 * g : q4;
        const uint32_t k_main = row_s * Y::kMain + ((c0 ^ Y::sw_main(row_s)) << 4);
        const uint32_t k_tail = kTailBaseM + row_s * Y::kTail + ((c0 ^ Y::sw_tail(row_s)) << 4);
        const uint32_t stat_w = (th * kHB + head0) * 4;
        uint32_t p_write[kA];
#pragma unroll
        for (int a = 0; a < kA; ++a)
          p_write[a] = lds_p + (FP8 ? p_chunk(head0, 2 * g + th) : p_chunk(head0 + 16 * a, 2 * th + (q4 & 1)) + (q4 >> 1) * 8);
        const uint32_t lds_w = lds_stat + wave * 2 * kScaleM;
        const uint32_t tok4 = (32 * th + 4 * g) * 4;
        uint32_t w_read = lds_w + tok4;
        asm volatile("" : "+v"(w_read));
        // what a masked position's raw product is replaced by (fp8: the sign of the scale is in q)
        const float masked_raw = !FP8 && c < 0.f ? INFINITY : -INFINITY;

        float ref[kA], l_run[kA], lq_run = 0.f, mt_all[kA], ref_exact[kA];
#pragma unroll
        for (int a = 0; a < kA; ++a) ref_exact[a] = __builtin_nanf("");
        auto head_max = [&](float x) { return FP8 ? half_max(x) : half_max(row_max(x)); };

        // One step: the weights of tile `it`, whose logits are in u, go to LDS in the operand order of PV, and S^T of
        // tile it + 1 is computed, with the arithmetic of the weights behind its matrix instructions.  (FIRST: no weights
        // yet.  LAST: no tile behind it and no S^T, whose matrix instructions would only hold up those of PV: 1,200 cycles fp8,
        // 600 bf16; a ring step of 40 sequences of six tiles, fp8, 37.0 -> 34.9 us, 32 of 4096 tokens bf16 48.7 -> 48.2.)
        float u[kE];       // logits over c (fp8: raw products times the token's scale), masked where a query keeps nothing
        float mu = 0.f;    // fp8: the largest
        int es = 0;        // fp8: every scale of the token half < 2^es
        auto step = [&](int it, auto first_tag, auto last_tag) {
          constexpr bool FIRST = decltype(first_tag)::value, LAST = decltype(last_tag)::value;
          const uint32_t st = stage_base(it + 1), pb = ((uint32_t)it & 1) * kPBytesM;
          const uint32_t am = st + k_main, at = st + k_tail;
          const uint32_t entry = LAST ? 1 : tile_entry(it + 1);
          if constexpr (FP8) {
            auto load_k = [&](int ks) -> i32x8 {
              const uint32_t ad = ks < 8 ? am ^ ((ks & 3) << 6) : at, imm = ks < 8 ? (ks >> 2) * 256 : 0;
              const i32x4 lo = *LDS_PTR(i32x4, ad + imm), hi = *LDS_PTR(i32x4, (ad ^ 16u) + imm);
              return i32x8{lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
            };
            constexpr int kRing = FIRST ? 2 : 3;
            i32x8 fr[kRing];
#pragma unroll
            for (int k = 0; k < (LAST ? 0 : kRing); ++k) fr[k] = load_k(k);
            f32x4 w[2], rw[2], sc[4];
            float sc_t = 0.f, rk = 0.f, ls0 = 0.f, ls1 = 0.f, lq0 = 0.f, lq1 = 0.f, e[2][2];
            int kk = 0;
            i32x4 pk;
            if constexpr (!FIRST) {
              w[0] = *LDS_PTR(f32x4, w_read);
              rw[0] = *LDS_PTR(f32x4, w_read + kScaleM);
              // Block exponent kk of the head's 32 weights: all are below 2^8 (see Weights above).
              const float mt = half_max(fmaf(mu, c, -ref[0]));
              mt_all[0] = fmaxf(mt_all[0], mt);
              int k = (int)ceilf(mt) - 8 + es;
              k = k < -126 ? -126 : k > 126 ? 126 : k;
              kk = mt == -INFINITY ? 0 : k;
              rk = ref[0] + (float)kk;
            }
            __builtin_amdgcn_sched_barrier(0);
            f32x16 s = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
            const uint32_t lsc = lds_scales + ((uint32_t)(it + 1) & (kStagesM - 1)) * kScaleM;
            // weights of elements 2 j, 2 j + 1 in three parts, which consecutive matrix instructions get of three pairs
            auto weights_e = [&](auto j_tag) {
              constexpr int j = decltype(j_tag)::value, i = 2 * j;
              e[j % 2][0] = __builtin_amdgcn_exp2f(fmaf(u[i], c, -rk));
              e[j % 2][1] = __builtin_amdgcn_exp2f(fmaf(u[i + 1], c, -rk));
            };
            auto weights_c = [&](auto j_tag) {
              constexpr int j = decltype(j_tag)::value, q = j / 2, k = (2 * j) & 3;
              const float e0 = e[j % 2][0], e1 = e[j % 2][1];
              ls0 += e0;
              ls1 += e1;
              pk[q] = __builtin_amdgcn_cvt_pk_fp8_f32(e0 * w[q & 1][k], e1 * w[q & 1][k + 1], k ? pk[q] : 0, k != 0);
              asm volatile("" : "+v"(ls0), "+v"(ls1));  // (here, and not collected behind the last matrix instruction)
            };
            auto weights_l = [&](auto j_tag) {
              constexpr int j = decltype(j_tag)::value, q = j / 2, k = (2 * j) & 3;
              const f32x2 b = __builtin_amdgcn_cvt_pk_f32_fp8(pk[q], k != 0);
              lq0 = fmaf(b[0], rw[q & 1][k], lq0);
              lq1 = fmaf(b[1], rw[q & 1][k + 1], lq1);
              asm volatile("" : "+v"(lq0), "+v"(lq1));
            };
            auto part = [&](auto m_tag) {
              constexpr int m = decltype(m_tag)::value, ks = m >> 1;
              if constexpr (LAST) {
              } else if constexpr ((m & 1) == 0) {
                s = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(fr[ks % kRing], qh[ks], s, 0, 0, 0, 127, 0, 127);
              } else {
                s = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(fr[ks % kRing], ql[ks], s, 0, 0, 0, 127, 0, 127 - kQLoShift);
                if constexpr (ks + kRing < kKS) fr[ks % kRing] = load_k(ks + kRing);
              }
              if constexpr (!FIRST) {
                if constexpr ((m & 1) == 0 && m < 16) weights_e(std::integral_constant<int, m / 2>{});
                if constexpr ((m & 1) == 1 && m < 16) weights_c(std::integral_constant<int, m / 2>{});
                if constexpr ((m & 1) == 0 && m >= 2) weights_l(std::integral_constant<int, m / 2 - 1>{});
                if constexpr (m == 2 || m == 6 || m == 10) w[((m + 2) / 4) & 1] = *LDS_PTR(f32x4, w_read + (m + 2) / 4 * 32);
                if constexpr (m == 3 || m == 7 || m == 11) rw[((m + 1) / 4) & 1] = *LDS_PTR(f32x4, w_read + kScaleM + (m + 1) / 4 * 32);
                if constexpr (m == 1)
                  *LDS_PTR(uint8_t, lds_kk + ((uint32_t)it & 1) * kStatM + th * kHB + head0) = (uint8_t)(127 + kk);  // (the same in both lanes of a head)
                if constexpr (m == 16) *LDS_PTR(i32x4, p_write[0] + pb) = pk;
                if constexpr (m == 17) {
                  l_run[0] += __builtin_amdgcn_ldexpf(ls0 + ls1, kk);
                  lq_run += __builtin_amdgcn_ldexpf(lq0 + lq1, kk);
                  asm volatile("" : "+v"(l_run[0]), "+v"(lq_run));
                }
              }
              if constexpr (m == 12 && !LAST) {
                sc_t = *LDS_PTR(float, lsc + lane * 4);
#pragma unroll
                for (int q = 0; q < 4; ++q) sc[q] = *LDS_PTR(f32x4, lsc + tok4 + q * 32);
              }
              if constexpr (m == 14 && !LAST) {
                // es: every scale of the token half < 2^es, es >= -100
                float mx = 0.f;
#pragma unroll
                for (int i = 0; i < kE; ++i) mx = fmaxf(mx, fabsf(sc[i >> 2][i & 3]));
                es = (int)(__builtin_bit_cast(uint32_t, half_max(mx)) >> 23) - 126;
                es = es < -100 ? -100 : es;
                asm volatile("" : "+v"(es));
              }
              if constexpr (m == 17 && !LAST) {
                // Weight scales of the tile for this wave (lane = token): the token's scale, raised to 2^(es - 10) so that
                // one far below the half's largest stays in the rounded sum; and their reciprocals.
                const float x = fmaxf(sc_t, __builtin_amdgcn_ldexpf(1.0f, es - 10));
                *LDS_PTR(float, lds_w + lane * 4) = x;
                *LDS_PTR(float, lds_w + kScaleM + lane * 4) = __builtin_amdgcn_rcpf(x);
              }
              __builtin_amdgcn_sched_barrier(0);
            };
            [&]<int... M>(std::integer_sequence<int, M...>) {
              (part(std::integral_constant<int, M>{}), ...);
            }(std::make_integer_sequence<int, 2 * kKS>{});
            if constexpr (!LAST) {
#pragma unroll
              for (int i = 0; i < kE; ++i) u[i] = s[i] * sc[i >> 2][i & 3];
            }
          } else {
            auto load_k = [&](int ks) {
              return *LDS_PTR(bf16x8, ks < 16 ? (am ^ ((ks & 3) << 6)) + (ks >> 2) * 256 : at ^ ((ks & 1) << 6));
            };
            constexpr int kRing = 8;
            bf16x8 fr[kRing];
#pragma unroll
            for (int ks = 0; ks < (LAST ? 0 : kRing); ++ks) fr[ks] = load_k(ks);
            float e[kE];
            if constexpr (!FIRST) {  // (while the first rows are on their way)
#pragma unroll
              for (int i = 0; i < kE; ++i) u[i] = fmaf(u[i], c, -ref[i >> 2]);
#pragma unroll
              for (int i = 0; i < kE; ++i) e[i] = __builtin_amdgcn_exp2f(u[i]);
            }
            __builtin_amdgcn_sched_barrier(0);
            f32x4 s[2] = {{0, 0, 0, 0}, {0, 0, 0, 0}};
            auto part = [&](auto m_tag) {
              constexpr int ks = decltype(m_tag)::value;
              if constexpr (!LAST) {
                s[0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fr[ks % kRing], qf[0][ks], s[0], 0, 0, 0);
                s[1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fr[ks % kRing], qf[1][ks], s[1], 0, 0, 0);
                if constexpr (ks + kRing < kKS) fr[ks % kRing] = load_k(ks + kRing);
              }
              if constexpr (!FIRST) {
                if constexpr (ks == 1 || ks == 3) {
                  constexpr int a = ks >> 1;
                  *LDS_PTR(bf16x4, p_write[a] + pb) = bf16x4{(__bf16)e[4 * a], (__bf16)e[4 * a + 1], (__bf16)e[4 * a + 2], (__bf16)e[4 * a + 3]};
                }
                if constexpr (ks >= 4 && ks < 12) {
                  constexpr int i = ks - 4;
                  l_run[i >> 2] += e[i];
                  mt_all[i >> 2] = fmaxf(mt_all[i >> 2], u[i]);
                  asm volatile("" : "+v"(l_run[i >> 2]), "+v"(mt_all[i >> 2]));  // (here, and not behind the last of them)
                }
              }
              __builtin_amdgcn_sched_barrier(0);
            };
            [&]<int... M>(std::integer_sequence<int, M...>) {
              (part(std::integral_constant<int, M>{}), ...);
            }(std::make_integer_sequence<int, kKS>{});
            if constexpr (!LAST) {
#pragma unroll
              for (int i = 0; i < kE; ++i) u[i] = s[i >> 2][i & 3];
            }
          }
          if constexpr (LAST) return;
          if (!(__builtin_amdgcn_readfirstlane(entry) & 1)) {  // uniform, one or two tiles of a sequence
            const int l = fresh_lane(), pos0 = sg.pos(it + 1);
#pragma unroll
            for (int a = 0; a < kA; ++a) {
              // length of the sequence that the lane's query sees (several queries: cut after its own token)
              const int head = sg.h0 + 32 * hg + (FP8 ? (l & 31) : (l & 15) + 16 * a);
              const int Lq = sg.L - (p.T - 1 - (head < p.H ? head : p.H - 1) / p.Hq);
#pragma unroll
              for (int i = 0; i < kE / kA; ++i) {
                const int j = pos0 + (FP8 ? 32 * th + (i >> 2) * 8 + 4 * (l >> 5) + (i & 3) : 16 * th + 4 * (l >> 4) + i);
                float& x = u[a * (kE / kA) + i];
                x = retained(j, Lq, sg.S, sg.W) ? x : masked_raw;
              }
            }
          }
          if constexpr (FP8) {
            mu = u[0];
#pragma unroll
            for (int i = 1; i < kE; ++i) mu = fmaxf(mu, u[i]);
          }
        };

#pragma unroll 1
        for (int attempt = 0; attempt < 2; ++attempt) {
          lq_run = 0.f;
#pragma unroll
          for (int a = 0; a < kA; ++a) {
            l_run[a] = 0.f;
            mt_all[a] = -INFINITY;
          }
          __syncthreads();  // 3: tile 0 is visible
          step(-1, std::true_type{}, std::false_type{});
#pragma unroll
          for (int a = 0; a < kA; ++a) {
            float mx = FP8 ? mu * c : -INFINITY;
            if constexpr (!FP8) {
#pragma unroll
              for (int i = 0; i < 4; ++i) mx = fmaxf(mx, u[4 * a + i] * c);
            }
            mx = head_max(mx);
            if (lane < (FP8 ? 32 : 16)) *LDS_PTR(float, lds_max + stat_w + a * 64) = mx;
          }
          __syncthreads();  // 4: also tile 1
#pragma unroll
          for (int a = 0; a < kA; ++a) {
            const uint32_t m0 = lds_max + (head0 + 16 * a) * 4;
            const float m2 = fmaxf(*LDS_PTR(float, m0), *LDS_PTR(float, m0 + kHB * 4));
            // an integer, so that weights against different references differ by exact powers of two
            ref[a] = ref_exact[a] == ref_exact[a] ? ref_exact[a] : (m2 == -INFINITY || m2 != m2) ? 0.f : ceilf(m2);
          }
#pragma unroll 1
          for (int it = 0; it + 1 < n; ++it) {
            step(it, std::false_type{}, std::false_type{});
            __syncthreads();  // weights of tile `it`, tile it + 2
          }
          step(n - 1, std::false_type{}, std::true_type{});
          __syncthreads();
          // (in step n - 1 these waves have nothing else to do, and no wave reads weight scales any more)
#pragma unroll
          for (int a = 0; a < kA; ++a) {
            const float l = FP8 ? half_sum(l_run[a]) : half_sum(row_sum(l_run[a]));
            const float m = FP8 ? mt_all[a] : head_max(mt_all[a]);
            const float lq = FP8 ? half_sum(lq_run) : l;
            if (lane < (FP8 ? 32 : 16)) {
              *LDS_PTR(float, lds_max + stat_w + a * 64) = m;
              *LDS_PTR(float, lds_stat + stat_w + a * 64) = l;
              *LDS_PTR(float, lds_stat + kStatM * 4 + stat_w + a * 64) = lq;
              *LDS_PTR(float, lds_stat + 2 * kStatM * 4 + stat_w + a * 64) = ref[a];
            }
          }
          __syncthreads();
          if (attempt > 0 || !out_of_range()) break;
#pragma unroll
          for (int a = 0; a < kA; ++a) {
            const uint32_t m0 = lds_max + (head0 + 16 * a) * 4;
            const float m3 = fmaxf(*LDS_PTR(float, m0), *LDS_PTR(float, m0 + kHB * 4));
            ref_exact[a] = m3 == -INFINITY ? 0.f : ref[a] + ceilf(m3);
          }
        }
      }
      const int lane = fresh_lane();
      if (wave == 0 && lane < p.H - sg.h0) {
        const float lse = n > 0 ? (stat(2, 0, lane) + __builtin_amdgcn_logf(stat(0, 0, lane) + stat(0, 1, lane))) * 0.6931471805599453f
                                : -INFINITY;
        if (sg.slot < 0) p.lse[(size_t)sg.b * p.H + sg.h0 + lane] = lse;
        else p.part_lse[(size_t)sg.slot * p.head_block + half * kHB + lane] = lse;
      }
      __syncthreads();  // the statistics have been read, the rows staged
    }
    return;
  }

  // =============================== loads and PV ===============================
  constexpr int kRowsPerWave = kT / kRoleWaves;  // 8 or 16
  for (int si = seg_lo; si < seg_hi; ++si) {
    SegM<FP8> sg;
    if (!begin_segment(si, sg)) continue;
    const int n = sg.n_tiles;
    f32x16 acc[2][4];
    if (n > 0) {
      const int lane = fresh_lane();
      const int n16 = lane & 15, q4 = lane >> 4, n32 = lane & 31, g = lane >> 5;
      // ---- tile loader: the wave fetches rows [kRowsPerWave * wave, ...) into stage it & 3, kept or not ----
      // (a tile lies inside one page, so its rows exist; what no query keeps is masked and cleared)
      // Loads 0 .. 7: 1 KB of value bytes each, four to an LDS base (the immediate offset counts on both sides and is
      // taken off the lane's); load 8: the rope parts; fp8, load 9: the scales (16 lanes).
      uint32_t dma_off[9];
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        const int r = kRowsPerWave * wave + (FP8 ? 2 * k + g : k);  // fp8: two rows, lanes 0..31 and 32..63
        dma_off[k] = (((FP8 ? n32 : lane) ^ Y::sw_main(r)) << 4) + (r - kRowsPerWave * wave) * Y::kRow - (k & 3) * 1024;
      }
      {
        constexpr int kTailChunks = Y::kTail / 16;
        const int r = lane / kTailChunks;
        dma_off[8] = r * Y::kRow + Y::kMain + (((lane % kTailChunks) ^ Y::sw_tail(kRowsPerWave * wave + r)) << 4);
      }
      auto load_piece = [&](uint64_t rows, uint64_t scales, uint32_t st, uint32_t lscale, auto k_tag) {
        constexpr int k = decltype(k_tag)::value;
        if constexpr (k < 8) {
          if constexpr ((k & 3) == 0) set_lds_base(st + wave * 8192 + k * 1024);
          load_lds16_at<(k & 3) * 1024>(rows, dma_off[k]);
        } else if constexpr (k == 8) {
          set_lds_base(st + kTailBaseM + wave * 1024);
          load_lds16_at<0>(rows, dma_off[8]);
        } else {
          set_lds_base(lscale);
          load_lds4_at(0xffffull, scales, lane * 4);
        }
      };
      auto issue_tile = [&](int it) {
        const uint64_t t = (uint32_t)__builtin_amdgcn_readfirstlane(tile_entry(it)) >> 1;
        uint64_t rows = (uint64_t)(uintptr_t)p.kv + wave * (kRowsPerWave * Y::kRow) + t * kStageM;
        uint64_t scales = FP8 ? (uint64_t)(uintptr_t)p.kv_scales + wave * (kRowsPerWave * 4) + t * kScaleM : 0;
        settle_address(rows, scales);
        const uint32_t lscale = lds_scales + ((uint32_t)it & (kStagesM - 1)) * kScaleM + wave * kRowsPerWave * 4;
        [&]<int... K>(std::integer_sequence<int, K...>) {
          (load_piece(rows, scales, stage_base(it), lscale, std::integral_constant<int, K>{}), ...);
        }(std::make_integer_sequence<int, kDma>{});
      };
      // `later` tiles were requested behind the one that has to be there
      auto wait_later = [&](int later) {
        if (later >= 3) wait_vm<3 * kDma>();
        else if (later == 2) wait_vm<2 * kDma>();
        else if (later == 1) wait_vm<kDma>();
        else wait_vm<0>();
      };
      // Of a tile's rows that the wave has fetched, those that no query keeps: values 0 (0 * NaN would poison PV), scales
      // the smallest normal number (a real one may be anything)
      auto clear_rows = [&](int it) {
        const int pos0 = sg.pos(it);
        if (sg.full(pos0)) return;
        const int lane = fresh_lane();
        constexpr int kChunks = Y::kMain / 16;
        const uint32_t st = stage_base(it);
#pragma unroll 1
        for (int k = lane; k < kRowsPerWave * kChunks; k += 64) {
          const int r = wave * kRowsPerWave + k / kChunks;
          if (!retained(pos0 + r, sg.L, sg.S, sg.Wu)) *LDS_PTR(u32x4, st + r * Y::kMain + (k % kChunks) * 16) = u32x4{0, 0, 0, 0};
        }
        if constexpr (FP8) {
          const int r = wave * kRowsPerWave + lane;
          if (lane < kRowsPerWave && !retained(pos0 + r, sg.L, sg.S, sg.Wu))
            *LDS_PTR(float, lds_scales + ((uint32_t)it & (kStagesM - 1)) * kScaleM + r * 4) = 1.1754944e-38f;
        }
      };
      // V^T, transposing reads.  bf16: 4 tokens x 16 columns per 16 lanes, rows 16 t + 8 k + 4 g + (n16 >> 2);
      // fp8: 8 tokens x 16 columns, rows 16 pt + 8 (ip >> 2) + 4 g + (ip & 3).  Columns 128 wave + 32 cb ..
      uint32_t v_main[FP8 ? 1 : 2];
      if constexpr (FP8) {
        const int ip = n16 >> 1, r = 8 * (ip >> 2) + 4 * g + (ip & 3);
        v_main[0] = r * Y::kMain + ((((q4 & 1) ^ Y::sw_main(r)) << 4) ^ ((wave & 1) << 7)) + (wave >> 1) * 256 + 8 * (lane & 1);
      } else {
        const int c_lane = (q4 & 1) * 2 + ((n16 & 3) >> 1);
#pragma unroll
        for (int k = 0; k < 2; ++k) {
          const int r = 8 * k + 4 * g + (n16 >> 2);
          v_main[k] = r * Y::kMain + ((c_lane ^ Y::sw_main(r)) << 4) + (n16 & 1) * 8 + wave * 256;
        }
      }

      // Q and tile 0 are what the first step waits for: the other tiles are requested behind the barriers that follow.
      issue_tile(0);
      wait_later(1);
      if constexpr (FP8) split_q();
      __syncthreads();  // 1: Q has arrived
      if (n > 1) issue_tile(1);
      __syncthreads();  // 2: Q has been read, its stages may be filled
#pragma unroll 1
      for (int attempt = 0; attempt < 2; ++attempt) {
        if (attempt > 0) {
          issue_tile(0);
          if (n > 1) issue_tile(1);
        }
        // V^T fragments of the tile whose PV comes next, requested while the one before is multiplied
        constexpr int kV1 = FP8 ? 4 : 8;
        std::conditional_t<FP8, i32x8, bf16x8> v[kV1];
        auto load_v = [&](uint32_t st, int j) {
          if constexpr (FP8) {
#pragma unroll
            for (int pt = 0; pt < 4; ++pt) {
              const i32x2 t = __builtin_amdgcn_ds_read_tr8_b64_v2i32(LDS_PTR(i32x2, ((st + v_main[0]) ^ (j << 5)) + pt * 16 * Y::kMain));
              v[j][2 * pt] = t[0];
              v[j][2 * pt + 1] = t[1];
            }
          } else {
            const uint32_t x = (j & 3) << 6, imm = (j >> 2) * 16 * Y::kMain;
            const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16(LDS_PTR(s16x4, ((st + v_main[0]) ^ x) + imm));
            const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16(LDS_PTR(s16x4, ((st + v_main[FP8 ? 0 : 1]) ^ x) + imm));
            v[j] = __builtin_bit_cast(bf16x8, s16x8{lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]});
          }
        };
        wait_later(n > 1 ? 1 : 0);
        clear_rows(0);
        __syncthreads();  // 3: tile 0 is visible
        if (n > 2) issue_tile(2);
        if (n > 3) issue_tile(3);
        const int later = n - 1 < 3 ? n - 1 : 3;
#pragma unroll
        for (int a = 0; a < 2; ++a)
#pragma unroll
          for (int cb = 0; cb < 4; ++cb)
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[a][cb][i] = 0.f;
        wait_later(later - 1);
        if (n > 1) clear_rows(1);
        __syncthreads();  // 4: tile 1
#pragma unroll
        for (int j = 0; j < kV1; ++j) load_v(stage_base(0), j);
        wait_later(later - 2);
        if (n > 2) clear_rows(2);
        __syncthreads();  // weights of tile 0, tile 2
        // Step it: PV of tile it and the V fragments of tile it + 1 here, the weights of tile it + 1 and S^T of tile it + 2
        // there.  Tile it has been read by all: tile it + 4 is requested into its stage, two steps before it is needed.
#pragma unroll 1
        for (int it = 0; it < n; ++it) {
          if (it + 4 < n) issue_tile(it + 4);
          const uint32_t st1 = stage_base(it + 1), pb = lds_p + ((uint32_t)it & 1) * kPBytesM;
          if constexpr (FP8) {
            i32x8 pf[2];
            int sb[2];
#pragma unroll
            for (int a = 0; a < 2; ++a) {
              const i32x4 lo = *LDS_PTR(i32x4, pb + p_chunk(32 * a + n32, 2 * g)), hi = *LDS_PTR(i32x4, pb + p_chunk(32 * a + n32, 2 * g + 1));
              pf[a] = i32x8{lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
              sb[a] = *LDS_PTR(uint8_t, lds_kk + ((uint32_t)it & 1) * kStatM + g * kHB + 32 * a + n32);  // (half g from lane (head, g))
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int j = 0; j < kV1; ++j) {
#pragma unroll
              for (int a = 0; a < 2; ++a)
                acc[a][j] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(v[j], pf[a], acc[a][j], 0, 0, 0, 127, 0, sb[a]);
              load_v(st1, j);
              __builtin_amdgcn_sched_barrier(0);
            }
          } else {
            bf16x8 pf[2][2];
#pragma unroll
            for (int t = 0; t < 2; ++t)
#pragma unroll
              for (int a = 0; a < 2; ++a) pf[a][t] = *LDS_PTR(bf16x8, pb + p_chunk(32 * a + n32, 2 * t + g));
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int j = 0; j < kV1; ++j) {
#pragma unroll
              for (int a = 0; a < 2; ++a)
                acc[a][j & 3] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(v[j], pf[a][j >> 2], acc[a][j & 3], 0, 0, 0);
              load_v(st1, j);  // (behind the last tile: what the stage holds, not used)
              __builtin_amdgcn_sched_barrier(0);
            }
          }
          // (here, and not behind the branches and the barrier that follow)
          asm volatile("" : "+v"(acc[0][0]), "+v"(acc[0][1]), "+v"(acc[0][2]), "+v"(acc[0][3]), "+v"(acc[1][0]), "+v"(acc[1][1]),
                       "+v"(acc[1][2]), "+v"(acc[1][3]));
          wait_later(it + 4 < n ? 1 : 0);
          if (it + 3 < n) clear_rows(it + 3);
          __syncthreads();
        }
        if (attempt > 0 || !out_of_range()) break;
      }
    } else {
#pragma unroll
      for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int cb = 0; cb < 4; ++cb)
#pragma unroll
          for (int i = 0; i < 16; ++i) acc[a][cb][i] = 0.f;
    }

    // ---- epilogue: normalise (fp8: by the rounded weights' sum), transpose through LDS, write 128 columns ----
    // Bound by the issue of one wave per SIMD (four columns a time through LDS), then by the 64 KB of rows that it writes.  The
    // output type and the empty segment are decided outside the loops over the accumulators (one branch per value: 4,500
    // cycles where it now takes 2,000), rows leave LDS eight requests at a time, and those of the first 32 heads while the
    // others are staged: 7,000 -> 4,550 cycles from the loop's end to the last store, 0.4 to 0.9 us per decode.
    const int lane = fresh_lane();
    const int n32 = lane & 31, g = lane >> 5;
    const bool final_out = sg.slot < 0;
    const int heads_here = p.H - sg.h0 < kHB ? p.H - sg.h0 : kHB;
    const size_t row0 = final_out ? (size_t)sg.b * p.H + sg.h0 : (size_t)sg.slot * p.head_block + half * kHB;
    constexpr int kOutMax = 128 * 4 + 16;
    const uint32_t ost = lds0 + wave * kHB * kOutMax;
    float inv[2];
#pragma unroll
    for (int a = 0; a < 2; ++a) {
      const float lq_tot = n > 0 ? stat(1, 0, 32 * a + n32) + stat(1, 1, 32 * a + n32) : 0.f;
      inv[a] = lq_tot != 0.f ? 1.0f / lq_tot : 0.f;
    }
    // 32 heads at a time: rows of `row` bytes, of which the wave has `data`, `per` of them to an instruction; `put` stages four columns
    auto write_rows = [&](auto row_tag, auto put) {
      constexpr int row = decltype(row_tag)::value, data = row / 4, per = 1024 / data, stride = data + 16;
      const uint32_t to = ost + n32 * stride + g * (data / 32);
      const int sub = lane / (data / 16), off = (lane & (data / 16 - 1)) * 16;
      const uint32_t from = ost + sub * stride + off;
      uint8_t* dst = (uint8_t*)(final_out ? p.out : p.part_o) + (row0 + sub) * row + wave * data + off;
#pragma unroll
      for (int a = 0; a < 2; ++a) {
#pragma unroll
        for (int cb = 0; cb < 4; ++cb)
#pragma unroll
          for (int i4 = 0; i4 < 4; ++i4)
            put(to + a * 32 * stride + (cb * 32 + i4 * 8) * (data / 128),
                f32x4{acc[a][cb][i4 * 4] * inv[a], acc[a][cb][i4 * 4 + 1] * inv[a], acc[a][cb][i4 * 4 + 2] * inv[a], acc[a][cb][i4 * 4 + 3] * inv[a]});
        constexpr int kBatch = 8;
#pragma unroll
        for (int k0 = 0; k0 < 32 / per; k0 += kBatch) {
          u32x4 r[kBatch];
#pragma unroll
          for (int k = 0; k < kBatch; ++k) r[k] = *LDS_PTR(u32x4, from + (32 * a + (k0 + k) * per) * stride);
#pragma unroll
          for (int k = 0; k < kBatch; ++k) {
            const int h = 32 * a + (k0 + k) * per;
            if (h + sub < heads_here) *(u32x4*)(dst + (size_t)h * row) = r[k];
          }
        }
      }
    };
    if (!p.out_fp32)
      write_rows(std::integral_constant<int, kV * 2>{},
                 [](uint32_t at, f32x4 x) { *LDS_PTR(bf16x4, at) = bf16x4{(__bf16)x[0], (__bf16)x[1], (__bf16)x[2], (__bf16)x[3]}; });
    else
      write_rows(std::integral_constant<int, kV * 4>{}, [](uint32_t at, f32x4 x) { *LDS_PTR(f32x4, at) = x; });
    __syncthreads();  // staging rows and tile table are free again before the next segment
  }
}

template <bool FP8>
static hipError_t set_lds_mid(int bytes) {
  return hipFuncSetAttribute(reinterpret_cast<const void*>(&decode_mid_kernel<FP8>), hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
}

hipError_t init_mid_kernels() {
  hipError_t e = set_lds_mid<false>(kLdsMidBf16);
  return e == hipSuccess ? set_lds_mid<true>(kLdsMidFp8) : e;
}

hipError_t launch_decode_mid(const DecodeParams& p, bool fp8, int n_units, hipStream_t stream) {
  if (n_units <= 0) return hipSuccess;
  if (p.xcds < 1 || (p.head_block != kHB && p.head_block != 2 * kHB)) return hipErrorInvalidValue;
  const dim3 grid(((n_units + p.xcds - 1) / p.xcds) * p.xcds * (p.head_block / kHB)), block(kWavesM * 64);
  if (fp8) hipLaunchKernelGGL(decode_mid_kernel<true>, grid, block, kLdsMidFp8, stream, p);
  else hipLaunchKernelGGL(decode_mid_kernel<false>, grid, block, kLdsMidBf16, stream, p);
  return hipGetLastError();
}

}  // namespace omniattn
