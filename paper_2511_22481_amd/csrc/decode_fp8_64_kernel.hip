// gfx950 kernel for sparse MLA decode over an fp8 (e4m3) latent cache, blocks of 64 head rows.
// (Paper section 3.2.1: softmax(q K_M^T * scale) V_M with M = sinks + recents.)
//
// Number formats are those of the kernel for blocks of 128 rows (decode_fp8_kernel.hip): the query in two
// e4m3 terms, weights in e4m3 with one block exponent per head and 32 tokens, normalised by their
// rounded sum.  That kernel gives each wave 32 heads of its own: every wave reads all of K and transposes
// all of V, and one wave per SIMD waits out a softmax that nothing covers; in the long loop it takes 7.5 K
// cycles per tile of 64 tokens where its matrix instructions take 3.3 K.  Here the four waves share 64 heads:
//   S^T  wave (th, hg): 32 tokens x 32 heads, the query (144 registers) as before;
//   P    the weights meet in LDS, in the operand order of PV;
//   PV   wave w: output columns 128 w .. of all 64 heads (128 accumulators instead of 256).
// V is transposed once per tile, K read twice, and the registers this frees let S^T of the next tile
// run ahead, so the softmax of a tile stands behind matrix instructions that do not wait for it: 3.14 K
// cycles per tile and 64 heads (6.3 K per 128) in the long loop, where its matrix instructions take 1.66 K and
// LDS is busy for 0.77 K.  What bounds it is the instruction issue of a lone wave per SIMD: 215 vector, 26
// matrix, 78 scalar and 58 LDS instructions a tile.
// us per decode with blocks of 128 -> 64 rows, each in its best partition, 128 rows per sequence unless stated: 32
// sequences of 8320 tokens 83 -> 73; 93 mixed 127 -> 124; 64 of 2176 59 -> 51, two queries each 91 -> 75;
// 128 of 2176, 64 rows 87 -> 56.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>
#include <utility>

#include "decode_common.h"

namespace omniattn {

namespace {

typedef __attribute__((ext_vector_type(2))) unsigned short u16x2;

constexpr int kHB = kHeadBlockFp8;       // 64
constexpr int kT = kTileFp8;
constexpr int kRowF = kQK, kMainF = 512, kTailF = 64;
constexpr int kTailBaseF = kT * kMainF;  // 32,768
constexpr int kStageF = kT * kRowF;      // 36,864
constexpr int kStagesF = 4;
constexpr int kWavesF = 4;
constexpr int kPRowF = 80;               // a head's weights of one tile: 64 bytes, padded to an odd multiple of 16
constexpr int kStatF = 2 * kHB;          // (token half, head)
constexpr int kScaleF = kT * 4;
// stages | weights | block exponents | per-head statistics (4) | tile table | token scales |
// per wave: weight scales of the tile at hand and their reciprocals
constexpr int kOffPF = kStagesF * kStageF;
constexpr int kOffKKF = kOffPF + kHB * kPRowF;
constexpr int kOffStatF = kOffKKF + kStatF * 4;
constexpr int kOffTilesF = kOffStatF + 4 * kStatF * 4;
constexpr int kOffScalesF = kOffTilesF + kMaxSegTiles * 4;
constexpr int kOffWScaleF = kOffScalesF + kStagesF * kScaleF;
constexpr int kLdsF = kOffWScaleF + kWavesF * 2 * kScaleF;
static_assert(kLdsF <= 160 * 1024, "LDS of one compute unit");

constexpr float kRefSlackF = 64.f;  // see the bf16 kernel: fixed softmax reference with retry
constexpr int kQLoShiftF = 4;       // see the fp8 kernel: the query's low term is stored 16 times too large

__host__ __device__ constexpr int swf_main(int r) { return ((r & 3) << 1) | ((r >> 2) & 1) | (((r >> 3) & 1) << 3); }
__host__ __device__ constexpr int swf_tail(int r) { return (r >> 2) & 3; }
// Q rows on their way through LDS: 1152 bytes, value and rope part apart, 32 rows to a stage
constexpr int kQMain = 1024, kQTail = 128, kQRow = 1152;
__host__ __device__ constexpr int swq_main(int r) { return ((r & 3) << 2) | ((r >> 2) & 3); }
__host__ __device__ constexpr int swq_tail(int r) { return (r >> 1) & 7; }

// Matrix instructions as assembly: only so does their place among the other instructions stay what is
// written.  Operands by register file: O^T (128 registers) and the query's low term (72) in accumulation
// registers; K, V^T, the weights, S^T and the query's high term in vector registers.  A vector-ALU
// read of a result needs 19 wait states (settle_*; checked on the generated code).  one, lo: E8M0 scales.
__device__ __forceinline__ void mfma_s_first(f32x16& s, i32x8 a, i32x8 b) {
  asm volatile("v_mfma_f32_32x32x64_f8f6f4 %0, %1, %2, 0" : "=&v"(s) : "v"(a), "v"(b));
}
__device__ __forceinline__ void mfma_s_hi(f32x16& s, i32x8 a, i32x8 b) {
  asm volatile("v_mfma_f32_32x32x64_f8f6f4 %0, %1, %2, %0" : "+v"(s) : "v"(a), "v"(b));
}
__device__ __forceinline__ void mfma_s_lo(f32x16& s, i32x8 a, i32x8 b, int one, int lo) {
  asm volatile("v_mfma_scale_f32_32x32x64_f8f6f4 %0, %1, %2, %0, %3, %4" : "+v"(s) : "v"(a), "a"(b), "v"(one), "v"(lo));
}
__device__ __forceinline__ void mfma_o(f32x16& acc, i32x8 a, i32x8 b, int one, int sb) {
  asm volatile("v_mfma_scale_f32_32x32x64_f8f6f4 %0, %1, %2, %0, %3, %4" : "+a"(acc) : "v"(a), "v"(b), "v"(one), "v"(sb));
}
__device__ __forceinline__ void settle_s(f32x16& s) { asm volatile("s_nop 15\n\ts_nop 3" : "+v"(s)); }
__device__ __forceinline__ void settle_o(f32x16 (&acc)[2][4]) {
  asm volatile("s_nop 15\n\ts_nop 3"
               : "+a"(acc[0][0]), "+a"(acc[0][1]), "+a"(acc[0][2]), "+a"(acc[0][3]), "+a"(acc[1][0]), "+a"(acc[1][1]),
                 "+a"(acc[1][2]), "+a"(acc[1][3]));
}

__device__ __forceinline__ float pair_max(float x) {
  float a = x, b = x;
  swap32(a, b);
  return fmaxf(a, b);
}
__device__ __forceinline__ float pair_sum(float x) {
  float a = x, b = x;
  swap32(a, b);
  return a + b;
}

}  // namespace

__global__ __launch_bounds__(kWavesF * 64, 1) void decode_fp8_64_kernel(DecodeParams p) {
  extern __shared__ __attribute__((aligned(16))) uint8_t lds_raw[];
  const uint32_t lds0 = (uint32_t)(uintptr_t)lds_raw;
  const uint32_t lds_p = lds0 + kOffPF, lds_kk = lds0 + kOffKKF, lds_stat = lds0 + kOffStatF;
  const uint32_t lds_tiles = lds0 + kOffTilesF, lds_scales = lds0 + kOffScalesF;
  const int tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int th = wave & 1, hg = wave >> 1;
  // Per-lane values are derived anew in each phase of a segment from a lane id that went through an
  // opaque move: computed once they would all stay alive across the loop, which has no registers for them.
  auto fresh_lane = [&]() {
    int l = tid & 63;
    asm volatile("" : "+v"(l));
    return l;
  };

  constexpr int kRowsPerWave = kT / kWavesF;  // 16
  constexpr int kDma = 10;  // direct loads per wave and tile: 8 of value bytes, 1 of rope bytes, 1 of scales

  const int per_xcd = (p.n_units + p.xcds - 1) / p.xcds;
  const int unit = ((int)blockIdx.x % p.xcds) * per_xcd + (int)blockIdx.x / p.xcds;
  if (unit >= p.n_units) return;
  auto uniform4 = [](u32x4 v) {
    return u32x4{(uint32_t)__builtin_amdgcn_readfirstlane(v.x), (uint32_t)__builtin_amdgcn_readfirstlane(v.y),
                 (uint32_t)__builtin_amdgcn_readfirstlane(v.z), (uint32_t)__builtin_amdgcn_readfirstlane(v.w)};
  };
  const u32x4* hdr = (const u32x4*)(p.units + unit);
  const u32x4 hdr0 = hdr[0], hdr1 = hdr[1], hdr2 = hdr[2];
  const int seg_lo = __builtin_amdgcn_readfirstlane(hdr0.x), seg_hi = __builtin_amdgcn_readfirstlane(hdr0.y);

  for (int si = seg_lo; si < seg_hi; ++si) {
    u32x4 sg_a = hdr1, sg_b = hdr2;
    if (si != seg_lo) {
      const u32x4* sp = (const u32x4*)(p.segs + si);
      sg_a = sp[0];
      sg_b = sp[1];
    }
    sg_a = uniform4(sg_a);
    sg_b = uniform4(sg_b);
    const DevSegment sg = {(int32_t)sg_a.x, (int32_t)sg_a.y, (int32_t)sg_a.z, (int32_t)sg_a.w,
                           (int32_t)sg_b.x, (int32_t)sg_b.y, (int32_t)sg_b.z, (int32_t)sg_b.w};
    const int lane = fresh_lane();
    const int n16 = lane & 15, n32 = lane & 31, g = lane >> 5;
    const int L = sg.L;
    const int h0 = sg.hb * kHB;
    const TileLayout tl = tile_layout(L, p.S, p.Wu, kT);
    const int n_tiles = sg.tile_hi - sg.tile_lo;
    const int L0 = L - (p.T - 1);
    const int sink_end = p.S < L0 ? p.S : L0;

    auto tile_pos = [&](int it) { return tl.logical(sg.tile_lo + it) * kT; };
    auto stage_base = [&](int it) -> uint32_t { return lds0 + ((uint32_t)it & (kStagesF - 1)) * kStageF; };
    auto tile_full = [&](int pos0) {
      return (pos0 + kT <= sink_end) || (pos0 >= L - p.W && pos0 + kT <= L0);
    };

    // ---- tile table: 64-token unit of the cache that holds the tile, bit 0 = every position kept ----
    constexpr int kTabPerThread = kMaxSegTiles / (kWavesF * 64);
    const int32_t* pt_row = p.page_table + (size_t)sg.b * p.max_pages;
    int page_of[kTabPerThread];
#pragma unroll
    for (int u = 0; u < kTabPerThread; ++u) {
      const int t = tid + u * kWavesF * 64;
      page_of[u] = 0;
      if (u * kWavesF * 64 < n_tiles) page_of[u] = pt_row[tile_pos(t < n_tiles ? t : n_tiles - 1) >> 7];
    }
#pragma unroll
    for (int u = 0; u < kTabPerThread; ++u) {
      const int t = tid + u * kWavesF * 64;
      if (t < n_tiles) {
        const int pos0 = tile_pos(t);
        *LDS_PTR(uint32_t, lds_tiles + t * 4) = ((uint32_t)page_of[u] * (kPage / kT) + ((pos0 / kT) & (kPage / kT - 1))) << 1 | (uint32_t)tile_full(pos0);
      }
    }
    __syncthreads();

    // ---- tile loader: wave w fetches rows [16 w, 16 w + 16) into stage it & 3, kept or not ----
    struct TileSrc {
      uint64_t rows, scales;  // the wave's first row and its scale (scalar registers)
      uint32_t st, lscale;    // LDS: the stage, the scales of the wave's rows
    };
    auto tile_entry = [&](int it) { return *LDS_PTR(uint32_t, lds_tiles + it * 4); };
    auto tile_src = [&](int it, uint32_t entry) -> TileSrc {
      const uint64_t t64 = __builtin_amdgcn_readfirstlane(entry) >> 1;
      TileSrc ts;
      ts.rows = (uint64_t)(uintptr_t)p.kv + wave * (kRowsPerWave * kRowF) + t64 * kStageF;
      ts.scales = (uint64_t)(uintptr_t)p.kv_scales + wave * (kRowsPerWave * 4) + t64 * kScaleF;
      ts.st = stage_base(it) + wave * 8192;
      ts.lscale = lds_scales + ((uint32_t)it & (kStagesF - 1)) * kScaleF + wave * kRowsPerWave * 4;
      return ts;
    };
    // Loads 0 .. 7: two rows each (row0 + 2 k for lanes 0..31, and the next, whose swizzles differ by
    // 2 (lane >> 5)), four to an LDS base: the immediate offset counts on both sides and is taken off the
    // lane's.  Load 8: the rope parts of the wave's 16 rows.  Load 9: their scales (16 lanes).
    // The lane's offsets are kept in registers; the loop has no instruction to spare for forming them.
    uint32_t dma_off[9];
#pragma unroll
    for (int k = 0; k < 8; ++k)
      dma_off[k] = ((n32 ^ (g << 1) ^ swf_main(2 * k)) << 4) + g * kRowF + (2 * k * kRowF - (k & 3) * 1024);
    dma_off[8] = (lane >> 2) * kRowF + kMainF + (((lane & 3) ^ ((lane >> 4) & 3)) << 4);
#pragma unroll
    for (int k = 0; k < 9; ++k) asm volatile("" : "+v"(dma_off[k]));
    const uint32_t lane4 = lane * 4;
    auto load_piece = [&](const TileSrc& ts, auto k_tag) {
      constexpr int k = decltype(k_tag)::value;
      if constexpr (k < 8) {
        if constexpr ((k & 3) == 0) set_lds_base(ts.st + k * 1024);
        load_lds16_at<(k & 3) * 1024>(ts.rows, dma_off[k]);
      } else if constexpr (k == 8) {
        set_lds_base(ts.st + kTailBaseF - wave * 7168);
        load_lds16_at<0>(ts.rows, dma_off[8]);
      } else {
        set_lds_base(ts.lscale);
        load_lds4_at(0xffffull, ts.scales, lane4);
      }
    };
    auto load_pieces = [&]<int... K>(const TileSrc& ts, std::integer_sequence<int, K...>) {
      (load_piece(ts, std::integral_constant<int, K>{}), ...);
    };
    auto issue_tile = [&](int it) {
      TileSrc ts = tile_src(it, tile_entry(it));
      settle_address(ts.rows, ts.scales);
      load_pieces(ts, std::make_integer_sequence<int, kDma>{});
    };

    // ---- Q: the block's 64 rows pass through stages 2 and 3 ----
    constexpr int kKS = kQK / 64;  // 9
    i32x8 qh[kKS], ql[kKS];
    float c_head = 0.f;
    if (n_tiles > 0) {
      const uint8_t* qbase = (const uint8_t*)p.q + (size_t)sg.b * p.H * kQRow;
      auto q_head = [&](int r) -> uint32_t { return h0 + r < p.H ? h0 + r : p.H - 1; };
      const uint32_t lds_q = lds0 + (2 + (wave >> 1)) * kStageF;  // (of the rows this wave fetches)
#pragma unroll
      for (int k = 0; k < 16; ++k) {  // wave w: rows 16 w .. 16 w + 15
        const int r = 16 * (wave & 1) + k;
        load_lds16<false>(lds_q + r * kQMain, qbase, q_head(16 * wave + k) * kQRow + ((lane ^ swq_main(r)) << 4));
      }
#pragma unroll
      for (int k = 0; k < 2; ++k) {
        const int r = 16 * (wave & 1) + 8 * k + (lane >> 3);
        load_lds16<false>(lds_q + kTailBaseF + (16 * (wave & 1) + 8 * k) * kQTail, qbase,
                          q_head(16 * wave + 8 * k + (lane >> 3)) * kQRow + kQMain + (((lane & 7) ^ swq_tail(r)) << 4));
      }
      issue_tile(0);
      if (n_tiles > 1) {
        issue_tile(1);
        wait_vm<2 * kDma>();
      } else {
        wait_vm<kDma>();
      }
      __syncthreads();
      // B operand of S^T: lane (head n32 of group hg, g) holds dims 64 ks + 32 g .. + 31, split in two e4m3 terms
      const uint32_t lq = lds0 + (2 + hg) * kStageF;
      auto q_chunk = [&](int c) -> u32x4 {  // 16 bytes = 8 dims
        return *LDS_PTR(u32x4, lq + (c < 64 ? n32 * kQMain + ((c ^ swq_main(n32)) << 4)
                                            : kTailBaseF + n32 * kQTail + (((c - 64) ^ swq_tail(n32)) << 4)));
      };
      auto q_raw = [&](int ks, int j) { return ks < 8 ? q_chunk(8 * ks + 4 * g + j) : q_chunk(64 + 4 * g + j); };
      u16x2 mx = {0, 0};
#pragma unroll
      for (int ks = 0; ks < kKS; ++ks)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const u32x4 r = q_raw(ks, j);
#pragma unroll
          for (int k = 0; k < 4; ++k) mx = __builtin_elementwise_max(mx, __builtin_bit_cast(u16x2, r[k] & 0x7fff7fffu));
        }
      // (bf16 magnitudes order like unsigned integers, and these convert to float exactly)
      const int m = (int)pair_max((float)(mx[0] > mx[1] ? mx[0] : mx[1]));
      int ex = m >> 7;
      ex = ex == 0 ? 0 : (ex > 254 ? 254 : ex) - 127 - 7;
      const float inv_s = __builtin_amdgcn_ldexpf(p.scale_log2 < 0.f ? -1.0f : 1.0f, -ex);
      c_head = __builtin_amdgcn_ldexpf(fabsf(p.scale_log2), ex);
      constexpr float kLo = (float)(1 << kQLoShiftF);
#pragma unroll
      for (int ks = 0; ks < kKS; ++ks)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const u32x4 r = q_raw(ks, j);
#pragma unroll
          for (int k2 = 0; k2 < 2; ++k2) {
            int hi = 0, lo = 0;
            {
              const float x0 = __builtin_bit_cast(float, r[2 * k2] << 16) * inv_s;
              const float x1 = __builtin_bit_cast(float, r[2 * k2] & 0xffff0000u) * inv_s;
              hi = __builtin_amdgcn_cvt_pk_fp8_f32(x0, x1, hi, false);
              const f32x2 back = __builtin_amdgcn_cvt_pk_f32_fp8(hi, false);
              lo = __builtin_amdgcn_cvt_pk_fp8_f32((x0 - back[0]) * kLo, (x1 - back[1]) * kLo, lo, false);
            }
            {
              const float x0 = __builtin_bit_cast(float, r[2 * k2 + 1] << 16) * inv_s;
              const float x1 = __builtin_bit_cast(float, r[2 * k2 + 1] & 0xffff0000u) * inv_s;
              hi = __builtin_amdgcn_cvt_pk_fp8_f32(x0, x1, hi, true);
              const f32x2 back = __builtin_amdgcn_cvt_pk_f32_fp8(hi, true);
              lo = __builtin_amdgcn_cvt_pk_fp8_f32((x0 - back[0]) * kLo, (x1 - back[1]) * kLo, lo, true);
            }
            qh[ks][j * 2 + k2] = hi;
            ql[ks][j * 2 + k2] = lo;
          }
        }
#pragma unroll
      for (int ks = 0; ks < kKS; ++ks) asm volatile("" : "+v"(qh[ks]), "+a"(ql[ks]));
      __syncthreads();  // Q has been read: its stages may be filled
      if (n_tiles > 2) issue_tile(2);
    }

    // ---- LDS addresses, relative to the stage ----
    // Kept per lane, relative to the stage; the swizzle-dependent part of a read's address is one XOR in
    // front of it (stage bases are multiples of 256 and the XORs touch bits 4 .. 7 only).
    const int row_s = 32 * th + n32;
    const uint32_t k_main = row_s * kMainF + (((2 * g) ^ swf_main(row_s)) << 4);  // K: chunks 4 ks + 2 g and the next
    const uint32_t k_tail = kTailBaseF + row_s * kTailF + (((2 * g) ^ swf_tail(row_s)) << 4);
    struct KAddr { uint32_t main, tail; };
    auto k_addr = [&](uint32_t st) -> KAddr { return {st + k_main, st + k_tail}; };
    auto load_k = [&](const KAddr& ka, int ks) -> i32x8 {
      const uint32_t a = ks < 8 ? ka.main ^ ((ks & 3) << 6) : ka.tail, imm = ks < 8 ? (ks >> 2) * 256 : 0;
      const i32x4 lo = *LDS_PTR(i32x4, a + imm), hi = *LDS_PTR(i32x4, (a ^ 16u) + imm);
      return i32x8{lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
    };
    // V^T, 8-bit transposing read: part pt of column block cb of lane l holds tokens 16 pt + 8 a + 4 g + b of
    // columns 128 wave + 32 cb .. (chunks 8 wave + 2 cb, + 1 of a row)
    const int ip = n16 >> 1, row_v = 8 * (ip >> 2) + 4 * g + (ip & 3);
    const uint32_t v_main = row_v * kMainF + (((((lane >> 4) & 1) ^ swf_main(row_v)) << 4) ^ ((wave & 1) << 7)) + (wave >> 1) * 256 + 8 * (lane & 1);
    auto load_v = [&](uint32_t va, int cb, int pt) -> i32x2 {
      return __builtin_amdgcn_ds_read_tr8_b64_v2i32(LDS_PTR(i32x2, (va ^ (cb << 5)) + pt * 16 * kMainF));
    };
    const uint32_t p_write = lds_p + (32 * hg + n32) * kPRowF + g * 32 + th * 16;
    const uint32_t p_read = lds_p + n32 * kPRowF + g * 32;
    const uint32_t kk_write = lds_kk + (th * kHB + 32 * hg + n32) * 4;
    const uint32_t kk_read = lds_kk + (g * kHB + n32) * 4;
    const uint32_t tok4 = (32 * th + 4 * g) * 4;  // the lane's tokens: 32 th + 8 q + 4 g .. + 3, q = 0..3
    const uint32_t lds_w = lds0 + kOffWScaleF + wave * 2 * kScaleF;
    const uint32_t stat_w = lds_stat + (th * kHB + 32 * hg + n32) * 4;
    const uint32_t stat_r = lds_stat + (32 * hg + n32) * 4;

    // block scales 2^0 and 2^-kQLoShift, held: written right in front of a matrix instruction they would
    // be read too early (two wait states, which nobody places in front of assembly)
    int one = 127, lo_scale = 127 - kQLoShiftF;
    asm volatile("s_nop 1" : "+v"(one), "+v"(lo_scale));
    float ref = 0.f, l_run = 0.f, lq_run = 0.f, mt_all = -INFINITY;
    float ref_exact = __builtin_nanf("");
    f32x16 acc[2][4];

#pragma unroll 1
    for (int attempt = 0; attempt < 2 && n_tiles > 0; ++attempt) {
      if (attempt > 0) {
        issue_tile(0);
        if (n_tiles > 1) issue_tile(1);
        if (n_tiles > 2) issue_tile(2);
      }
#pragma unroll
      for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int cb = 0; cb < 4; ++cb)
#pragma unroll
          for (int i = 0; i < 16; ++i) acc[a][cb][i] = 0.f;
      l_run = lq_run = 0.f;
      mt_all = -INFINITY;

      f32x16 s;  // S^T of the tile ahead
      f32x16 u;  // S^T times the token's scale, of the tile at hand
      float mu = -INFINITY;  // the lane's largest u
      int es = 0;            // exponent bound of its scales

      // Element i of a lane: token 32 th + (i / 4) * 8 + 4 g + i % 4 of the tile.
      // A tile that is not kept whole (uniform, one or two of a sequence).  First, what no query keeps: scales
      // replaced by the smallest normal number (every wave writes the same), value rows cleared
      // (0 * NaN would poison PV).
      auto clear_scales = [&](int it, int pos0) {
        const int l = fresh_lane();
        if (!retained(pos0 + l, L, p.S, p.Wu))
          *LDS_PTR(float, lds_scales + ((uint32_t)it & (kStagesF - 1)) * kScaleF + l * 4) = 1.1754944e-38f;
      };
      auto clear_rows = [&](int it, int pos0) {
        const int l = fresh_lane();
        const uint32_t st = stage_base(it);
        for (int k = l; k < kRowsPerWave * 32; k += 64) {
          const int r = wave * kRowsPerWave + (k >> 5);
          if (!retained(pos0 + r, L, p.S, p.Wu)) *LDS_PTR(u32x4, st + r * kMainF + (k & 31) * 16) = u32x4{0, 0, 0, 0};
        }
      };
      // Then, per query: logits of what it does not keep.
      auto mask_logits = [&](int pos0) {
        const int l = fresh_lane();
        // length of the sequence that the lane's query sees (several queries: cut after its own token)
        const int head = h0 + 32 * hg + (l & 31);
        const int Lq = L - (p.T - 1 - (head < p.H ? head : p.H - 1) / p.Hq);
        mu = -INFINITY;
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          const int j = pos0 + 32 * th + (i >> 2) * 8 + 4 * (l >> 5) + (i & 3);
          u[i] = retained(j, Lq, p.S, p.W) ? u[i] : -INFINITY;
          mu = fmaxf(mu, u[i]);
        }
      };
      // es: every scale of the token half < 2^es, es >= -100 (from the lane's 16 tokens and its partner's)
      auto half_exp = [&](const f32x4 (&sc)[4]) -> int {
        float m = 0.f;
#pragma unroll
        for (int i = 0; i < 16; ++i) m = fmaxf(m, fabsf(sc[i >> 2][i & 3]));
        const int es = (int)(__builtin_bit_cast(uint32_t, pair_max(m)) >> 23) - 126;
        return es < -100 ? -100 : es;
      };
      // Weight scales of the half for this wave's use (lane = token of the tile) and their reciprocals: the
      // token's scale, raised to 2^(es - 10) so that one far below the half's largest stays in the rounded sum.
      auto put_weight_scales = [&](float sc, int es) {
        const float w = fmaxf(sc, __builtin_amdgcn_ldexpf(1.0f, es - 10));
        *LDS_PTR(float, lds_w + lane4) = w;
        *LDS_PTR(float, lds_w + kScaleF + lane4) = __builtin_amdgcn_rcpf(w);
      };
      auto scale_quad = [&](int q, f32x4 sc) {
#pragma unroll
        for (int i = 4 * q; i < 4 * q + 4; ++i) {
          u[i] = s[i] * sc[i & 3];
          mu = fmaxf(mu, u[i]);
        }
      };
      // ---- tile 0: S^T, reference ----
      {
        const int later = n_tiles - 1;
        if (later >= 2) wait_vm<2 * kDma>();
        else if (later == 1) wait_vm<kDma>();
        else wait_vm<0>();
        __syncthreads();
        const KAddr ka0 = k_addr(stage_base(0));
#pragma unroll
        for (int ks = 0; ks < kKS; ++ks) {
          const i32x8 k8 = load_k(ka0, ks);
          if (ks == 0) mfma_s_first(s, k8, qh[0]);
          else mfma_s_hi(s, k8, qh[ks]);
          mfma_s_lo(s, k8, ql[ks], one, lo_scale);
        }
        settle_s(s);
        const int pos0 = tile_pos(0);
        const bool part = !tile_full(pos0);
        if (part) clear_scales(0, pos0);
        if (part) clear_rows(0, pos0);  // (of a tile's bytes, K is masked, and V is read behind more barriers)
        const float sc_t = *LDS_PTR(float, lds_scales + lane4);
        mu = -INFINITY;
        f32x4 sc[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) sc[q] = *LDS_PTR(f32x4, lds_scales + tok4 + q * 32);
#pragma unroll
        for (int q = 0; q < 4; ++q) scale_quad(q, sc[q]);
        if (part) mask_logits(pos0);
        const float mx = pair_max(mu * c_head);
        if (g == 0) *LDS_PTR(float, stat_w) = mx;
        if (later >= 2) wait_vm<kDma>();
        else wait_vm<0>();
        __syncthreads();  // (also: tile 1 is visible)
        const float m2 = fmaxf(*LDS_PTR(float, stat_r), *LDS_PTR(float, stat_r + kHB * 4));
        ref = ref_exact == ref_exact ? ref_exact : (m2 == -INFINITY || m2 != m2) ? 0.f : ceilf(m2);
        es = half_exp(sc);
        put_weight_scales(sc_t, es);
      }
      const int t3 = n_tiles > 3 ? 3 : n_tiles - 1;
      TileSrc ts = tile_src(t3, tile_entry(t3));
      settle_address(ts.rows, ts.scales);

      // One iteration per tile, one stream of 26 matrix instructions: S^T of tile it + 1 (18, a dependent chain),
      // behind them the weights of tile it, the loads of tile it + 3 and the operand requests; then PV of
      // tile it (8), behind them the logits of tile it + 1 are scaled.  Both barriers lie inside the
      // stream, so that the matrix pipeline does not drain at them:
      //   A  (behind S^T 1) every wave is done with PV of tile it - 1: its stage may be loaded, the weights' slots
      //      written;
      //   B  (behind S^T 13) the weights of tile it and all of tile it + 2 are visible.
      // The first K fragments of tile it + 2 are requested behind the last PV instructions.
      // (Behind the last tile S^T is computed once more from what the stage holds and not used: a copy of the
      // loop body without it makes the compiler move accumulators between registers.)
      constexpr int kRing = 3;
      i32x8 fr[kRing];
      f32x4 w[2], rw[2];
      {
        const KAddr ka = k_addr(stage_base(1));
#pragma unroll
        for (int k = 0; k < kRing; ++k) fr[k] = load_k(ka, k);
        w[0] = *LDS_PTR(f32x4, lds_w + tok4);
        rw[0] = *LDS_PTR(f32x4, lds_w + kScaleF + tok4);
      }
      auto iteration = [&](const int it) {
        const bool next = it + 1 < n_tiles;
        const uint32_t st = stage_base(it), st1 = stage_base(it + 1);
        i32x8 v[4], pf[2];
        i32x4 pk;
        f32x4 sc[4];
        float ls0 = 0.f, ls1 = 0.f, lq0 = 0.f, lq1 = 0.f, rk = 0.f, sc_t = 0.f;
        int kk = 0, sb[2];
        uint32_t entry1 = 0, entry4 = 0;
        bool part = false;
        const KAddr ka = k_addr(st1);
        const uint32_t va = st + v_main;
        const uint32_t scales = lds_scales + ((uint32_t)(it + 1) & (kStagesF - 1)) * kScaleF;
        const int t4 = it + 4 < n_tiles ? it + 4 : n_tiles - 1;
        const bool more = it + 3 < n_tiles;
        // Weights of elements 2 j, 2 j + 1 in three parts, which consecutive matrix instructions get of three
        // different pairs: a lone wave waits out the latency of every dependent instruction, so what stands
        // together should not depend on each other.
        float e[3][2];
        auto weights_e = [&](auto j_tag) {
          constexpr int j = decltype(j_tag)::value, i = 2 * j;
          e[j % 3][0] = __builtin_amdgcn_exp2f(fmaf(u[i], c_head, -rk));
          e[j % 3][1] = __builtin_amdgcn_exp2f(fmaf(u[i + 1], c_head, -rk));
        };
        auto weights_c = [&](auto j_tag) {
          constexpr int j = decltype(j_tag)::value, q = j / 2, k = (2 * j) & 3;
          const float e0 = e[j % 3][0], e1 = e[j % 3][1];
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
        auto step = [&](auto m_tag) {
          constexpr int m = decltype(m_tag)::value, ks = m >> 1;
          if constexpr (m == 0) mfma_s_first(s, fr[0], qh[0]);
          else if constexpr ((m & 1) == 0) mfma_s_hi(s, fr[ks % kRing], qh[ks]);
          else mfma_s_lo(s, fr[ks % kRing], ql[ks], one, lo_scale);
          if constexpr ((m & 1) == 1 && ks + kRing < kKS) fr[ks % kRing] = load_k(ka, ks + kRing);
          if constexpr (m == 0) {
            // Block exponent kk of the head's 32 weights: the largest lands in [2^7, 2^8).
            const float mt = pair_max(fmaf(mu, c_head, -ref));
            mt_all = fmaxf(mt_all, mt);
            int k = (int)ceilf(mt) - 8 + es;
            k = k < -126 ? -126 : k > 126 ? 126 : k;
            kk = mt == -INFINITY ? 0 : k;
            rk = ref + (float)kk;
          }
          if constexpr (m == 1) {
            asm volatile("" : : : "memory");
            __builtin_amdgcn_s_barrier();  // A (its waves' LDS reads have been used: nothing to wait for)
            asm volatile("" : : : "memory");
          }
          if constexpr (m >= 1 && m < 9) weights_e(std::integral_constant<int, m - 1>{});
          if constexpr (m >= 2 && m < 10) weights_c(std::integral_constant<int, m - 2>{});
          if constexpr (m >= 3 && m < 11) weights_l(std::integral_constant<int, m - 3>{});
          if constexpr (m == 2 || m == 4 || m == 6) {  // weight scales of quad m / 2 (first used behind m + 2)
            constexpr int q = m / 2;
            w[q & 1] = *LDS_PTR(f32x4, lds_w + tok4 + q * 32);
          }
          if constexpr (m == 3 || m == 5 || m == 7) {  // (its reciprocals: behind m + 2)
            constexpr int q = m / 2;
            rw[q & 1] = *LDS_PTR(f32x4, lds_w + kScaleF + tok4 + q * 32);
          }
          if constexpr (m == 10) {
            *LDS_PTR(i32x4, p_write) = pk;
            *LDS_PTR(int, kk_write) = 127 + kk;  // (the same in both lanes of a head)
          }
          if constexpr (m == 2 || m == 5 || m == 8 || m == 11) {  // three loads each, the last one
            if (more) {
              constexpr int k = m - 2;
              load_piece(ts, std::integral_constant<int, k>{});
              if constexpr (k + 1 < kDma) load_piece(ts, std::integral_constant<int, k + 1>{});
              if constexpr (k + 2 < kDma) load_piece(ts, std::integral_constant<int, k + 2>{});
            }
          }
          if constexpr (m == 10) {
            entry1 = tile_entry(next ? it + 1 : it);
            entry4 = tile_entry(t4);
          }
          if constexpr (m == 12) part = next && !(__builtin_amdgcn_readfirstlane(entry1) & 1);
          if constexpr (m >= 9 && m < 13) {
            constexpr int cb = m - 9;
#pragma unroll
            for (int pt = 0; pt < 4; ++pt) {
              const i32x2 t = load_v(va, cb, pt);
              v[cb][2 * pt] = t[0];
              v[cb][2 * pt + 1] = t[1];
            }
          }
          if constexpr (m == 13) {
            if (it + 3 < n_tiles) wait_vm<kDma>();
            else wait_vm<0>();
            __syncthreads();  // B
#pragma unroll
            for (int a = 0; a < 2; ++a) {
              const i32x4 lo = *LDS_PTR(i32x4, p_read + a * 32 * kPRowF), hi = *LDS_PTR(i32x4, p_read + a * 32 * kPRowF + 16);
              pf[a] = i32x8{lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
              sb[a] = *LDS_PTR(int, kk_read + a * 32 * 4);  // (half g from lane (head, g))
            }
          }
          if constexpr (m == 14) {
            l_run += __builtin_amdgcn_ldexpf(ls0 + ls1, kk);
            lq_run += __builtin_amdgcn_ldexpf(lq0 + lq1, kk);
            asm volatile("" : "+v"(l_run), "+v"(lq_run));
            if (part) {
              const int pos1 = tile_pos(it + 1);
              clear_scales(it + 1, pos1);
              clear_rows(it + 1, pos1);
            }
            sc_t = *LDS_PTR(float, scales + lane4);
#pragma unroll
            for (int q = 0; q < 4; ++q) sc[q] = *LDS_PTR(f32x4, scales + tok4 + q * 32);
          }
          if constexpr (m == 15) ts = tile_src(t4, entry4);
          if constexpr (m == 16) {
            es = half_exp(sc);
            asm volatile("" : "+v"(es));
          }
          if constexpr (m == 17) put_weight_scales(sc_t, es);
          __builtin_amdgcn_sched_barrier(0);
        };
        [&]<int... M>(std::integer_sequence<int, M...>) {
          (step(std::integral_constant<int, M>{}), ...);
        }(std::make_integer_sequence<int, 2 * kKS>{});
        mu = -INFINITY;
        const KAddr kn = k_addr(stage_base(it + 2));
        auto pv = [&](auto m_tag) {
          constexpr int m = decltype(m_tag)::value, a = m >> 2, cb = m & 3;
          mfma_o(acc[a][cb], v[cb], pf[a], one, sb[a]);
          if constexpr (m == 2) asm volatile("s_nop 11" : "+v"(s));  // nothing reads S^T ahead of this point
          if constexpr (m >= 3 && m < 7) {
            scale_quad(m - 3, sc[m - 3]);
            asm volatile("" : "+v"(mu));
          }
          if constexpr (m >= 4 && m < 4 + kRing) fr[m - 4] = load_k(kn, m - 4);
          if constexpr (m == 4) {
            w[0] = *LDS_PTR(f32x4, lds_w + tok4);
            rw[0] = *LDS_PTR(f32x4, lds_w + kScaleF + tok4);
          }
          __builtin_amdgcn_sched_barrier(0);
        };
        [&]<int... M>(std::integer_sequence<int, M...>) {
          (pv(std::integral_constant<int, M>{}), ...);
        }(std::make_integer_sequence<int, 8>{});
        if (part) mask_logits(tile_pos(it + 1));
        settle_address(ts.rows, ts.scales);
      };
#pragma unroll 1
      for (int it = 0; it < n_tiles; ++it) iteration(it);
      settle_o(acc);

      // ---- per-head statistics of both token halves ----
      const float l_q = pair_sum(l_run), lq_q = pair_sum(lq_run);
      __syncthreads();  // (PV has read its operands; the statistics' slots were last read in the first tile)
      if (g == 0) {
        *LDS_PTR(float, stat_w) = mt_all;
        *LDS_PTR(float, stat_w + kStatF * 4) = l_q;
        *LDS_PTR(float, stat_w + 2 * kStatF * 4) = lq_q;
        *LDS_PTR(float, stat_w + 3 * kStatF * 4) = ref;
      }
      __syncthreads();
      // (every wave looks at all 64 heads, so all take the same way)
      const float m2 = fmaxf(*LDS_PTR(float, lds_stat + lane * 4), *LDS_PTR(float, lds_stat + (kHB + lane) * 4));
      const bool off = m2 > kRefSlackF || (m2 < -kRefSlackF && m2 != -INFINITY);
      if (attempt > 0 || !__any(off)) break;
      const float m3 = fmaxf(*LDS_PTR(float, stat_r), *LDS_PTR(float, stat_r + kHB * 4));
      ref_exact = m3 == -INFINITY ? 0.f : ref + ceilf(m3);
    }

    // ---- epilogue: normalise by the rounded weights' sum, transpose through LDS, write 128 columns ----
    auto stat = [&](int k, int half, int h) { return *LDS_PTR(float, lds_stat + (k * kStatF + half * kHB + h) * 4); };
    const int lane_e = fresh_lane();
    const int n16e = lane_e & 15, n32e = lane_e & 31, ge = lane_e >> 5;
    const bool final_out = sg.slot < 0;
    const int heads_here = p.H - h0 < kHB ? p.H - h0 : kHB;
    if (wave == 0 && lane_e < heads_here) {
      const float lse = n_tiles > 0 ? (stat(3, 0, lane_e) + __builtin_amdgcn_logf(stat(1, 0, lane_e) + stat(1, 1, lane_e))) * 0.6931471805599453f
                                    : -INFINITY;
      if (final_out) p.lse[(size_t)sg.b * p.H + h0 + lane_e] = lse;
      else p.part_lse[(size_t)sg.slot * kHB + lane_e] = lse;
    }
    const size_t row0 = final_out ? (size_t)sg.b * p.H + h0 : (size_t)sg.slot * kHB;
    constexpr int kOutMax = 128 * 4 + 16;
    const uint32_t ost = lds0 + wave * kHB * kOutMax;
#pragma unroll
    for (int a = 0; a < 2; ++a) {
      const float lq_tot = n_tiles > 0 ? stat(2, 0, 32 * a + n32e) + stat(2, 1, 32 * a + n32e) : 0.f;
      const float inv = lq_tot != 0.f ? 1.0f / lq_tot : 0.f;
      auto value = [&](int cb, int i) { return n_tiles > 0 ? acc[a][cb][i] * inv : 0.f; };
#pragma unroll
      for (int cb = 0; cb < 4; ++cb)
#pragma unroll
        for (int i4 = 0; i4 < 4; ++i4) {
          const int col = cb * 32 + i4 * 8 + ge * 4;
          const f32x4 v = {value(cb, i4 * 4), value(cb, i4 * 4 + 1), value(cb, i4 * 4 + 2), value(cb, i4 * 4 + 3)};
          if (!p.out_fp32)
            *LDS_PTR(bf16x4, ost + (32 * a + n32e) * (128 * 2 + 16) + col * 2) = bf16x4{(__bf16)v[0], (__bf16)v[1], (__bf16)v[2], (__bf16)v[3]};
          else
            *LDS_PTR(f32x4, ost + (32 * a + n32e) * kOutMax + col * 4) = v;
        }
    }
    if (!p.out_fp32) {
      uint8_t* dst = (uint8_t*)(final_out ? p.out : p.part_o) + row0 * (kV * 2) + wave * 256 + n16e * 16;
#pragma unroll
      for (int k = 0; k < kHB / 4; ++k) {
        const int h = 4 * k + (lane_e >> 4);
        if (h < heads_here) *(u32x4*)(dst + (size_t)h * (kV * 2)) = *LDS_PTR(u32x4, ost + h * (128 * 2 + 16) + n16e * 16);
      }
    } else {
      uint8_t* dst = (uint8_t*)(final_out ? p.out : p.part_o) + row0 * (kV * 4) + wave * 512 + n32e * 16;
#pragma unroll
      for (int k = 0; k < kHB / 2; ++k) {
        const int h = 2 * k + ge;
        if (h < heads_here) *(u32x4*)(dst + (size_t)h * (kV * 4)) = *LDS_PTR(u32x4, ost + h * kOutMax + n32e * 16);
      }
    }
    __syncthreads();  // staging rows and page table are free again before the next segment
  }
}

hipError_t init_fp8_64_kernel() {
  return hipFuncSetAttribute(reinterpret_cast<const void*>(&decode_fp8_64_kernel), hipFuncAttributeMaxDynamicSharedMemorySize, kLdsF);
}

hipError_t launch_decode_fp8_64(const DecodeParams& p, int n_units, hipStream_t stream) {
  if (n_units <= 0) return hipSuccess;
  if (p.xcds < 1 || p.head_block != kHB) return hipErrorInvalidValue;
  const dim3 grid(((n_units + p.xcds - 1) / p.xcds) * p.xcds), block(kWavesF * 64);
  hipLaunchKernelGGL(decode_fp8_64_kernel, grid, block, kLdsF, stream, p);
  return hipGetLastError();
}

}  // namespace omniattn
