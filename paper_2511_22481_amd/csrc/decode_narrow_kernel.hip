// gfx950 kernel for sparse MLA decode with few head rows per sequence (one head-sharded rank, or
// few sequences whose heads are dealt to several work units): blocks of 32 head rows, bf16 or fp8
// cache.  (Paper section 3.2.1: softmax(q K_M^T * scale) V_M with M = sinks + recents.)
//
// The kernels for full head blocks give each wave 32 heads of its own, so with 32 or fewer rows one
// wave works and three repeat it: every wave reads every K row and transposes every V row out of LDS.
// Here the four waves of a work group share the arithmetic of one block of 32 head rows, and a tile
// passes through LDS once:
//   S^T   wave (th, hh) computes the logits of token half th and head half hh (16x16 matrix
//         instructions, K from the LDS tile, Q of 16 heads in registers);
//   P     the softmax weights of the tile meet in LDS (2 KB), already in the operand order of
//   PV    where wave w accumulates output columns 128 w .. 128 w + 127 of all 32 heads.
// That leaves the loop bound by the cache rows it streams, 1.4 us per tile and compute unit (6.7 TB/s
// chip-wide; a kernel for full head blocks takes 2.1 us bf16 at 16 heads).  Four LDS stages of 36,864 bytes (32
// bf16 or 64 fp8 tokens) are filled by direct global->LDS loads, three tiles ahead of the one in
// use, with two barriers per tile.  It is written with compiler builtins; bf16: all K fragments of a tile, and its V
// fragments, are requested ahead of the matrix instructions that use them (128 sequences of 2176 tokens, 16 heads: 60.7 -> 58.4
// us; one sequence of 128 heads 15.0 -> 14.6; four of 16 heads 10.7 -> 10.4; their start is quicker since, see there).
// us per decode against blocks of 128 rows: 128 sequences of 2176 kept tokens, 16 heads bf16 88 -> 59, fp8 94 -> 43; one
// sequence of 128 heads 26 -> 14.9.  (64 heads are decode_mid_kernel's.)
// Softmax reference (fixed per segment, second run if a logit leaves its range), weight formats,
// masking and partial rows are those of the kernels for full head blocks.  The 8-bit product of 128 dims aligns
// each 64 of them to their largest, as the one of 64 dims does: the logits carry the same error.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "decode_common.h"

namespace omniattn {

namespace {

constexpr int kWavesN = 4;
constexpr int kStagesN = 4;
constexpr int kStageN = 36864;
constexpr int kTailBaseN = 32768;
constexpr int kPRow = 80;  // a head's weights of one tile: 64 bytes, padded to an odd multiple of 16
constexpr int kStatN = 2 * kHeadsPerWave;  // (token half, head)
// stages | weights | block exponents | per-head statistics (4) | fp8: token scales, a copy per wave | tile table
constexpr int kOffP = kStagesN * kStageN;
constexpr int kOffKK = kOffP + kHeadsPerWave * kPRow;
constexpr int kOffStat = kOffKK + kStatN * 4;
constexpr int kOffTiles = kOffStat + 4 * kStatN * 4;
constexpr int kOffScales = kOffTiles + kMaxSegTiles * 4;
constexpr int kScaleStageN = kTileFp8 * 4;
constexpr int kLdsNarrowBf16 = kOffScales;
constexpr int kLdsNarrowFp8 = kOffScales + kWavesN * kStagesN * kScaleStageN;
static_assert(kLdsNarrowFp8 <= 160 * 1024, "LDS of one compute unit");

constexpr float kRefSlackN = 64.f;  // see the bf16 kernel: fixed softmax reference with retry

// LDS layout of a stage: the value part of the rows, then their rope parts; 16-byte chunks XORed with a
// function of the row, as in the kernels for full head blocks (16 consecutive rows at one chunk index
// fall into 16 different bank groups, and so do the pieces of a transposing read).
template <bool FP8>
struct Lay;
template <>
struct Lay<false> {
  static constexpr int kTok = kTile, kMain = 1024, kTail = 128, kRow = 1152;
  __host__ __device__ static constexpr int sw_main(int r) { return ((r & 3) << 2) | ((r >> 2) & 3); }
  __host__ __device__ static constexpr int sw_tail(int r) { return (r >> 1) & 7; }
};
template <>
struct Lay<true> {
  static constexpr int kTok = kTileFp8, kMain = 512, kTail = 64, kRow = 576;
  __host__ __device__ static constexpr int sw_main(int r) { return ((r & 3) << 1) | ((r >> 2) & 1) | (((r >> 3) & 1) << 3); }
  __host__ __device__ static constexpr int sw_tail(int r) { return (r >> 2) & 3; }
};

// A lane's value combined with those of lanes l ^ 16, l ^ 32 and l ^ 48 (the four lanes of a head in
// the 16x16 result layout).
__device__ __forceinline__ float quad_max(float x) {
  float a = x, b = x;
  swap16(a, b);
  a = b = fmaxf(a, b);
  swap32(a, b);
  return fmaxf(a, b);
}
__device__ __forceinline__ float quad_sum(float x) {
  float a = x, b = x;
  swap16(a, b);
  a = b = a + b;
  swap32(a, b);
  return a + b;
}

}  // namespace

template <bool FP8>
__global__ __launch_bounds__(kWavesN * 64, 1) void decode_narrow_kernel(DecodeParams p) {
  using Y = Lay<FP8>;
  extern __shared__ __attribute__((aligned(16))) uint8_t lds_raw[];
  const uint32_t lds0 = (uint32_t)(uintptr_t)lds_raw;
  const uint32_t lds_p = lds0 + kOffP, lds_kk = lds0 + kOffKK, lds_stat = lds0 + kOffStat;
  const uint32_t lds_tiles = lds0 + kOffTiles, lds_scales = lds0 + kOffScales;
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int th = wave & 1, hh = wave >> 1;
  const int n16 = lane & 15, q4 = lane >> 4;
  const int n32 = lane & 31, g = lane >> 5;

  constexpr int kRowsPerWave = Y::kTok / kWavesN;  // 8 or 16
  // direct loads per wave and tile: eight of 1 KB of value bytes, one of rope bytes, fp8: one of scales
  constexpr int kMainLoads = kRowsPerWave * Y::kMain / 1024;
  constexpr int kDmaPerTile = kMainLoads + 1 + (FP8 ? 1 : 0);
  static_assert(kMainLoads == 8 && kRowsPerWave * Y::kTail == 1024);

  // unit mapping as in the kernels for full head blocks: consecutive units share an XCD
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
    const int L = sg.L;
    const int h0 = sg.hb * kHeadsPerWave;
    const int head_s = h0 + 16 * hh + n16;  // the head whose logits this lane computes
    const int head_q = head_s < p.H ? head_s : p.H - 1;  // (past the last: repeats it, never written)
    const TileLayout tl = tile_layout(L, p.S, p.Wu, Y::kTok);
    const int n_tiles = sg.tile_hi - sg.tile_lo;
    const int L0 = L - (p.T - 1);
    const int sink_end = p.S < L0 ? p.S : L0;
    // length of the sequence that the lane's query sees (several queries: cut after its own token)
    const int Lq = L - (p.T - 1 - head_q / p.Hq);

    auto tile_pos = [&](int it) { return tl.logical(sg.tile_lo + it) * Y::kTok; };
    auto stage_base = [&](int it) -> uint32_t { return lds0 + ((uint32_t)it & (kStagesN - 1)) * kStageN; };
    auto tile_full = [&](int pos0) {
      return (pos0 + Y::kTok <= sink_end) || (pos0 >= L - p.W && pos0 + Y::kTok <= L0);
    };

    // ---- tile table (unit of the cache that holds the tile, bit 0 = every position kept) and Q ----
    // A call of a few tiles per unit is a chain of round trips: unit header, page-table entries, rows.  The entries go straight
    // to the table and the block's 32 query rows (1152 bytes each, through stage 3, laid out like bf16 cache rows) right behind
    // them, so that Q travels with them and is read, and split, while the first tiles are on their way; then each thread turns
    // its own entries into the table's.  us per decode, entries through registers and Q requested with tile 0 -> now: one
    // sequence, 128 heads, 2176 tokens 14.92 -> 14.54 (fp8 15.22 -> 15.02), four of 576 tokens, 16 heads 10.30 -> 10.17
    // (fp8 11.68 -> 11.32); 128 of 2176, 16 heads, 59, take the time they took.
    // (A segment without tiles reads no entry: its row of the table may hold nothing valid.  Query rows past the last head
    // repeat it; their results are never written.)
    constexpr int kTabPerThread = kMaxSegTiles / (kWavesN * 64);
    constexpr int kQLoads = 9;
    const uint32_t lds_q = lds0 + 3 * kStageN;
    using QY = Lay<false>;
    if (n_tiles > 0) {
      const uint8_t* pt_row = (const uint8_t*)(p.page_table + (size_t)sg.b * p.max_pages);
#pragma unroll
      for (int u = 0; u < kTabPerThread; ++u) {
        const int t = tid + u * kWavesN * 64, t0 = (u * kWavesN + wave) * 64;
        if (t0 < n_tiles) load_lds4(lds_tiles + t0 * 4, pt_row, (uint32_t)(tile_pos(t < n_tiles ? t : n_tiles - 1) >> 7) << 2);
      }
      const uint8_t* qbase = (const uint8_t*)p.q + (size_t)sg.b * p.H * QY::kRow;
      auto q_head = [&](int r) -> uint32_t { return h0 + r < p.H ? h0 + r : p.H - 1; };
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        const int r = 8 * wave + k;
        load_lds16<false>(lds_q + r * QY::kMain, qbase, q_head(r) * QY::kRow + ((lane ^ QY::sw_main(r)) << 4));
      }
      const int r = 8 * wave + (lane >> 3);
      load_lds16<false>(lds_q + kTailBaseN + wave * 1024, qbase, q_head(r) * QY::kRow + QY::kMain + (((lane & 7) ^ QY::sw_tail(r)) << 4));
      wait_vm<kQLoads>();
#pragma unroll
      for (int u = 0; u < kTabPerThread; ++u) {
        const int t = tid + u * kWavesN * 64;
        if (t < n_tiles) {
          const int pos0 = tile_pos(t);
          const uint32_t page = *LDS_PTR(uint32_t, lds_tiles + t * 4);
          *LDS_PTR(uint32_t, lds_tiles + t * 4) = (page * (kPage / Y::kTok) + ((pos0 / Y::kTok) & (kPage / Y::kTok - 1))) << 1 | (uint32_t)tile_full(pos0);
        }
      }
      __syncthreads();
    }

    // ---- tile loader: wave w fetches rows [w * kRowsPerWave, ...) into stage it & 3 ----
    // All rows of a tile are fetched, kept or not (a tile lies inside one page, so they exist); what
    // is not kept is masked and cleared when the tile is used.
    auto issue_tile = [&](int it) {
      const uint64_t unit_of_cache = (uint32_t)__builtin_amdgcn_readfirstlane(*LDS_PTR(uint32_t, lds_tiles + it * 4)) >> 1;
      const uint8_t* gbase = p.kv + unit_of_cache * kStageN;
      const uint32_t st = stage_base(it);
      const int row0 = wave * kRowsPerWave;
#pragma unroll
      for (int k = 0; k < kMainLoads; ++k) {
        const int row = FP8 ? row0 + 2 * k + g : row0 + k;  // fp8: two rows, lanes 0..31 and 32..63
        const uint32_t pos = (FP8 ? lane & 31 : lane) ^ Y::sw_main(row);
        load_lds16<true>(st + wave * 8192 + k * 1024, gbase, row * Y::kRow + (pos << 4));
      }
      constexpr int kTailChunks = Y::kTail / 16;
      const int row = row0 + lane / kTailChunks;
      load_lds16<true>(st + kTailBaseN + wave * 1024, gbase,
                       row * Y::kRow + Y::kMain + (((lane % kTailChunks) ^ Y::sw_tail(row)) << 4));
      if constexpr (FP8)
        load_lds4(lds_scales + (wave * kStagesN + (it & (kStagesN - 1))) * kScaleStageN,
                  (const uint8_t*)(p.kv_scales + unit_of_cache * Y::kTok), lane << 2);
    };
    // this wave's share of tile `it` has arrived; later tiles (at most two were requested) may be in flight
    auto wait_tile = [&](int it) {
      const int later = n_tiles - 1 - it;
      if (later >= 2) wait_vm<2 * kDmaPerTile>();
      else if (later == 1) wait_vm<kDmaPerTile>();
      else wait_vm<0>();
    };

    // Q, which is older than the tiles, is read (and split) while they are on their way.
    if (n_tiles > 0) {
      issue_tile(0);
      if (n_tiles > 1) issue_tile(1);
      if (n_tiles > 2) issue_tile(2);
      if (n_tiles > 2) wait_vm<3 * kDmaPerTile>();
      else if (n_tiles == 2) wait_vm<2 * kDmaPerTile>();
      else wait_vm<kDmaPerTile>();
      __syncthreads();
    }
    // The B operand of S^T, 16 heads.  bf16: lane (head n16, q4) holds dims 32 ks + 8 q4 .. + 7, ks = 0..17.
    // fp8: dims 128 ks + 32 q4 .. + 31, ks = 0..4 (ks = 4: q4 >= 2 is past the row and zero), as two
    // e4m3 terms (see decode_mid_kernel.hip).
    constexpr int kKS = FP8 ? 5 : kQK / 32;
    bf16x8 qf[FP8 ? 1 : kKS];
    i32x8 qh[FP8 ? kKS : 1], ql[FP8 ? kKS : 1];
    u32x4 raw[FP8 ? kKS : 1][4];
    float c_head = p.scale_log2;  // logits are raw products times c_head, in the log2 domain
    {
      const int r = 16 * hh + n16;
      auto q_chunk = [&](int c) -> u32x4 {
        return *LDS_PTR(u32x4, lds_q + (c < 64 ? r * QY::kMain + ((c ^ QY::sw_main(r)) << 4)
                                               : kTailBaseN + r * QY::kTail + (((c - 64) ^ QY::sw_tail(r)) << 4)));
      };
      if constexpr (FP8) {
#pragma unroll
        for (int ks = 0; ks < kKS; ++ks)
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            raw[ks][j] = u32x4{0, 0, 0, 0};
            if (ks < 4) raw[ks][j] = q_chunk(16 * ks + 4 * q4 + j);
            else if (q4 < 2) raw[ks][j] = q_chunk(64 + 4 * q4 + j);
          }
      } else {
#pragma unroll
        for (int ks = 0; ks < kKS; ++ks) qf[ks] = __builtin_bit_cast(bf16x8, q_chunk(4 * ks + q4));
      }
    }
    if constexpr (FP8) {
      // split of the query row: q = 2^ex (hi + lo / 16), row maximum in [128, 256) (see decode_common.h)
      float mx_q = 0.f;
#pragma unroll
      for (int ks = 0; ks < kKS; ++ks)
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
          for (int k = 0; k < 4; k += 2) mx_q = bf16_max4(mx_q, raw[ks][j][k], raw[ks][j][k + 1]);
      const int ex = split_q_exponent(__builtin_bit_cast(uint32_t, quad_max(mx_q)) >> 16);
      const float scale = __builtin_amdgcn_ldexpf(1.0f, ex), inv = __builtin_amdgcn_ldexpf(1.0f, -ex);
      c_head = split_q_factor(p.scale_log2, ex);
      const uint32_t sign = p.scale_log2 < 0.f ? 0x80008000u : 0u;
#pragma unroll
      for (int ks = 0; ks < kKS; ++ks)
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
          for (int k2 = 0; k2 < 2; ++k2) {
            const u32x2 t = split_q4(raw[ks][j][k2 * 2] ^ sign, raw[ks][j][k2 * 2 + 1] ^ sign, scale, inv);
            qh[ks][j * 2 + k2] = t[0];
            ql[ks][j * 2 + k2] = t[1];
          }
    }

    // ---- LDS addresses (relative to the stage) ----
    constexpr int kGroups = FP8 ? 2 : 1;  // groups of 16 tokens whose logits the wave computes
    const int row_s = (FP8 ? 32 : 16) * th + n16;  // its first group's token row of the A operand
    uint32_t am[kGroups], at[kGroups];
#pragma unroll
    for (int a = 0; a < kGroups; ++a) {
      const int r = row_s + 16 * a;
      const int c0 = FP8 ? 2 * q4 : q4;
      am[a] = r * Y::kMain + ((c0 ^ Y::sw_main(r)) << 4);
      at[a] = kTailBaseN + r * Y::kTail + (((FP8 ? 2 * (q4 & 1) : q4) ^ Y::sw_tail(r)) << 4);
    }
    // V^T, transposing reads: 4 tokens x 16 columns (bf16) or 8 tokens x 16 columns (fp8) per 16 lanes
    uint32_t vb[2];
    if constexpr (FP8) {
      const int ip = n16 >> 1;
      const int r = 8 * (ip >> 2) + 4 * g + (ip & 3);
      vb[0] = r * Y::kMain + (((q4 & 1) ^ Y::sw_main(r)) << 4) + 8 * (lane & 1);
      vb[1] = 0;
    } else {
      const int c_lane = (q4 & 1) * 2 + ((n16 & 3) >> 1);
#pragma unroll
      for (int k = 0; k < 2; ++k) {
        const int r = 8 * k + 4 * g + (n16 >> 2);
        vb[k] = r * Y::kMain + ((c_lane ^ Y::sw_main(r)) << 4) + (n16 & 1) * 8;
      }
    }
    // weights: head row n, operand lane g at 32 g (fp8) or token half t at 32 t, g at 16 g (bf16)
    const uint32_t p_write = lds_p + (16 * hh + n16) * kPRow + (FP8 ? (q4 & 1) * 32 + th * 16 + (q4 >> 1) * 4
                                                                   : th * 32 + (q4 & 1) * 16 + (q4 >> 1) * 8);
    const uint32_t p_read = lds_p + n32 * kPRow + g * (FP8 ? 32 : 16);
    const uint32_t stat_w = lds_stat + (th * kHeadsPerWave + 16 * hh + n16) * 4;
    const uint32_t stat_r = lds_stat + (16 * hh + n16) * 4;  // (token half 1: + kHeadsPerWave * 4)

    // what a masked position's raw product is replaced by (fp8: the sign of the scale is in q)
    const float masked_raw = !FP8 && c_head < 0.f ? INFINITY : -INFINITY;
    float ref = 0.f, l_run = 0.f, lq_run = 0.f, mt_all = -INFINITY;
    float ref_exact = __builtin_nanf("");
    float l_tot = 0.f, lq_tot = 0.f, ref_out = 0.f;  // of head n32
    f32x16 acc[4];
    if (n_tiles == 0)
#pragma unroll
      for (int cb = 0; cb < 4; ++cb)
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[cb][i] = 0.f;

#pragma unroll 1
    for (int attempt = 0; attempt < 2 && n_tiles > 0; ++attempt) {
      if (attempt > 0) {
        issue_tile(0);
        if (n_tiles > 1) issue_tile(1);
        if (n_tiles > 2) issue_tile(2);
      }
#pragma unroll
      for (int cb = 0; cb < 4; ++cb)
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[cb][i] = 0.f;
      l_run = lq_run = 0.f;
      mt_all = -INFINITY;

#pragma unroll 1
      for (int it = 0; it < n_tiles; ++it) {
        wait_tile(it);
        // tile it is visible; every wave is done with tile it - 1 (its stage) and with its weights
        __syncthreads();
        const uint32_t st = stage_base(it);
        const int pos0 = tile_pos(it);
        const bool full = tile_full(pos0);

        // ---- bf16: K fragments, all of them ahead of the first matrix instruction; left to itself the compiler reads,
        // waits and multiplies one by one.  The next tile's requests go out while they arrive.  (fp8: 2 % slower so.) ----
        bf16x8 kf[FP8 ? 1 : kKS];
        if constexpr (!FP8) {
#pragma unroll
          for (int ks = 0; ks < kKS; ++ks)
            kf[ks] = *LDS_PTR(bf16x8, st + (ks < 16 ? (am[0] ^ ((ks & 3) << 6)) + (ks >> 2) * 256 : at[0] ^ ((ks & 1) << 6)));
          __builtin_amdgcn_sched_barrier(0);
        }
        if (it + 3 < n_tiles) issue_tile(it + 3);
        // V^T fragments of the wave's 128 columns; bf16: also ahead of the weights (a tile that is not kept whole: again,
        // once its cleared rows are visible)
        std::conditional_t<FP8, i32x8, bf16x8> v[FP8 ? 4 : 8];
        auto load_v = [&]() {
          if constexpr (FP8) {
#pragma unroll
            for (int cb = 0; cb < 4; ++cb) {
              const int cg = 4 * wave + cb;  // its 32 columns are chunks 2 cg, 2 cg + 1 of a row
              const uint32_t a = st + (vb[0] ^ ((cg & 7) << 5)) + (cg >> 3) * 256;
#pragma unroll
              for (int pt = 0; pt < 4; ++pt) {
                const i32x2 t = __builtin_amdgcn_ds_read_tr8_b64_v2i32(LDS_PTR(i32x2, a + pt * 16 * Y::kMain));
                v[cb][2 * pt] = t[0];
                v[cb][2 * pt + 1] = t[1];
              }
            }
          } else {
#pragma unroll
            for (int j = 0; j < 8; ++j) {
              const uint32_t a = st + (j >> 2) * 16 * Y::kMain + wave * 256, x = (j & 3) << 6;
              const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16(LDS_PTR(s16x4, a + (vb[0] ^ x)));
              const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16(LDS_PTR(s16x4, a + (vb[1] ^ x)));
              v[j] = __builtin_bit_cast(bf16x8, s16x8{lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]});
            }
          }
        };
        __builtin_amdgcn_sched_barrier(0);

        // ---- S^T ----
        f32x4 s[kGroups];
        if constexpr (FP8) {
#pragma unroll
          for (int a = 0; a < kGroups; ++a) {
            s[a] = f32x4{0, 0, 0, 0};
#pragma unroll
            for (int ks = 0; ks < kKS; ++ks) {
              const uint32_t ad = st + (ks < 4 ? (am[a] ^ ((ks & 1) << 7)) + (ks >> 1) * 256 : at[a]);
              const i32x4 lo = *LDS_PTR(i32x4, ad), hi = *LDS_PTR(i32x4, ad ^ 16u);
              const i32x8 k8 = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
              s[a] = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(k8, qh[ks], s[a], 0, 0, 0, 127, 0, 127);
              s[a] = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(k8, ql[ks], s[a], 0, 0, 0, 127, 0, 127 - kQLoShift);
            }
          }
        } else {
          f32x4 s1 = {0, 0, 0, 0};
          s[0] = f32x4{0, 0, 0, 0};
#pragma unroll
          for (int ks = 0; ks < kKS; ks += 2) {
            s[0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf[ks], qf[ks], s[0], 0, 0, 0);
            s1 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf[ks + 1], qf[ks + 1], s1, 0, 0, 0);
          }
          s[0] += s1;
          load_v();
        }
        // element i of group a: token tok0 + 16 a + i of the tile
        const int tok0 = (FP8 ? 32 : 16) * th + 4 * q4;

        // ---- what is not kept: logits -inf; value rows cleared (0 * NaN would poison PV) ----
        uint32_t valid = ~0u;
        f32x4 sc[kGroups];
        float sc_max = 0.f;
        if constexpr (FP8) {
          const uint32_t sb = lds_scales + (wave * kStagesN + (it & (kStagesN - 1))) * kScaleStageN;
#pragma unroll
          for (int a = 0; a < kGroups; ++a) sc[a] = *LDS_PTR(f32x4, sb + (tok0 + 16 * a) * 4);
          sc_max = *LDS_PTR(float, sb + lane * 4);
        }
        if (!full) {  // uniform, one or two tiles of a sequence
          valid = 0;
#pragma unroll
          for (int a = 0; a < kGroups; ++a)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
              const int j = pos0 + tok0 + 16 * a + i;
              valid |= (uint32_t)retained(j, Lq, p.S, p.W) << (4 * a + i);
              // (a position no query keeps: the smallest normal scale, as a real one may be anything)
              if constexpr (FP8) sc[a][i] = retained(j, L, p.S, p.Wu) ? sc[a][i] : 1.1754944e-38f;
            }
          if constexpr (FP8) sc_max = retained(pos0 + lane, L, p.S, p.Wu) ? sc_max : 1.1754944e-38f;
          constexpr int kChunks = Y::kMain / 16;
          for (int k = lane; k < kRowsPerWave * kChunks; k += 64) {
            const int r = wave * kRowsPerWave + k / kChunks;
            if (!retained(pos0 + r, L, p.S, p.Wu)) *LDS_PTR(u32x4, st + r * Y::kMain + (k % kChunks) * 16) = u32x4{0, 0, 0, 0};
          }
        }

        // ---- softmax weights of the wave's 16 heads and token half ----
#pragma unroll
        for (int a = 0; a < kGroups; ++a)
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const float u = FP8 ? s[a][i] * sc[a][i] : s[a][i];
            s[a][i] = (valid >> (4 * a + i)) & 1 ? u : masked_raw;
          }
        float mx = -INFINITY;
        if (FP8 || it == 0) {
#pragma unroll
          for (int a = 0; a < kGroups; ++a)
#pragma unroll
            for (int i = 0; i < 4; ++i) mx = fmaxf(mx, FP8 ? s[a][i] : s[a][i] * c_head);
          mx = quad_max(FP8 ? mx * c_head : mx);
        }
        if (it == 0) {
          // the segment's reference: an integer at or above the first tile's largest logit
          if (q4 == 0) *LDS_PTR(float, stat_w) = mx;
          __syncthreads();
          const float m2 = fmaxf(*LDS_PTR(float, stat_r), *LDS_PTR(float, stat_r + kHeadsPerWave * 4));
          ref = ref_exact == ref_exact ? ref_exact : (m2 == -INFINITY || m2 != m2) ? 0.f : ceilf(m2);
        }
        if constexpr (FP8) {
          // every token scale of the tile < 2^es; weight scales at least 2^(es - 10) (see decode_mid_kernel.hip)
          uint32_t m = __builtin_bit_cast(uint32_t, sc_max) & 0x7fffffffu;
#define OA_ROW_SHR_MAX(n)                                                                             \
  {                                                                                                   \
    const uint32_t o = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)m, 0x110 + (n), 0xf, 0xf, true); \
    m = m > o ? m : o;                                                                                \
  }
          OA_ROW_SHR_MAX(1) OA_ROW_SHR_MAX(2) OA_ROW_SHR_MAX(4) OA_ROW_SHR_MAX(8)
#undef OA_ROW_SHR_MAX
          const uint32_t r0 = __builtin_amdgcn_readlane(m, 15), r1 = __builtin_amdgcn_readlane(m, 31);
          const uint32_t r2 = __builtin_amdgcn_readlane(m, 47), r3 = __builtin_amdgcn_readlane(m, 63);
          const uint32_t r01 = r0 > r1 ? r0 : r1, r23 = r2 > r3 ? r2 : r3;
          int es = (int)((r01 > r23 ? r01 : r23) >> 23) - 126;
          es = es < -100 ? -100 : es;
          const float floor_w = __builtin_amdgcn_ldexpf(1.0f, es - 10);
          // block exponent of the head's 32 weights: all are below 2^8 (see decode_mid_kernel.hip)
          const float mt = mx - ref;
          int kk = mt == -INFINITY ? 0 : (int)ceilf(mt) - 8 + es;
          kk = mt == -INFINITY ? 0 : kk < -126 ? -126 : kk > 126 ? 126 : kk;
          mt_all = fmaxf(mt_all, mt);
          const float rk = ref + (float)kk;
          float ls = 0.f, lq = 0.f;
#pragma unroll
          for (int a = 0; a < kGroups; ++a) {
            float e[4], w[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
              e[i] = __builtin_amdgcn_exp2f(fmaf(s[a][i], c_head, -rk));
              ls += e[i];
              w[i] = fmaxf(sc[a][i], floor_w);
            }
            int pk = 0;
            pk = __builtin_amdgcn_cvt_pk_fp8_f32(e[0] * w[0], e[1] * w[1], pk, false);
            pk = __builtin_amdgcn_cvt_pk_fp8_f32(e[2] * w[2], e[3] * w[3], pk, true);
            const f32x2 b0 = __builtin_amdgcn_cvt_pk_f32_fp8(pk, false), b1 = __builtin_amdgcn_cvt_pk_f32_fp8(pk, true);
            lq = fmaf(b0[0], __builtin_amdgcn_rcpf(w[0]), lq);
            lq = fmaf(b0[1], __builtin_amdgcn_rcpf(w[1]), lq);
            lq = fmaf(b1[0], __builtin_amdgcn_rcpf(w[2]), lq);
            lq = fmaf(b1[1], __builtin_amdgcn_rcpf(w[3]), lq);
            *LDS_PTR(int, p_write + a * 8) = pk;
          }
          l_run += __builtin_amdgcn_ldexpf(ls, kk);
          lq_run += __builtin_amdgcn_ldexpf(lq, kk);
          if (q4 == 0) *LDS_PTR(int, lds_kk + (th * kHeadsPerWave + 16 * hh + n16) * 4) = 127 + kk;
        } else {
          bf16x4 pv;
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const float t = fmaf(s[0][i], c_head, -ref);
            mt_all = fmaxf(mt_all, t);
            const float e = __builtin_amdgcn_exp2f(t);
            l_run += e;
            pv[i] = (__bf16)e;
          }
          *LDS_PTR(bf16x4, p_write) = pv;
        }
        __syncthreads();  // the tile's weights are visible (and its cleared rows)

        // ---- PV: columns 128 wave .. + 127 of all 32 heads ----
        if (FP8 || !full) load_v();
        if constexpr (FP8) {
          const i32x4 p0 = *LDS_PTR(i32x4, p_read), p1 = *LDS_PTR(i32x4, p_read + 16);
          const i32x8 pf = {p0[0], p0[1], p0[2], p0[3], p1[0], p1[1], p1[2], p1[3]};
          const int sb = *LDS_PTR(int, lds_kk + (g * kHeadsPerWave + n32) * 4);  // (half g from lane (head, g))
#pragma unroll
          for (int cb = 0; cb < 4; ++cb)
            acc[cb] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(v[cb], pf, acc[cb], 0, 0, 0, 127, 0, sb);
        } else {
          const bf16x8 pf0 = *LDS_PTR(bf16x8, p_read), pf1 = *LDS_PTR(bf16x8, p_read + 32);
#pragma unroll
          for (int j = 0; j < 8; ++j) acc[j & 3] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(v[j], j < 4 ? pf0 : pf1, acc[j & 3], 0, 0, 0);
        }
      }

      // ---- per-head statistics of both token halves ----
      const float mt_q = quad_max(mt_all), l_q = quad_sum(l_run), lq_q = FP8 ? quad_sum(lq_run) : l_q;
      __syncthreads();  // (the statistics' slots were last read in the first tile; also: PV has read its operands)
      if (q4 == 0) {
        *LDS_PTR(float, stat_w) = mt_q;
        *LDS_PTR(float, stat_w + kStatN * 4) = l_q;
        *LDS_PTR(float, stat_w + 2 * kStatN * 4) = lq_q;
        *LDS_PTR(float, stat_w + 3 * kStatN * 4) = ref;
      }
      __syncthreads();
      auto stat = [&](int k, int half) { return *LDS_PTR(float, lds_stat + (k * kStatN + half * kHeadsPerWave + n32) * 4); };
      const float m2 = fmaxf(stat(0, 0), stat(0, 1));
      l_tot = stat(1, 0) + stat(1, 1);
      lq_tot = stat(2, 0) + stat(2, 1);
      ref_out = stat(3, 0);
      // (every wave looks at all 32 heads, so all take the same way)
      const bool off = m2 > kRefSlackN || (m2 < -kRefSlackN && m2 != -INFINITY);
      if (attempt > 0 || !__any(off)) break;
      const float m3 = fmaxf(*LDS_PTR(float, stat_r), *LDS_PTR(float, stat_r + kHeadsPerWave * 4));
      ref_exact = m3 == -INFINITY ? 0.f : ref + ceilf(m3);
    }

    // ---- epilogue: normalise, transpose through LDS, write the wave's 128 columns ----
    // (all tiles have been read: the barriers above; a segment without tiles left the stages alone)
    const float inv = (n_tiles > 0 && lq_tot != 0.f) ? 1.0f / lq_tot : 0.f;
    const float lse = n_tiles > 0 ? (ref_out + __builtin_amdgcn_logf(l_tot)) * 0.6931471805599453f : -INFINITY;
    const bool final_out = sg.slot < 0;
    const int heads_here = p.H - h0 < kHeadsPerWave ? p.H - h0 : kHeadsPerWave;
    if (wave == 0 && lane < heads_here) {
      if (final_out) p.lse[(size_t)sg.b * p.H + h0 + lane] = lse;
      else p.part_lse[(size_t)sg.slot * kHeadsPerWave + lane] = lse;
    }
    const size_t row0 = final_out ? (size_t)sg.b * p.H + h0 : (size_t)sg.slot * kHeadsPerWave;
    constexpr int kOutMax = 128 * 4 + 16;
    const uint32_t ost = lds0 + wave * kHeadsPerWave * kOutMax;
    // Rows of `row` bytes, of which the wave has `data`, `per` of them to an instruction; `put` stages four columns.  The output type is
    // decided outside, and rows leave LDS four requests at a time: a lone wave per SIMD would wait out each (eight at a time:
    // 16 heads 0.8 % slower, half of what they read is not written).  us per decode, one by one -> now: four of 576 tokens, 16 heads
    // 10.15 -> 10.07 (fp8 11.29 -> 11.13), one sequence, 128 heads, fp8 15.02 -> 14.82 (bf16, 14.5, and 128 of 2176, 16 heads: nothing
    // beyond what two runs differ by).
    auto write_rows = [&](auto row_tag, auto put) {
      constexpr int row = decltype(row_tag)::value, data = row / 4, per = 1024 / data, stride = data + 16, kBatch = 4;
      const int sub = lane / (data / 16), off = (lane & (data / 16 - 1)) * 16;
#pragma unroll
      for (int cb = 0; cb < 4; ++cb)
#pragma unroll
        for (int i4 = 0; i4 < 4; ++i4)
          put(ost + n32 * stride + (cb * 32 + i4 * 8 + g * 4) * (data / 128),
              f32x4{acc[cb][i4 * 4] * inv, acc[cb][i4 * 4 + 1] * inv, acc[cb][i4 * 4 + 2] * inv, acc[cb][i4 * 4 + 3] * inv});
      uint8_t* dst = (uint8_t*)(final_out ? p.out : p.part_o) + (row0 + sub) * row + wave * data + off;
#pragma unroll
      for (int k0 = 0; k0 < kHeadsPerWave / per; k0 += kBatch) {
        if (k0 * per >= heads_here) break;  // uniform
        u32x4 r[kBatch];
#pragma unroll
        for (int k = 0; k < kBatch; ++k) r[k] = *LDS_PTR(u32x4, ost + ((k0 + k) * per + sub) * stride + off);
#pragma unroll
        for (int k = 0; k < kBatch; ++k) {
          const int h = (k0 + k) * per;
          if (h + sub < heads_here) *(u32x4*)(dst + (size_t)h * row) = r[k];
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
static hipError_t set_lds_narrow(int bytes) {
  return hipFuncSetAttribute(reinterpret_cast<const void*>(&decode_narrow_kernel<FP8>),
                             hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
}

hipError_t init_narrow_kernels() {
  hipError_t e = set_lds_narrow<false>(kLdsNarrowBf16);
  return e == hipSuccess ? set_lds_narrow<true>(kLdsNarrowFp8) : e;
}

hipError_t launch_decode_narrow(const DecodeParams& p, bool fp8, int n_units, hipStream_t stream) {
  if (n_units <= 0) return hipSuccess;
  if (p.xcds < 1 || p.head_block != kHeadsPerWave) return hipErrorInvalidValue;
  const dim3 grid(((n_units + p.xcds - 1) / p.xcds) * p.xcds), block(kWavesN * 64);
  if (fp8) hipLaunchKernelGGL(decode_narrow_kernel<true>, grid, block, kLdsNarrowFp8, stream, p);
  else hipLaunchKernelGGL(decode_narrow_kernel<false>, grid, block, kLdsNarrowBf16, stream, p);
  return hipGetLastError();
}

}  // namespace omniattn
