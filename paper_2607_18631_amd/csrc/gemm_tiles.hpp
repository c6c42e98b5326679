// Device code shared by the forward grouped-GEMM kernels (the ring kernel of gemm.hip and the
// phase kernel of gemm_phase.hip): the launch's tile table, tile decoding and the slice copies.
#pragma once
#include "common.hpp"
#include "gemm_device.hpp"
#include "kernels.hpp"
#include "tile_rule.hpp"

namespace moe {

// Persistent launch of kernel `fn` (nth threads, lds bytes of dynamic LDS) on the problem; `occ`
// caches the kernel's occupancy per device (gemm.hip).
hipError_t launch_persistent(const void* fn, OccCache& occ, int nth, size_t lds, int bm, int outn,
                             const GemmProblem& p, hipStream_t stream);

// The phase kernel on bm x 256 tiles (bm = 256 or 320), epilogue p.epi (gemm_phase.hip).
hipError_t launch_phase_gemm(int bm, const GemmProblem& p, hipStream_t stream);

// epilogues whose weight tile pairs gate rows [0, N) with up rows [N, 2N)
constexpr bool swiglu_pairs(int epi) { return epi == EPI_SWIGLU || epi == EPI_SWIGLU_BWD; }

// ---------------------------------------------------------------------------------------
// Tile table, tile decoding, slice copies, epilogue
// ---------------------------------------------------------------------------------------

// Tiles of one launch: `groups` row segments of BM-row tiles x tiles_n output tiles each,
// plus tiles_x tiles of the optional extra group, `total` in all.  s_off / s_tp live in LDS.
// With a K split (ksplit > 1, one group, no extra group) the tile space is ksplit copies of
// the (m, n) tiles, chunk c covering K slices [c * kchunk, min(nk, (c + 1) * kchunk)); chunk is
// the slowest index, so the workgroups of one XCD work on one K chunk of the weights.
struct TileSpace {
  int groups, tiles_n, tiles_x, total;
  int bmx;                   // m-tile height of the extra group
  int base_total;            // (m, n) tiles
  int nk, kchunk;            // K slices; slices per chunk
  int seg_stride;            // > 0: group g owns rows [g * seg_stride, g * seg_stride + s_off[g])
  const int* s_off;          // [groups + 1] row offsets clamped to [0, max_rows] (or valid lengths)
  const int* s_tp;           // [groups + 1] first tile of each group; s_tp[groups] = grouped tiles
  __device__ int seg_begin(int g) const { return seg_stride > 0 ? g * seg_stride : s_off[g]; }
  __device__ int seg_end(int g) const { return seg_stride > 0 ? g * seg_stride + s_off[g] : s_off[g + 1]; }
};

// Build the launch's tile table in LDS (every thread of the block calls this).
template <int NTH, int BM, int BK>
__device__ TileSpace build_tile_space(const GemmProblem& p, int outn, int* s_off, int* s_tp, int* s_tmp) {
  const int tid = threadIdx.x;
  TileSpace ts;
  ts.tiles_n = (p.N + outn - 1) / outn;
  int groups = p.groups;
  ts.seg_stride = 0;
  if (p.offsets && p.seg_stride > 0) {
    // equal-stride segments: the valid length of each, clamped to [0, seg_stride] (the
    // launcher keeps groups * seg_stride <= max_rows)
    ts.seg_stride = p.seg_stride;
    for (int g = tid; g < groups; g += NTH) s_off[g] = min(max(p.offsets[g], 0), p.seg_stride);
  } else if (p.offsets) {
    // clamp to [0, max_rows]: any offsets content keeps every access inside the buffers
    const int cap = (int)p.max_rows;
    for (int g = tid; g <= groups; g += NTH) s_off[g] = min(max(p.offsets[g], 0), cap);
  } else {
    groups = 1;
    if (tid == 0) { s_off[0] = 0; s_off[1] = (int)p.rows_single; }
  }
  __syncthreads();
  constexpr int PER = (kMaxGroups + NTH - 1) / NTH;
  int loc[PER];
  int lsum = 0;
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    int g = tid * PER + i;
    int m = g >= groups ? 0 : ts.seg_stride > 0 ? s_off[g] : max(s_off[g + 1] - s_off[g], 0);
    loc[i] = ((m + BM - 1) / BM) * ts.tiles_n;
    lsum += loc[i];
  }
  int excl;
  const int total_r = block_exclusive_scan<NTH>(lsum, s_tmp, excl);
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    int g = tid * PER + i;
    if (g < groups) s_tp[g] = excl;
    excl += loc[i];
  }
  if (tid == 0) s_tp[groups] = total_r;
  __syncthreads();
  // the extra group's tiles sit among the grouped ones (see extra_position)
  ts.bmx = (p.rows2_tile > 0 && p.rows2_tile < BM) ? p.rows2_tile : BM;
  ts.tiles_x = p.rows2 > 0 ? ((p.rows2 + ts.bmx - 1) / ts.bmx) * ts.tiles_n : 0;
  ts.base_total = total_r + ts.tiles_x;
  ts.nk = (p.K + BK - 1) / BK;
  const int ksplit = p.ksplit > 1 ? p.ksplit : 1;
  ts.kchunk = (ts.nk + ksplit - 1) / ksplit;
  ts.total = ts.base_total * ksplit;
  ts.groups = groups;
  ts.s_off = s_off;
  ts.s_tp = s_tp;
  return ts;
}

// One tile: token rows [row0, min(row0 + BM, row_end)) of operand X against output tile ni
// of the weights W, results into Y.
struct TileDesc {
  int row0, row_end, ni;
  int kb, ke, kc;            // K slices [kb, ke) of K chunk kc
  const int32_t* rows;       // gathered rows: tile row r is X row rows[row0 + r] (else row0 + r)
  const int32_t* stok;       // EPI_SCATTER: token of each row (nullptr: the row itself)
  const float* sw;           // EPI_SCATTER: weight of each row (nullptr: 1)
  const bf16_t* X;
  const bf16_t* W;
  void* Y;
};

#ifndef MOE_EXTRA_BLOCKS
#define MOE_EXTRA_BLOCKS 1
#endif
// Where the extra group's (shared expert's) tiles sit among the grouped ones: x_before = extra
// tiles before position t, extra = position t is one.  Workgroup i runs on XCD i % 8 and an XCD
// takes G / 8 consecutive positions per round of the persistent grid, so the extra tiles are
// spread over whole such blocks: every block is all-extra or all-grouped (the last extra block
// may be part-filled, its other positions grouped), which keeps the tiles an XCD runs together
// on shared token and weight panels, while HBM-bound expert blocks and compute-bound shared
// blocks still run side by side on the chip.  Problems with fewer full blocks than extra blocks
// (or grids that are not whole rounds of the 8 XCDs) spread tile by tile.
__device__ __forceinline__ void extra_position(const TileSpace& ts, int t, int& x_before, bool& extra) {
  const int S = ts.tiles_x, T = ts.base_total;
  const int G = gridDim.x;
  const int BS = (MOE_EXTRA_BLOCKS && G % 8 == 0) ? G / 8 : 1;
  const int nbf = T / BS;                                 // full blocks
  const int sb = (S + BS - 1) / BS;                       // blocks the extra tiles fill
  if (S == 0 || BS == 1 || sb > nbf) {
    x_before = (int)((int64_t)t * S / T);
    extra = (int)((int64_t)(t + 1) * S / T) > x_before;
    return;
  }
  const int b = t / BS, o = t - b * BS;
  // extra blocks among the full ones: block b is one iff floor((b+1) sb / nbf) > floor(b sb / nbf)
  const int before = (int)((int64_t)min(b, nbf) * sb / nbf);
  const bool xblock = b < nbf && (int)((int64_t)(b + 1) * sb / nbf) > before;
  const int first = before * BS;                          // extra tiles in earlier blocks
  extra = xblock && first + o < S;
  x_before = min(S, first + (xblock ? o : 0));
}

// A tile's coordinates: rows [row0, row_end) of group g (-1: the extra group), output tile ni,
// K slices [kb, ke) of K chunk kc.  Computed by any thread on its own (no wave-uniform input).
struct TileCode {
  int row0, row_end, ni, kb, ke, kc, g;
};

template <int BM>
__device__ __forceinline__ TileCode tile_code(const GemmProblem& p, const TileSpace& ts, int tile) {
  TileCode c;
  c.kc = tile / ts.base_total;
  tile -= c.kc * ts.base_total;
  c.kb = c.kc * ts.kchunk;
  c.ke = min(ts.nk, c.kb + ts.kchunk);
  int x_before;
  bool extra;
  extra_position(ts, tile, x_before, extra);
  int row0g, local;
  if (extra) {
    row0g = 0;
    c.row_end = p.rows2;
    local = x_before;
    c.g = -1;
  } else {
    const int t = tile - x_before;                        // index among the grouped tiles
    int lo = 0, hi = ts.groups;                           // s_tp[groups] == grouped tiles > t
    while (hi - lo > 1) {
      int mid = (lo + hi) >> 1;
      if (ts.s_tp[mid] <= t) lo = mid; else hi = mid;
    }
    c.g = lo;
    row0g = ts.seg_begin(lo);
    c.row_end = ts.seg_end(lo);
    local = t - ts.s_tp[lo];
  }
  const int bmg = extra ? ts.bmx : BM;                  // m-tile height of this group
  const int mt = (c.row_end - row0g + bmg - 1) / bmg;
  constexpr int BAND = band_m(BM);
  // banded order: bands of up to BAND m-tiles; inside a band m-fastest, then n.  The
  // 32 adjacent tiles one XCD runs at a time then share BAND token panels and
  // 32 / BAND weight panels (groups with few m-tiles reduce to plain m-fastest order)
  const int band = local / (BAND * ts.tiles_n);
  const int bm0 = band * BAND;
  const int bmt = min(BAND, mt - bm0);
  const int in_band = local - band * BAND * ts.tiles_n;
  const int mi = bm0 + in_band % bmt;
  c.ni = in_band / bmt;
  c.row0 = row0g + mi * bmg;
  if (bmg < BM) c.row_end = min(c.row0 + bmg, c.row_end);   // the extra group's shorter tiles
  return c;
}

// The tile of a wave-uniform code (values moved to scalar registers) with its operand pointers.
__device__ __forceinline__ TileDesc tile_desc(const GemmProblem& p, TileCode c) {
  TileDesc d;
  d.row0 = __builtin_amdgcn_readfirstlane(c.row0);
  d.row_end = __builtin_amdgcn_readfirstlane(c.row_end);
  d.ni = __builtin_amdgcn_readfirstlane(c.ni);
  d.kb = __builtin_amdgcn_readfirstlane(c.kb);
  d.ke = __builtin_amdgcn_readfirstlane(c.ke);
  d.kc = __builtin_amdgcn_readfirstlane(c.kc);
  const int g = __builtin_amdgcn_readfirstlane(c.g);
  if (g < 0) {
    d.W = p.W2;
    d.X = p.X2;
    d.Y = p.Y2;
    d.rows = nullptr;
    d.stok = nullptr;
    d.sw = nullptr;
  } else {
    d.W = p.W + (int64_t)g * p.w_group_stride;
    d.X = p.X;
    d.Y = p.Y;
    d.rows = p.row_index;
    d.stok = p.scatter_token;
    d.sw = p.scatter_weight;
  }
  return d;
}

// Tiles a workgroup decodes once at its start (one thread per tile) and keeps in LDS; the
// position of its round r is r G + slot in even rounds, r G + G - 1 - slot in odd ones.
constexpr int kTileList = 64;
__device__ __forceinline__ int round_position(int r, int slot) {
  const int G = gridDim.x;
  return r * G + ((r & 1) ? G - 1 - slot : slot);
}

// Copies of one K slice of a tile into a ring slot, spread over NW waves.  Per tile, a
// wave-uniform base (scalar registers) per copy instruction and a fixed per-lane 32-bit byte
// offset (row * ld + logical chunk), so a full slice's copies cost one scalar add each and
// no vector ALU.  The W instruction j is uniformly in the gate or the up half of a SwiGLU
// tile.  Token rows past the tile's end and weight rows past N are clamped to the last valid
// row.
template <int BM, int BN, int BK, int NW, int EPI>
struct CopyPlan {
  using Z = Swz<BK>;
  static constexpr int RPI = 1024 / (BK * 2);              // rows one wave instruction fills
  static constexpr int LX = BM / RPI / NW, LW = BN / RPI / NW;
  static constexpr int L = LX + LW;                        // vector-memory ops per wave per slice
  static_assert(LX >= 1 && LW >= 1 && (BM / RPI) % NW == 0 && (BN / RPI) % NW == 0, "tile too small");

  // The lanes past K as a scalar mask, or compared from the lane's chunk at each copy.  On 320-row tiles the allocator
  // fits only one of the two without copies of fragments around the K loop's back edge: 16 experts of 629 rows, d = 4768,
  // F = 3416, SwiGLU backward 660 us with the mask and 792 without, SwiGLU 742 and 593.
  static constexpr bool PAST_MASK = EPI == EPI_SWIGLU_BWD;

  const char* xbase;
  const char* wsb[LW];
  uint32_t xoff[LX], woff[LW];
  int xchunk[LX], wchunk[LW];
  uint64_t past;                                           // lanes whose chunk of the partial last slice lies past K

  __device__ __forceinline__ void setup(const GemmProblem& p, const TileDesc& t, int wave, int lane) {
    const int li_row = lane / Z::CPR, li_pc = lane % Z::CPR;
    const int K = p.K;
    const int last = t.row_end - 1 - t.row0;
    if (t.rows) {
      // gathered rows: the lane's own source row (the launcher keeps x_rows * ldx * 2 < 2^32)
      xbase = reinterpret_cast<const char*>(t.X);
      const int top = (int)p.x_rows - 1;
#pragma unroll
      for (int j = 0; j < LX; ++j) {
        const int r = (wave + NW * j) * RPI + li_row;
        xchunk[j] = li_pc ^ Z::f(r);
        const int src = min(max(t.rows[t.row0 + min(r, last)], 0), top);
        xoff[j] = (uint32_t)((int64_t)src * p.ldx * 2 + xchunk[j] * 16);
      }
    } else {
      xbase = reinterpret_cast<const char*>(t.X + (int64_t)t.row0 * p.ldx);
#pragma unroll
      for (int j = 0; j < LX; ++j) {
        const int r = (wave + NW * j) * RPI + li_row;         // tile row
        xchunk[j] = li_pc ^ Z::f(r);
        xoff[j] = (uint32_t)(min(r, last) * p.ldx * 2 + xchunk[j] * 16);
      }
    }
    // every copy of a lane has the same chunk (the swizzle repeats every 16 rows)
    if constexpr (PAST_MASK) past = __ballot((K - 1) / BK * BK + xchunk[0] * 8 >= K);
#pragma unroll
    for (int j = 0; j < LW; ++j) {
      const int r = (wave + NW * j) * RPI + li_row;
      wchunk[j] = li_pc ^ Z::f(r);
      if (swiglu_pairs(EPI)) {
        const int half = ((wave + NW * j) * RPI) >= BN / 2;  // uniform per instruction
        const int f0 = t.ni * (BN / 2);
        const int f = min(f0 + (r - half * (BN / 2)), p.N - 1);
        wsb[j] = reinterpret_cast<const char*>(t.W + ((int64_t)f0 + half * p.N) * K);
        woff[j] = (uint32_t)((f - f0) * K * 2 + wchunk[j] * 16);
      } else {
        const int f0 = t.ni * BN;
        const int f = min(f0 + r, p.N - 1);
        wsb[j] = reinterpret_cast<const char*>(t.W + (int64_t)f0 * K);
        woff[j] = (uint32_t)((f - f0) * K * 2 + wchunk[j] * 16);
      }
    }
  }

  // copy K slice kt into the ring slot at dst (L vector-memory ops of this wave)
  __device__ __forceinline__ void issue(bf16_t* dst, int kt, int wave) const {
    const int k0b = kt * BK * 2;                           // byte offset of the slice
#pragma unroll
    for (int j = 0; j < LX; ++j)
      dma16(reinterpret_cast<const bf16_t*>(xbase + k0b + xoff[j]), dst + (wave + NW * j) * 512);
#pragma unroll
    for (int j = 0; j < LW; ++j)
      dma16(reinterpret_cast<const bf16_t*>(wsb[j] + k0b + woff[j]), dst + BM * BK + (wave + NW * j) * 512);
  }

  // Copy J of K slice kt into the ring slot at dst through a scalar base (the instruction's
  // uniform row block plus the slice's byte offset) and the lane's 32-bit offset: no 64-bit
  // per-lane address arithmetic and no per-lane 64-bit bases held across the K loop.  The
  // compiler does not see these copies; the K loop orders them with its own vmcnt waits and
  // barriers.
  template <int J>
  __device__ __forceinline__ void issue_one_sv(bf16_t* dst, int kt, int wave) const {
    const int k0b = kt * BK * 2;
    if constexpr (J < LX) {
      dma16_sv(xbase + k0b, xoff[J], dst + (wave + NW * J) * 512);
    } else {
      constexpr int JW = J - LX;
      dma16_sv(wsb[JW] + k0b, woff[JW], dst + BM * BK + (wave + NW * JW) * 512);
    }
  }
  template <int J = 0>
  __device__ __forceinline__ void issue_sv(bf16_t* dst, int kt, int wave) const {
    if constexpr (J < L) {
      issue_one_sv<J>(dst, kt, wave);
      issue_sv<J + 1>(dst, kt, wave);
    }
  }

  // Copy J of K slice kt for the phase loop.  KT: slice kt is the last and K is no multiple of BK; the
  // lanes whose chunk lies past K fetch 16 zero bytes instead (both operands), so the partial slice
  // needs no clean-up in LDS.
  template <bool KT, int J>
  __device__ __forceinline__ void issue_block(bf16_t* dst, int kt, int wave, int K) const {
    if constexpr (!KT) {
      issue_one_sv<J>(dst, kt, wave);
    } else {
      const uint64_t base = (uint64_t)(J < LX ? xbase : wsb[J < LX ? 0 : J - LX]) + kt * BK * 2;
      const uint32_t off = J < LX ? xoff[J < LX ? J : 0] : woff[J < LX ? 0 : J - LX];
      // added in halves: for a 64-bit sum the compiler holds every offset widened to 64 bits over the K loop, and
      // reloads them from scratch between its MFMAs
      uint32_t lo = (uint32_t)base;
      asm volatile("" : "+s"(lo));
      const uint32_t sum = lo + off;
      const char* src = reinterpret_cast<const char*>((uint64_t)((uint32_t)(base >> 32) + (sum < off)) << 32 | sum);
      bool dead;
      if constexpr (PAST_MASK) dead = __builtin_amdgcn_inverse_ballot_w64(past);
      else dead = kt * BK + xchunk[0] * 8 >= K;
      if (dead) src = reinterpret_cast<const char*>(g_zero_chunk);
      dma16_v(src, dst + (J < LX ? (wave + NW * J) * 512 : BM * BK + (wave + NW * (J - LX)) * 512));
    }
  }
  // the partial last slice (K % BK != 0): chunks past K are fetched from K-8 and zeroed later
  __device__ __forceinline__ void issue_tail(bf16_t* dst, int kt, int wave, int K) const {
    const int k0 = kt * BK;
#pragma unroll
    for (int j = 0; j < LX; ++j) {
      const int back = max(k0 + xchunk[j] * 8 - (K - 8), 0) * 2;
      dma16(reinterpret_cast<const bf16_t*>(xbase + k0 * 2 + xoff[j] - back), dst + (wave + NW * j) * 512);
    }
#pragma unroll
    for (int j = 0; j < LW; ++j) {
      const int back = max(k0 + wchunk[j] * 8 - (K - 8), 0) * 2;
      dma16(reinterpret_cast<const bf16_t*>(wsb[j] + k0 * 2 + woff[j] - back), dst + BM * BK + (wave + NW * j) * 512);
    }
  }
};

// row stride (floats) of the EPI_SCATTER staging block: 32 columns and padding that spreads the banks
constexpr int kScatterLd = 36;

}  // namespace moe
