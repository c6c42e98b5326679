// Tiles of the backward GEMMs (gemm_bwd.hip, gemm_phase_bwd.hpp): the segment table and its decoding.
#pragma once
#include <type_traits>

#include "common.hpp"
#include "gemm_device.hpp"
#include "kernels.hpp"
#include "tile_rule.hpp"

namespace moe {

// The phase kernel on bm x 256 tiles: row segments (bm = 256 or 320) and K segments with bf16
// results (bm = 256).  gemm_phase_bwd.hpp.
hipError_t launch_phase_bwd(int bm, const GemmBwdProblem& p, hipStream_t stream);

// One tile: output rows [m0, m_end) x columns [n0, N) of group g, K range [kbeg, kbeg + klen).
struct BTile {
  int g, m0, m_end, n0, kbeg, klen;
};

// Segment table in LDS: begin s_off / length s_len of every group (clamped to the row bound) and, for
// row segments, the first tile s_tp of each; tn output tiles per m-tile.  Returns the launch's tile
// count.  Every thread of the block calls this.
template <int MODE, int NTH, int BM>
__device__ __forceinline__ int bwd_tile_table(const GemmBwdProblem& p, int tn, int* s_off, int* s_len, int* s_tp,
                                              int* s_tmp) {
  const int tid = threadIdx.x, groups = p.groups;
  const int cap = (int)p.max_rows;
  for (int g = tid; g < groups; g += NTH) {
    int b, e;
    if (p.seg_stride > 0) {
      b = g * p.seg_stride;
      e = b + min(max(p.offsets[g], 0), p.seg_stride);
    } else {
      b = min(max(p.offsets[g], 0), cap);
      e = min(max(p.offsets[g + 1], b), cap);
    }
    s_off[g] = b;
    s_len[g] = e - b;
  }
  __syncthreads();
  if constexpr (MODE == BWD_KSEG) return groups * ((p.M + BM - 1) / BM) * tn;
  // tiles per group = ceil(len / BM) * tn, prefix-summed into s_tp (first tile of g)
  constexpr int PER = (kMaxGroups + NTH - 1) / NTH;
  int loc[PER], lsum = 0;
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    const int g = tid * PER + i;
    loc[i] = g < groups ? ((s_len[g] + BM - 1) / BM) * tn : 0;
    lsum += loc[i];
  }
  int excl;
  const int total = block_exclusive_scan<NTH>(lsum, s_tmp, excl);
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    const int g = tid * PER + i;
    if (g < groups) s_tp[g] = excl;
    excl += loc[i];
  }
  if (tid == 0) s_tp[groups] = total;
  __syncthreads();
  return total;
}

template <int MODE, int BM, int BN>
__device__ __forceinline__ BTile bwd_decode(const GemmBwdProblem& p, int tile, int tn, const int* s_off,
                                            const int* s_len, const int* s_tp) {
  BTile t;
  if constexpr (MODE == BWD_ROWS) {
    int lo = 0, hi = p.groups;
    while (hi - lo > 1) {
      const int mid = (lo + hi) >> 1;
      if (s_tp[mid] <= tile) lo = mid; else hi = mid;
    }
    t.g = __builtin_amdgcn_readfirstlane(lo);
    const int local = tile - __builtin_amdgcn_readfirstlane(s_tp[t.g]);
    const int len = __builtin_amdgcn_readfirstlane(s_len[t.g]);
    const int tm = (len + BM - 1) / BM;
    const int mi = local % tm, ni = local / tm;           // m-fastest: tiles of one weight panel adjacent
    const int b = __builtin_amdgcn_readfirstlane(s_off[t.g]);
    t.m0 = b + mi * BM;
    t.m_end = b + len;
    t.n0 = ni * BN;
    t.kbeg = 0;
    t.klen = p.K;
  } else {
    const int tm = (p.M + BM - 1) / BM;
    t.g = tile / (tm * tn);
    const int local = tile - t.g * tm * tn;
    const TileMN o = wgrad_order(local, tm, tn, p.Yf != nullptr);
    t.m0 = o.m * BM;
    t.m_end = p.M;
    t.n0 = o.n * BN;
    t.kbeg = __builtin_amdgcn_readfirstlane(s_off[t.g]);
    t.klen = __builtin_amdgcn_readfirstlane(s_len[t.g]);
  }
  return t;
}

// The zeros of a weight-gradient tile of a group without rows: BM x 256 from row m0, column n0 of y, by the block's
// 512 threads, two 512-byte row pieces per instruction, BM / 16 instructions of a wave.  Rows of whole 128-byte lines
// nontemporal like the results: a few tokens on many experts write mostly zeros, and temporal ones push the weights out of
// the last-level cache (13 tokens, 32 experts of 2944 x 1344: the next forward's up-projection 100 us against 65,
// the step 512 against 488).  Rows that do not start on a line temporal: nontemporal part lines cost more than that
// (2 tokens, 96 experts of 2984 x 1408: the step 890 us nontemporal, 854 temporal, 988 through the accumulators in
// 256-byte pieces; 4 tokens, 64 experts of 1000 x 2008: 505, 470, 541).
template <int BM>
__device__ __forceinline__ void store_zero_tile(bf16_t* y, int64_t ld, int m0, int m_end, int n0, int N, int wave, int lane) {
  const int col = n0 + (lane & 31) * 8;
  auto rows = [&](auto nt) {
#pragma unroll 4
    for (int it = 0; it < BM / 16; ++it) {
      const int row = m0 + wave * (BM / 8) + it * 2 + (lane >> 5);
      u32x4* dst = reinterpret_cast<u32x4*>(y + (int64_t)row * ld + col);
      if (row < m_end && col < N) {
        if constexpr (decltype(nt)::value) __builtin_nontemporal_store(u32x4{0, 0, 0, 0}, dst);
        else *dst = u32x4{0, 0, 0, 0};
      }
    }
  };
  if (ld % 64 == 0) rows(std::true_type{});
  else rows(std::false_type{});
}

}  // namespace moe
