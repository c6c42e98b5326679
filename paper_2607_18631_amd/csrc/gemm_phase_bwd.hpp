// The large-tile backward GEMMs on the phase-pipelined K loop (phase_loop.hpp):
//   row segments (dA, dX, the router's dx): K-major token rows against an MN-major weight;
//   K segments (per-expert weight gradients): both operands MN-major, one M x N output per group,
//   reduced over the group's rows.
// Part of gemm_bwd.hip, which has the problem and the smaller tiles.
//
// What bounds them, and what was measured (8192 tokens, d = 7168, 32 experts and a shared one of F = 2048;
// before: 32 x 32 x 16 MFMAs, one slice of copy lead, results staged in LDS):
//  - routed dX 503 -> 456 us, dA 275 -> 228, shared dX 409 -> 359, dA 218 -> 180: as the forward, power and
//    copy latency.
//  - routed dW13 853 -> 683, dW2 430 -> 370 (14336 tiles of 4-5 slices each, 128 KB of results per tile).
//    The next tile's first two slices stream in behind the last two of this one, and its first slice runs
//    over the stores still in flight.  Without any store the launch takes 516 us: the stores, 1.9 GB, add 204, as loads
//    wait behind stores in the same in-order counter.  At most two slices per group: the ring kernel's (wgrad_on_ring).
//  - shared dW13 454 -> 434, dW2 221 -> 214 (K = 8192).
#pragma once
#include <type_traits>

#include "common.hpp"
#include "gemm_bwd_tiles.hpp"
#include "gemm_device.hpp"
#include "kernels.hpp"
#include "phase_loop.hpp"

namespace moe {
namespace {

// Slice copies of both operands of a tile, one 64-row block per instruction and wave.  K-major: element
// (r, k) at base + r ld + k; MN-major: (k, r) at base + k ld + r.  Rows past the tile's last valid one
// are clamped to it (never stored), k past the range is fetched as zeros (the partial last slice).
// An MN-major lane's offset is its k-row's plus the clamped row, computed at each copy (three VALU
// instructions): one offset per block held over the K loop left the weight gradients short of
// registers, and a reload inside the loop waits for every copy in flight.
template <int FM, bool XMN>
struct PhaseCopy {
  const char *xbase, *wbase;                               // element (0, 0) of the tile's K range
  const char *xnext, *wnext;                               // of the next tile's
  int64_t xadv, wadv;                                      // bytes from slice to slice
  int xlast, wlast, xlast_next, wlast_next;                // last valid row (K-major) / 8-row chunk start (MN-major)
  uint32_t xoff[XMN ? 1 : FM];                             // per lane: K-major offsets per block
  uint32_t xrow, wrow;                                     // per lane: offset of the lane's k-row (MN-major)
  int row, lc;                                             // LDS row of the lane in its block, first row of its chunk
  int xk;                                                  // k of the lane's X chunk in its slice

  __device__ __forceinline__ void init(int64_t ldx, int64_t ldw, int wave, int lane) {
    row = 8 * wave + (lane >> 3);
    lc = ((lane & 7) ^ mn_swz(row)) * 8;
    xrow = row * (uint32_t)ldx * 2;
    wrow = row * (uint32_t)ldw * 2;
    xadv = XMN ? 64 * ldx * 2 : 128;
    wadv = 64 * ldw * 2;
    xk = XMN ? row : ((lane & 7) ^ Swz<64>::f(row)) * 8;
  }
  // K-major X: the offsets of the tile's blocks
  __device__ __forceinline__ void rows(int64_t ldx) {
    if constexpr (!XMN) {
#pragma unroll
      for (int j = 0; j < FM; ++j) xoff[j] = min(64 * j + row, xlast) * (uint32_t)ldx * 2 + xk * 2;
    }
  }
  template <int J>
  __device__ __forceinline__ uint32_t offset(int last) const {
    if constexpr (J < FM && !XMN) {
      return xoff[J < FM && !XMN ? J : 0];
    } else {
      asm volatile("" : "+s"(last));                       // computed here, not hoisted out of the K loop
      return (J < FM ? xrow : wrow) + min(64 * (J < FM ? J : J - FM) + lc, last) * 2;
    }
  }
  template <bool KT, int J>
  __device__ __forceinline__ void issue_block(bf16_t* dst, int kt, int wave, int K) const {
    const char* base = J < FM ? xbase + kt * xadv : wbase + kt * wadv;
    const uint32_t off = offset<J>(J < FM ? xlast : wlast);
    bf16_t* d = dst + J * 64 * 64 + wave * 512;
    if constexpr (KT) {
      const char* src = base + off;
      if (kt * 64 + (J < FM ? xk : row) >= K) src = reinterpret_cast<const char*>(g_zero_chunk);
      dma16_v(src, d);
    } else {
      dma16_sv(base, off, d);
    }
  }
  template <int J>
  __device__ __forceinline__ void issue_next(int on, bf16_t* dst, int kt, int wave) const {
    const char* base = J < FM ? xnext + kt * xadv : wnext + kt * wadv;
    dma16_sv_if(on, base, offset<J>(J < FM ? xlast_next : wlast_next), dst + J * 64 * 64 + wave * 512);
  }
};

template <int BM, int MODE, bool KTAIL>
__global__ __launch_bounds__(512, 1) void k_phase_bwd(GemmBwdProblem p) {
  constexpr bool KSEG = MODE == BWD_KSEG;
  using PT = PhaseTile<BM, KSEG, true, false>;
  constexpr int BN = PT::BN, BK = PT::BK, FM = PT::FM, NTH = 512;
  constexpr int SPB = kStoresPerBlock;
  static_assert(!KSEG || BM / 16 == FM * SPB, "store_zero_tile leaves as many stores as a full tile's results");
  extern __shared__ __align__(16) uint8_t smem[];
  bf16_t* ring = reinterpret_cast<bf16_t*>(smem);          // [2][SLICE]
  __shared__ int s_off[kMaxGroups];
  __shared__ int s_len[kMaxGroups];
  __shared__ int s_tp[KSEG ? 1 : kMaxGroups + 1];
  __shared__ int s_tmp[NTH / 64];

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / 4, wn = wave % 4;
  const int tn = (p.N + BN - 1) / BN;
  const int total = bwd_tile_table<MODE, NTH, BM>(p, tn, s_off, s_len, s_tp, s_tmp);
  int tile = first_tile_slot();
  if (tile >= total) return;
  const int G = gridDim.x;

  PT pt;
  pt.init(ring, wave, lane);
  PhaseCopy<FM, KSEG> cp;
  cp.init(p.ldx, p.ldw, wave, lane);
  auto xptr = [&](const BTile& t) {
    return reinterpret_cast<const char*>(KSEG ? p.X + (int64_t)t.kbeg * p.ldx + t.m0 : p.X + (int64_t)t.m0 * p.ldx);
  };
  auto wptr = [&](const BTile& t) {
    return reinterpret_cast<const char*>(KSEG ? p.W + (int64_t)t.kbeg * p.ldw + t.n0
                                              : p.W + (int64_t)t.g * p.w_group_stride + t.n0);
  };
  auto xend = [&](const BTile& t) { return t.m_end - (KSEG ? 8 : 1) - t.m0; };
  auto wend = [&](const BTile& t) { return p.N - 8 - t.n0; };
  auto setup = [&](const BTile& t) {
    cp.xbase = xptr(t);
    cp.wbase = wptr(t);
    cp.xlast = xend(t);
    cp.wlast = wend(t);
    cp.rows(p.ldx);
  };
  auto phases = [&](const BTile& t) { return KSEG ? FM : max(2, min(FM, (t.m_end - t.m0 + 63) / 64)); };
  auto slices = [&](const BTile& t) { return (t.klen + BK - 1) / BK; };
  auto full = [&](const BTile& t) { return t.m0 + BM <= t.m_end && t.n0 + BN <= p.N; };
  // the copies that go out before the previous tile's epilogue: slices 0 and 1
  auto issue_first = [&](const BTile& t, int nl, int s0) {
    if (nl == 0) return;
    phase_first_slice<KTAIL>(pt, cp, phases(t), nl, t.klen, s0);
    if (nl > 1) {
      if constexpr (KSEG) phase_second_slice<FM, KTAIL>(pt, cp, nl, t.klen, s0);
      else with_phases<FM>(phases(t), [&](auto pc) { phase_second_slice<decltype(pc)::value, KTAIL>(pt, cp, nl, t.klen, s0); });
    }
  };

  BTile td = bwd_decode<MODE, BM, BN>(p, tile, tn, s_off, s_len, s_tp);
  setup(td);
  int nl = slices(td), s0 = 0;
  issue_first(td, nl, s0);
  if constexpr (KSEG) wait_vmcnt<0>();                     // the first slice counts on a full tile's stores behind them
  int nst = 0;                                             // full 32-row blocks stored after the copies
  while (true) {
    f32x4 acc[FM][2][4];
#pragma unroll
    for (int a = 0; a < FM; ++a)
#pragma unroll
      for (int r = 0; r < 2; ++r)
#pragma unroll
        for (int b = 0; b < 4; ++b) acc[a][r][b] = f32x4{0.f, 0.f, 0.f, 0.f};
    tile += G;
    const bool more = tile < total;
    const BTile cur = td;
    const int cur_nl = nl;
    int stream = 0;
    if constexpr (KSEG) {
      // every block is computed (the tiles are full except at the edge of M), which leaves one K loop.  A
      // weight gradient's tiles have few slices (an expert's rows / 64), so the next tile's first two
      // stream in behind this one's last (when both have three or more).
      if (more) td = bwd_decode<MODE, BM, BN>(p, tile, tn, s_off, s_len, s_tp);
      const int nnl = more ? slices(td) : 0;
      stream = __builtin_amdgcn_readfirstlane(nl >= 3 && nnl >= 3);
      if (nl > 0) {
        cp.xnext = xptr(td);
        cp.wnext = wptr(td);
        cp.xlast_next = xend(td);
        cp.wlast_next = wend(td);
        phase_wait_first<FM, SPB, PT>(nl, nst);
        phase_loop<FM, FM, KTAIL, false, FM * SPB, true>(pt, cp, acc, nl, cur.klen, s0, stream);
        if (stream) {
          cp.xbase = cp.xnext;
          cp.wbase = cp.wnext;
          cp.xlast = cp.xlast_next;
          cp.wlast = cp.wlast_next;
          s0 = (s0 + nl) & 1;
        }
      }
      nl = nnl;
    } else {
      const int live = min(BM / 32, (cur.m_end - cur.m0 + 31) / 32);
      const int na = __builtin_amdgcn_readfirstlane(max(0, (live - wm + 1) / 2));   // live blocks of this wave
      with_phases<FM>(phases(cur), [&](auto pc) {
        constexpr int P = decltype(pc)::value;
        phase_wait_first<P, SPB, PT>(nl, nst);
        if (na >= P) phase_loop<P, P, KTAIL, false, 0, false>(pt, cp, acc, nl, cur.klen);
        else if (P > 2 || na == 1) phase_loop<P, P - 1, KTAIL, false, 0, false>(pt, cp, acc, nl, cur.klen);
        else if constexpr (P == 2) phase_loop<P, 0, KTAIL, false, 0, false>(pt, cp, acc, nl, cur.klen);
      });
      if (more) td = bwd_decode<MODE, BM, BN>(p, tile, tn, s_off, s_len, s_tp);
    }
    if (!stream) {
      lds_barrier();                                       // every wave is done with the ring
      if (more) {
        setup(td);
        issue_first(td, nl, s0);
      }
    }
    bf16_t* y = p.Y + (KSEG ? (int64_t)cur.g * p.y_group_stride : 0);
    const int row0 = cur.m0 + wm * 32, col0 = cur.n0 + wn * 64;
    if (KSEG && cur_nl == 0) {
      store_zero_tile<BM>(y, p.ldy, cur.m0, cur.m_end, cur.n0, p.N, wave, lane);
    } else {
#pragma unroll
      for (int a = 0; a < FM; ++a)
        if (row0 + a * 64 < cur.m_end) store_block<KSEG>(acc[a], y, p.ldy, row0 + a * 64, cur.m_end, col0, p.N, lane);
    }
    // at least SPB stores for each 32-row block that lies inside the output (K segments: the first slice
    // counts on all of a full tile's, so an edge tile leaves nothing in flight)
    nst = col0 + 64 > p.N ? 0 : max(0, min(FM, (cur.m_end - row0 + 32) / 64));
    if (KSEG && !full(cur)) {
      nst = 0;
      wait_vmcnt<0>();
    }
    nst = __builtin_amdgcn_readfirstlane(nst);
    if (!more) break;
  }
}

template <int BM, int MODE, bool KTAIL>
hipError_t launch(const GemmBwdProblem& p, hipStream_t stream) {
  static OccCache occ;
  const void* fn = reinterpret_cast<const void*>(&k_phase_bwd<BM, MODE, KTAIL>);
  const size_t lds = (size_t)2 * (BM + 256) * 64 * sizeof(bf16_t);
  const size_t lds_static = (MODE == BWD_ROWS ? 3 : 2) * (kMaxGroups + 1) * sizeof(int) + 64;
  if (lds + lds_static > (size_t)lds_limit()) return hipErrorInvalidConfiguration;
  hipError_t err;
  const int per_cu = kernel_occupancy(occ, fn, 512, lds, err);
  if (err != hipSuccess) return err;
  const int64_t tn = (p.N + 255) / 256;
  const int64_t upper = MODE == BWD_ROWS ? tn * ((p.max_rows + BM - 1) / BM + p.groups)
                                         : (int64_t)p.groups * ((p.M + BM - 1) / BM) * tn;
  const int64_t resident = (int64_t)cu_count() * per_cu;
  int64_t grid = upper < resident ? upper : resident;
  if (grid >= 8) grid -= grid % 8;
  if (grid < 1) grid = 1;
  GemmBwdProblem arg = p;
  void* args[] = {&arg};
  hipError_t e = hipLaunchKernel(fn, dim3((unsigned)grid), dim3(512), args, lds, stream);
  return e != hipSuccess ? e : hipGetLastError();
}

}  // namespace

hipError_t launch_phase_bwd(int bm, const GemmBwdProblem& p, hipStream_t stream) {
  if (p.mode == BWD_KSEG) {
    if (bm != 256 || p.Yf) return hipErrorInvalidValue;
    return launch<256, BWD_KSEG, true>(p, stream);         // the rows of a group are any number
  }
  const bool kt = p.K % 64 != 0;
  if (bm == 256) return kt ? launch<256, BWD_ROWS, true>(p, stream) : launch<256, BWD_ROWS, false>(p, stream);
  // 320 rows with K-tail code would reload spilled registers inside its K loop
  if (bm == 320 && !kt) return launch<320, BWD_ROWS, false>(p, stream);
  return hipErrorInvalidValue;
}

}  // namespace moe
