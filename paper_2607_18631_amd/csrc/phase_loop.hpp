// The phase-pipelined K loop of the large-tile GEMMs (gemm_phase.hip, gemm_phase_bwd.hpp): a BM x 256
// tile (BM = 256 or 320) of 8 waves, 2 (token rows) x 4 (weight rows), each 32 rows of every 64-row token
// block x 64 weight rows, on v_mfma_f32_16x16x32_bf16.
#pragma once
#include <type_traits>

#include "common.hpp"
#include "gemm_device.hpp"

namespace moe {

// When a phase-pipelined tile copies what.  A K slice runs P phases, one 64-row token block each
// (P = the tile's live blocks, 2 .. FM).  Phase t = i P + a multiplies block a of slice i; the two
// LDS slots hold slices i and i + 1.  Block b of a slice is in registers once its phase has run,
// the weight rows once phase 0 has, so the copies that refill their places two slices later go
// out in the next phases: X_b(s) in phase (s - 2) P + b + 1, W_w(s) in phase (s - 2) P + wrel(w).
// A wave issues them in that order (X before W inside a phase), which fixes how many newer copies
// may still be in flight when a given one has to have landed: the vmcnt of each phase.
template <int P, int LW>
struct PhasePlan {
  // weight copies (LW = 4 per slice and wave): two in each of phases 1 and 2 (all four in phase 1, or one
  // per phase, measured within 1%)
  static constexpr int wrel(int w) { return P <= 2 ? 1 : 1 + w / 2; }
  static constexpr int xtime(int s, int b) { return (s - 2) * P + b + 1; }
  static constexpr int wtime(int s, int w) { return (s - 2) * P + wrel(w); }
  // copies issued before phase t0 and after the one with issue time t, kind (0 = X, 1 = W) and index
  // w, of slices up to smax
  static constexpr int newer(int t, int kind, int w, int t0, int smax) {
    int n = 0;
    for (int s = 0; s <= smax; ++s) {
      for (int b = 0; b < P; ++b) {
        const int u = xtime(s, b);
        if (u < t0 && u > t) ++n;
      }
      for (int v = 0; v < LW; ++v) {
        const int u = wtime(s, v);
        if (u < t0 && (u > t || (u == t && (kind == 0 || v > w)))) ++n;
      }
    }
    return n;
  }
  // vmcnt before phase a of a slice with R slices after it (the largest R: that many or more): what the phase
  // reads for the next one -- block a + 1, or block 0 and the weights of the next slice -- landed
  static constexpr int vmcnt(int a, int R) {
    const int i = 8, t0 = i * P + a, smax = i + R;
    if (a + 1 < P) return newer(xtime(i, a + 1), 0, 0, t0, smax);
    if (R == 0) return -1;                                 // nothing is read after the last phase
    const int nx = newer(xtime(i + 1, 0), 0, 0, t0, smax);
    const int nw = newer(wtime(i + 1, LW - 1), 1, LW - 1, t0, smax);
    return nx < nw ? nx : nw;
  }
};

// The tile's LDS and this wave's fragments in it.  A ring slot holds one K slice: FM token blocks of
// 64 rows, then 4 weight blocks of 64 rows, 8 KB each (one copy instruction per wave).  A K-major
// block is [64 rows][64 k], row r's 16-byte chunk c at c ^ f(r) (Swz); fragments by ds_read_b128.  An
// MN-major block (the operand's rows run along memory) is [64 k][64 rows], chunk c of k-row k at
// c ^ g(k), fragments by two ds_read_b64_tr_b16: within each 16-lane group that instruction hands
// lane i element (i & 3) of the 8-byte pieces the group's lanes 4 j + (i >> 2), j = 0 .. 3, point at, so
// lane 4 j + q of group G points at k-row 8 G + 4 h + j, rows 4 q .. 4 q + 3, and lane i receives row i at
// k = 8 G + 4 h + 0 .. 3: the MFMA operand layout.  g(k) = 2 (bit 1 of k) + 4 (bit 3 of k) puts the eight
// k-rows that 32 lanes read 32 bytes of into different eighths of a 256-byte bank cycle.
// PAIRS (SwiGLU): the wave's weight fragments are two of gate rows and the two matching up rows.
__device__ __forceinline__ int mn_swz(int k) { return (k & 2) | ((k >> 1) & 4); }

template <int BM_, bool XMN_, bool WMN_, bool PAIRS>
struct PhaseTile {
  static constexpr int BM = BM_, BN = 256, BK = 64, FM = BM / 64, FN = 4, KS = 2, LW = 4;
  static constexpr bool XMN = XMN_, WMN = WMN_;
  static constexpr int SLICE = (BM + BN) * BK;            // bf16 elements per ring slot
  static constexpr int BLK = 64 * BK;                     // elements per block
  static_assert(!(PAIRS && WMN), "gate / up pairs are K-major");
  bf16_t* ring;                                           // [2][SLICE]
  int wave;
  int xl[2], wl[WMN ? FN : KS];                           // this lane's fragment offsets (elements)

  __device__ __forceinline__ void init(bf16_t* r, int w, int lane) {
    ring = r;
    wave = w;
    const int wm = wave / 4, wn = wave % 4, c15 = lane & 15, q = lane >> 4;
    // MN-major: k-row 8 G + j of the K-step, rows 16 m + 4 (lane & 3) of the block
    const int krow = 8 * q + (c15 >> 2), piece = c15 & 3;
    auto mn = [&](int m) { return krow * 64 + (((m * 2 + (piece >> 1)) ^ mn_swz(krow)) << 3) + (piece & 1) * 4; };
    auto km = [&](int ks) { return c15 * BK + (((ks * 4 + q) ^ Swz<BK>::f(c15)) << 3); };
#pragma unroll
    for (int i = 0; i < 2; ++i) xl[i] = XMN ? mn(wm * 2 + i) : km(i) + wm * 32 * BK;
    if constexpr (WMN) {
#pragma unroll
      for (int b = 0; b < FN; ++b) wl[b] = BM * BK + wn * BLK + mn(b);
    } else {
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) wl[ks] = (BM + wn * (PAIRS ? 32 : 64)) * BK + km(ks);
    }
  }
  // the ring slot of a slice, as an element offset
  __device__ __forceinline__ static int slot(int s) { return s * SLICE; }
  __device__ __forceinline__ bf16x8 tr(int off) const {
    typedef short v4s __attribute__((ext_vector_type(4)));
    typedef __attribute__((address_space(3))) v4s lds_v4s;
    const v4s a = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4s*)(ring + off));
    const v4s b = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4s*)(ring + off + 4 * 64));
    return __builtin_bit_cast(bf16x8, __builtin_shufflevector(a, b, 0, 1, 2, 3, 4, 5, 6, 7));
  }
  // K-step ks of 16-row half r of the wave's part of token block a
  __device__ __forceinline__ bf16x8 read_x(int sl, int a, int ks, int r) const {
    if constexpr (XMN) return tr(slot(sl) + xl[r] + a * BLK + ks * 32 * 64);
    else return *reinterpret_cast<const bf16x8*>(ring + slot(sl) + xl[ks] + a * BLK + r * 16 * BK);
  }
  // K-step ks of the wave's 16-row weight fragment b
  __device__ __forceinline__ bf16x8 read_w(int sl, int b, int ks) const {
    if constexpr (WMN) return tr(slot(sl) + wl[b] + ks * 32 * 64);
    else return *reinterpret_cast<const bf16x8*>(ring + slot(sl) + wl[ks] +
                                                 (PAIRS && b >= 2 ? BN / 2 + (b - 2) * 16 : b * 16) * BK);
  }
};

// Copies before the loop.  Slice 0 (into slot s0): the tile's ph live token blocks and the weights.
template <bool KTAIL, class PT, class CP>
__device__ __forceinline__ void phase_first_slice(const PT& pt, const CP& cp, int ph, int nl, int K, int s0 = 0) {
  bf16_t* dst = pt.ring + pt.slot(s0);
  auto all = [&](auto kt) {
    constexpr bool KT = decltype(kt)::value;
    static_for<PT::FM>([&](auto a) {
      if (decltype(a)::value < ph) cp.template issue_block<KT, decltype(a)::value>(dst, 0, pt.wave, K);
    });
    static_for<PT::LW>([&](auto w) { cp.template issue_block<KT, PT::FM + decltype(w)::value>(dst, 0, pt.wave, K); });
  };
  if (KTAIL && nl == 1) all(std::bool_constant<KTAIL>{});
  else all(std::false_type{});
}
// Slice 1 (nl > 1) as far as the plan issues it before phase 0, in the plan's order, and how many copies
// of a wave that is.
template <int P, int LW>
constexpr int phase_second_count() {
  int n = P - 1;
  for (int w = 0; w < LW; ++w) n += PhasePlan<P, LW>::wrel(w) < P;
  return n;
}
template <int P, bool KTAIL, class PT, class CP>
__device__ __forceinline__ void phase_second_slice(const PT& pt, const CP& cp, int nl, int K, int s0 = 0) {
  bf16_t* dst = pt.ring + pt.slot(s0 ^ 1);
  auto all = [&](auto kt) {
    constexpr bool KT = decltype(kt)::value;
    static_for<P - 1>([&](auto tc) {
      constexpr int T = decltype(tc)::value + 1;           // phase T - P: block T - 1, weights with wrel = T
      cp.template issue_block<KT, T - 1>(dst, 1, pt.wave, K);
      static_for<PT::LW>([&](auto w) {
        if constexpr (PhasePlan<P, PT::LW>::wrel(decltype(w)::value) == T)
          cp.template issue_block<KT, PT::FM + decltype(w)::value>(dst, 1, pt.wave, K);
      });
    });
  };
  if (KTAIL && nl == 2) all(std::bool_constant<KTAIL>{});
  else all(std::false_type{});
}

// Wait for slice 0 with slice 1's first copies (nl > 1) and at least SPB * nst stores issued after it.
template <int P, int SPB, class PT>
__device__ __forceinline__ void phase_wait_first(int nl, int nst) {
  constexpr int N1 = phase_second_count<P, PT::LW>();
  static_for<PT::FM + 1>([&](auto kc) {
    constexpr int k = decltype(kc)::value;
    if (nst == k) {
      if (nl > 1) wait_vmcnt<N1 + SPB * k>();
      else wait_vmcnt<SPB * k>();
    }
  });
}

// The K loop over nl slices with P phases each, the first NA of them live for this wave (every wave
// copies and meets every barrier).  cp.issue_block<KT, J>(dst, kt, wave, K) issues the wave's copy of block
// J of slice kt (token blocks 0 .. FM - 1, then weight blocks), KT: of the partial last slice.
// Slice i lives in ring slot (s0 + i) & 1; slice 0 has landed for this wave, and slice 1 is in flight
// unless SECOND asks for its copies here.
// STREAM (wave-uniform `stream` set; both tiles have three slices or more): the last two slices issue
// slices 0 and 1 of the next tile, cp.issue_next<J>(on, dst, kt, wave), as far as the plan has them
// before the next tile's phase 0; and up to ST stores issued after slice 1's copies may stay in flight
// over a first slice that RMAX or more follow.
template <int P, int NA, bool KTAIL, bool SECOND, int ST, bool STREAM, class PT, class CP>
__device__ __forceinline__ void phase_loop(const PT& pt, const CP& cp, f32x4 (&acc)[PT::FM][2][PT::FN], int nl, int K,
                                           int s0 = 0, int stream = 0) {
  constexpr int FN = PT::FN, KS = PT::KS, LW = PT::LW, FM = PT::FM;
  using PP = PhasePlan<P, LW>;
  constexpr int RMAX = KTAIL ? 3 : 2;                      // R = RMAX: RMAX or more slices follow
  bf16x8 fx[2][2][KS], fw[FN][KS];                         // token fragments double-buffered by phase
  // copy number C of phase A of slice i (the block of the phase before, then weight rows), if it has one
  auto issue_copy = [&](auto ac, auto rc, auto cc, int i, int sl) {
    constexpr int A = decltype(ac)::value, R = decltype(rc)::value, C = decltype(cc)::value;
    constexpr int T = C > 0 ? PP::wrel(C > 0 ? C - 1 : 0) : 0;
    constexpr bool HERE = C == 0 || T % P == A;
    constexpr int S = C == 0 ? (A == 0 ? 1 : 2) : (T == P ? 1 : 2);   // for slice i + S
    constexpr int J = C == 0 ? (A == 0 ? P - 1 : A - 1) : FM + C - 1;
    bf16_t* dst = pt.ring + pt.slot(S == 1 ? sl ^ 1 : sl);
    if constexpr (HERE && R >= S)
      cp.template issue_block<(KTAIL && R < RMAX && S == R), J>(dst, i + S, pt.wave, K);
    if constexpr (STREAM) {
      if constexpr (HERE && R < S) cp.template issue_next<J>(stream, dst, S - R - 1, pt.wave);
    }
  };
  // One slice (slot sl).  MFMA m of a phase: K-step m / 8, weight fragment (m % 8) / 2, token half m % 2;
  // behind it go the reads whose registers it leaves free and, spread out, the phase's copies.
  auto slice = [&](auto rc, int i) {
    constexpr int R = decltype(rc)::value;
    const int sl = (s0 + i) & 1;
    static_for<P>([&](auto ac) {
      constexpr int A = decltype(ac)::value;
      constexpr bool LAST = A + 1 == P;
      constexpr bool READS = !LAST || R > 0;               // something is read for the next phase
      constexpr int VM = READS ? PP::vmcnt(A, R) : 0;      // and with the next tile's copies behind this one's:
      constexpr int VMS = READS ? PP::vmcnt(A, RMAX) : 0;
      constexpr int XB = A & 1;                            // buffer of this phase's token fragments
      constexpr int NB = LAST ? 0 : XB ^ 1;                // of the next phase's
      constexpr bool READX = NA > 0 && (LAST ? R > 0 : A + 1 < NA);
      constexpr bool READW = NA > 0 && LAST && R > 0;
      constexpr bool SYNC = READS || STREAM;
      __builtin_amdgcn_sched_barrier(0);
      if constexpr (SYNC) {
        if constexpr (READS && STREAM && R == RMAX) wait_vmcnt_sel<VM + ST, VM>(i);
        else if constexpr (READS && STREAM) wait_vmcnt_sel<VMS, VM>(stream - 1);
        else if constexpr (READS) wait_vmcnt<VM>();
        raw_barrier();
        __builtin_amdgcn_sched_barrier(0);
      }
      static_for<KS * FN * 2>([&](auto mc) {
        constexpr int m = decltype(mc)::value;
        constexpr int ks = m / (FN * 2), b = m % (FN * 2) / 2, r = m % 2;
        if constexpr (A < NA) {
          acc[A][r][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fw[b][ks], fx[XB][r][ks], acc[A][r][b], 0, 0, 0);
          __builtin_amdgcn_sched_barrier(0);
        }
        if constexpr (READX) {
          const int nsl = LAST ? sl ^ 1 : sl, na = LAST ? 0 : A + 1;
          if constexpr (NB != XB) {                        // into the free buffer: at once
            if constexpr (m < 4) fx[NB][m % 2][m / 2] = pt.read_x(nsl, na, m / 2, m % 2);
          } else if constexpr (m % (FN * 2) == FN * 2 - 1) {   // over this phase's: behind their last use
            fx[NB][0][ks] = pt.read_x(nsl, na, ks, 0);
            fx[NB][1][ks] = pt.read_x(nsl, na, ks, 1);
          }
        }
        if constexpr (READW && r == 1) fw[b][ks] = pt.read_w(sl ^ 1, b, ks);
        if constexpr (SYNC && m % 2 == 0 && m / 2 <= LW) issue_copy(ac, rc, std::integral_constant<int, m / 2>{}, i, sl);
        __builtin_amdgcn_sched_barrier(0);
      });
    });
  };
  lds_barrier();                                           // slice 0 landed for every wave
  if constexpr (SECOND)
    if (nl > 1) phase_second_slice<P, KTAIL>(pt, cp, nl, K, s0);
  if constexpr (NA > 0) {
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
#pragma unroll
      for (int b = 0; b < FN; ++b) fw[b][ks] = pt.read_w(s0, b, ks);
#pragma unroll
      for (int r = 0; r < 2; ++r) fx[0][r][ks] = pt.read_x(s0, 0, ks, r);
    }
    // nothing in flight on entry to the loop: the compiler's waits at its head are the stricter of the
    // entry's and the back edge's read order, and the entry's made every slice wait for weight fragments
    // it does not need yet
    __builtin_amdgcn_s_waitcnt(0xc07f);                    // lgkmcnt(0)
  }
  // The slot of the loop's last slices follows from nl alone, which is the same for every tile of a forward launch: not
  // hidden from the compiler, their LDS addresses are computed once per launch, spilled, and reloaded between
  // the MFMAs, each reload waiting for the copies in flight (43 on a 320-row tile, 3 this way; 32 experts of
  // 320 rows, F = 640, d = 6144: down-projection 146 -> 128 us).
  if constexpr (!STREAM) asm volatile("" : "+s"(s0));
  int i = 0;
  for (; i < nl - RMAX; ++i) slice(std::integral_constant<int, RMAX>{}, i);
  if constexpr (RMAX == 3)
    if (i == nl - 3) {
      slice(std::integral_constant<int, 2>{}, i);
      ++i;
    }
  if (i == nl - 2) {
    slice(std::integral_constant<int, 1>{}, i);
    ++i;
  }
  if (i == nl - 1) slice(std::integral_constant<int, 0>{}, i);
}

// ---- results to memory without a trip through LDS memory ----
// In the MFMA layout lane (c, q) holds columns 4 q .. 4 q + 3 of row c of each 16 x 16 fragment.  Two neighbouring
// fragments, packed to bf16, become one 16-byte piece per lane by exchanging the first's odd with the
// second's even 16-lane rows: columns 8 (q >> 1) .. + 7 of fragment q & 1, i.e. piece 2 (q & 1) + (q >> 1) of the
// pair's four.  Its own inverse (for loads).
__device__ __forceinline__ u32x4 swap_pieces(u32x4 v) {
  const auto x = __builtin_amdgcn_permlane16_swap(v.x, v.z, false, false);
  const auto y = __builtin_amdgcn_permlane16_swap(v.y, v.w, false, false);
  return u32x4{x[0], y[0], x[1], y[1]};
}
__device__ __forceinline__ u32x4 pack_pieces(f32x4 b0, f32x4 b1) {
  return swap_pieces(u32x4{pack_bf16x2(b0[0], b0[1]), pack_bf16x2(b0[2], b0[3]), pack_bf16x2(b1[0], b1[1]),
                           pack_bf16x2(b1[2], b1[3])});
}
// Both pairs of a 16-row x 64-column block (pieces p01 of columns 0 .. 31, p23 of 32 .. 63): p01 takes the whole
// lines of rows 0 .. 7 (lane (c, q): row c & 7, pieces 4 .. 7 in the lanes with c >= 8), p23 those of rows 8 .. 15.
__device__ __forceinline__ void whole_lines(u32x4& p01, u32x4& p23) {
  u32x4 lo, hi;
#pragma unroll
  for (int i = 0; i < 4; ++i) {                            // row_ror:8 swaps the halves of a 16-lane row
    lo[i] = __builtin_amdgcn_update_dpp(p01[i], p23[i], 0x128, 0xf, 0xc, false);
    hi[i] = __builtin_amdgcn_update_dpp(p23[i], p01[i], 0x128, 0xf, 0x3, false);
  }
  p01 = lo;
  p23 = hi;
}
// Lane l <- lane src / 4: neighbouring lanes then hold neighbouring pieces of a row.  The memory pipeline takes
// a 16-byte-per-lane store four lanes (64 bytes) at a time, and four lanes in four rows cost it four
// times as much: with the pieces stored where they were, the down-projection of 16384 tokens, 128 experts
// of F = 768 took 420 us, permuted 411, staged through LDS 392-397.
__device__ __forceinline__ u32x4 permute_lanes(u32x4 v, int src) {
#pragma unroll
  for (int i = 0; i < 4; ++i) v[i] = __builtin_amdgcn_ds_bpermute(src, v[i]);
  return v;
}
__device__ __forceinline__ int piece_lane(int c, int p) { return (((p & 1) * 2 + ((p >> 1) & 1)) * 16 + c) * 4; }
// sources for whole lines (lane l: row l >> 3, piece l & 7) and for a pair's 64-byte rows (row l >> 2, piece l & 3)
__device__ __forceinline__ int line_src(int lane) { return piece_lane((lane >> 3) + 2 * (lane & 4), lane & 3); }
__device__ __forceinline__ int pair_src(int lane) { return piece_lane(lane >> 2, lane & 3); }
// and back: where lane (c, q)'s piece of a pair was loaded
__device__ __forceinline__ int pair_dst(int lane) {
  const int q = lane >> 4;
  return ((lane & 15) * 4 + (q & 1) * 2 + (q >> 1)) * 4;
}

// Stores of store_block for a block inside its bounds: what a wait may count on behind the copies before it.
constexpr int kStoresPerBlock = 4;

// Store 16 bytes at a wave-uniform base plus the lane's 32-bit byte offset.
template <bool NT>
__device__ __forceinline__ void st16_at(char* base, uint32_t off, u32x4 v) {
  u32x4* dst = reinterpret_cast<u32x4*>(base + off);
  if constexpr (NT) __builtin_nontemporal_store(v, dst);
  else *dst = v;
}

// The bf16 results of one 32-row x 64-column block (acc[r][b]) to rows rbase .. of Y, columns col0 ..; rows
// from row_end and columns from ncol on are not stored.  A block inside both costs exactly kStoresPerBlock stores.
template <bool NT>
__device__ __forceinline__ void store_block(const f32x4 (&acc)[2][4], bf16_t* Y, int64_t ld, int rbase, int row_end,
                                            int col0, int ncol, int lane) {
  char* base = reinterpret_cast<char*>(Y + (int64_t)rbase * ld + col0);
  const int lr = lane >> 3, lc = (lane & 7) * 8;           // row (of eight) and column this lane stores
  const uint32_t off = (lr * (uint32_t)ld + lc) * 2;
  const int src = line_src(lane);
  const bool full = rbase + 32 <= row_end && col0 + 64 <= ncol;
  static_assert(kStoresPerBlock == 2 * 2, "row halves x line halves below");
#pragma unroll
  for (int r = 0; r < 2; ++r) {
    u32x4 v[2] = {pack_pieces(acc[r][0], acc[r][1]), pack_pieces(acc[r][2], acc[r][3])};
    whole_lines(v[0], v[1]);
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const u32x4 w = permute_lanes(v[h], src);
      char* b = base + (int64_t)(r * 16 + h * 8) * ld * 2;
      if (full) st16_at<NT>(b, off, w);
      else if (rbase + r * 16 + h * 8 + lr < row_end && col0 + lc < ncol) st16_at<NT>(b, off, w);
    }
  }
}

}  // namespace moe
