// The large-tile grouped GEMM: 256 x 256 and 320 x 256 tiles (token rows x weight rows) on
// v_mfma_f32_16x16x32_bf16, fp32 accumulation.  The problem, the tile table, the tile order and the
// slice copies are the ring kernel's (gemm.hip, gemm_tiles.hpp).
//
// What bounds these tiles is power and the latency of the slice copies, and the kernel is built
// around both (measured on 8192 x 4096 x 7168, one group, random data, back to back):
//  - MFMA shape.  A register-only loop of 16 x 16 x 32 MFMAs on random operands sustains 2050-2100
//    TFLOP/s at 2.0-2.08 GHz, the same loop of 32 x 32 x 16 ones 1815-1830 at 1.8 GHz: under full
//    matrix load the clock is what the power limit leaves, and the smaller shape takes less power
//    per flop.  Keeping the weight operand over two consecutive MFMAs takes 2% less than keeping
//    the token operand.
//  - Copy lead.  With a K slice consumed K-step by K-step, its LDS slot is busy until the last
//    step, and a copy has one slice (~1.1 us) to land, less than the latency past the L2.  Here a
//    slice is consumed one 64-row token block at a time ("phase") against weight fragments that
//    stay in registers for the whole slice, so a block's place in LDS is free after its phase and
//    the weights' place after the first: in the same two slots copies go out ~1.5 slices ahead.
//    The price is a barrier per phase instead of one per slice.
//  - Read placement.  The next phase's token fragments are read at the start of a phase into a
//    second buffer, the next slice's weight fragments right behind the last MFMA that uses each
//    register, every MFMA pinned in order.  Reading both behind whole K-steps left the MFMAs
//    waiting for LDS at every barrier (301,500 cycles per 112-slice tile against 270,000; 229,400
//    is the MFMAs alone).
// Up-projection of the benchmark's layer (8192 tokens, d = 7168, 32 experts and a shared one of
// F = 2048) 845 -> 765 us, down-projection 465 -> 420; 4096 tokens x 8 experts of 14336 wide: 1600 ->
// 1500 and 812 -> 778; the single group above 1347 -> 1450 TFLOP/s.
#include <type_traits>

#include "common.hpp"
#include "gemm_device.hpp"
#include "gemm_tiles.hpp"
#include "kernels.hpp"

namespace moe {
namespace {
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
  // vmcnt before phase a of a slice with R slices after it (R = 2: two or more): what the phase
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

// Epilogue of the phase kernel.  Lane (c = lane & 15, q = lane >> 4) holds, in acc[a][r][b], token row
// trow + 64 a + 16 r + c of the tile and output features fcol + 16 b + 4 q .. + 3 (SwiGLU: gate in
// b, up in b + FN / 2).  The bf16 results of one 32-row block go through the wave's staging area
// `st` and come back as 16-byte pieces of whole rows, so a store instruction writes whole rows of
// the wave's columns; piece c of staged row r sits at piece c ^ (r % pieces), which spreads the
// rows one write instruction touches over the banks.
constexpr int kPhaseStage = 32 * 72;                     // bf16 elements per wave (32 x 36 floats)

// 32 staged rows of OUTW columns -> rows [rbase, rbase + 32) of Y (row stride ld), from column col0
template <int OUTW>
__device__ __forceinline__ void flush_stage(const bf16_t* st, bf16_t* Y, int64_t ld, int rbase, int row_end, int col0,
                                            int ncol, int lane) {
  constexpr int CPRW = OUTW / 8;
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  __builtin_amdgcn_wave_barrier();
#pragma unroll
  for (int it = 0; it < 32 * CPRW / 64; ++it) {
    const int idx = it * 64 + lane;
    const int rr = idx / CPRW, c = idx % CPRW;
    const int row = rbase + rr, col = col0 + c * 8;
    const u32x4 v = ld16(st + rr * OUTW + ((c ^ (rr % CPRW)) << 3));
    if (row < row_end && col < ncol) st16(Y + (int64_t)row * ld + col, v);
  }
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  __builtin_amdgcn_wave_barrier();
}

template <int EPI, int FM, int FN>
__device__ __forceinline__ void phase_epilogue(const GemmProblem& p, const f32x4 (&acc)[FM][2][FN], const TileDesc& t,
                                               int trow, int fcol, int lane, bf16_t* st) {
  const int c15 = lane & 15, q = lane >> 4;
  constexpr int FO = swiglu_pairs(EPI) ? FN / 2 : FN;     // output fragments per row block
  constexpr int OUTW = FO * 16, CPRW = OUTW / 8;
  // where the lane's 4 columns of fragment b, row r16 + c15, are staged
  auto at = [&](int r, int b) {
    const int row = r * 16 + c15;
    return st + row * OUTW + (((b * 2 + (q >> 1)) ^ (row % CPRW)) << 3) + 4 * (q & 1);
  };
#pragma unroll
  for (int a = 0; a < FM; ++a) {
    const int rbase = t.row0 + trow + a * 64;            // first row of the 32-row block
    if (rbase >= t.row_end) continue;                     // wave-uniform
    if constexpr (EPI == EPI_BF16 || EPI == EPI_SWIGLU) {
#pragma unroll
      for (int r = 0; r < 2; ++r)
#pragma unroll
        for (int b = 0; b < FO; ++b) {
          f32x4 o = acc[a][r][b];
          if constexpr (EPI == EPI_SWIGLU) {
#pragma unroll
            for (int e = 0; e < 4; ++e) o[e] = o[e] * __builtin_amdgcn_rcpf(1.0f + __expf(-o[e])) * acc[a][r][b + FO][e];
          }
          uint2 v;
          v.x = pack_bf16x2(o[0], o[1]);
          v.y = pack_bf16x2(o[2], o[3]);
          *reinterpret_cast<uint2*>(at(r, b)) = v;
        }
      flush_stage<OUTW>(st, reinterpret_cast<bf16_t*>(t.Y), p.ldy, rbase, t.row_end, fcol, p.N, lane);
    } else if constexpr (EPI == EPI_SWIGLU_BWD) {
      // recomputed gate h and up u: dh = dA u silu'(h), du = dA silu(h), a = silu(h) u
#pragma unroll
      for (int r = 0; r < 2; ++r) {
        const int row = rbase + r * 16 + c15;
        if (row >= t.row_end) continue;
        bf16_t* yrow = reinterpret_cast<bf16_t*>(t.Y) + (int64_t)row * p.ldy;
        const bf16_t* darow = p.dact + (int64_t)row * p.N;
        bf16_t* arow = p.act_out + (int64_t)row * p.N;
#pragma unroll
        for (int b = 0; b < FO; ++b) {
          const int col = fcol + b * 16 + 4 * q;
          if (col >= p.N) continue;
          const uint2 dav = *reinterpret_cast<const uint2*>(darow + col);
          const float da[4] = {bf16_to_f32(dav.x & 0xffffu), bf16_to_f32(dav.x >> 16), bf16_to_f32(dav.y & 0xffffu),
                               bf16_to_f32(dav.y >> 16)};
          float dh[4], du[4], av[4];
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const float h = acc[a][r][b][e], u = acc[a][r][b + FO][e];
            const float sg = __builtin_amdgcn_rcpf(1.0f + __expf(-h));
            const float silu = h * sg;
            av[e] = silu * u;
            du[e] = da[e] * silu;
            dh[e] = da[e] * u * sg * (1.0f + h * (1.0f - sg));
          }
          uint2 v;
          v.x = pack_bf16x2(dh[0], dh[1]);
          v.y = pack_bf16x2(dh[2], dh[3]);
          *reinterpret_cast<uint2*>(yrow + col) = v;
          v.x = pack_bf16x2(du[0], du[1]);
          v.y = pack_bf16x2(du[2], du[3]);
          *reinterpret_cast<uint2*>(yrow + p.N + col) = v;
          v.x = pack_bf16x2(av[0], av[1]);
          v.y = pack_bf16x2(av[2], av[3]);
          *reinterpret_cast<uint2*>(arow + col) = v;
        }
      }
    } else {
      // EPI_SCATTER: 32 rows x 32 columns at a time through the staging area (rows of 36 floats), two
      // rows of 32 consecutive columns per atomic instruction; see scatter_tile
      float* lw = reinterpret_cast<float*>(st);
      const int hi = lane >> 5, r32 = lane & 31;
      const int nrow = min(32, t.row_end - rbase);
      int tok = -1;
      float w = 0.f;
      if (r32 < nrow) {
        tok = t.stok ? t.stok[rbase + r32] : rbase + r32;
        w = t.sw ? t.sw[rbase + r32] : 1.0f;
        if (tok < 0 || tok >= p.scatter_rows) tok = -1;
      }
#pragma unroll
      for (int bp = 0; bp < FN / 2; ++bp) {
        const int col0 = fcol + bp * 32;
        if (col0 >= p.N) continue;
#pragma unroll
        for (int r = 0; r < 2; ++r)
#pragma unroll
          for (int h = 0; h < 2; ++h)
            *reinterpret_cast<f32x4*>(lw + (r * 16 + c15) * kScatterLd + h * 16 + 4 * q) = acc[a][r][2 * bp + h];
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_wave_barrier();
        const int col = col0 + r32;
#pragma unroll
        for (int j = 0; j < 16; ++j) {
          const int rl = 2 * j + hi;                       // block row of this lane
          const int tj0 = __builtin_amdgcn_readlane(tok, 2 * j), tj1 = __builtin_amdgcn_readlane(tok, 2 * j + 1);
          const float wj0 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(w), 2 * j));
          const float wj1 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(w), 2 * j + 1));
          const int tk = hi ? tj1 : tj0;
          const float wk = hi ? wj1 : wj0;
          const float v = lw[rl * kScatterLd + r32];
          if (tk >= 0 && col < p.N) unsafeAtomicAdd(reinterpret_cast<float*>(t.Y) + (int64_t)tk * p.ldy + col, wk * v);
        }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_wave_barrier();
      }
    }
  }
}

template <int BM, int EPI, bool KTAIL>
__global__ __launch_bounds__(512, 1) void k_phase_gemm(GemmProblem p) {
  constexpr int BN = 256, BK = 64, WGM = 2, WGN = 4, NW = 8, NTH = 512;
  using Z = Swz<BK>;
  constexpr int FM = BM / 64;                             // 32-row token blocks per wave
  constexpr int WN = BN / WGN, FN = WN / 16, KS = BK / 32;
  constexpr int OUTN = swiglu_pairs(EPI) ? BN / 2 : BN;
  constexpr int SLICE = (BM + BN) * BK;                   // bf16 elements per ring slot
  using CP = CopyPlan<BM, BN, BK, NW, EPI>;
  constexpr int LX = CP::LX, LW = CP::LW;
  static_assert(LX == FM && LW == 4, "one copy per wave and 64-row block");
  static_assert(NW * kPhaseStage <= SLICE, "epilogue staging fits one ring slot");

  extern __shared__ __align__(16) uint8_t smem[];
  bf16_t* ring = reinterpret_cast<bf16_t*>(smem);         // [2][BM + BN][BK]: X rows then W rows
  __shared__ int s_off[kMaxGroups + 1];
  __shared__ int s_tp[kMaxGroups + 1];
  __shared__ int s_tmp[NTH / 64];
  __shared__ int s_list[kTileList][8];

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / WGN, wn = wave % WGN;
  const TileSpace ts = build_tile_space<NTH, BM, BK>(p, OUTN, s_off, s_tp, s_tmp);

  const int slot = first_tile_slot();
  int round = 0;
  int tile = slot;
  if (tile >= ts.total) return;
  for (int r = tid; r < kTileList; r += NTH) {
    const int pos = round_position(r, slot);
    if (pos < ts.total) {
      const TileCode c = tile_code<BM>(p, ts, pos);
      s_list[r][0] = c.row0; s_list[r][1] = c.row_end; s_list[r][2] = c.ni; s_list[r][3] = c.kb;
      s_list[r][4] = c.ke; s_list[r][5] = c.kc; s_list[r][6] = c.g;
    }
  }
  __syncthreads();
  auto fetch_tile = [&](int r, int pos) -> TileDesc {
    TileCode c;
    if (r < kTileList) {
      c.row0 = s_list[r][0]; c.row_end = s_list[r][1]; c.ni = s_list[r][2]; c.kb = s_list[r][3];
      c.ke = s_list[r][4]; c.kc = s_list[r][5]; c.g = s_list[r][6];
    } else {
      c = tile_code<BM>(p, ts, pos);
    }
    return tile_desc(p, c);
  };

  CP cp;
  const int nl = ts.nk;                                   // K slices (no K split on these tiles)
  // phases of a tile: its live 64-row blocks, at least two (a block's place has to be free for two
  // phases before the block that refills it is read)
  auto phases = [&](const TileDesc& t) { return max(2, min(FM, (t.row_end - t.row0 + 63) / 64)); };

  // LDS fragment offsets of this lane (elements): K-step ks of token block 0 / of the weight rows
  int xl[KS], wl[KS];
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) {
    const int l15 = lane & 15;
    const int o = l15 * BK + (((ks * 4 + (lane >> 4)) ^ Z::f(l15)) << 3);
    xl[ks] = o + wm * 32 * BK;
    wl[ks] = o + (BM + wn * (swiglu_pairs(EPI) ? 32 : WN)) * BK;
  }
  // weight fragment b's first row after fragment 0's (SwiGLU: two of gate rows, two of up rows)
  auto wfrag = [](int b) { return (swiglu_pairs(EPI) && b >= FN / 2 ? BN / 2 + (b - FN / 2) * 16 : b * 16) * BK; };

  TileDesc td = fetch_tile(0, tile);
  cp.setup(p, td, wave, lane);
  auto issue_first = [&](int ph) {                        // slice 0 of the tile
    cp.template issue_pipe<KTAIL, 0, LX>(ring, 0, wave, p.K, ph);
    cp.template issue_pipe_w<KTAIL, 0>(ring, 0, wave, p.K);
  };
  int nph = phases(td);
  issue_first(nph);

  const int fcol = (swiglu_pairs(EPI) ? wn * (BN / 2 / WGN) : wn * WN);
  while (true) {
    f32x4 acc[FM][2][FN];
#pragma unroll
    for (int a = 0; a < FM; ++a)
#pragma unroll
      for (int r = 0; r < 2; ++r)
#pragma unroll
        for (int b = 0; b < FN; ++b) acc[a][r][b] = f32x4{0.f, 0.f, 0.f, 0.f};
    bf16x8 fx[2][2][KS], fw[FN][KS];                      // token fragments double-buffered by phase

    // the K loop with P phases per slice, the first NA of them live for this wave
    auto k_loop = [&](auto pc, auto nac) {
      constexpr int P = decltype(pc)::value, NA = decltype(nac)::value;
      using PP = PhasePlan<P, LW>;
      auto read_x = [&](auto buf, int sl, int a, int ks, int r) {
        fx[decltype(buf)::value][r][ks] =
            *reinterpret_cast<const bf16x8*>(ring + sl * SLICE + xl[ks] + (a * 64 + r * 16) * BK);
      };
      auto read_w = [&](int sl, int b, int ks) {
        fw[b][ks] = *reinterpret_cast<const bf16x8*>(ring + sl * SLICE + wl[ks] + wfrag(b));
      };
      // copy number C of the phase (the block of the phase before, then weight rows), if it has one
      auto issue_copy = [&](auto ac, auto rc, auto cc, int i, int sl) {
        constexpr int A = decltype(ac)::value, R = decltype(rc)::value, C = decltype(cc)::value;
        if constexpr (C == 0) {
          constexpr int BX = A == 0 ? P - 1 : A - 1;       // block refilled in this phase
          constexpr int SX = A == 0 ? 1 : 2;               // for slice i + SX
          if constexpr (R >= SX)
            cp.template issue_pipe_one<KTAIL, BX>(ring + (SX == 1 ? sl ^ 1 : sl) * SLICE, i + SX, wave, p.K);
        } else {
          constexpr int W = C - 1;
          constexpr int T = PP::wrel(W);
          constexpr int SW = T == P ? 1 : 2;               // phase P is phase 0 of the next slice
          if constexpr (T % P == A && R >= SW)
            cp.template issue_pipe_one<KTAIL, LX + W>(ring + (SW == 1 ? sl ^ 1 : sl) * SLICE, i + SW, wave, p.K);
        }
      };
      // one slice (slot sl); R = slices after it (2: two or more).  MFMA m of a phase: K-step m / 8,
      // weight fragment (m % 8) / 2, token fragment m % 2; behind it go the reads whose registers it
      // leaves free and, spread out, the phase's copies.
      auto slice = [&](auto rc, int i, int sl) {
        constexpr int R = decltype(rc)::value;
        static_for<P>([&](auto ac) {
          constexpr int A = decltype(ac)::value;
          constexpr int VM = PP::vmcnt(A, R);
          constexpr bool LAST = A + 1 == P;
          constexpr int XB = A & 1;                        // buffer of this phase's token fragments
          constexpr int NB = LAST ? 0 : XB ^ 1;            // of the next phase's
          constexpr bool READX = NA > 0 && (LAST ? R > 0 : A + 1 < NA);
          constexpr bool READW = NA > 0 && LAST && R > 0;
          using nb = std::integral_constant<int, NB>;
          __builtin_amdgcn_sched_barrier(0);
          if constexpr (VM >= 0) {
            wait_vmcnt<(VM >= 0 ? VM : 0)>();
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
              if constexpr (NB != XB) {                    // into the free buffer: at once
                if constexpr (m < 4) read_x(nb{}, nsl, na, m / 2, m % 2);
              } else {                                     // over this phase's: behind their last use
                if constexpr (m % (FN * 2) == FN * 2 - 1) {
                  read_x(nb{}, nsl, na, ks, 0);
                  read_x(nb{}, nsl, na, ks, 1);
                }
              }
            }
            if constexpr (READW && r == 1) read_w(sl ^ 1, b, ks);
            if constexpr (VM >= 0 && m % 2 == 0 && m / 2 <= LW) issue_copy(ac, rc, std::integral_constant<int, m / 2>{}, i, sl);
            __builtin_amdgcn_sched_barrier(0);
          });
        });
      };
      // slice 0 landed (and every earlier store: loads and stores share the counter)
      wait_vmcnt<0>();
      lds_barrier();
      if (nl > 1) {
        // slice 1 up to phase -1, in the order of the plan
        static_for<P>([&](auto tc) {
          constexpr int T = decltype(tc)::value;           // phase T - P: X_{T-1}(1), W with wrel = T
          if constexpr (T >= 1) {
            cp.template issue_pipe_one<KTAIL, T - 1>(ring + SLICE, 1, wave, p.K);
            static_for<LW>([&](auto w) {
              constexpr int W = decltype(w)::value;
              if constexpr (PP::wrel(W) == T) cp.template issue_pipe_one<KTAIL, LX + W>(ring + SLICE, 1, wave, p.K);
            });
          }
        });
      }
      if constexpr (NA > 0) {
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
          for (int b = 0; b < FN; ++b) read_w(0, b, ks);
          for (int r = 0; r < 2; ++r) read_x(std::integral_constant<int, 0>{}, 0, 0, ks, r);
        }
      }
      int i = 0;
      for (; i < nl - 2; ++i) slice(std::integral_constant<int, 2>{}, i, i & 1);
      if (nl > 1) {
        slice(std::integral_constant<int, 1>{}, i, i & 1);
        ++i;
      }
      slice(std::integral_constant<int, 0>{}, i, i & 1);
    };
    const int live_blocks = min(BM / 32, (td.row_end - td.row0 + 31) / 32);
    const int na = __builtin_amdgcn_readfirstlane(max(0, (live_blocks - wm + 1) / 2));   // live blocks of this wave
    with_phases<FM>(nph, [&](auto pc) {
      constexpr int P = decltype(pc)::value;
      if (na >= P) k_loop(pc, pc);
      else if (P > 2 || na == 1) k_loop(pc, std::integral_constant<int, P - 1>{});
      else if constexpr (P == 2) k_loop(pc, std::integral_constant<int, 0>{});
    });

    const TileDesc cur_td = td;
    ++round;
    tile = round_position(round, slot);
    const bool more = tile < ts.total;
    lds_barrier();
    if (more) {
      td = fetch_tile(round, tile);
      cp.setup(p, td, wave, lane);
      nph = phases(td);
      issue_first(nph);
    }
    // the other ring slot is idle until the next tile's first barrier: a staging area per wave
    phase_epilogue<EPI, FM, FN>(p, acc, cur_td, wm * 32, cur_td.ni * OUTN + fcol, lane, ring + SLICE + wave * kPhaseStage);
    if (!more) break;
  }
}


template <int BM, int EPI>
hipError_t launch_phase(const GemmProblem& p, hipStream_t stream) {
  if (p.K < 8 || p.ksplit > 1) return hipErrorInvalidValue;
  const size_t lds = (size_t)2 * (BM + 256) * 64 * sizeof(bf16_t);
  const int outn = swiglu_pairs(EPI) ? 128 : 256;
  if (p.K % 64 == 0) {
    static OccCache occ;
    return launch_persistent(reinterpret_cast<const void*>(&k_phase_gemm<BM, EPI, false>), occ, 512, lds, BM, outn, p,
                             stream);
  }
  static OccCache occ;
  return launch_persistent(reinterpret_cast<const void*>(&k_phase_gemm<BM, EPI, true>), occ, 512, lds, BM, outn, p,
                           stream);
}

template <int BM>
hipError_t launch_epi(const GemmProblem& p, hipStream_t stream) {
  switch (p.epi) {
    case EPI_BF16: return launch_phase<BM, EPI_BF16>(p, stream);
    case EPI_SWIGLU: return launch_phase<BM, EPI_SWIGLU>(p, stream);
    case EPI_SWIGLU_BWD: return launch_phase<BM, EPI_SWIGLU_BWD>(p, stream);
    default: break;
  }
  if constexpr (BM == 256)
    if (p.epi == EPI_SCATTER) return launch_phase<BM, EPI_SCATTER>(p, stream);
  return hipErrorInvalidValue;
}

}  // namespace

hipError_t launch_phase_gemm(int bm, const GemmProblem& p, hipStream_t stream) {
  if (bm == 256) return launch_epi<256>(p, stream);
  if (bm == 320) return launch_epi<320>(p, stream);
  return hipErrorInvalidValue;
}

}  // namespace moe
