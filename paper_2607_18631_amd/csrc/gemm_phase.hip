// The large-tile grouped GEMM: 256 x 256 and 320 x 256 tiles (token rows x weight rows) on
// v_mfma_f32_16x16x32_bf16, fp32 accumulation.  The problem, the tile table, the tile order and the
// slice copies are the ring kernel's (gemm.hip, gemm_tiles.hpp).
//
// What bounds these tiles is power and the latency of the slice copies, and the kernel is built
// around both (measured on 8192 x 4096 x 7168, one group, random data, back to back):
//  - MFMA shape.  A register-only loop of 16 x 16 x 32 MFMAs (probe/stream.hip, operands of 8 random bits)
//    sustains 2330 TFLOP/s, the same loop of 32 x 32 x 16 ones 1905 (with all mantissa bits random 2050-2100 and
//    1815-1830): under full matrix load the clock is what the power limit leaves, and the smaller shape takes
//    less power per flop.  Keeping the weight operand over two consecutive MFMAs takes 2% less than keeping
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
// F = 2048) 845 -> 750 us, down-projection 465 -> 410; 4096 tokens x 8 experts of 14336 wide: 1600 ->
// 1495 and 812 -> 765; the single group above 1347 -> 1450 TFLOP/s.
#include <type_traits>

#include "common.hpp"
#include "gemm_device.hpp"
#include "gemm_tiles.hpp"
#include "kernels.hpp"
#include "phase_loop.hpp"

namespace moe {
namespace {
// Epilogue of the phase kernel.  Lane (c = lane & 15, q = lane >> 4) holds, in acc[a][r][b], token row
// trow + 64 a + 16 r + c of the tile and output features fcol + 16 b + 4 q .. + 3 (SwiGLU: gate in
// b, up in b + FN / 2).  The SwiGLU epilogues exchange their bf16 results between lanes into row pieces and
// store them straight from registers, so the second ring slot takes the next tile's slice 1 before the
// epilogue (16384 tokens, 128 experts of F = 768: 790 -> 690 us; the benchmark's up-projection 795 ->
// 755).  EPI_BF16, with twice the results per tile, stages each 32-row block in that slot (`st`): with the
// exchange and the early copies the down-projections were 2-5% slower (392 against 411 us).
// EPI_SCATTER stages there too.
constexpr int kPhaseStage = 32 * 72;                     // bf16 elements per wave (32 x 36 floats)

// stores a wave issues per 32-row block whose rows all lie inside the tile (SwiGLU epilogues)
template <int EPI>
constexpr int stores_per_block() {
  return EPI == EPI_SWIGLU ? 2 : 6;
}

template <int EPI, int FM, int FN>
__device__ __forceinline__ void phase_epilogue(const GemmProblem& p, const f32x4 (&acc)[FM][2][FN], const TileDesc& t,
                                               int trow, int fcol, int lane, bf16_t* st) {
  const int c15 = lane & 15, q = lane >> 4;
  constexpr int FO = swiglu_pairs(EPI) ? FN / 2 : FN;     // output fragments per row block
  static_assert(FN == 4, "two pairs of fragments");
  const int prow = lane >> 2, pcol = (lane & 3) * 8;      // of a pair's 16 rows x 32 columns, this lane's piece
#pragma unroll
  for (int a = 0; a < FM; ++a) {
    const int rbase = t.row0 + trow + a * 64;            // first row of the 32-row block
    if (rbase >= t.row_end) continue;                     // wave-uniform
    if constexpr (EPI == EPI_BF16) {
      constexpr int LD = 64;                               // staged columns; piece c of row r at c ^ (r & 7)
#pragma unroll
      for (int r = 0; r < 2; ++r)
#pragma unroll
        for (int b = 0; b < FN; ++b) {
          const f32x4 o = acc[a][r][b];
          uint2 v;
          v.x = pack_bf16x2(o[0], o[1]);
          v.y = pack_bf16x2(o[2], o[3]);
          *reinterpret_cast<uint2*>(st + (r * 16 + c15) * LD + (((b * 2 + (q >> 1)) ^ (c15 & 7)) << 3) + 4 * (q & 1)) = v;
        }
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
      __builtin_amdgcn_wave_barrier();
      const int lr = lane >> 3, lc = lane & 7;
#pragma unroll
      for (int h = 0; h < 4; ++h) {
        const int row = rbase + h * 8 + lr, col = fcol + lc * 8;
        const u32x4 v = ld16(st + (h * 8 + lr) * LD + ((lc ^ lr) << 3));
        if (row < t.row_end && col < p.N) st16(reinterpret_cast<bf16_t*>(t.Y) + (int64_t)row * p.ldy + col, v);
      }
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
      __builtin_amdgcn_wave_barrier();
    } else if constexpr (EPI == EPI_SWIGLU) {
      const bool full = rbase + 32 <= t.row_end && fcol + 32 <= p.N;
      char* base = reinterpret_cast<char*>(reinterpret_cast<bf16_t*>(t.Y) + (int64_t)rbase * p.ldy + fcol);
      const uint32_t off = (prow * (uint32_t)p.ldy + pcol) * 2;
#pragma unroll
      for (int r = 0; r < 2; ++r) {
        f32x4 o[2];
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const float g = acc[a][r][h][e];
            o[h][e] = g * __builtin_amdgcn_rcpf(1.0f + __expf(-g)) * acc[a][r][h + FO][e];
          }
        const u32x4 v = permute_lanes(pack_pieces(o[0], o[1]), pair_src(lane));
        char* b = base + (int64_t)r * 16 * p.ldy * 2;
        if (full) st16_at<false>(b, off, v);
        else if (rbase + r * 16 + prow < t.row_end && fcol + pcol < p.N) st16_at<false>(b, off, v);
      }
    } else if constexpr (EPI == EPI_SWIGLU_BWD) {
      // recomputed gate h and up u: dh = dA u silu'(h), du = dA silu(h), a = silu(h) u
#pragma unroll
      for (int r = 0; r < 2; ++r) {
        const int row = rbase + r * 16 + prow, col = fcol + pcol;
        const bool in = row < t.row_end && col < p.N;
        u32x4 dav = {0, 0, 0, 0};
        if (in) dav = ld16(p.dact + (int64_t)row * p.N + col);
        dav = swap_pieces(permute_lanes(dav, pair_dst(lane)));   // dA of this lane's features
        f32x4 dh[2], du[2], av[2];
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const uint32_t w = dav[2 * h + (e >> 1)];
            const float da = bf16_to_f32((e & 1) ? w >> 16 : w & 0xffffu);
            const float g = acc[a][r][h][e], u = acc[a][r][h + FO][e];
            const float sg = __builtin_amdgcn_rcpf(1.0f + __expf(-g));
            const float silu = g * sg;
            av[h][e] = silu * u;
            du[h][e] = da * silu;
            dh[h][e] = da * u * sg * (1.0f + g * (1.0f - sg));
          }
        const int src = pair_src(lane);
        const u32x4 vh = permute_lanes(pack_pieces(dh[0], dh[1]), src), vu = permute_lanes(pack_pieces(du[0], du[1]), src),
                    va = permute_lanes(pack_pieces(av[0], av[1]), src);
        if (in) {
          bf16_t* yrow = reinterpret_cast<bf16_t*>(t.Y) + (int64_t)row * p.ldy + col;
          st16(yrow, vh);
          st16(yrow + p.N, vu);
          st16(p.act_out + (int64_t)row * p.N + col, va);
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
  using PT = PhaseTile<BM, false, false, swiglu_pairs(EPI)>;
  constexpr int BN = PT::BN, BK = PT::BK, WGN = 4, NW = 8, NTH = 512, FM = PT::FM, FN = PT::FN;
  constexpr int WN = BN / WGN, SLICE = PT::SLICE;
  constexpr int OUTN = swiglu_pairs(EPI) ? BN / 2 : BN;
  using CP = CopyPlan<BM, BN, BK, NW, EPI>;
  static_assert(CP::LX == FM && CP::LW == PT::LW, "one copy per wave and 64-row block");
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

  PT pt;
  pt.init(ring, wave, lane);

  TileDesc td = fetch_tile(0, tile);
  cp.setup(p, td, wave, lane);
  // the copies that go out before the previous tile's epilogue: slice 0, and slice 1 where the epilogue does
  // not stage its results in that slot
  constexpr bool EARLY = swiglu_pairs(EPI);
  int nph = 0;
  auto issue_first = [&]() {
    nph = phases(td);
    phase_first_slice<KTAIL>(pt, cp, nph, nl, p.K);
    if constexpr (EARLY)
      if (nl > 1) with_phases<FM>(nph, [&](auto pc) { phase_second_slice<decltype(pc)::value, KTAIL>(pt, cp, nl, p.K); });
  };
  issue_first();
  int nst = 0;                                            // full 32-row blocks the wave stored after them

  const int fcol = (swiglu_pairs(EPI) ? wn * (BN / 2 / WGN) : wn * WN);
  while (true) {
    f32x4 acc[FM][2][FN];
#pragma unroll
    for (int a = 0; a < FM; ++a)
#pragma unroll
      for (int r = 0; r < 2; ++r)
#pragma unroll
        for (int b = 0; b < FN; ++b) acc[a][r][b] = f32x4{0.f, 0.f, 0.f, 0.f};
    const int live_blocks = min(BM / 32, (td.row_end - td.row0 + 31) / 32);
    const int na = __builtin_amdgcn_readfirstlane(max(0, (live_blocks - wm + 1) / 2));   // live blocks of this wave
    with_phases<FM>(nph, [&](auto pc) {
      constexpr int P = decltype(pc)::value;
      constexpr int SPB = stores_per_block<EPI>();
      if constexpr (EARLY) phase_wait_first<P, SPB, PT>(nl, nst);
      else wait_vmcnt<0>();
      if (na >= P) phase_loop<P, P, KTAIL, !EARLY, 0, false>(pt, cp, acc, nl, p.K);
      else if (P > 2 || na == 1) phase_loop<P, P - 1, KTAIL, !EARLY, 0, false>(pt, cp, acc, nl, p.K);
      else if constexpr (P == 2) phase_loop<P, 0, KTAIL, !EARLY, 0, false>(pt, cp, acc, nl, p.K);
    });

    const TileDesc cur_td = td;
    ++round;
    tile = round_position(round, slot);
    const bool more = tile < ts.total;
    lds_barrier();
    if (more) {
      td = fetch_tile(round, tile);
      cp.setup(p, td, wave, lane);
      issue_first();
    }
    const int col0 = cur_td.ni * OUTN + fcol;
    phase_epilogue<EPI, FM, FN>(p, acc, cur_td, wm * 32, col0, lane, ring + SLICE + wave * kPhaseStage);
    // a lower bound of the stores just issued: blocks whose rows and columns all lie inside
    constexpr int OUTW = swiglu_pairs(EPI) ? WN / 2 : WN;
    nst = col0 + OUTW <= p.N ? max(0, min(FM, (cur_td.row_end - cur_td.row0 - wm * 32 + 32) / 64)) : 0;
    nst = __builtin_amdgcn_readfirstlane(nst);
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
