// Grouped GEMM on gfx950 bf16 MFMA (v_mfma_f32_32x32x16_bf16), fp32 accumulation.
//
//   Y[r, n] = sum_k X[r, k] * W_g[n, k]     for every group g, every row r in [offs[g], offs[g+1])
//
// One launch serves every group (local expert) of a batch: the row segment of group g
// is [offsets[g], offsets[g+1]) -- the monotone [E+1] row-offset array of the paper's
// kernel-generation section -- read from device memory, so the row counts never travel
// to the host.  Each workgroup builds the launch's tile table in LDS (ceil(m_g / BM) x
// n-tiles per group, one block-wide prefix sum), decodes the tiles it will run into a short
// list (one thread per tile), and then walks them persistently.
// Tiles of one group are ordered m-fastest, so the m-tiles sharing a weight tile are
// adjacent, and adjacent tiles go to workgroups of the same XCD (workgroup i runs on XCD
// i mod 8): a weight tile is fetched from HBM once per XCD L2, not once per m-tile.
//
// Data movement: K is consumed in BK-wide slices through a STAGES-deep LDS ring.  Slices
// are copied global -> LDS by the direct-to-LDS loads of gfx950 (global_load_lds_dwordx4:
// lane i of a wave instruction writes bytes [16 i, 16 i + 16) after the wave's LDS base),
// issued STAGES-1 slices ahead, so HBM/L2 latency hides behind the MFMAs of the slices in
// between and no VGPR staging is needed; a slice's copies go out one per MFMA of the K-step
// that follows the barrier that frees their ring slot.  A slice is consumed after `s_waitcnt vmcnt`
// (this wave's copies of it have landed) and a workgroup barrier (everyone's have).
// The barrier also orders the reuse of a ring slot: the slot refilled in iteration kt was
// last read in iteration kt-1, which every wave has finished once it passes the barrier.
//
// LDS layout of a slice: [rows][BK] bf16, row r's 16-byte chunk c stored at chunk
// c ^ f(r), f(r) = (r / (16 / CPR)) % CPR with CPR = BK / 8 chunks per row.  The 16 lanes of
// one ds_read_b128 phase read one logical chunk of 16 consecutive rows and hit 16
// distinct 16-byte bank groups.  The swizzle is applied on the global side: a lane
// fetches the logical chunk that belongs at its fixed LDS position.
//
// Operand roles: the weight tile is the MFMA A operand (rows = output features) and the
// token tile the B operand (columns = tokens), so each lane ends with 4 consecutive
// output features of one token: 8-byte bf16 stores along the output row.
//
// Edges: token rows past the group's end and weight rows past N are clamped to the last
// valid row (their results are never stored); a K tail (K % BK != 0) is fetched from
// clamped addresses and its chunks past K are zeroed in LDS before use.  The 32-row token
// blocks of a tile alternate over the waves, and a wave runs no MFMA for its blocks past
// the group's end, so the ragged last m-tile of an expert costs MFMA time in proportion to
// its live rows (the per-expert row counts of a routed batch scatter around the mean,
// which leaves most experts with one mostly empty m-tile).
//
// Variants of the same body: equal-stride row segments [g * seg_stride, + count_g) (the
// masked-decode form of the same section: capacity offsets plus valid counts); gathered
// token rows (the permute folded into the prologue: row r of the tile is X row
// row_index[r]); and the scatter epilogue (the weighted combine folded into the epilogue:
// rows added, times their gate, into float32 token rows with atomics).
//
// This file holds the ring kernel (tiles of 64 x 64 to 256 x 128) and the choice of tiles; the
// 256 x 256 and 320 x 256 tiles run in gemm_phase.hip.
#include <type_traits>

#include "common.hpp"
#include "gemm_device.hpp"
#include "gemm_tiles.hpp"
#include "kernels.hpp"
#include "tile_rule.hpp"

namespace moe {

// device properties, queried once per device (std::call_once on the first launch there)
struct DevInfo {
  std::once_flag once;
  int cus = 256;
  int lds = 65536;
};
static DevInfo g_dev[kMaxDevices];

static const DevInfo* dev_info() {
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return nullptr;
  DevInfo& d = g_dev[dev];
  std::call_once(d.once, [&] {
    int n = 0, l = 0;
    if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess && n > 0) d.cus = n;
    if (hipDeviceGetAttribute(&l, hipDeviceAttributeMaxSharedMemoryPerBlock, dev) == hipSuccess && l > 0) d.lds = l;
  });
  return &d;
}
int cu_count() {
  const DevInfo* d = dev_info();
  return d ? d->cus : 256;
}
int lds_limit() {
  const DevInfo* d = dev_info();
  return d ? d->lds : 65536;
}

int kernel_occupancy(OccCache& c, const void* fn, int nth, size_t lds, hipError_t& err) {
  err = hipSuccess;
  int dev = 0;
  if ((err = hipGetDevice(&dev)) != hipSuccess) return 0;
  if (dev < 0 || dev >= kMaxDevices) {
    err = hipErrorInvalidDevice;
    return 0;
  }
  std::call_once(c.once[dev], [&] {
    int occ = 0;
    hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e == hipSuccess) e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&occ, fn, nth, lds);
    c.err[dev] = e;
    c.per_cu[dev] = occ > 0 ? occ : 1;
  });
  err = c.err[dev];
  return err == hipSuccess ? c.per_cu[dev] : 0;
}

// Persistent launch of kernel `fn` (nth threads, lds bytes of dynamic LDS): grid = the
// smaller of an upper bound of the launch's tile count and the resident workgroups, rounded
// down to whole rounds of the 8 XCDs.  `occ` caches the kernel's occupancy per device.
hipError_t launch_persistent(const void* fn, OccCache& occ, int nth, size_t lds, int bm, int outn,
                             const GemmProblem& p, hipStream_t stream) {
  const size_t lds_static = 2 * (kMaxGroups + 1) * sizeof(int) + kTileList * 8 * sizeof(int) + 64;
  if (lds + lds_static > (size_t)lds_limit()) return hipErrorInvalidConfiguration;
  hipError_t err;
  const int per_cu = kernel_occupancy(occ, fn, nth, lds, err);
  if (err != hipSuccess) return err;
  const int64_t tiles_n = (p.N + outn - 1) / outn;
  const int64_t groups = p.offsets ? p.groups : 1;
  const int64_t rows = p.offsets ? p.max_rows : p.rows_single;
  const int bmx = (p.rows2_tile > 0 && p.rows2_tile < bm) ? p.rows2_tile : bm;
  const int64_t upper = tiles_n * ((rows + bm - 1) / bm + groups + (p.rows2 + bmx - 1) / bmx) *
                        (p.ksplit > 1 ? p.ksplit : 1);
  const int64_t resident = (int64_t)cu_count() * per_cu;
  int64_t grid = upper < resident ? upper : resident;
  if (grid >= 8) grid -= grid % 8;
  if (grid < 1) grid = 1;
  GemmProblem arg = p;
  void* args[] = {&arg};
  hipError_t e = hipLaunchKernel(fn, dim3((unsigned)grid), dim3(nth), args, lds, stream);
  return e != hipSuccess ? e : hipGetLastError();
}

namespace {

// First W-tile row of fragment b of a wave whose sub-tile is column block wn of WGN (each
// wave owns the gate rows and the matching up rows of its features in a SwiGLU tile).
template <int EPI, int BN, int WGN, int FN>
__device__ __forceinline__ int frag_wrow(int wn, int b) {
  if (swiglu_pairs(EPI)) {
    constexpr int HALF_W = BN / 2 / WGN;
    return (b < FN / 2) ? wn * HALF_W + b * 32 : BN / 2 + wn * HALF_W + (b - FN / 2) * 32;
  }
  return wn * (BN / WGN) + b * 32;
}

// silu(g) = g / (1 + e^-g) is taken as g * rcp(1 + e^-g) (v_rcp_f32, 1 ulp) in every epilogue: the
// result is rounded to bf16 next, and an IEEE division costs ~10 VALU instructions per element.
// Store one wave's FM x FN accumulator fragments of tile t.  Lane holds token row
// trow + astride a + (lane & 31) and output features fcol + 32 b + 8 q + 4 (lane >> 5) + 0..3.
// SwiGLU pairs fragment b (gate) with b + FN/2 (up): Y = bf16(silu(gate) * up).
template <int EPI, int FM, int FN>
__device__ __forceinline__ void store_tile(const GemmProblem& p, const f32x16 (&acc)[FM][FN], const TileDesc& t,
                                           int trow, int astride, int fcol, int lane) {
#pragma unroll
  for (int a = 0; a < FM; ++a) {
    const int row = t.row0 + trow + a * astride + (lane & 31);
    if (row >= t.row_end) continue;
    if (EPI == EPI_SWIGLU_BWD) {
      // recomputed gate h and up u: dh = dA u silu'(h), du = dA silu(h), a = silu(h) u
      bf16_t* yrow = reinterpret_cast<bf16_t*>(t.Y) + (int64_t)row * p.ldy;
      const bf16_t* darow = p.dact + (int64_t)row * p.N;
      bf16_t* arow = p.act_out + (int64_t)row * p.N;
#pragma unroll
      for (int b = 0; b < FN / 2; ++b) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int col = fcol + b * 32 + 8 * q + 4 * (lane >> 5);
          if (col >= p.N) continue;
          const uint2 dav = *reinterpret_cast<const uint2*>(darow + col);
          const float da[4] = {bf16_to_f32(dav.x & 0xffffu), bf16_to_f32(dav.x >> 16), bf16_to_f32(dav.y & 0xffffu),
                               bf16_to_f32(dav.y >> 16)};
          float dh[4], du[4], av[4];
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const float h = acc[a][b][4 * q + e], u = acc[a][b + FN / 2][4 * q + e];
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
    } else if (EPI == EPI_SWIGLU) {
      bf16_t* yrow = reinterpret_cast<bf16_t*>(t.Y) + (int64_t)row * p.ldy;
#pragma unroll
      for (int b = 0; b < FN / 2; ++b) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int col = fcol + b * 32 + 8 * q + 4 * (lane >> 5);
          if (col >= p.N) continue;
          float o[4];
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            float gt = acc[a][b][4 * q + e], up = acc[a][b + FN / 2][4 * q + e];
            o[e] = gt * __builtin_amdgcn_rcpf(1.0f + __expf(-gt)) * up;
          }
          uint2 v;
          v.x = pack_bf16x2(o[0], o[1]);
          v.y = pack_bf16x2(o[2], o[3]);
          *reinterpret_cast<uint2*>(yrow + col) = v;
        }
      }
    } else if (EPI == EPI_BF16) {
      bf16_t* yrow = reinterpret_cast<bf16_t*>(t.Y) + (int64_t)row * p.ldy;
#pragma unroll
      for (int b = 0; b < FN; ++b) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int col = fcol + b * 32 + 8 * q + 4 * (lane >> 5);
          if (col >= p.N) continue;
          uint2 v;
          v.x = pack_bf16x2(acc[a][b][4 * q + 0], acc[a][b][4 * q + 1]);
          v.y = pack_bf16x2(acc[a][b][4 * q + 2], acc[a][b][4 * q + 3]);
          *reinterpret_cast<uint2*>(yrow + col) = v;
        }
      }
    } else {
      float* yrow = reinterpret_cast<float*>(t.Y) + t.kc * p.y_split_stride + (int64_t)row * p.ldy;
      const bool vec = (p.ldy % 4 == 0) && (p.y_split_stride % 4 == 0);   // 16-byte aligned rows
#pragma unroll
      for (int b = 0; b < FN; ++b) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int col = fcol + b * 32 + 8 * q + 4 * (lane >> 5);
          if (vec && col + 3 < p.N) {
            const f32x4 v = {acc[a][b][4 * q], acc[a][b][4 * q + 1], acc[a][b][4 * q + 2], acc[a][b][4 * q + 3]};
            *reinterpret_cast<f32x4*>(yrow + col) = v;
          } else {
#pragma unroll
            for (int e = 0; e < 4; ++e)
              if (col + e < p.N) yrow[col + e] = acc[a][b][4 * q + e];
          }
        }
      }
    }
  }
}

// EPI_BF16 / EPI_SWIGLU through LDS: a lane's MFMA results are 4-column pieces of one row, so
// storing them straight from registers writes 16-byte pieces of 32 rows per instruction.
// Each 32-row block of the wave's sub-tile instead goes to a wave-private LDS area (`st`, 32 rows
// of OUTW bf16) and comes back as 16-byte pieces of whole rows: a store instruction then writes
// 64 / (OUTW / 8) full rows of OUTW columns.  The 16-byte piece c of staged row r sits at piece
// c ^ (r % (OUTW / 8)), which spreads the 32 rows one write instruction touches over the banks.
template <int EPI, int FM, int FN, int OUTW>
__device__ __forceinline__ void store_tile_staged(const GemmProblem& p, const f32x16 (&acc)[FM][FN],
                                                  const TileDesc& t, int trow, int astride, int fcol, int lane,
                                                  bf16_t* st) {
  static_assert(EPI == EPI_BF16 || EPI == EPI_SWIGLU, "staged epilogue: bf16 results");
  constexpr int CPRW = OUTW / 8;                          // 16-byte pieces per staged row
  constexpr int FO = EPI == EPI_SWIGLU ? FN / 2 : FN;     // output fragments per row block
  static_assert(FO * 32 == OUTW && (32 * CPRW) % 64 == 0, "staged row width");
  const int hi = lane >> 5, r = lane & 31;
#pragma unroll
  for (int a = 0; a < FM; ++a) {
    const int rbase = t.row0 + trow + a * astride;       // first row of the 32-row block
    if (rbase >= t.row_end) continue;                     // wave-uniform
#pragma unroll
    for (int b = 0; b < FO; ++b)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        float o[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          if (EPI == EPI_SWIGLU) {
            const float gt = acc[a][b][4 * q + e], up = acc[a][b + FN / 2][4 * q + e];
            o[e] = gt * __builtin_amdgcn_rcpf(1.0f + __expf(-gt)) * up;
          } else {
            o[e] = acc[a][b][4 * q + e];
          }
        }
        uint2 v;
        v.x = pack_bf16x2(o[0], o[1]);
        v.y = pack_bf16x2(o[2], o[3]);
        *reinterpret_cast<uint2*>(st + r * OUTW + (((b * 4 + q) ^ (r % CPRW)) << 3) + 4 * hi) = v;
      }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int it = 0; it < 32 * CPRW / 64; ++it) {
      const int idx = it * 64 + lane;
      const int rr = idx / CPRW, c = idx % CPRW;
      const int row = rbase + rr, col = fcol + c * 8;
      const u32x4 v = ld16(st + rr * OUTW + ((c ^ (rr % CPRW)) << 3));
      if (row < t.row_end && col < p.N)
        st16(reinterpret_cast<bf16_t*>(t.Y) + (int64_t)row * p.ldy + col, v);
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_wave_barrier();
  }
}

// EPI_SCATTER: the gate-weighted combine folded into the epilogue.  In the MFMA layout a lane
// holds 4-column pieces of one token row, so adding the fragment straight from registers
// would touch 32 rows (cache lines) per instruction; each 32 x 32 fragment instead goes
// through a wave-private LDS block `lw` (32 rows of 36 floats, the padding spreads the banks)
// and comes back two rows per instruction, 32 consecutive columns each, so every float32
// atomic instruction covers two cache lines.  Row r of the tile adds w(r) * row into token
// row tok(r) of Y (see TileDesc::stok / sw).
template <int FM, int FN>
__device__ __forceinline__ void scatter_tile(const GemmProblem& p, const f32x16 (&acc)[FM][FN], const TileDesc& t,
                                             int trow, int astride, int fcol, int lane, float* lw) {
  const int hi = lane >> 5, r32 = lane & 31;
#pragma unroll
  for (int a = 0; a < FM; ++a) {
    const int rbase = t.row0 + trow + a * astride;               // first row of the 32-row block
    if (rbase >= t.row_end) continue;                            // wave-uniform
    const int nrow = min(32, t.row_end - rbase);
    // token and weight of the block's rows, one per lane (lanes 0..31)
    int tok = -1;
    float w = 0.f;
    if (r32 < nrow) {
      tok = t.stok ? t.stok[rbase + r32] : rbase + r32;
      w = t.sw ? t.sw[rbase + r32] : 1.0f;
      if (tok < 0 || tok >= p.scatter_rows) tok = -1;
    }
#pragma unroll
    for (int b = 0; b < FN; ++b) {
      const int col0 = fcol + b * 32;
      if (col0 >= p.N) continue;                                 // N % 8 == 0: whole 32-col pieces or none
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const f32x4 v = {acc[a][b][4 * q], acc[a][b][4 * q + 1], acc[a][b][4 * q + 2], acc[a][b][4 * q + 3]};
        *reinterpret_cast<f32x4*>(lw + r32 * kScatterLd + 8 * q + 4 * hi) = v;
      }
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
      __builtin_amdgcn_wave_barrier();
      const int col = col0 + r32;
#pragma unroll
      for (int j = 0; j < 16; ++j) {
        const int rl = 2 * j + hi;                               // block row of this lane
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


// One K-step's MFMAs with the next slice's copies between them: MFMA M (token fragment M / FN,
// weight fragment M % FN) then copy M, while either remains.  Issuing a slice's copies in one
// block held every wave's MFMA issue behind ~50 address and copy instructions right after the
// slice barrier; spread this way the MFMA pipe keeps running (DeepSeek-V3 layer: up-projection
// 945 -> 908 us, down-projection 510 -> 498 us; Mixtral -6 / -7%; skewed up-projection -8%).
template <int M, int NA, int FN, int FM, int L, class CP>
__device__ __forceinline__ void mfma_copy_steps(f32x16 (&acc)[FM][FN], const bf16x8 (&fw)[FN], const bf16x8 (&fx)[FM],
                                                const CP& cp, bf16_t* dst, int kt, int wave) {
  if constexpr (M < NA * FN || M < L) {
    if constexpr (M < NA * FN)
      acc[M / FN][M % FN] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fw[M % FN], fx[M / FN], acc[M / FN][M % FN], 0, 0, 0);
    if constexpr (M < L) cp.template issue_one_sv<M>(dst, kt, wave);
    __builtin_amdgcn_sched_barrier(0);
    mfma_copy_steps<M + 1, NA, FN, FM, L>(acc, fw, fx, cp, dst, kt, wave);
  }
}

template <int FM, int FN>
__device__ __forceinline__ void zero_acc(f32x16 (&acc)[FM][FN]) {
#pragma unroll
  for (int a = 0; a < FM; ++a)
#pragma unroll
    for (int b = 0; b < FN; ++b)
#pragma unroll
      for (int q = 0; q < 16; ++q) acc[a][b][q] = 0.f;
}

// ---------------------------------------------------------------------------------------
// The kernel: every wave copies, reads and multiplies
// ---------------------------------------------------------------------------------------

// BM token rows x BN weight rows per tile, WGM x WGN waves (each a (BM/WGM) x (BN/WGN)
// sub-tile), BK-wide K slices through a STAGES-deep ring.
template <int BM, int BN, int BK, int STAGES, int WGM, int WGN, int EPI, bool KTAIL>
__global__ __launch_bounds__(64 * WGM * WGN, 1) void k_grouped_gemm(GemmProblem p) {
  using Z = Swz<BK>;
  constexpr int NW = WGM * WGN, NTH = 64 * NW;
  constexpr int WM = BM / WGM, WN = BN / WGN;             // per-wave sub-tile
  constexpr int FM = WM / 32, FN = WN / 32;               // 32x32 fragments per wave
  constexpr int OUTN = (swiglu_pairs(EPI)) ? BN / 2 : BN;
  constexpr int SLICE = (BM + BN) * BK;                   // bf16 elements per ring slot
  using CP = CopyPlan<BM, BN, BK, NW, EPI>;
  constexpr int L = CP::L;
  static_assert(FM >= 1 && FN >= 1, "tile too small");
  static_assert(!swiglu_pairs(EPI) || (FN % 2 == 0 && (BN / 2 / WGN) % 32 == 0), "SwiGLU pairs gate and up fragments");
  static_assert(STAGES >= 2 && (STAGES - 2) * L < 64, "ring depth");

  extern __shared__ __align__(16) uint8_t smem[];
  bf16_t* ring = reinterpret_cast<bf16_t*>(smem);         // [STAGES][BM + BN][BK]: X rows then W rows
  __shared__ int s_off[kMaxGroups + 1];
  __shared__ int s_tp[kMaxGroups + 1];
  __shared__ int s_tmp[NTH / 64];
  __shared__ int s_list[kTileList][8];

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / WGN, wn = wave % WGN;
  const TileSpace ts = build_tile_space<NTH, BM, BK>(p, OUTN, s_off, s_tp, s_tmp);
  const int G = gridDim.x;
  const int K = p.K;
  const int nk = (K + BK - 1) / BK;
  const int nk_full = K / BK;
  constexpr bool ktail = KTAIL;                           // K % BK != 0 (launcher-checked)

  CP cp;
  auto issue_any = [&](int kt, int st) {
    if constexpr (KTAIL) {
      if (kt >= nk_full) cp.issue_tail(ring + st * SLICE, kt, wave, K);
      else cp.issue(ring + st * SLICE, kt, wave);
    } else {
      cp.issue_sv(ring + st * SLICE, kt, wave);
    }
  };

  // The current tile runs K slices kb .. kb + nl - 1; its i-th slice lives in ring slot
  // i % STAGES.  sync_slice(i) makes slice i readable by every wave and (issue) refills the ring
  // slot that slice i-1 used (i may be nl: then it only waits for every copy and synchronises).
  int kb = 0, nl = nk;
  auto sync_slice = [&](int i, bool issue = true) {
    const int after = min(STAGES - 2, nl - 1 - i);       // slices issued after i
    if (STAGES >= 4 && after >= 2) wait_vmcnt<(STAGES >= 4 ? 2 * L : 0)>();
    else if (STAGES >= 3 && after >= 1) wait_vmcnt<(STAGES >= 3 ? L : 0)>();
    else wait_vmcnt<0>();
    lds_barrier();
    if (issue && i + STAGES - 1 < nl) issue_any(kb + i + STAGES - 1, (i + STAGES - 1) % STAGES);
    const int kt = kb + i;
    if (ktail && i < nl && kt == nk - 1) {
      // zero the chunks past K of the last slice (their copies came from clamped addresses)
      bf16_t* z = ring + (i % STAGES) * SLICE;
      for (int idx = tid; idx < (BM + BN) * Z::CPR; idx += NTH) {
        const int r = idx / Z::CPR, pc = idx % Z::CPR;
        const int c = pc ^ Z::f(r);
        if (kt * BK + c * 8 >= K) st16(z + r * BK + pc * 8, u32x4{0, 0, 0, 0});
      }
      lds_barrier();
    }
  };

  // Token rows: fragment a of wave (wm, wn) holds the tile's 32-row block a * WGM + wm, so the
  // row blocks alternate over the waves.  A tile whose segment ends early (the ragged last
  // m-tile of a group) leaves every wave with fewer live blocks; a wave multiplies only its
  // live ones (NA of FM, uniform per wave and tile), and the blocks past the end cost no MFMA.
  constexpr int KS = BK / 16;                             // MFMA K-steps per slice
  int wrow_l[FN], xrow_l[FM], wf_l[FN], xf_l[FM];
#pragma unroll
  for (int b = 0; b < FN; ++b) {
    const int r = frag_wrow<EPI, BN, WGN, FN>(wn, b) + (lane & 31);
    wrow_l[b] = BM * BK + r * BK;
    wf_l[b] = Z::f(r);
  }
#pragma unroll
  for (int a = 0; a < FM; ++a) {
    const int r = (a * WGM + wm) * 32 + (lane & 31);
    xrow_l[a] = r * BK;
    xf_l[a] = Z::f(r);
  }
  const int hi = lane >> 5;
  bf16x8 fw[2][FN], fx[2][FM];
  // read the fragments of K-step ks of ring slot st (the first NA token fragments)
  auto load_frags = [&](auto na, int buf, int st, int ks) {
    constexpr int NA = decltype(na)::value;
    const bf16_t* base = ring + st * SLICE;
    const int c = ks * 2 + hi;
    if constexpr (NA > 0) {
#pragma unroll
      for (int b = 0; b < FN; ++b)
        fw[buf][b] = *reinterpret_cast<const bf16x8*>(base + wrow_l[b] + ((c ^ wf_l[b]) << 3));
#pragma unroll
      for (int a = 0; a < NA; ++a)
        fx[buf][a] = *reinterpret_cast<const bf16x8*>(base + xrow_l[a] + ((c ^ xf_l[a]) << 3));
    }
  };

  // Round r of the persistent grid: the workgroup with first slot `slot` takes position
  // r G + slot in even rounds and r G + (G - 1 - slot) in odd ones (a snake order).  Tiles of a
  // routed expert cost in proportion to its live 32-row blocks; the snake pairs a workgroup's
  // positions from opposite ends of the tile sequence, so the per-workgroup sums of 4 rounds
  // scatter less.  An XCD still takes a contiguous block of positions in every round.
  const int slot = first_tile_slot();
  int round = 0;
  int tile = slot;
  if (tile >= ts.total) return;
  // this workgroup's tiles, decoded in parallel (the per-tile decode is ~2,500 cycles of integer
  // divisions and an LDS binary search, on the critical path between two tiles)
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
  TileDesc td = fetch_tile(0, tile);
  cp.setup(p, td, wave, lane);
  kb = td.kb;
  nl = td.ke - td.kb;
#pragma unroll
  for (int s = 0; s < STAGES - 1; ++s)
    if (s < nl) issue_any(kb + s, s);

  const int fcol = (swiglu_pairs(EPI) ? wn * (BN / 2 / WGN) : wn * WN);
  while (true) {
    f32x16 acc[FM][FN];
    zero_acc(acc);

    // the K loop of one tile with NA live token fragments
    auto k_loop = [&](auto na) {
      constexpr int NA = decltype(na)::value;
      sync_slice(0);
      load_frags(na, 0, 0, 0);
      // Slice i: K-steps 0 .. KS-2 read the next step's fragments during this step's MFMAs.  The
      // last step's fragments are already in registers, so it first publishes slice i + 1 (vmcnt
      // wait + barrier) and reads that slice's first fragments, then runs its MFMAs; with
      // WITH_COPIES it also refills the ring slot slice i used (slice i + STAGES), one copy per
      // MFMA.  After the final slice the fragment reads touch a stale ring slot, harmlessly, to
      // keep the loop free of branches.  The slices that issue no copies run as a loop of their
      // own: a uniform branch between the two MFMA sequences inside one loop body made the
      // register allocator spill the accumulators.
      auto slice_body = [&](int i, auto with_copies) {
        constexpr bool WC = decltype(with_copies)::value;
        const int st = i % STAGES;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
          const int cur = ks & 1;
          if (ks + 1 < KS) {
            load_frags(na, cur ^ 1, st, ks + 1);
#pragma unroll
            for (int a = 0; a < NA; ++a)
#pragma unroll
              for (int b = 0; b < FN; ++b)
                acc[a][b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fw[cur][b], fx[cur][a], acc[a][b], 0, 0, 0);
            // scheduling: an MFMA first (its operands were read during the previous step), then
            // the next step's LDS reads two at a time between MFMAs, so every read has several
            // MFMAs of this step to hide its latency behind
            if constexpr (NA > 0) sched_step<NA + FN, NA * FN>();
          } else if constexpr (KTAIL) {
            // K tail: the copies go out right after the barrier (the last slice's copies take
            // clamped addresses and its chunks past K are zeroed inside sync_slice)
            sync_slice(i + 1);
            load_frags(na, cur ^ 1, (i + 1) % STAGES, 0);
#pragma unroll
            for (int a = 0; a < NA; ++a)
#pragma unroll
              for (int b = 0; b < FN; ++b)
                acc[a][b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fw[cur][b], fx[cur][a], acc[a][b], 0, 0, 0);
            if constexpr (NA > 0) sched_step<NA + FN, NA * FN>();
          } else {
            sync_slice(i + 1, false);
            load_frags(na, cur ^ 1, (i + 1) % STAGES, 0);
            __builtin_amdgcn_sched_barrier(0);
            if constexpr (WC) {
              mfma_copy_steps<0, NA, FN, FM, L>(acc, fw[cur], fx[cur], cp, ring + st * SLICE, kb + i + STAGES, wave);
            } else {
#pragma unroll
              for (int a = 0; a < NA; ++a)
#pragma unroll
                for (int b = 0; b < FN; ++b)
                  acc[a][b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fw[cur][b], fx[cur][a], acc[a][b], 0, 0, 0);
            }
            __builtin_amdgcn_sched_barrier(0);
          }
        }
      };
      if constexpr (KTAIL) {
        for (int i = 0; i < nl; ++i) slice_body(i, std::false_type{});
      } else {
        int i = 0;
        for (; i < nl - STAGES; ++i) slice_body(i, std::true_type{});
        for (; i < nl; ++i) slice_body(i, std::false_type{});
      }
    };
    const int live_blocks = min(BM / 32, (td.row_end - td.row0 + 31) / 32);
    const int na = __builtin_amdgcn_readfirstlane(max(0, (live_blocks - wm + WGM - 1) / WGM));
    with_count<FM>(na, k_loop);

    // next tile: start its copies before this tile's epilogue (every wave is done with the ring)
    const TileDesc cur_td = td;
    ++round;
    tile = round_position(round, slot);
    const bool more = tile < ts.total;
    lds_barrier();
    if (more) {
      td = fetch_tile(round, tile);
      cp.setup(p, td, wave, lane);
      kb = td.kb;
      nl = td.ke - td.kb;
#pragma unroll
      for (int s = 0; s < STAGES - 1; ++s)
        if (s < nl) issue_any(kb + s, s);
    }
    if constexpr (EPI == EPI_SCATTER) {
      // the last ring slot is idle until the next tile's first barrier: one LDS block per wave
      static_assert(NW * 32 * kScatterLd * 4 <= SLICE * 2, "scatter staging fits one ring slot");
      float* lw = reinterpret_cast<float*>(ring + (STAGES - 1) * SLICE) + wave * 32 * kScatterLd;
      scatter_tile<FM, FN>(p, acc, cur_td, wm * 32, WGM * 32, cur_td.ni * OUTN + fcol, lane, lw);
    } else if constexpr ((EPI == EPI_BF16 || EPI == EPI_SWIGLU) &&
                         NW * 32 * (EPI == EPI_SWIGLU ? WN / 2 : WN) <= SLICE) {
      // whole-row stores staged through the last ring slot (idle until the next tile's first barrier)
      constexpr int OUTW = EPI == EPI_SWIGLU ? WN / 2 : WN;
      bf16_t* st = ring + (STAGES - 1) * SLICE + wave * 32 * OUTW;
      store_tile_staged<EPI, FM, FN, OUTW>(p, acc, cur_td, wm * 32, WGM * 32, cur_td.ni * OUTN + fcol, lane, st);
    } else {
      store_tile<EPI, FM, FN>(p, acc, cur_td, wm * 32, WGM * 32, cur_td.ni * OUTN + fcol, lane);
    }
    if (!more) break;
  }
}

template <int BM, int BN, int BK, int STAGES, int WGM, int WGN, int EPI, bool KTAIL>
hipError_t launch_kernel(const GemmProblem& p, hipStream_t stream) {
  static OccCache occ;
  const void* fn = reinterpret_cast<const void*>(&k_grouped_gemm<BM, BN, BK, STAGES, WGM, WGN, EPI, KTAIL>);
  return launch_persistent(fn, occ, 64 * WGM * WGN, (size_t)STAGES * (BM + BN) * BK * sizeof(bf16_t), BM,
                           swiglu_pairs(EPI) ? BN / 2 : BN, p, stream);
}

template <int BM, int BN, int BK, int STAGES, int WGM, int WGN, int EPI>
hipError_t launch_tile(const GemmProblem& p, hipStream_t stream) {
  if (p.K < 8) return hipErrorInvalidValue;
  if (p.K % BK == 0) return launch_kernel<BM, BN, BK, STAGES, WGM, WGN, EPI, false>(p, stream);
  return launch_kernel<BM, BN, BK, STAGES, WGM, WGN, EPI, true>(p, stream);
}

template <int EPI>
hipError_t launch_cfg(Tile tile, const GemmProblem& p, hipStream_t stream) {
  switch (tile) {
    case TILE_128X256: return launch_tile<128, 256, 64, 3, 2, 4, EPI>(p, stream);
    case TILE_256X128:
      if constexpr (EPI == EPI_BF16) return launch_tile<256, 128, 64, 3, 4, 2, EPI>(p, stream);
      break;
    case TILE_256X256: return launch_phase_gemm(256, p, stream);
    case TILE_320X256: return launch_phase_gemm(320, p, stream);
    // few rows per group (decode-like): 64 x 128 tiles, 4 waves, 3-slot ring, two workgroups per CU
    case TILE_64X128: return launch_tile<64, 128, 64, 3, 2, 2, EPI>(p, stream);
  }
  return hipErrorInvalidValue;
}

}  // namespace

hipError_t launch_grouped_gemm(const GemmProblem& p, hipStream_t stream) {
  if (p.ksplit > 1 && (p.epi != EPI_F32 || p.offsets != nullptr || p.rows2 > 0)) return hipErrorInvalidValue;
  // gathered rows: the per-lane 32-bit source offsets must reach every row of X
  if (p.row_index && (p.x_rows < 1 || p.x_rows * p.ldx * 2 >= (int64_t(1) << 32))) return hipErrorInvalidValue;
  // equal-stride segments must fit the row bound
  if (p.seg_stride > 0 && (p.offsets == nullptr || (int64_t)p.groups * p.seg_stride > p.max_rows))
    return hipErrorInvalidValue;
  GemmProblem q = p;
  q.rows2_tile = 0;
  auto tile = [&](FwdEpilogue epi) {
    const FwdSizes sizes{cu_count(), p.N, p.K, p.offsets ? p.groups : 1, p.rows_hint, p.rows2};
    const Tile t = fwd_tile(sizes, epi);
    if (p.epi != EPI_SWIGLU_BWD) q.rows2_tile = extra_group_rows(sizes, epi, t);
    return t;
  };
  switch (p.epi) {
    case EPI_SWIGLU: return launch_cfg<EPI_SWIGLU>(tile(FWD_SWIGLU), q, stream);
    case EPI_SWIGLU_BWD:                                   // the forward up-projection's tiles (same operand shapes)
      if (!p.dact || !p.act_out || p.rows2 > 0 || p.ldy != 2 * (int64_t)p.N) return hipErrorInvalidValue;
      return launch_cfg<EPI_SWIGLU_BWD>(tile(FWD_SWIGLU), q, stream);
    case EPI_BF16: return launch_cfg<EPI_BF16>(tile(FWD_BF16), q, stream);
    case EPI_SCATTER:
      if (p.scatter_rows < 1) return hipErrorInvalidValue;
      return launch_cfg<EPI_SCATTER>(tile(FWD_SCATTER), q, stream);
    case EPI_F32:
    {
      const TileShape ft = f32_tile(p.offsets ? p.max_rows : p.rows_single, p.N);
      if (ft.bn == 256) return launch_tile<128, 256, 64, 3, 2, 4, EPI_F32>(p, stream);
      if (ft.bn == 128) return launch_tile<64, 128, 64, 3, 2, 2, EPI_F32>(p, stream);
      return launch_tile<64, 64, 64, 3, 2, 2, EPI_F32>(p, stream);
    }
    default: return hipErrorInvalidValue;
  }
}

}  // namespace moe

