// GEMMs of more than 128 bf16 rows (prefill chunks, wide verify batches) over
// matrices wide or deep enough: Y = X[M][K] @ W[K][N] on 2-D output tiles, with
// the operands of kernels_gemm.hip (both in MFMA fragment order) and its
// summation order, bit for bit: per reduction slice four partial sums, one per
// residue class of the k-blocks mod 4, added in class order, then the slices in
// slice order.
//
// The streaming kernel gives each of its four waves one class, so a workgroup
// re-reads its activation rows for every run of 6 column blocks: fine while
// the weight stream is what is waited for, and 430-600 TFLOP/s on 2048 rows.
// Here a workgroup owns a tile of up to 256 rows x 192 columns, its eight
// waves 64 x 64 (two a SIMD: 64 accumulators, 64 totals and, with the slices
// added in registers, 64 sums fit their 256 registers) or 64 x 96, and the
// classes run one after another.  Operand tiles go from memory straight into a
// ring of four LDS stages (global_load_lds, 1 KiB a wave: fragment order is what
// such a load writes), so a stage costs no registers and one barrier.
//
// What bounds it: the operand tiles on their way into LDS.  With 256x128 tiles
// a 2048-row gate/up took 388 us; its loads alone took 296, its MFMAs alone 227
// (1.6 PFLOP/s, this card's matrix rate), its LDS reads 120, and rings of 3 to
// 8 stages or another order of the tiles over the dies changed nothing.  So the
// tile is as large as the registers allow, 256x192 (28 KiB a k-block for 1.5
// times the work of 24 KiB): that product 388 -> 365 us, gate/up at 512 rows
// 107 -> 86, 1024 rows 187 -> 170, QKV at 1024 rows 117 -> 94.  Against the
// streaming kernel, 7B shapes, us: 2048 rows QKV 477 -> 230, O 153 -> 68,
// gate/up 620 -> 365, down 319 -> 167; 256 rows QKV 42 -> 40, O 28 -> 24 (with
// the finishing pass), gate/up 75 -> 65, LM head 119 -> 76.  Fragments read a
// step ahead of their MFMAs were no faster.  Where its tiles are too large for
// the matrix the streaming kernel stays (gemm_wide_takes).
#include <hip/hip_ext.h>

#include <algorithm>

#include "common.h"
#include "gemm_epilogue.h"
#include "kernels.h"

namespace {

constexpr int XCDS = 8;

template <int N>
struct Int {
  static constexpr int value = N;
};

// s_waitcnt vmcnt(N) lgkmcnt(0): all but the N youngest loads into LDS have
// landed, and every LDS read issued so far has its data (an MFMA may be
// scheduled past the barrier that follows; the read that feeds it must not
// still be in flight when the barrier lets its buffer be refilled).
template <int N>
__device__ __forceinline__ void wait_vm() {
  __builtin_amdgcn_s_waitcnt(0x0070 | (N & 15) | ((N >> 4) << 14));
}
__device__ __forceinline__ void wg_barrier() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}
// 16 bytes per lane, 1 KiB per wave, straight from memory into LDS.
__device__ __forceinline__ void dma_tile(const char* src, char* lds) {
  __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)src,
                                   (__attribute__((address_space(3))) void*)lds, 16, 0, 0);
}

constexpr int NS = 4;  // ring stages

// Waves WM x WN, each MT 16-row tiles x CB column blocks.  SL: the workgroup
// runs all reduction slices and adds them (otherwise it runs the one its place
// in the grid names).  AL: every class is a multiple of NS k-blocks, so a class
// always starts at ring position 0.
template <typename T, int KIND, int WM, int WN, int MT, int CB, bool SL, bool AL>
__global__ __launch_bounds__(64 * WM * WN, (WM * WN + 3) / 4) void gemm_wide_kernel(const GemmShape sh, const GemmEpi e,
                                                                                   int nrb, int ncb) {
  constexpr int VEC = ET<T>::VEC;
  constexpr int NW = WM * WN;
  constexpr int TA = WM * MT, TB = WN * CB, NT = TA + TB;  // 1 KiB tiles per stage
  constexpr int P = (NT + NW - 1) / NW;                    // of them per wave
  // one array per stage, and every use of one names it at compile time: the
  // compiler then knows which loads a read of a stage has to wait for
  constexpr int SB = NT * 1024;
  __shared__ __attribute__((aligned(1024))) char s0[SB], s1[SB], s2[SB], s3[SB];
  __shared__ RowMeta rm[KIND == EPI_QKV ? 16 * TA : 1];

  if (sh.skip && *sh.skip == 0) return;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / WN, wn = wave % WN;
  const int kblocks = sh.K / (4 * VEC);
  const int nbc = sh.nb_count ? sh.nb_count : sh.N / 16;
  // column runs are dealt to the dies in contiguous ranges, row blocks fastest
  const int zs = SL ? 1 : sh.splits;
  const int total = nrb * ncb * zs;
  const int xcd = blockIdx.x % XCDS, q = total / XCDS, rem = total % XCDS;
  const int idx = xcd * q + min(xcd, rem) + (int)blockIdx.x / XCDS;
  const int mb0 = (idx % nrb) * TA, cb0 = ((idx / nrb) % ncb) * TB, split = idx / (nrb * ncb);

  if constexpr (KIND == EPI_QKV) {
    for (int i = tid; i < 16 * TA; i += 64 * NW) {
      const int row = 16 * mb0 + i;
      RowMeta t{-1, 0, -1};
      if (row < sh.M) t = RowMeta{e.kvoff[row], e.pos[row], e.qrow[row]};
      rm[i] = t;
    }
  }
  // this wave's share of a stage: tiles wave, wave + NW, ... (past the last:
  // the last one again); rows and columns past the edge read the last tile
  const int kps = kblocks / sh.splits;
  const char* base[P];
  uint32_t step[P];  // bytes between consecutive k-blocks (an operand panel is under 4 GiB)
#pragma unroll
  for (int p = 0; p < P; ++p) {
    const int t = min(wave + NW * p, NT - 1);
    if (t < TA) {
      step[p] = (uint32_t)sh.x_mtiles * 1024;
      base[p] = (const char*)sh.X + (int64_t)min(mb0 + t, sh.x_mtiles - 1) * 1024;
    } else {
      const int c = sh.nb_off + min(cb0 + t - TA, nbc - 1);
      step[p] = NB * 1024;
      base[p] = (const char*)sh.W + ((int64_t)(c / NB) * kblocks * NB + c % NB) * 1024;
    }
    base[p] += (int64_t)(split * kps) * step[p];
  }
  const uint32_t lane16 = lane * 16;
  auto issue = [&](char* buf, uint32_t kb) __attribute__((always_inline)) {
#pragma unroll
    for (int p = 0; p < P; ++p)
      dma_tile(base[p] + (kb * step[p] + lane16), buf + min(wave + NW * p, NT - 1) * 1024);
  };

  f32x4 acc[MT][CB], tot[MT][CB], sum[SL ? MT : 1][SL ? CB : 1];
  const f32x4 zero = f32x4{0.f, 0.f, 0.f, 0.f};
  const f32x4 nzero = f32x4{-0.f, -0.f, -0.f, -0.f};  // nzero + x is x, bit for bit
  // Loads run NS - 1 stages ahead of the sums, over the k-blocks in the order
  // of the summation: in each slice the residue classes mod 4 one after
  // another.  Past the end they repeat k-block 0 (nothing reads it).
  const int slices = SL ? sh.splits : 1;
  int lbase = 0, lcls = 0, lkb = 0;
  const int lend = slices * kps, cls_n = min(4, kps);
  auto next_kb = [&]() __attribute__((always_inline)) {  // no branches: it sits between a barrier and the stage's loads
    const int kb = lbase < lend ? lbase + lkb : 0;
    const int nk = lkb + 4, c1 = lcls + 1;
    const bool wrap = nk >= kps, last = c1 >= cls_n;
    lkb = wrap ? (last ? 0 : c1) : nk;
    lcls = wrap ? (last ? 0 : c1) : lcls;
    lbase += wrap && last ? kps : 0;
    return (uint32_t)kb;
  };
  auto buf = [&](auto i) __attribute__((always_inline)) -> char* {
    constexpr int k = decltype(i)::value % NS;
    if constexpr (k == 0) return s0;
    else if constexpr (k == 1) return s1;
    else if constexpr (k == 2) return s2;
    else return s3;
  };
  // one stage: its own loads have landed (NS - 2 later stages still in
  // flight), every wave is past the stage before, whose buffer is refilled
  auto step_k = [&](auto i) __attribute__((always_inline)) {
    constexpr int I = decltype(i)::value;
    wait_vm<P * (NS - 2)>();
    wg_barrier();
    issue(buf(Int<I + NS - 1>{}), next_kb());
    const char* b = buf(i);
    int4 fa[MT], fb[CB];
#pragma unroll
    for (int j = 0; j < CB; ++j) fb[j] = ld16(b + (TA + wn * CB + j) * 1024 + lane16);
#pragma unroll
    for (int k = 0; k < MT; ++k) fa[k] = ld16(b + (wm * MT + k) * 1024 + lane16);
#pragma unroll
    for (int k = 0; k < MT; ++k)
#pragma unroll
      for (int j = 0; j < CB; ++j) acc[k][j] = mfma_kb<T>(fa[k], fb[j], acc[k][j]);
  };
  // the n k-blocks of one class, the first of them in ring position PH
  auto round = [&](auto ph) __attribute__((always_inline)) {
    constexpr int PH = decltype(ph)::value;
    step_k(Int<PH>{});
    step_k(Int<PH + 1>{});
    step_k(Int<PH + 2>{});
    step_k(Int<PH + 3>{});
  };
  auto run_class = [&](auto ph, int n) __attribute__((always_inline)) {
    constexpr int PH = decltype(ph)::value;
    int r = n / NS;
    if constexpr (AL) {
      for (; r > 0; --r) round(ph);
    } else {
      // a first round on its own: only its waits have to cover every history
      // of the ring that leads here
      if (r > 0) {
        round(ph);
        while (--r > 0) round(ph);
      }
      r = n % NS;
      if (r > 0) step_k(Int<PH>{});
      if (r > 1) step_k(Int<PH + 1>{});
      if (r > 2) step_k(Int<PH + 2>{});
    }
  };
  issue(s0, next_kb());
  issue(s1, next_kb());
  issue(s2, next_kb());
  int phase = 0;
#pragma unroll 1
  for (int sl = 0; sl < slices; ++sl) {
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
      for (int j = 0; j < CB; ++j) tot[i][j] = nzero;
#pragma unroll 1
    for (int c = 0; c < 4; ++c) {
#pragma unroll
      for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int j = 0; j < CB; ++j) acc[i][j] = zero;
      const int n = (kps - c + 3) / 4;
      if constexpr (AL) {
        run_class(Int<0>{}, n);
      } else {
        if (phase == 0) run_class(Int<0>{}, n);
        else if (phase == 1) run_class(Int<1>{}, n);
        else if (phase == 2) run_class(Int<2>{}, n);
        else run_class(Int<3>{}, n);
      }
      if constexpr (!AL) phase = (phase + n) % NS;
#pragma unroll
      for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int j = 0; j < CB; ++j) tot[i][j] = tot[i][j] + acc[i][j];
    }
    if constexpr (SL) {
#pragma unroll
      for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int j = 0; j < CB; ++j) sum[i][j] = sl == 0 ? tot[i][j] : sum[i][j] + tot[i][j];
    }
  }
  wait_vm<0>();  // no load may land after the workgroup's LDS is released

  wg_barrier();  // every wave is past its last read of a stage
  float* tw = reinterpret_cast<float*>(s0) + wave * 256;
  float* part = KIND == EPI_PARTIAL ? e.part + (int64_t)split * sh.M * sh.N : nullptr;
#pragma unroll
  for (int i = 0; i < MT; ++i) {
    const int mb = mb0 + wm * MT + i;
    if (16 * mb >= sh.M) break;  // wave-uniform
    // the rotary entries of a row tile's blocks are requested together
    f32x4 cs[KIND == EPI_QKV ? CB : 1], sn[KIND == EPI_QKV ? CB : 1];
    if constexpr (KIND == EPI_QKV) {
      const int hd = e.hd, bh = hd / 16;
#pragma unroll
      for (int j = 0; j < CB; ++j) {
        const int blk = sh.nb_off + min(cb0 + wn * CB + j, nbc - 1);
        cs[j] = f32x4{1.f, 1.f, 1.f, 1.f};
        sn[j] = zero;
        if (blk < 2 * e.H * bh) {  // wave-uniform
#pragma unroll
          for (int r = 0; r < 4; ++r) {  // rows past M read position 0
            const int64_t ti = (int64_t)rm[16 * (wm * MT + i) + 4 * (lane >> 4) + r].pos * (hd / 2) + 8 * (blk % bh) + (lane & 7);
            cs[j][r] = e.rcos[ti];
            sn[j][r] = e.rsin[ti];
          }
        }
      }
    }
#pragma unroll
    for (int j = 0; j < CB; ++j) {
      const int cj = cb0 + wn * CB + j;
      if (cj >= nbc) break;  // wave-uniform
      f32x4 v;
      if constexpr (SL) v = sum[i][j];
      else v = tot[i][j];
      constexpr int jq = KIND == EPI_QKV ? 1 : 0;
      store_tile<T, KIND>(sh, e, mb, sh.nb_off + cj, v, part, tw, jq ? rm + 16 * (wm * MT + i) : rm, cs[jq ? j : 0],
                          sn[jq ? j : 0], lane);
    }
  }
}

// Output tiles: rows x 16-column blocks per workgroup, and the time of one
// round of a launch with them on 256 CUs (us, K = 4096).
enum Tile { XL, BIG, MED, SQ, SML };
constexpr int TILE_ROWS[] = {256, 256, 256, 128, 128};
constexpr int TILE_BLKS[] = {12, 8, 6, 8, 6};

int tiles_of(Tile t, int M, int nbc) {
  return (M + TILE_ROWS[t] - 1) / TILE_ROWS[t] * ((nbc + TILE_BLKS[t] - 1) / TILE_BLKS[t]);
}

// Unsplit launches: the tile with the fewest rounds, weighted by the measured
// time of a round.  256-row tiles run one workgroup per CU (90 us a round with
// 192 columns, 64 with 128, 57 with 96), 128-row tiles two (74 and 65 us, or
// 46 and 43 us when the launch has at most one per CU).  The 192-column tile
// exists for reductions of whole rounds of the ring only (K a multiple of 512:
// the general one would spill).
Tile pick_tile(int M, int nbc, int kps) {
  auto cost = [&](Tile t) {
    const int n = tiles_of(t, M, nbc);
    switch (t) {
      case XL: return kps % 16 == 0 ? (n + 255) / 256 * 90 : 1 << 30;
      case BIG: return (n + 255) / 256 * 64;
      case MED: return (n + 255) / 256 * 57;
      case SQ: return n <= 256 ? 46 : (n + 511) / 512 * 74;
      default: return n <= 256 ? 43 : (n + 511) / 512 * 65;
    }
  };
  Tile best = XL;
  for (Tile t : {BIG, MED, SQ, SML})
    if (cost(t) < cost(best)) best = t;
  return best;
}

// Split-K shapes.  With at least 192 256x128 tiles a launch fills the chip by
// itself: each workgroup runs its slices one after another and adds them in
// registers (at 2048 x 4096 x 4096 65 us against 91 us with the slices side
// by side, and the consumer reads one partial instead of four).  Smaller ones
// put the slices side by side, on 256-row tiles if that makes 256 workgroups.
constexpr int SLICES_IN_WG_TILES = 192;
bool slices_in_wg(int M, int nbc) { return tiles_of(BIG, M, nbc) >= SLICES_IN_WG_TILES; }

}  // namespace

int gemm_wide_tile(int M, int nbc, int kps, int splits) {
  if (splits == 1) return pick_tile(M, nbc, kps);
  return slices_in_wg(M, nbc) || tiles_of(BIG, M, nbc) * splits >= 256 ? BIG : SQ;
}

namespace {

// Time of a launch in us, from what a CU takes in (1 KiB tiles, 16 rows or
// columns by a k-block) and its output tiles, in rounds of 256 workgroups.
// Fitted to 991 launches of 129 to 2048 rows, 64 to 32000 columns and K from
// 256 to 16384 on both kernels: a CU takes in about 70 GB/s, a streaming
// workgroup reduces and stores an output tile in 0.1 us (its four waves meet in
// LDS), one of this kernel's (eight waves, no reduction) in 0.0125 us.  Picked
// by it no launch is more than 4% slower than on the streaming kernel, 13 are
// on this one.
double launch_us(double fixed, int wgs, int kblocks, int row_tiles, int blocks, double in_us, double out_us) {
  return fixed + (wgs + 255) / 256 * ((double)kblocks * (row_tiles + blocks) * in_us + row_tiles * blocks * out_us);
}
double stream_us(int M, int nbc, int kps, int splits, int x_mtiles) {
  const StreamPlan p = gemm_stream_plan(M, nbc, splits, x_mtiles);
  return launch_us(2.0, p.row_blocks * p.runs * splits, kps, p.row_tiles, p.run, 14.0 / 1024, 0.1);
}
double wide_us(int M, int nbc, int kps, int splits) {
  const bool sl = splits > 1 && slices_in_wg(M, nbc);
  const Tile t = (Tile)gemm_wide_tile(M, nbc, kps, splits);
  return launch_us(3.5, tiles_of(t, M, nbc) * (sl ? 1 : splits), sl ? kps * splits : kps, TILE_ROWS[t] / 16, TILE_BLKS[t],
                   15.0 / 1024, 0.0125);
}

template <typename T, int KIND, int WM, int WN, int MT, int CB, bool SL>
void go(const GemmShape& s, const GemmEpi& e, hipStream_t st, hipEvent_t ea, hipEvent_t eb) {
  const int nbc = s.nb_count ? s.nb_count : s.N / 16;
  const int nrb = (s.M + 16 * WM * MT - 1) / (16 * WM * MT), ncb = (nbc + WN * CB - 1) / (WN * CB);
  const int kps = s.K / (4 * ET<T>::VEC) / s.splits;
  const dim3 grid(nrb * ncb * (SL ? 1 : s.splits)), wg(64 * WM * WN);
  const bool al = kps % (4 * NS) == 0;
  if (ea || eb) {
    if (al)
      hipExtLaunchKernelGGL((gemm_wide_kernel<T, KIND, WM, WN, MT, CB, SL, true>), grid, wg, 0, st, ea, eb, 0, s, e,
                            nrb, ncb);
    else if constexpr (CB < 6)
      hipExtLaunchKernelGGL((gemm_wide_kernel<T, KIND, WM, WN, MT, CB, SL, false>), grid, wg, 0, st, ea, eb, 0, s,
                            e, nrb, ncb);
    return;
  }
  if (al)
    hipLaunchKernelGGL((gemm_wide_kernel<T, KIND, WM, WN, MT, CB, SL, true>), grid, wg, 0, st, s, e, nrb, ncb);
  else if constexpr (CB < 6)
    hipLaunchKernelGGL((gemm_wide_kernel<T, KIND, WM, WN, MT, CB, SL, false>), grid, wg, 0, st, s, e, nrb, ncb);
}

template <int KIND>
void go_unsplit(const GemmShape& s, const GemmEpi& e, hipStream_t st, hipEvent_t ea, hipEvent_t eb) {
  switch (gemm_wide_tile(s.M, s.nb_count ? s.nb_count : s.N / 16, s.K / (4 * ET<bf16_t>::VEC), 1)) {
    case XL: go<bf16_t, KIND, 4, 2, 4, 6, false>(s, e, st, ea, eb); break;
    case BIG: go<bf16_t, KIND, 4, 2, 4, 4, false>(s, e, st, ea, eb); break;
    case MED: go<bf16_t, KIND, 4, 2, 4, 3, false>(s, e, st, ea, eb); break;
    case SQ: go<bf16_t, KIND, 4, 2, 2, 4, false>(s, e, st, ea, eb); break;
    default: go<bf16_t, KIND, 4, 2, 2, 3, false>(s, e, st, ea, eb); break;
  }
}

template <int KIND>
void go_slices(const GemmShape& s, const GemmEpi& e, hipStream_t st, hipEvent_t ea, hipEvent_t eb) {
  go<bf16_t, KIND, 4, 2, 4, 4, true>(s, e, st, ea, eb);
}

}  // namespace

bool gemm_wide_fits(int K, int x_mtiles) { return (int64_t)K * 16 * x_mtiles * 2 < (int64_t)1 << 32 && K < 1 << 24; }

bool gemm_wide_takes(int dtype, int M, int nbc, int K, int splits, int x_mtiles) {
  // up to 128 rows the streaming kernel is faster (QKV at 128 rows 33 us
  // against 37 us)
  if (dtype != DT_BF16 || M <= 128 || !gemm_wide_fits(K, x_mtiles)) return false;
  // Matrices too small for its tiles to reach most CUs, and those whose
  // columns the streaming kernel deals in shorter runs, stay on that one, us:
  // 256 rows 768 x 256 3.8 / 5.8, 1024 x 4096 14.7 / 15.6, 8192 x 4096 30.6 /
  // 39.4, 5120 x 13824 68 / 77; 512 rows 2048 x 256 5.5 / 6.6.
  const int kps = K / 32 / splits;
  return wide_us(M, nbc, kps, splits) <= stream_us(M, nbc, kps, splits, x_mtiles);
}

bool gemm_wide_sums_slices(int M, int nbc, int kind) {
  return (kind == EPI_PARTIAL || kind == EPI_F32 || kind == EPI_SILU) && slices_in_wg(M, nbc);
}

void launch_gemm_wide(const GemmShape& s, const GemmEpi& e, hipStream_t st, hipEvent_t ea, hipEvent_t eb) {
  const int nbc = s.nb_count ? s.nb_count : s.N / 16;
  if (s.splits > 1 && gemm_wide_sums_slices(s.M, nbc, e.kind)) {
    if (e.kind == EPI_PARTIAL) go_slices<EPI_PARTIAL>(s, e, st, ea, eb);
    else if (e.kind == EPI_F32) go_slices<EPI_F32>(s, e, st, ea, eb);
    else go_slices<EPI_SILU>(s, e, st, ea, eb);
  } else if (e.kind == EPI_PARTIAL) {
    if (gemm_wide_tile(s.M, nbc, s.K / (4 * ET<bf16_t>::VEC) / s.splits, s.splits) == BIG)
      go<bf16_t, EPI_PARTIAL, 4, 2, 4, 4, false>(s, e, st, ea, eb);
    else
      go<bf16_t, EPI_PARTIAL, 4, 2, 2, 4, false>(s, e, st, ea, eb);
  } else if (e.kind == EPI_F32) {
    go_unsplit<EPI_F32>(s, e, st, ea, eb);
  } else if (e.kind == EPI_SILU) {
    go_unsplit<EPI_SILU>(s, e, st, ea, eb);
  } else if (e.kind == EPI_SWIGLU) {
    go_unsplit<EPI_SWIGLU>(s, e, st, ea, eb);
  } else if (e.kind == EPI_QKV) {  // launch_gemm refuses every other kind
    go_unsplit<EPI_QKV>(s, e, st, ea, eb);
  }
}
