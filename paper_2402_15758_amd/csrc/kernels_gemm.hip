// Skinny GEMMs on MFMA for the decode step: Y = X[M][K] @ W[K][N] with M the
// number of tree nodes (or draft rows) and W streamed from HBM exactly once.
//
// Both operands are stored in MFMA fragment order, so every operand load of
// a wave is one contiguous 1 KiB (64 lanes x 16 bytes):
//   * W (repacked at load): layout group g of 4 column blocks stores its
//     tiles as [g][kb][4][1 KiB];
//   * X (written tiled by the kernel that produces it): tile (kb, mb) of
//     16 rows x KB reduction indices at ((kb * mtiles + mb) * 64 + lane).
//
// Work split.  A launch runs GEMM_WGS / splits workgroups per reduction slice
// (more only when a matrix has over CB_MAX column blocks per workgroup), and
// the 16-column blocks are dealt out in contiguous runs whose lengths differ
// by at most one, so every CU streams the same number of weight bytes and
// the activation tiles a workgroup reads are reused across its whole run.
// A workgroup = 4 wave64s; its waves take interleaved k-blocks and are summed
// through LDS in wave order.  The steady-state loop issues the loads of
// stage s + PF unconditionally, so the wait before stage s only covers that
// stage's own loads.  Split-K slices are written as partials and summed in
// slice order by their consumer (the next norm) or by a finishing pass that
// applies the epilogue.  Every row's arithmetic depends only on (N, K): the
// same row gives identical bits whether a launch carries 1 or 256 rows.
#include <hip/hip_ext.h>

#include <algorithm>

#include "common.h"
#include "gemm_epilogue.h"
#include "kernels.h"

// The GEMM kernels take GemmShape and GemmEpi by value: a plain block of
// pointers and integers well inside the kernel-argument limit.
static_assert(sizeof(GemmShape) + sizeof(GemmEpi) + 4 * sizeof(int) <= 512, "GEMM kernel-argument block");
static_assert(alignof(GemmShape) <= 8 && alignof(GemmEpi) <= 8, "GEMM kernel-argument alignment");

namespace {

constexpr int CB_MAX = 8;    // column blocks per workgroup, upper bound
constexpr int CB_MAX_MB8 = 6;  // with 128-row tiles: runs of up to 6 blocks fit the registers without spills
constexpr int RED_TILES = 32;  // 16x16 output tiles per wave in one LDS reduction round (4 x 32 KiB)
constexpr int GEMM_WGS = 256;  // one workgroup per CU per reduction slice
constexpr int GEMM_XCDS = 8;   // accelerator dies; workgroups are dealt to them round-robin
// Matrices at least this wide run unsplit (their epilogue needs whole sums and
// they fill the GPU on their own); narrower ones split the reduction until a
// launch has at least SPLIT_TARGET_WGS 64-column groups' worth of work.
constexpr int SPLIT_MIN_COLS_NO = 8192;
constexpr int SPLIT_TARGET_WGS = 256;

// ---------------------------------------------------------------------------
// Weight repacking (load time).  Packed column block c, lane column cl:
//   PACK_NATURAL: column 16 c + cl.
//   PACK_QKV: sections Q, K, V of H * hd / 16 blocks each; block q of head h
//     holds, for Q and K, rotary dims 8q + cl (cl < 8) and hd/2 + 8q + cl - 8
//     (cl >= 8), so both halves of a rotary pair sit in lanes cl and cl ^ 8;
//     V keeps dims 16q + cl.
//   PACK_GU: gate column 8c + cl (cl < 8) and up column 8c + cl - 8 (cl >= 8).
// ---------------------------------------------------------------------------
template <typename T>
__global__ void repack_kernel(const T* __restrict__ s0, const T* __restrict__ s1, const T* __restrict__ s2, int K,
                              int n_src, int kind, int H, int hd, T* __restrict__ dst, int nblocks) {
  constexpr int VEC = ET<T>::VEC, KB = 4 * VEC;
  const int kblocks = K / KB;
  const int64_t tid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t total = (int64_t)nblocks * kblocks * 64;
  if (tid >= total) return;
  const int lane = (int)(tid & 63);
  const int64_t tile = tid >> 6;
  const int kb = (int)(tile % kblocks);
  const int c = (int)(tile / kblocks);
  const int cl = lane & 15;
  const T* src = s0;
  int col;
  if (kind == PACK_QKV) {
    const int per_sec = H * hd / 16;
    const int sec = c / per_sec, within = c % per_sec;
    const int h = within / (hd / 16), q = within % (hd / 16);
    const int dim = sec < 2 ? (cl < 8 ? 8 * q + cl : hd / 2 + 8 * q + cl - 8) : 16 * q + cl;
    src = sec == 0 ? s0 : (sec == 1 ? s1 : s2);
    col = h * hd + dim;
  } else if (kind == PACK_GU) {
    src = cl < 8 ? s0 : s1;
    col = 8 * c + (cl & 7);
  } else {
    col = 16 * c + cl;
  }
  const int k0 = kb * KB + (lane >> 4) * VEC;
  T* d = dst + ((((int64_t)(c / NB) * kblocks + kb) * NB + c % NB) * 64 + lane) * VEC;
#pragma unroll
  for (int e = 0; e < VEC; ++e) d[e] = src[(int64_t)(k0 + e) * n_src + col];
}

template <typename T>
__device__ __forceinline__ int4 ldw(const T* p) {
  typedef int i32x4 __attribute__((ext_vector_type(4)));
  const i32x4 v = __builtin_nontemporal_load(reinterpret_cast<const i32x4*>(p));
  return int4{v.x, v.y, v.z, v.w};
}

// One workgroup's run of CB column blocks starting at block cb0, rows
// [16 mb0, 16 (mb0 + MB)), reduction slice [kbeg, kend).  red: LDS of
// [4][MB][CB][64] f32x4.
// Epilogue of gemm_run for column blocks [J0, J0 + JN) of the run: the waves'
// partial sums are added in wave order through LDS, then stored.
template <typename T, int MB, int CB, int J0, int JN>
__device__ __forceinline__ void gemm_epilogue(const GemmShape& sh, const GemmEpi& e, int kind, int cb0, int mb0,
                                              const f32x4 (&acc)[MB][CB], f32x4* red, const RowMeta* rm,
                                              float* stage, int wave, int lane, int split) {
  const int g = lane >> 4, c16 = lane & 15;
  // this wave's output tiles: items it = wave, wave + 4, ... of MB * JN
  constexpr int ITEMS = (MB * JN + 3) / 4;
  // QKV: the rotary table entries of every element are requested first, so
  // that their round trip overlaps the reduction below
  float cs[ITEMS][4], sn[ITEMS][4];
  if (kind == EPI_QKV) {
#pragma unroll
    for (int k = 0; k < ITEMS; ++k) {
      const int it = wave + 4 * k;
      const int i = it / JN, j = J0 + it % JN;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        cs[k][r] = 1.f;
        sn[k][r] = 0.f;
        const int lr = 16 * i + 4 * g + r;
        const int row = 16 * mb0 + lr;
        const int q = (cb0 + j) % (e.hd / 16);
        const bool rot = (cb0 + j) < 2 * e.H * (e.hd / 16);
        if (it < MB * JN && row < sh.M && rot) {
          const int64_t ti = (int64_t)rm[lr].pos * (e.hd / 2) + 8 * q + (c16 & 7);
          cs[k][r] = e.rcos[ti];
          sn[k][r] = e.rsin[ti];
        }
      }
    }
  }
#pragma unroll
  for (int i = 0; i < MB; ++i)
#pragma unroll
    for (int jj = 0; jj < JN; ++jj) red[((wave * MB + i) * JN + jj) * 64 + lane] = acc[i][J0 + jj];
  __syncthreads();
  f32x4 vv[ITEMS], vpp[ITEMS];
#pragma unroll
  for (int k = 0; k < ITEMS; ++k) {
    const int it = wave + 4 * k;
    if (it < MB * JN) {  // wave-uniform
      const int i = it / JN, j = it % JN;
      f32x4 v = red[((0 * MB + i) * JN + j) * 64 + lane];
#pragma unroll
      for (int w = 1; w < 4; ++w) v = v + red[((w * MB + i) * JN + j) * 64 + lane];
      vv[k] = v;
#pragma unroll
      for (int r = 0; r < 4; ++r) vpp[k][r] = dpp_mov<DPP_ROR8>(v[r]);  // lane column c16 ^ 8
    }
  }
  if (kind == EPI_QKV) {
    if constexpr (sizeof(T) == 2) {
      // each 16x16 tile goes through the wave's LDS tile, then 32 lanes store
      // 8 consecutive outputs of one row each
      T* tw = reinterpret_cast<T*>(stage + wave * 256);
#pragma unroll
      for (int k = 0; k < ITEMS; ++k) {
        const int it = wave + 4 * k;
        if (it >= MB * JN) break;  // wave-uniform
        const int i = it / JN, blk = cb0 + J0 + it % JN;
#pragma unroll
        for (int r = 0; r < 4; ++r)
          tw[(4 * g + r) * 16 + c16] = ET<T>::from_f(qkv_value(e, blk, c16, vv[k][r], vpp[k][r], cs[k][r], sn[k][r]));
        __builtin_amdgcn_wave_barrier();
        if (lane < 32) {
          const int lr = 16 * i + (lane & 15);
          const int4 v = *reinterpret_cast<const int4*>(tw + (lane & 15) * 16 + 8 * (lane >> 4));
          if (16 * mb0 + lr < sh.M) qkv_store16<T>(e, rm[lr], blk, lane >> 4, v);
        }
        __builtin_amdgcn_wave_barrier();
      }
      return;
    }
#pragma unroll
    for (int k = 0; k < ITEMS; ++k) {
      const int it = wave + 4 * k;
      const int i = it / JN, j = J0 + it % JN;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int lr = 16 * i + 4 * g + r;
        const int row = 16 * mb0 + lr;
        if (it < MB * JN && row < sh.M) qkv_store<T>(e, rm[lr], cb0 + j, c16, vv[k][r], vpp[k][r], cs[k][r], sn[k][r]);
      }
    }
    return;
  }
  if (kind == EPI_F32 || kind == EPI_PARTIAL) {
    // float outputs: the tile goes through the wave's LDS tile, then each lane
    // stores 4 consecutive columns of one row (16 rows x 64 bytes)
    float* tw = stage + wave * 256;
    float* base;
    int64_t ld;
    if (kind == EPI_F32) {
      base = e.out_f;
      ld = e.ldo;
    } else {
      base = e.part + (int64_t)split * sh.M * sh.N;
      ld = sh.N;
    }
#pragma unroll
    for (int k = 0; k < ITEMS; ++k) {
      const int it = wave + 4 * k;
      if (it >= MB * JN) break;  // wave-uniform
      const int i = it / JN, blk = cb0 + J0 + it % JN;
#pragma unroll
      for (int r = 0; r < 4; ++r) tw[(4 * g + r) * 16 + c16] = vv[k][r];
      __builtin_amdgcn_wave_barrier();
      const int row = 16 * (mb0 + i) + (lane >> 2);
      const f32x4 v = *reinterpret_cast<const f32x4*>(tw + (lane >> 2) * 16 + 4 * (lane & 3));
      if (row < sh.M) *reinterpret_cast<f32x4_any*>(base + (int64_t)row * ld + 16 * blk + 4 * (lane & 3)) = v;
      __builtin_amdgcn_wave_barrier();
    }
    return;
  }
  if constexpr (sizeof(T) == 2) {
    if (kind == EPI_SWIGLU) {
      // the 16 x 8 outputs of a tile (gate columns c16 < 8 times their up
      // partners) are 16 rows of 8 consecutive tiled elements: one 16-byte
      // store per row
      T* tw = reinterpret_cast<T*>(stage + wave * 256);
#pragma unroll
      for (int k = 0; k < ITEMS; ++k) {
        const int it = wave + 4 * k;
        if (it >= MB * JN) break;  // wave-uniform
        const int i = it / JN, blk = cb0 + J0 + it % JN;
        if (c16 < 8) {
#pragma unroll
          for (int r = 0; r < 4; ++r) tw[(4 * g + r) * 8 + c16] = ET<T>::from_f(silu_f(vv[k][r]) * vpp[k][r]);
        }
        __builtin_amdgcn_wave_barrier();
        if (lane < 16) {
          const int row = 16 * (mb0 + i) + lane;
          const int4 v = *reinterpret_cast<const int4*>(tw + lane * 8);
          if (row < sh.M) *reinterpret_cast<int4*>((T*)e.out_t + tiled_index<T>(e.o_mtiles, row, 8 * blk)) = v;
        }
        __builtin_amdgcn_wave_barrier();
      }
      return;
    }
  }
#pragma unroll
  for (int k = 0; k < ITEMS; ++k) {
    const int it = wave + 4 * k;
    const int i = it / JN, j = J0 + it % JN;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int row = 16 * (mb0 + i) + 4 * g + r;
      if (it < MB * JN && row < sh.M)
        epi_elem<T>(e, kind, sh.N, sh.M, split, row, cb0 + j, c16, vv[k][r], vpp[k][r]);
    }
  }
}

template <typename T, int MB, int CB, int PF>
__device__ __forceinline__ void gemm_run(const GemmShape& sh, const GemmEpi& e, int kind, int cb0, int mb0, int kbeg,
                                         int kend, f32x4* red, const RowMeta* rm, float* stage, int split) {
  constexpr int VEC = ET<T>::VEC;
  // The wave index is made provably wave-uniform so that every branch of the
  // k-loop below is a scalar branch: an MFMA ignores EXEC, so it must never
  // sit in a lane-predicated region.
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int kblocks = sh.K / (4 * VEC);
  const T* X = (const T*)sh.X + (int64_t)lane * VEC;
  const T* Wl = (const T*)sh.W + (int64_t)lane * VEC;
  int64_t wofs[CB];
#pragma unroll
  for (int j = 0; j < CB; ++j) {
    const int c = cb0 + j;
    wofs[j] = ((int64_t)(c / NB) * kblocks * NB + c % NB) * 64 * VEC;
  }

  f32x4 acc[MB][CB];
#pragma unroll
  for (int i = 0; i < MB; ++i)
#pragma unroll
    for (int j = 0; j < CB; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

  int4 bw[PF][CB], bx[PF][MB];
  auto load = [&](int s, int kb) {
#pragma unroll
    for (int j = 0; j < CB; ++j) bw[s][j] = ldw(Wl + wofs[j] + (int64_t)kb * NB * 64 * VEC);
#pragma unroll
    for (int i = 0; i < MB; ++i) bx[s][i] = ld16(X + ((int64_t)kb * sh.x_mtiles + mb0 + i) * 64 * VEC);
  };
  auto mma = [&](int s) {
#pragma unroll
    for (int i = 0; i < MB; ++i)
#pragma unroll
      for (int j = 0; j < CB; ++j) acc[i][j] = mfma_kb<T>(bx[s][i], bw[s][j], acc[i][j]);
  };
  // wave w takes k-blocks kbeg + w, kbeg + w + 4, ... (nk of them)
  const int kfirst = kbeg + wave;
  const int nk = kfirst < kend ? (kend - kfirst + 3) / 4 : 0;
  if (nk >= PF) {
#pragma unroll
    for (int s = 0; s < PF; ++s) load(s, kfirst + 4 * s);
    int it = 0;
    for (; it + 2 * PF <= nk; it += PF) {
#pragma unroll
      for (int s = 0; s < PF; ++s) {
        mma(s);
        load(s, kfirst + 4 * (it + PF + s));
      }
    }
    // stages it .. it+PF-1 are loaded; rem (< PF) k-blocks remain after them
    const int rem = nk - it - PF;
#pragma unroll
    for (int s = 0; s < PF; ++s) {
      mma(s);
      if (s < rem) load(s, kfirst + 4 * (it + PF + s));
    }
#pragma unroll
    for (int s = 0; s < PF - 1; ++s)
      if (s < rem) mma(s);
  } else {
    for (int t = 0; t < nk; ++t) {
      load(0, kfirst + 4 * t);
      mma(0);
    }
  }

  // the four waves' partial sums meet in LDS, JR column blocks at a time
  constexpr int JR = CB < RED_TILES / MB ? CB : RED_TILES / MB;
  gemm_epilogue<T, MB, CB, 0, JR>(sh, e, kind, cb0, mb0, acc, red, rm, stage, wave, lane, split);
  if constexpr (CB > JR) {
    __syncthreads();  // the first round's reads of red are done
    gemm_epilogue<T, MB, CB, JR, CB - JR>(sh, e, kind, cb0, mb0, acc, red, rm, stage, wave, lane, split);
  }
}

// Workgroup -> (row block, column run, split).  Workgroups are dealt to the
// 8 XCDs round-robin by linear id.  When a launch has several row blocks and
// its (run, split) count is a multiple of 8, consecutive workgroups of one
// XCD take the row blocks of one weight run, so every run's weight tiles are
// fetched from HBM once into that XCD's L2 and re-read from there; otherwise
// the linear order is used.  The mapping moves no arithmetic.  Two row blocks
// of 64 (65 to 128 rows, runs of 7 or 8 blocks) at 96 rows, linear -> mapped,
// us: LM head 7B 94.7 -> 75.6, 13B 115 -> 90, gate/up 13B 104 -> 81.
struct GemmTile {
  int rb, run, split;
};
// X, Y: grid.x and grid.y (X > 1 and grid.y * grid.z a multiple of 8).
__device__ __forceinline__ GemmTile gemm_tile_xcd(int X, int Y) {
  const int L = blockIdx.x + X * (blockIdx.y + Y * blockIdx.z);  // linear dispatch id
  const int xcd = L % GEMM_XCDS, k = L / GEMM_XCDS;
  const int r = (k / X) * GEMM_XCDS + xcd;
  return GemmTile{k % X, r % Y, r / Y};
}

// grid = (row blocks of 16 MB, workgroups per slice, splits).  Workgroups
// [0, nbig) own CBA column blocks, the others CBA - 1.
template <typename T, int MB, int CBA, bool XCD_MAP>
__global__ __launch_bounds__(256) void gemm_kernel(const GemmShape sh, const GemmEpi e, int kind, int nbig, int gx,
                                                   int gy) {
  constexpr int PF = MB == 1 ? 4 : (MB >= 8 ? 2 : 3);
  constexpr int JR = CBA < RED_TILES / MB ? CBA : RED_TILES / MB;
  if (sh.skip && *sh.skip == 0) return;
  __shared__ f32x4 red[4 * MB * JR * 64];
  const int kblocks = sh.K / (4 * ET<T>::VEC);
  const int kps = kblocks / sh.splits;
  const GemmTile tl = XCD_MAP ? gemm_tile_xcd(gx, gy) : GemmTile{(int)blockIdx.x, (int)blockIdx.y, (int)blockIdx.z};
  const int kbeg = tl.split * kps;
  const int kend = kbeg + kps;
  const int b = tl.run;
  const int mb0 = tl.rb * MB;
  // QKV epilogue targets of this workgroup's rows (visible after the k-loop's
  // barrier)
  __shared__ RowMeta rm[16 * MB];
  __shared__ __attribute__((aligned(16))) float stage[4 * 256];  // a 16x16 output tile per wave
  if (kind == EPI_QKV && threadIdx.x < 16 * MB) {
    const int row = 16 * mb0 + threadIdx.x;
    RowMeta t{-1, 0, -1};
    if (row < sh.M) t = RowMeta{e.kvoff[row], e.pos[row], e.qrow[row]};
    rm[threadIdx.x] = t;
  }
  if (b < nbig) {
    gemm_run<T, MB, CBA, PF>(sh, e, kind, sh.nb_off + b * CBA, mb0, kbeg, kend, red, rm, stage, tl.split);
  } else {
    if constexpr (CBA > 1)
      gemm_run<T, MB, CBA - 1, PF>(sh, e, kind, sh.nb_off + nbig * CBA + (b - nbig) * (CBA - 1), mb0, kbeg, kend,
                                   red, rm, stage, tl.split);
  }
}

// Sum split-K partials in split order and apply the epilogue (one thread
// per output element of the launch's column blocks).
template <typename T>
__global__ void gemm_finish_kernel(const GemmShape sh, const GemmEpi e, int kind, const float* __restrict__ part) {
  if (sh.skip && *sh.skip == 0) return;
  const int nbc = sh.nb_count ? sh.nb_count : sh.N / 16;
  const int64_t tid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t total = (int64_t)sh.M * nbc * 16;
  if (tid >= total) return;
  const int c16 = (int)(tid & 15);
  const int blk = sh.nb_off + (int)((tid >> 4) % nbc);
  const int row = (int)((tid >> 4) / nbc);
  // every slice is requested before the first is added
  float pv[GEMM_MAX_SPLITS], pp[GEMM_MAX_SPLITS];
#pragma unroll
  for (int s = 0; s < GEMM_MAX_SPLITS; ++s) {
    if (s < sh.splits) {
      const float* p = part + ((int64_t)s * sh.M + row) * sh.N + 16 * blk;
      pv[s] = p[c16];
      pp[s] = p[c16 ^ 8];
    }
  }
  float v = pv[0], vp = pp[0];
#pragma unroll
  for (int s = 1; s < GEMM_MAX_SPLITS; ++s) {
    if (s < sh.splits) {
      v = v + pv[s];
      vp = vp + pp[s];
    }
  }
  epi_elem<T>(e, kind, sh.N, sh.M, 0, row, blk, c16, v, vp);
}

template <typename T, int MB, int CBA>
void gemm_launch(const GemmShape& s, const GemmEpi& e, int kind, const StreamPlan& p, hipStream_t st, hipEvent_t ea,
                 hipEvent_t eb) {
  const int gx = p.row_blocks, gy = p.runs, nbig = p.long_runs;
  dim3 grid(gx, gy, s.splits);
  if (p.mapped) {
    if constexpr (MB >= 4) {  // smaller tiles are for launches of one row block
      if (ea || eb)
        hipExtLaunchKernelGGL((gemm_kernel<T, MB, CBA, true>), grid, dim3(256), 0, st, ea, eb, 0, s, e, kind, nbig, gx,
                              gy);
      else
        hipLaunchKernelGGL((gemm_kernel<T, MB, CBA, true>), grid, dim3(256), 0, st, s, e, kind, nbig, gx, gy);
      return;
    }
  }
  if (ea || eb)
    hipExtLaunchKernelGGL((gemm_kernel<T, MB, CBA, false>), grid, dim3(256), 0, st, ea, eb, 0, s, e, kind, nbig, gx,
                          gy);
  else
    hipLaunchKernelGGL((gemm_kernel<T, MB, CBA, false>), grid, dim3(256), 0, st, s, e, kind, nbig, gx, gy);
}

template <typename T, int MB>
void gemm_mb(const GemmShape& s, const GemmEpi& e, int kind, const StreamPlan& p, hipStream_t st, hipEvent_t ea,
             hipEvent_t eb) {
  switch (p.run) {
    case 1: gemm_launch<T, MB, 1>(s, e, kind, p, st, ea, eb); break;
    case 2: gemm_launch<T, MB, 2>(s, e, kind, p, st, ea, eb); break;
    case 3: gemm_launch<T, MB, 3>(s, e, kind, p, st, ea, eb); break;
    case 4: gemm_launch<T, MB, 4>(s, e, kind, p, st, ea, eb); break;
    case 5: gemm_launch<T, MB, 5>(s, e, kind, p, st, ea, eb); break;
    case 6: gemm_launch<T, MB, 6>(s, e, kind, p, st, ea, eb); break;
    default:
      if constexpr (MB < 8) {  // 128-row tiles take runs of up to CB_MAX_MB8 blocks
        if (p.run == 7)
          gemm_launch<T, MB, 7>(s, e, kind, p, st, ea, eb);
        else
          gemm_launch<T, MB, 8>(s, e, kind, p, st, ea, eb);
      }
      break;
  }
}

int gemm_blocks(const GemmShape& s) { return s.nb_count ? s.nb_count : s.N / 16; }

template <typename T>
void launch_finish(const GemmShape& s, const GemmEpi& e, hipStream_t st, hipEvent_t ev_stop) {
  const int64_t total = (int64_t)s.M * gemm_blocks(s) * 16;
  const dim3 grid((unsigned)((total + 255) / 256));
  if (ev_stop)
    hipExtLaunchKernelGGL((gemm_finish_kernel<T>), grid, dim3(256), 0, st, nullptr, ev_stop, 0, s, e, e.kind,
                          (const float*)e.part);
  else
    hipLaunchKernelGGL((gemm_finish_kernel<T>), grid, dim3(256), 0, st, s, e, e.kind, (const float*)e.part);
}

template <typename T>
void gemm_t(const GemmShape& s, const GemmEpi& e, hipStream_t st, hipEvent_t ev_start, hipEvent_t ev_stop) {
  const StreamPlan p = gemm_stream_plan(s.M, gemm_blocks(s), s.splits, s.x_mtiles);
  const bool finish = s.splits > 1 && e.kind != EPI_PARTIAL;
  const int kind = finish ? EPI_PARTIAL : e.kind;
  hipEvent_t eb = finish ? nullptr : ev_stop;
  switch (p.row_tiles) {
    case 1: gemm_mb<T, 1>(s, e, kind, p, st, ev_start, eb); break;
    case 2: gemm_mb<T, 2>(s, e, kind, p, st, ev_start, eb); break;
    case 4: gemm_mb<T, 4>(s, e, kind, p, st, ev_start, eb); break;
    default: gemm_mb<T, 8>(s, e, kind, p, st, ev_start, eb); break;
  }
  if (finish) launch_finish<T>(s, e, st, ev_stop);
}

template <typename T>
__global__ void tile_rows_kernel(const T* __restrict__ src, int M, int K, T* __restrict__ dst, int mtiles) {
  const int64_t tid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (tid >= (int64_t)M * K) return;
  const int r = (int)(tid / K), c = (int)(tid % K);
  copy_tiled<T>(dst, mtiles, r, c, src[tid]);
}

// Both operands of one product in a single launch (the static-scratch GEMM):
// workgroups [0, nw) pack STAGE_KB k-blocks of a 64-column group of w each,
// the others tile x.  Rows are read 16 bytes a lane, a k-block's 4 KiB in one
// go, and the columns gathered from LDS: lanes that fetch a column each read
// 2 bytes at a row's stride eight times over.
constexpr int STAGE_KB = 4;
template <typename T>
__global__ __launch_bounds__(256) void stage_operands_kernel(const T* __restrict__ x, int M, int K, T* __restrict__ xd,
                                                             int mtiles, const T* __restrict__ w, int N,
                                                             T* __restrict__ wd, int nw) {
  constexpr int VEC = ET<T>::VEC, KB = 4 * VEC, PPR = 64 / VEC;  // 16-byte pieces of a 64-column row
  constexpr int PITCH = 64 + VEC;
  __shared__ __attribute__((aligned(16))) T tile[STAGE_KB][KB * PITCH];
  const int kblocks = K / KB, tid = threadIdx.x;
  if ((int)blockIdx.x >= nw) {  // x: one 16-byte piece a thread, consecutive rows side by side in the tiles
    const int64_t i = (int64_t)(blockIdx.x - nw) * 256 + tid;
    if (i >= (int64_t)M * (K / VEC)) return;
    const int r = (int)(i % M), q = (int)(i / M);
    st16(xd + tiled_index<T>(mtiles, r, q * VEC), ld16(x + (int64_t)r * K + q * VEC));
    return;
  }
  const int kgroups = (kblocks + STAGE_KB - 1) / STAGE_KB;
  const int grp = blockIdx.x / kgroups, kb0 = blockIdx.x % kgroups * STAGE_KB, n = min(STAGE_KB, kblocks - kb0);
  const int row = tid / PPR, piece = tid % PPR;  // KB rows x PPR pieces = 256
  int4 v[STAGE_KB];
#pragma unroll
  for (int k = 0; k < STAGE_KB; ++k)
    if (k < n) v[k] = ld16(w + ((int64_t)(kb0 + k) * KB + row) * N + grp * 64 + piece * VEC);
#pragma unroll
  for (int k = 0; k < STAGE_KB; ++k)
    if (k < n) st16(&tile[k][row * PITCH + piece * VEC], v[k]);
  __syncthreads();
  const int lane = tid & 63, col = 16 * (tid >> 6) + (lane & 15), k0 = (lane >> 4) * VEC;
#pragma unroll
  for (int k = 0; k < STAGE_KB; ++k) {
    if (k >= n) break;
    int4 o;
    T* e = reinterpret_cast<T*>(&o);
#pragma unroll
    for (int j = 0; j < VEC; ++j) e[j] = tile[k][(k0 + j) * PITCH + col];
    st16(wd + (((int64_t)grp * kblocks + kb0 + k) * 256 + tid) * VEC, o);
  }
}

}  // namespace

void launch_tile_rows(int dtype, const void* src, int M, int K, void* dst, int mtiles, hipStream_t st) {
  const int64_t total = (int64_t)M * K;
  dim3 grid((unsigned)((total + 255) / 256));
  if (dtype == DT_BF16)
    hipLaunchKernelGGL(tile_rows_kernel<bf16_t>, grid, dim3(256), 0, st, (const bf16_t*)src, M, K, (bf16_t*)dst, mtiles);
  else
    hipLaunchKernelGGL(tile_rows_kernel<float>, grid, dim3(256), 0, st, (const float*)src, M, K, (float*)dst, mtiles);
}

void launch_stage_operands(int dtype, const void* x, int M, int K, void* xd, int mtiles, const void* w, int N, void* wd,
                           hipStream_t st) {
  if (((uintptr_t)x | (uintptr_t)w) & 15) {  // the caller's matrices may start anywhere; their rows are whole pieces
    launch_tile_rows(dtype, x, M, K, xd, mtiles, st);
    launch_repack(dtype, PACK_NATURAL, w, nullptr, nullptr, K, N, wd, 1, 64, st);
    return;
  }
  const int VEC = dtype == DT_BF16 ? 8 : 4, kblocks = K / (4 * VEC);
  const int nw = N / 64 * ((kblocks + STAGE_KB - 1) / STAGE_KB);
  const int nx = (int)(((int64_t)M * (K / VEC) + 255) / 256);
  if (dtype == DT_BF16)
    hipLaunchKernelGGL(stage_operands_kernel<bf16_t>, dim3(nw + nx), dim3(256), 0, st, (const bf16_t*)x, M, K,
                       (bf16_t*)xd, mtiles, (const bf16_t*)w, N, (bf16_t*)wd, nw);
  else
    hipLaunchKernelGGL(stage_operands_kernel<float>, dim3(nw + nx), dim3(256), 0, st, (const float*)x, M, K, (float*)xd,
                       mtiles, (const float*)w, N, (float*)wd, nw);
}

StreamPlan gemm_stream_plan(int M, int nbc, int splits, int x_mtiles) {
  // runs per slice: GEMM_WGS / splits, at least ceil(nbc / CB_MAX), at most
  // one per column block
  StreamPlan p{};
  p.runs = std::min(std::max((GEMM_WGS + splits - 1) / splits, (nbc + CB_MAX - 1) / CB_MAX), nbc);
  p.run = (nbc + p.runs - 1) / p.runs;
  // Rows per workgroup: every output element's arithmetic is the same for
  // any tile (the waves split the reduction, not the rows), so the choice only
  // trades weight re-reads against activation traffic.  Above 64 rows a
  // 128-row tile halves the weight re-reads when the buffer holds whole tiles.
  p.row_tiles = M <= 16 ? 1 : (M <= 32 ? 2 : 4);
  if (M > 64 && p.run <= CB_MAX_MB8 && (M + 127) / 128 * 8 <= x_mtiles) {
    p.row_tiles = 8;
    // A 128-row workgroup holds one CU on its own.  When runs of up to
    // CB_MAX_MB8 blocks let the whole launch (row blocks x runs x splits) fit
    // one workgroup per CU, deal the columns that way: a single round beats
    // two rounds of shorter runs, each re-reading the activation tiles.
    const int gx = (M + 127) / 128;
    const int fewer = std::max((nbc + CB_MAX_MB8 - 1) / CB_MAX_MB8, GEMM_WGS / (gx * splits));
    if (fewer < p.runs && gx * fewer * splits <= GEMM_WGS) {
      p.runs = fewer;
      p.run = (nbc + fewer - 1) / fewer;
    }
  }
  p.long_runs = nbc - p.runs * (p.run - 1);
  p.row_blocks = (M + 16 * p.row_tiles - 1) / (16 * p.row_tiles);
  p.mapped = p.row_blocks > 1 && p.runs * splits % GEMM_XCDS == 0;
  return p;
}

int gemm_pick_splits(int n_cols, int K, int dtype) {
  // Wide matrices have enough column blocks to fill the GPU on their own;
  // narrow ones split the reduction so that >= 256 workgroups stream weights.
  const int KB = dtype == DT_BF16 ? 32 : 16;
  const int kblocks = K / KB;
  if (n_cols >= SPLIT_MIN_COLS_NO) return 1;
  const int groups = n_cols / 64;
  int s = 1;
  while (groups * s < SPLIT_TARGET_WGS && s < GEMM_MAX_SPLITS && kblocks % (2 * s) == 0 && kblocks / (2 * s) >= 16) s *= 2;
  return s;
}

int gemm_partials(int dtype, int M, int n_cols, int K, int x_mtiles, int kind) {
  const int splits = gemm_pick_splits(n_cols, K, dtype), nbc = n_cols / 16;
  if (kind != EPI_PARTIAL && (splits == 1 || gemm_rows_takes(dtype, M, nbc, K, splits, kind))) return 0;
  if (gemm_wide_takes(dtype, M, nbc, K, splits, x_mtiles)) {
    if (kind != EPI_PARTIAL && gemm_wide_sums_slices(M, nbc, kind)) return 0;
    if (gemm_wide_sums_slices(M, nbc, EPI_PARTIAL)) return 1;
  }
  return splits;
}

int64_t gemm_partial_rows(int dtype, int max_M, int n_cols, int K, int kind) {
  // A buffer of over 4 GiB keeps all its launches on the streaming kernel;
  // below that the route of more than 16 rows depends on whole 64-row blocks
  // alone, so the last row of each block stands for it.
  const int mtiles = (max_M + 127) / 128 * 8;
  int64_t most = 0;
  for (int M = std::min(64, max_M); M > 0; M = M == max_M ? 0 : std::min(M + 64, max_M)) {
    const bool huge = !gemm_wide_fits(K, mtiles);
    const int parts = huge ? gemm_pick_splits(n_cols, K, dtype) : gemm_partials(dtype, M, n_cols, K, mtiles, kind);
    most = std::max(most, (int64_t)parts * M);
  }
  return most;
}

bool launch_gemm(int dtype, const GemmShape& s, const GemmEpi& e, hipStream_t st, hipEvent_t ev_start,
                 hipEvent_t ev_stop) {
  if (s.M <= 0) return true;
  if (gemm_rows_takes(dtype, s.M, gemm_blocks(s), s.K, s.splits, e.kind)) {
    launch_gemm_rows(dtype, s, e, st, ev_start, ev_stop);
    return true;
  }
  switch (e.kind) {
    case EPI_F32: case EPI_SILU: case EPI_SWIGLU: case EPI_QKV: case EPI_PARTIAL: break;
    default: return false;  // EPI_ZIN is for launches of a few rows
  }
  if (gemm_wide_takes(dtype, s.M, gemm_blocks(s), s.K, s.splits, s.x_mtiles)) {
    const bool finish = s.splits > 1 && e.kind != EPI_PARTIAL && !gemm_wide_sums_slices(s.M, gemm_blocks(s), e.kind);
    if (finish) {
      GemmEpi p = e;
      p.kind = EPI_PARTIAL;
      launch_gemm_wide(s, p, st, ev_start, nullptr);
      GemmShape f = s;
      if (gemm_wide_sums_slices(s.M, gemm_blocks(s), EPI_PARTIAL)) f.splits = 1;  // one summed partial was written
      launch_finish<bf16_t>(f, e, st, ev_stop);
    } else {
      launch_gemm_wide(s, e, st, ev_start, ev_stop);
    }
    return true;
  }
  if (dtype == DT_BF16)
    gemm_t<bf16_t>(s, e, st, ev_start, ev_stop);
  else
    gemm_t<float>(s, e, st, ev_start, ev_stop);
  return true;
}

void launch_repack(int dtype, int kind, const void* src0, const void* src1, const void* src2, int K, int n_src,
                   void* dst, int H, int hd, hipStream_t st) {
  const int n_packed = kind == PACK_QKV ? 3 * n_src : (kind == PACK_GU ? 2 * n_src : n_src);
  const int nblocks = n_packed / 16;
  const int KB = dtype == DT_BF16 ? 32 : 16;
  const int64_t total = (int64_t)nblocks * (K / KB) * 64;
  dim3 grid((unsigned)((total + 255) / 256));
  if (dtype == DT_BF16)
    hipLaunchKernelGGL(repack_kernel<bf16_t>, grid, dim3(256), 0, st, (const bf16_t*)src0, (const bf16_t*)src1,
                       (const bf16_t*)src2, K, n_src, kind, H, hd, (bf16_t*)dst, nblocks);
  else
    hipLaunchKernelGGL(repack_kernel<float>, grid, dim3(256), 0, st, (const float*)src0, (const float*)src1,
                       (const float*)src2, K, n_src, kind, H, hd, (float*)dst, nblocks);
}
