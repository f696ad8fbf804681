// Split-K GEMMs of a few rows in one launch (M <= 16: the draft's trigram
// encoder, down projection and head MLPs).  The streaming kernel runs one
// workgroup per reduction slice and leaves the slices to a finishing launch:
// with a few rows a pass over some hundred KiB that costs as much as a fifth of
// the product (3.8 us next to 15-20 us at 7B width).  Where the consumer adds the slices
// anyway (the norms after O and down) it stays the faster one, 11.7 us against
// 13.1 a launch in greedy decoding at 7B width.
//
// Here a workgroup owns one 16-column block and the whole reduction: four
// waves per slice (up to four slices side by side, 16 waves), each summing the
// k-blocks of one residue class, then the classes in class order and the
// slices in slice order -- the streaming kernel's sums, bit for bit -- and the
// epilogue on the result.  The activations are staged in LDS, only the rows
// there are: fetched as whole 16-row fragments they would double the bytes
// that enter a CU.  Bound by the weight stream.
#include <hip/hip_ext.h>

#include "common.h"
#include "gemm_epilogue.h"
#include "kernels.h"

namespace {

constexpr int MAX_LDS_X = 126 << 10;  // activation rows staged, bytes (33 KiB more hold the sums)
constexpr int SIDE = 4;               // slices side by side

template <typename T, int KIND, int WAVES>
__global__ __launch_bounds__(64 * WAVES) void gemm_rows_kernel(const GemmShape sh, const GemmEpi e) {
  constexpr int VEC = ET<T>::VEC, PF = 4;
  if (sh.skip && *sh.skip == 0) return;
  extern __shared__ __attribute__((aligned(16))) char xs[];  // [K / VEC][M] 16-byte pieces
  __shared__ f32x4 red[GEMM_MAX_SPLITS * 4 * 64];
  __shared__ __attribute__((aligned(16))) float stage[256];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int g = lane >> 4, r = lane & 15;
  const int kblocks = sh.K / (4 * VEC), kps = kblocks / sh.splits, M = sh.M;
  const int blk = sh.nb_off + blockIdx.x;
  const char* W = (const char*)sh.W + ((int64_t)(blk / NB) * kblocks * NB + blk % NB) * 1024 + lane * 16;
  const int cls = wave & 3;
  const int n = (kps - cls + 3) / 4;  // k-blocks of this wave in each of its slices
  const bool have = r < M;
  int4 w[PF];
  auto load = [&](int slot, int slice, int i) {
    typedef int i32x4 __attribute__((ext_vector_type(4)));
    const i32x4 v = __builtin_nontemporal_load(
        reinterpret_cast<const i32x4*>(W + (int64_t)(slice * kps + cls + 4 * i) * NB * 1024));
    w[slot] = int4{v.x, v.y, v.z, v.w};
  };
  int slice = wave / 4;
#pragma unroll
  for (int p = 0; p < PF; ++p)
    if (p < n) load(p, slice, p);
  // the rows: piece (kb, g, r) of the tiled activations goes to (4 kb + g) M + r
  for (int i = tid; i < kblocks * 4 * M; i += 64 * WAVES) {
    const int q = i / M, row = i % M;
    st16(xs + (int64_t)i * 16, ld16((const char*)sh.X + ((int64_t)(q >> 2) * sh.x_mtiles * 64 + (q & 3) * 16 + row) * 16));
  }
  __syncthreads();
  for (; slice < sh.splits; slice += WAVES / 4) {
    if (slice >= WAVES / 4) {
#pragma unroll
      for (int p = 0; p < PF; ++p)
        if (p < n) load(p, slice, p);
    }
    f32x4 acc = f32x4{0.f, 0.f, 0.f, 0.f};
    const char* x = xs + ((int64_t)(4 * (slice * kps + cls) + g) * M + r) * 16;
    const int64_t xstep = (int64_t)16 * M * 16;
    for (int i = 0; i < n; i += PF) {
#pragma unroll
      for (int p = 0; p < PF; ++p) {
        if (i + p < n) {  // wave-uniform
          int4 xv = int4{0, 0, 0, 0};
          if (have) xv = ld16(x + (i + p) * xstep);
          acc = mfma_kb<T>(xv, w[p], acc);
          if (i + p + PF < n) load(p, slice, i + p + PF);
        }
      }
    }
    red[(slice * 4 + cls) * 64 + lane] = acc;
  }
  __syncthreads();
  if (wave != 0) return;
  f32x4 v;
  for (int s = 0; s < sh.splits; ++s) {
    f32x4 t = red[(s * 4) * 64 + lane];
#pragma unroll
    for (int c = 1; c < 4; ++c) t = t + red[(s * 4 + c) * 64 + lane];
    v = s == 0 ? t : v + t;
  }
  store_tile<T, KIND>(sh, e, 0, blk, v, e.part, stage, nullptr, f32x4{}, f32x4{}, lane);
}

template <typename T, int KIND, int WAVES>
void go(const GemmShape& s, const GemmEpi& e, hipStream_t st, hipEvent_t ea, hipEvent_t eb) {
  const dim3 grid(s.nb_count ? s.nb_count : s.N / 16), wg(64 * WAVES);
  const size_t lds = (size_t)s.K * s.M * sizeof(T);
  if (ea || eb)
    hipExtLaunchKernelGGL((gemm_rows_kernel<T, KIND, WAVES>), grid, wg, lds, st, ea, eb, 0, s, e);
  else
    hipLaunchKernelGGL((gemm_rows_kernel<T, KIND, WAVES>), grid, wg, lds, st, s, e);
}

template <typename T, int KIND>
void go_waves(const GemmShape& s, const GemmEpi& e, hipStream_t st, hipEvent_t ea, hipEvent_t eb) {
  if (s.splits >= SIDE)
    go<T, KIND, 4 * SIDE>(s, e, st, ea, eb);
  else
    go<T, KIND, 8>(s, e, st, ea, eb);
}

template <typename T>
void go_kind(const GemmShape& s, const GemmEpi& e, hipStream_t st, hipEvent_t ea, hipEvent_t eb) {
  switch (e.kind) {
    case EPI_F32: go_waves<T, EPI_F32>(s, e, st, ea, eb); break;
    case EPI_ZIN: go_waves<T, EPI_ZIN>(s, e, st, ea, eb); break;
    default: go_waves<T, EPI_SILU>(s, e, st, ea, eb); break;
  }
}

}  // namespace

bool gemm_rows_takes(int dtype, int M, int nbc, int K, int splits, int kind) {
  if (splits <= 1 || splits > GEMM_MAX_SPLITS || M > 16) return false;
  if (kind != EPI_F32 && kind != EPI_SILU && kind != EPI_ZIN) return false;
  const int es = dtype == DT_BF16 ? 2 : 4;
  const int64_t rows = (int64_t)M * K * es, weights = (int64_t)16 * K * es;
  if (rows > MAX_LDS_X) return false;
  if (nbc <= 256) {
    // One round.  With most CUs busy the weights stream at the card's rate
    // either way (256 blocks, K = 4096 bf16, one row: 9.0 us against 10.2 with
    // the slices side by side and the finishing launch).  With fewer blocks one
    // CU takes in what `splits` of them would: worth the launch saved (1.5 to 4
    // us, more the more columns it has) while a block is short.  Against the
    // split launches, us, one row, bf16: 64 columns K = 2048 3.4 / 4.2, K = 4096
    // 6.3 / 4.6, K = 32768 24 / 8.4; 2560 columns K = 3072 6.0 / 7.4, K = 6144
    // 10.9 / 9.9; fp32 (four MFMAs a k-block): 512 columns K = 1024 4.4 / 5.0,
    // K = 2048 7.9 / 5.3.
    return nbc >= 224 || weights + rows / 2 <= (dtype == DT_BF16 ? 104 << 10 : 80 << 10) + 64 * es * nbc;
  }
  // More rounds: the last may not be mostly empty (320 blocks of K = 15360: 33
  // us against 28 + 4), and two workgroups have to fit a CU's LDS for one round
  // to start under the other (480 blocks, 16 rows of bf16: K = 1280 7.3 / 8.6
  // us, K = 1536 10.4 / 9.2).
  const int rounds = (nbc + 255) / 256;
  return 10 * (rounds * 256 - nbc) <= nbc && rows <= 46 << 10;
}

void launch_gemm_rows(int dtype, const GemmShape& s, const GemmEpi& e, hipStream_t st, hipEvent_t ea, hipEvent_t eb) {
  if (dtype == DT_BF16)
    go_kind<bf16_t>(s, e, st, ea, eb);
  else
    go_kind<float>(s, e, st, ea, eb);
}
