// Output stage shared by the GEMM kernels: what one 16x16 output tile (or one
// element of it) becomes under each epilogue.
#pragma once
#include "common.h"
#include "kernels.h"

namespace {

constexpr int NB = 4;  // 16-column blocks per weight-layout group

// Four floats of a row-major output, which may be a caller's and start at any
// float: still one 16-byte store (global stores take 4-byte alignment).
typedef float f32x4_any __attribute__((ext_vector_type(4), aligned(4)));

// ---------------------------------------------------------------------------
// Epilogue of one output element: v is packed column 16 blk + c16 of `row`,
// vp the same row's value at lane column c16 ^ 8 (the other half of a rotary
// or gate/up pair).
// ---------------------------------------------------------------------------
template <typename T>
__device__ __forceinline__ void epi_elem(const GemmEpi& e, int kind, int N, int M, int split, int row, int blk,
                                         int c16, float v, float vp) {
  const int col = 16 * blk + c16;
  if (kind == EPI_PARTIAL) {
    e.part[((int64_t)split * M + row) * N + col] = v;
  } else if (kind == EPI_F32) {
    e.out_f[(int64_t)row * e.ldo + col] = v;
  } else if (kind == EPI_SILU) {
    store_tiled<T>((T*)e.out_t, e.o_mtiles, row, col, silu_f(v));
  } else if (kind == EPI_SWIGLU) {
    if (c16 < 8) store_tiled<T>((T*)e.out_t, e.o_mtiles, row, 8 * blk + c16, silu_f(v) * vp);
  } else if (kind == EPI_QKV) {
    const int hd = e.hd;
    const int blk_head = hd / 16;
    const int sec_blks = e.H * blk_head;
    const int sec = blk / sec_blks, rem = blk % sec_blks;
    const int h = rem / blk_head, q = rem % blk_head;
    if (sec < 2) {
      const bool first = c16 < 8;
      const int i = 8 * q + (c16 & 7);
      const int pos = e.pos[row];
      const float c = e.rcos[(int64_t)pos * (hd / 2) + i];
      const float s = e.rsin[(int64_t)pos * (hd / 2) + i];
      // first half: x1 cos - x2 sin; second half: x2 cos + x1 sin
      const float o = first ? v * c - vp * s : v * c + vp * s;
      const int dim = first ? i : i + hd / 2;
      if (sec == 0) {
        const int qr = e.qrow[row];
        if (qr >= 0) ((T*)e.qout)[(int64_t)qr * e.ldq + h * hd + dim] = ET<T>::from_f(o);
      } else {
        const int64_t off = e.kvoff[row];
        if (off >= 0) ((T*)e.kbase)[off + h * e.head_stride + dim] = ET<T>::from_f(o);
      }
    } else {
      const int64_t off = e.kvoff[row];
      if (off >= 0) ((T*)e.vbase)[off + h * e.head_stride + 16 * q + c16] = ET<T>::from_f(v);
    }
  }
}

// Per-row targets of the QKV epilogue, staged in LDS before the k-loop.
struct RowMeta {
  int64_t kvoff;  // K/V element offset (-1: skip)
  int pos;        // rotary position
  int qrow;       // Q output row (-1: skip)
};

// QKV epilogue of one element with its rotary cos/sin already loaded (the
// same arithmetic as epi_elem's EPI_QKV branch).
template <typename T>
__device__ __forceinline__ void qkv_store(const GemmEpi& e, const RowMeta& rm, int blk, int c16, float v, float vp,
                                          float c, float s) {
  const int hd = e.hd;
  const int blk_head = hd / 16;
  const int sec_blks = e.H * blk_head;
  const int sec = blk / sec_blks, rem = blk % sec_blks;
  const int h = rem / blk_head, q = rem % blk_head;
  if (sec < 2) {
    const bool first = c16 < 8;
    const int i = 8 * q + (c16 & 7);
    const float o = first ? v * c - vp * s : v * c + vp * s;
    const int dim = first ? i : i + hd / 2;
    if (sec == 0) {
      if (rm.qrow >= 0) ((T*)e.qout)[(int64_t)rm.qrow * e.ldq + h * hd + dim] = ET<T>::from_f(o);
    } else if (rm.kvoff >= 0) {
      ((T*)e.kbase)[rm.kvoff + h * e.head_stride + dim] = ET<T>::from_f(o);
    }
  } else if (rm.kvoff >= 0) {
    ((T*)e.vbase)[rm.kvoff + h * e.head_stride + 16 * q + c16] = ET<T>::from_f(v);
  }
}

// The same element's value before the store: rotated Q/K or plain V.
__device__ __forceinline__ float qkv_value(const GemmEpi& e, int blk, int c16, float v, float vp, float c, float s) {
  const int sec = blk / (e.H * (e.hd / 16));
  if (sec == 2) return v;
  return c16 < 8 ? v * c - vp * s : v * c + vp * s;
}

// 8 consecutive outputs of one row of a QKV tile as one 16-byte store: half 0
// holds lane columns 0..7 of block blk, half 1 columns 8..15.
template <typename T>
__device__ __forceinline__ void qkv_store16(const GemmEpi& e, const RowMeta& rm, int blk, int half, int4 v) {
  const int hd = e.hd;
  const int blk_head = hd / 16;
  const int sec_blks = e.H * blk_head;
  const int sec = blk / sec_blks, rem = blk % sec_blks;
  const int h = rem / blk_head, q = rem % blk_head;
  const int dim = sec < 2 ? (half ? hd / 2 : 0) + 8 * q : 16 * q + 8 * half;
  if (sec == 0) {
    if (rm.qrow >= 0) *reinterpret_cast<int4*>((T*)e.qout + (int64_t)rm.qrow * e.ldq + h * hd + dim) = v;
  } else if (rm.kvoff >= 0) {
    T* base = (T*)(sec == 1 ? e.kbase : e.vbase);
    *reinterpret_cast<int4*>(base + rm.kvoff + h * e.head_stride + dim) = v;
  }
}

// Store one 16x16 output tile (row block mb, column block blk): v in MFMA
// layout (lane (g, c16): rows 4g .. 4g+3, column c16).  tw: 1 KiB of LDS of
// this wave.  rm: row targets of the tile's 16 rows (QKV).
template <typename T, int KIND>
__device__ __forceinline__ void store_tile(const GemmShape& sh, const GemmEpi& e, int mb, int blk, f32x4 v, float* part,
                                           float* tw, const RowMeta* rm, f32x4 cs, f32x4 sn, int lane) {
  const int g = lane >> 4, c16 = lane & 15;
  if constexpr (KIND == EPI_F32 || KIND == EPI_PARTIAL) {
    float* base = KIND == EPI_F32 ? e.out_f : part;
    const int64_t ld = KIND == EPI_F32 ? e.ldo : sh.N;
#pragma unroll
    for (int r = 0; r < 4; ++r) tw[(4 * g + r) * 16 + c16] = v[r];
    __builtin_amdgcn_wave_barrier();
    const int row = 16 * mb + (lane >> 2);
    const f32x4 o = *reinterpret_cast<const f32x4*>(tw + (lane >> 2) * 16 + 4 * (lane & 3));
    if (row < sh.M) *reinterpret_cast<f32x4_any*>(base + (int64_t)row * ld + 16 * blk + 4 * (lane & 3)) = o;
    __builtin_amdgcn_wave_barrier();
    return;
  }
  if constexpr (KIND == EPI_ZIN) {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int row = 16 * mb + 4 * g + r, col = 16 * blk + c16;
      if (row < sh.M)
        store_tiled<T>((T*)e.out_t, e.o_mtiles, row, sh.N + col, e.out_f[(int64_t)row * e.ldo + col] + v[r]);
    }
    return;
  }
  f32x4 vp;  // lane column c16 ^ 8
#pragma unroll
  for (int r = 0; r < 4; ++r) vp[r] = dpp_mov<DPP_ROR8>(v[r]);
  if constexpr (sizeof(T) == 2 && KIND == EPI_SWIGLU) {
    T* tt = reinterpret_cast<T*>(tw);
    if (c16 < 8) {
#pragma unroll
      for (int r = 0; r < 4; ++r) tt[(4 * g + r) * 8 + c16] = ET<T>::from_f(silu_f(v[r]) * vp[r]);
    }
    __builtin_amdgcn_wave_barrier();
    if (lane < 16) {
      const int row = 16 * mb + lane;
      const int4 o = *reinterpret_cast<const int4*>(tt + lane * 8);
      if (row < sh.M) *reinterpret_cast<int4*>((T*)e.out_t + tiled_index<T>(e.o_mtiles, row, 8 * blk)) = o;
    }
    __builtin_amdgcn_wave_barrier();
  } else if constexpr (KIND == EPI_QKV) {
    T* tt = reinterpret_cast<T*>(tw);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      if constexpr (sizeof(T) == 2)
        tt[(4 * g + r) * 16 + c16] = ET<T>::from_f(qkv_value(e, blk, c16, v[r], vp[r], cs[r], sn[r]));
      else if (16 * mb + 4 * g + r < sh.M)
        qkv_store<T>(e, rm[4 * g + r], blk, c16, v[r], vp[r], cs[r], sn[r]);
    }
    if constexpr (sizeof(T) == 2) {
      __builtin_amdgcn_wave_barrier();
      if (lane < 32) {
        const int4 o = *reinterpret_cast<const int4*>(tt + (lane & 15) * 16 + 8 * (lane >> 4));
        if (16 * mb + (lane & 15) < sh.M) qkv_store16<T>(e, rm[lane & 15], blk, lane >> 4, o);
      }
      __builtin_amdgcn_wave_barrier();
    }
  } else {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int row = 16 * mb + 4 * g + r;
      if (row < sh.M) epi_elem<T>(e, KIND, sh.N, sh.M, 0, row, blk, c16, v[r], vp[r]);
    }
  }
}

}  // namespace
