// Page-resolved rows of the tree attention's window, shared by the kernels
// that start a pass.
#pragma once
#include "kernels.h"

// Entry k < W is position n - W + k (committed), entry W + j the slot of tree
// node j (position n + j) of `count`; entries before position 0 or past the
// tree are zero.  All threads of the workgroup.
__device__ __forceinline__ void window_rows(const int* __restrict__ ptab, int n, int count, int ps, int64_t page_stride,
                                            int hd, int64_t* __restrict__ rowtab) {
  constexpr int W = TREE_ATTN_WINDOW;
  for (int rr = threadIdx.x; rr < TREE_ATTN_TAIL_ROWS; rr += blockDim.x) {
    const int p = rr < W ? n - W + rr : n + rr - W;
    int64_t off = 0;
    if (p >= 0 && (rr < W || rr - W < count)) off = (int64_t)ptab[p / ps] * page_stride + (int64_t)(p % ps) * hd;
    rowtab[rr] = off;
  }
}
