// Row sums of the sparse matrix (gfx950): the sliced ELLPACK copy, one row per
// lane, and the row-tiled CSR arrays, products staged in LDS.
#pragma once

#include "device.hpp"

namespace gir {

// ---------------------------------------------------------------------------
// source-vector accessors of the SpMV gather
// ---------------------------------------------------------------------------

// v = round_to_basis(src * inv): the next basis vector built from the
// unnormalised vector of the previous iteration.
template <typename T, typename S>
struct XScaled {
  const T* src;
  T inv;
  __device__ __forceinline__ T operator()(int c) const { return Basis<S, T>::round(src[c] * inv); }
};

template <typename T>
struct XPlain {
  const T* src;
  __device__ __forceinline__ T operator()(int c) const { return src[c]; }
};

// prod[i] = vals[p0 + i] * x(col[p0 + i]) for i < len (a tile staged in LDS).
// The loads of SPMV_UNROLL nonzeros per thread are issued before their
// gathers, and the gathers before the products, so a tile costs two memory
// round trips per batch instead of one per nonzero.  Each product is rounded
// on its own (no fused multiply-add with the row sum).
template <typename T, typename XF>
__device__ __forceinline__ void stage_products(const Csr& A, int p0, int len, const XF& xf, T* prod) {
  const T* vals = (const T*)A.vals;
  for (int i0 = 0; i0 < len; i0 += BLOCK * SPMV_UNROLL) {
    int cc[SPMV_UNROLL];
    T vv[SPMV_UNROLL], xv[SPMV_UNROLL];
#pragma unroll
    for (int k = 0; k < SPMV_UNROLL; ++k) {
      const int i = i0 + (int)threadIdx.x + k * BLOCK;
      const int ic = i < len ? i : len - 1;
      cc[k] = A.col[p0 + ic];
      vv[k] = vals[p0 + ic];
    }
#pragma unroll
    for (int k = 0; k < SPMV_UNROLL; ++k) xv[k] = xf(cc[k]);
#pragma unroll
    for (int k = 0; k < SPMV_UNROLL; ++k) {
      const int i = i0 + (int)threadIdx.x + k * BLOCK;
      if (i < len) prod[i] = vv[k] * xv[k];
    }
  }
}

// One row of the sliced ELLPACK copy, summed in column order by the lane that
// owns it (the same order, and so the same bits, as the tiled CSR kernels).
// Loads of U entries are issued before their gathers; padding entries past
// the row length are loaded (valid addresses) but not added.
// LAYOUT 1: 32-bit columns; 2: 16-bit offsets from the row (rows past n: from
// row 0); 3: the slice's shared offsets (a wave-uniform load), every slot
// added -- an absent entry adds 0 * x[c] = +-0 to a sum that started at +0,
// which leaves it unchanged (x finite), so the bits match the CSR row sum --
// and the gathered index clamped to [0, n) (absent neighbours, rows past n).
template <typename T, int LAYOUT, int U, typename XF>
__device__ __forceinline__ T sell_row_cols(const Csr& A, const XF& xf, int s, int r, int lane, int base, int K) {
#pragma clang fp contract(off)
  const T* vals = (const T*)A.svals;
  const int len = LAYOUT == 3 ? K : (r < A.n ? A.rowptr[r + 1] - A.rowptr[r] : 0);
  const int rr = r < A.n ? r : 0;
  const int* soff = A.scol + base / SELL_C;
  T sum = T(0);
  for (int k0 = 0; k0 < K; k0 += U) {
    int cc[U];
    T vv[U], xv[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int k = k0 + u < K ? k0 + u : K - 1;
      if constexpr (LAYOUT == 3) cc[u] = min(max(r + soff[k], 0), A.n - 1);
      else if constexpr (LAYOUT == 2) cc[u] = rr + (int)A.scol16[base + SELL_C * k + lane];
      else cc[u] = A.scol[base + SELL_C * k + lane];
      vv[u] = vals[base + SELL_C * k + lane];
    }
#pragma unroll
    for (int u = 0; u < U; ++u) xv[u] = xf(cc[u]);
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const T p = vv[u] * xv[u];
      if (k0 + u < len) sum = sum + p;
    }
  }
  return sum;
}

// The entries whose loads go out together follow the slice's width K (a
// wave-uniform value): rounds of U in {5, 7, 9} entries, the U that loads the
// fewest padded entries (ceil(K / U) U), the larger U on ties -- a 27-point
// row in three rounds of 9, a 13-point one in two of 7, a 19-point one in
// four of 5 (measured: 27-point 128^3 SpMV + projection 124 -> 119 us with 9
// instead of 5; rounds of 9 on 5-, 13- and 19-entry rows, which load 4, 5
// and 8 entries for nothing, ran 5-15 % slower).
__device__ __forceinline__ int sell_round(int K) {
  const int l5 = (K + 4) / 5 * 5, l7 = (K + 6) / 7 * 7, l9 = (K + 8) / 9 * 9;
  return (l9 <= l7 && l9 <= l5) ? 9 : (l7 <= l5 ? 7 : 5);
}

template <typename T, int LAYOUT, bool WIDE, typename XF>
__device__ __forceinline__ T sell_row_k(const Csr& A, const XF& xf, int s, int r, int lane) {
  const int base = A.sptr[s];
  const int K = (A.sptr[s + 1] - base) / SELL_C;
  // WIDE (shared offsets, slices wider than 9): no index registers per entry,
  // so a slice 10..27 wide issues all its loads in one round (27-point 128^3
  // SpMV + projection 94 -> 93 us fp32, 76 -> 69 us with a bf16 basis, against
  // rounds of 9; 19-point fp64 SpMV 77 -> 73 us).  A template choice: the
  // wide rounds' registers would cost the narrow stencils occupancy (7-point
  // 150^3 one-reduction SpMV 184 -> 221 us when compiled in).
  if constexpr (LAYOUT == 3 && WIDE) {
    if (K > 9 && K <= 14) return sell_row_cols<T, LAYOUT, 14>(A, xf, s, r, lane, base, K);
    if (K > 14 && K <= 19) return sell_row_cols<T, LAYOUT, 19>(A, xf, s, r, lane, base, K);
    if (K > 19 && K <= 27) return sell_row_cols<T, LAYOUT, 27>(A, xf, s, r, lane, base, K);
  }
  const int U = sell_round(K);
  if (U == 5) return sell_row_cols<T, LAYOUT, 5>(A, xf, s, r, lane, base, K);
  if (U == 7) return sell_row_cols<T, LAYOUT, 7>(A, xf, s, r, lane, base, K);
  return sell_row_cols<T, LAYOUT, 9>(A, xf, s, r, lane, base, K);
}

// The layout and the round size are chosen once per slice (wave-uniform
// branches), not per load: a load under a branch is waited for at the
// branch's end.
template <typename T, bool WIDE = false, typename XF>
__device__ __forceinline__ T sell_row(const Csr& A, const XF& xf, int s, int r, int lane) {
  if (A.shared) return sell_row_k<T, 3, WIDE>(A, xf, s, r, lane);
  return A.d16 ? sell_row_k<T, 2, false>(A, xf, s, r, lane) : sell_row_k<T, 1, false>(A, xf, s, r, lane);
}

// SpMV over the sliced ELLPACK copy: the block takes a contiguous range of
// slices, its waves take every fourth of them, each lane one row; epi(r, y)
// per row as in spmv_tiles.
template <typename T, bool WIDE = false, typename XF, typename EPI>
__device__ __forceinline__ void sell_rows(const Csr& A, const XF& xf, EPI& epi) {
  const int lane = threadIdx.x & (WAVE - 1);
  const int wid = __builtin_amdgcn_readfirstlane(threadIdx.x / WAVE);
  const int B = gridDim.x, lb = logical_block();
  const int s0 = (int)((long)A.nslices * lb / B);
  const int s1 = (int)((long)A.nslices * (lb + 1) / B);
  for (int s = s0 + wid; s < s1; s += NWAVES) {
    const int r = s * SELL_C + lane;
    const T y = sell_row<T, WIDE>(A, xf, s, r, lane);
    if (r < A.n) epi(r, y);
  }
}

// Row-tiled CSR SpMV: a block takes a contiguous range of tiles; per tile the
// nonzeros are streamed with coalesced loads, multiplied by the gathered x and
// staged in LDS, then each thread sums one row in column order.  epi(r, y) is
// called once per row by the thread owning it.
template <typename T, typename XF, typename EPI>
__device__ __forceinline__ void spmv_tiles(const Csr& A, const XF& xf, EPI& epi, T* prod, T* red) {
  const T* vals = (const T*)A.vals;
  const int B = gridDim.x, lb = logical_block();
  const int t0 = (int)((long)A.ntiles * lb / B);
  const int t1 = (int)((long)A.ntiles * (lb + 1) / B);
  for (int t = t0; t < t1; ++t) {
    const int r0 = A.tile_row[t], r1 = A.tile_row[t + 1];
    const int p0 = A.rowptr[r0], p1 = A.rowptr[r1];
    const int len = p1 - p0;
    if (len <= TILE_NNZ) {
      stage_products<T>(A, p0, len, xf, prod);
      __syncthreads();
      for (int rr = threadIdx.x; rr < r1 - r0; rr += BLOCK) {
        const int r = r0 + rr;
        const int q0 = A.rowptr[r] - p0, q1 = A.rowptr[r + 1] - p0;
        T s = T(0);
        for (int q = q0; q < q1; ++q) s += prod[q];
        epi(r, s);
      }
      __syncthreads();
    } else {
      // a single row longer than a tile: block-wide dot product
      T s = T(0);
      for (int i = threadIdx.x; i < len; i += BLOCK) s += vals[p0 + i] * xf(A.col[p0 + i]);
      s = block_sum(s, red);
      if (threadIdx.x == 0) epi(r0, s);
      __syncthreads();
    }
  }
}

}  // namespace gir
