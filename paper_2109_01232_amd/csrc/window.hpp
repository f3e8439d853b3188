// The part of x a block's SpMV reads, as a window in LDS (shared-offset rows).
#pragma once

#include "spmv.hpp"

namespace gir {

// The rows of x a block's SpMV reads, in LDS: the set of 64-row chunks its
// slices' offsets reach, in ascending order, so that neighbouring chunks lie
// side by side and entry (slice, k) of lane l is at off[pair] + l.  Chunks
// outside the matrix are zeros (their values are zeros too).  Every row is
// then loaded once a block and iteration, all loads in flight together,
// instead of once per entry in dependent rounds (27-point rows: three rounds
// of nine).
constexpr int WIN_BITS = 8192;  // chunks between the first and the last

// CHUNKS, PAIRS, SLICES: capacity of the block's chunks, (slice, offset) pairs, slices
template <int CHUNKS_, int PAIRS_, int SLICES_>
struct WindowMap {
  static constexpr int CHUNKS = CHUNKS_, PAIRS = PAIRS_, SLICES = SLICES_;
  int off[PAIRS];  // more pairs: in a larger place of the caller's
  int chunk[CHUNKS];
  unsigned int bits[WIN_BITS / 32];
  int before[WIN_BITS / 32];  // set bits of the words before
  int pair[SLICES + 1];       // first pair of each slice
  int first;                  // chunk of bit 0
  int chunks;                 // 0: the block does not fit, the rows are gathered one by one
  int own;                    // place of the block's own first chunk
  __device__ __forceinline__ bool wide() const { return pair[SLICES] > PAIRS; }
};

// Built once per cycle by the whole block of NT threads (all call it) for
// slices s0 .. s0 + ns - 1, in at most `most` chunks; layout with shared offsets.
// more: place of `room` > PAIRS pairs' entries, used where PAIRS are too few.
template <int NT, typename W_>
__device__ __forceinline__ void window_build(W_& W, const Csr& A, int s0, int ns, int most, int* more = nullptr,
                                             int room = W_::PAIRS) {
  const int lane = threadIdx.x & (WAVE - 1), wid = threadIdx.x / WAVE;  // a wave takes a slice, a lane an offset
  for (int i = threadIdx.x; i < WIN_BITS / 32; i += NT) W.bits[i] = 0;
  for (int s = threadIdx.x; s <= W_::SLICES; s += NT) W.pair[s] = (A.sptr[s0 + min(s, ns)] - A.sptr[s0]) / SELL_C;
  if (threadIdx.x == 0) {
    W.first = s0;
    W.chunks = A.shared && (A.sptr[s0 + ns] - A.sptr[s0]) / SELL_C <= room;
  }
  __syncthreads();
  if (!W.chunks) return;
  // offset of pair p of slice s
  auto offset = [&](int s, int p) { return A.scol[A.sptr[s0 + s] / SELL_C + p - W.pair[s]]; };
  for (int s = threadIdx.x; s < ns; s += NT)
    if (W.pair[s + 1] > W.pair[s]) atomicMin(&W.first, s0 + s + (offset(s, W.pair[s]) >> 6));  // ascending offsets
  __syncthreads();
  bool fits = true;
  auto mark = [&](int c) {
    const int b = c - W.first;
    if (b < WIN_BITS) atomicOr(&W.bits[b >> 5], 1u << (b & 31));
    else fits = false;
  };
  for (int s = wid; s < ns; s += NT / WAVE) {
    if (lane == 0) mark(s0 + s);
    for (int p = W.pair[s] + lane; p < W.pair[s + 1]; p += WAVE) {
      const int o = offset(s, p), c = s0 + s + (o >> 6);
      mark(c);
      if (o & 63) mark(c + 1);
    }
  }
  fits = __syncthreads_and(fits);
  if (threadIdx.x < WAVE) {
    constexpr int PER = WIN_BITS / 32 / WAVE;
    int cnt[PER], sum = 0;
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      cnt[i] = sum;
      sum += __popc(W.bits[threadIdx.x * PER + i]);
    }
    int incl = sum;
    for (int o = 1; o < WAVE; o *= 2) {
      const int y = __shfl_up(incl, o, WAVE);
      if ((int)threadIdx.x >= o) incl += y;
    }
#pragma unroll
    for (int i = 0; i < PER; ++i) W.before[threadIdx.x * PER + i] = incl - sum + cnt[i];
    if (threadIdx.x == WAVE - 1) W.chunks = fits && incl <= min(most, W_::CHUNKS) ? incl : 0;
  }
  __syncthreads();
  if (!W.chunks) return;
  auto place = [&](int c) {
    const int b = c - W.first;
    return W.before[b >> 5] + __popc(W.bits[b >> 5] & ((1u << (b & 31)) - 1));
  };
  for (int i = threadIdx.x; i < WIN_BITS / 32; i += NT)
    for (unsigned int m = W.bits[i], k = 0; m; m &= m - 1, ++k) W.chunk[W.before[i] + k] = W.first + 32 * i + __ffs(m) - 1;
  int* const off = W.wide() ? more : W.off;
  for (int s = wid; s < ns; s += NT / WAVE)
    for (int p = W.pair[s] + lane; p < W.pair[s + 1]; p += WAVE) {
      const int o = offset(s, p);
      off[p] = place(s0 + s + (o >> 6)) * SELL_C + (o & 63);
    }
  if (threadIdx.x == 0) W.own = place(s0);
  __syncthreads();
}

// Row sums of slice s from the window, in the order of sell_row; vals: the
// slice's values (LDS or memory), 64 per entry; U entries' loads go out together.
template <typename T, int U = 9, typename W_>
__device__ __forceinline__ T window_row(const W_& W, const int* off, const T* x, const T* vals, int s, int lane) {
#pragma clang fp contract(off)
  const int p0 = W.pair[s], K = W.pair[s + 1] - p0;
  T sum = T(0);
  for (int k0 = 0; k0 < K; k0 += U) {
    T vv[U], xv[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int k = k0 + u < K ? k0 + u : K - 1;
      vv[u] = vals[SELL_C * k + lane];
      xv[u] = x[off[p0 + k] + lane];
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const T p = vv[u] * xv[u];
      if (k0 + u < K) sum = sum + p;
    }
  }
  return sum;
}
template <typename T, int U = 9, typename W_>
__device__ __forceinline__ T window_row(const W_& W, const T* x, const T* vals, int s, int lane) {
  return window_row<T, U>(W, W.off, x, vals, s, lane);
}

}  // namespace gir
