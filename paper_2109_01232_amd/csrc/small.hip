// Kernels of the LDS-resident inner cycle (see small.hpp).
#include <hip/hip_runtime.h>

#include <algorithm>

#include "exchange.hpp"
#include "spmv.hpp"
#include "window.hpp"

namespace gir {

namespace {

// The partial sums of one exchange: block b, wave w write their sums of the
// columns w + 7 q as one line of 16 values.  A line has one writer and is
// written by one store, so it changes hands once (words of several blocks in
// one line: 3.0 instead of 1.1 us per exchange of 16 blocks), and a reader
// that looks too early takes the line from the writer: POLL_WAIT (times 64
// clocks) after its own store it looks for the first time, about when the
// others' stores have arrived (1.8 -> 1.1 us).
constexpr int POLL_WAIT = 12;
constexpr int LINE = 16;

template <typename T>
__device__ __forceinline__ word_t* line_of(word_t* words, int P, int wid, int b) {
  return words + ((size_t)wid * P + b) * (LINE * small_words_per_value<T>());
}

// the wave's sums of acc[q], q < nq: its columns' partial sums
template <typename T, int SLOTS>
__device__ __forceinline__ void publish(word_t* words, int P, int wid, int lane, unsigned int tag, T (&acc)[SLOTS],
                                        int nq) {
  constexpr int LANES = WAVE / SLOTS;
  const T v = lane_sums<SLOTS>(acc);
  const int q = lane / LANES;
  if (lane % LANES == 0 && q < nq) put_value(line_of<T>(words, P, wid, blockIdx.x) + small_words_per_value<T>() * q, v, tag);
}

// out[q], q < nq: the sums over the P blocks, in every lane, and kept in
// all[wid + 7 q].  SLOTS lanes take a line's values side by side, 64 / SLOTS
// blocks at once; a pass has up to eight such loads in flight.
template <typename T, int SLOTS>
__device__ __forceinline__ bool collect(word_t* words, int P, int wid, int lane, unsigned int tag, T (&out)[SLOTS],
                                        T* all, int nq) {
  constexpr int WV = small_words_per_value<T>();
  constexpr int W = SLOTS, NB = WAVE / W;
  constexpr int G = 8 / WV;
  const int q = lane % W, bl = lane / W;
  const word_t* p = line_of<T>(words, P, wid, 0) + WV * q;
  T sum = T(0);
  for (int b0 = 0; b0 < P; b0 += NB * G) {
    word_t w[G][WV];
    const bool ok = poll([&] {
      bool right = true;
#pragma unroll
      for (int g = 0; g < G; ++g) {
        const int b = b0 + NB * g + bl;
        if (NB * g + b0 < P)
#pragma unroll
          for (int h = 0; h < WV; ++h) w[g][h] = get_word(p + (unsigned)((b < P ? b : P - 1) * LINE * WV + h));
      }
#pragma unroll
      for (int g = 0; g < G; ++g)
        if (NB * g + b0 < P)
#pragma unroll
          for (int h = 0; h < WV; ++h) right = right && ((unsigned int)w[g][h] == tag || q >= nq);
      return right;
    });
    if (!ok) return false;
#pragma unroll
    for (int g = 0; g < G; ++g)
      if (NB * g + b0 < P && NB * g + b0 + bl < P && q < nq) sum += word_value(w[g], T(0));
  }
  sum = lane_sum<W>(sum);
  // lane q holds the sum of value q; hand each to every lane
  if (lane < nq) all[wid + SMALL_NW * lane] = sum;
#pragma unroll
  for (int i = 0; i < SLOTS; ++i) out[i] = read_lane(sum, i);
  return true;
}

// one value a block, in a line of its own: the sum over the blocks
template <typename T>
__device__ __forceinline__ bool collect_one(const word_t* words, int P, int lane, unsigned int tag, T& out) {
  constexpr int WV = small_words_per_value<T>();
  constexpr int L = SMALL_MAX_P / WAVE;
  word_t w[L][WV];
  const bool ok = poll([&] {
    bool all = true;
#pragma unroll
    for (int l = 0; l < L; ++l) {
      const int b = lane + WAVE * l;
      if (WAVE * l < P)
#pragma unroll
        for (int h = 0; h < WV; ++h) w[l][h] = get_word(words + (unsigned)((b < P ? b : P - 1) * LINE + h));
    }
#pragma unroll
    for (int l = 0; l < L; ++l)
      if (WAVE * l < P)
#pragma unroll
        for (int h = 0; h < WV; ++h) all = all && (unsigned int)w[l][h] == tag;
    return all;
  });
  if (!ok) return false;
  T s = T(0);
#pragma unroll
  for (int l = 0; l < L; ++l)
    if (lane + WAVE * l < P) s += word_value(w[l], T(0));
  out = lane_sum<1>(s);
  return true;
}

// A block's rows of V in memory (the single phases): column c, local row i, 0 past n.
template <typename T, typename S>
struct VGlobal {
  const S* v;  // column 0 at the block's first row
  long ldv;
  int left;    // rows of the block below n
  __device__ __forceinline__ T operator()(int c, int i) const {
    return i < left ? Basis<S, T>::load(v + (size_t)c * ldv + i) : T(0);
  }
};

// Sweeps of a block's rows: wave w has the columns c = w + 7 q, lane l the
// rows l + 64 i.  QB columns x IB rows are loaded together, without branches:
// a column past j reads column 0, a row past the block's reads the lane's
// first (the results are not used, or multiplied by 0).
constexpr int QB = 4, IB = 4;

// partial sums of V[:, c]^T w, published
template <typename T, int SLOTS, typename VF>
__device__ __forceinline__ void small_dots(word_t* words, int P, unsigned int tag, const VF& V, const T* w, int rows,
                                           int j, int wid, int lane) {
  const int nq = wid <= j ? (j - wid) / SMALL_NW + 1 : 0;
  T acc[SLOTS];
#pragma unroll
  for (int q = 0; q < SLOTS; ++q) acc[q] = T(0);
  for (int i0 = lane; i0 < rows; i0 += IB * WAVE) {
    T wv[IB];
    int at[IB];
#pragma unroll
    for (int i = 0; i < IB; ++i) {
      const bool in = i0 + WAVE * i < rows;
      at[i] = in ? i0 + WAVE * i : lane;
      wv[i] = in ? w[at[i]] : T(0);
    }
#pragma unroll
    for (int q0 = 0; q0 < SLOTS; q0 += QB) {
      if (q0 < nq) {
        T v[QB][IB];
#pragma unroll
        for (int q = 0; q < QB; ++q)
#pragma unroll
          for (int i = 0; i < IB; ++i) v[q][i] = V(q0 + q < nq ? wid + SMALL_NW * (q0 + q) : 0, at[i]);
#pragma unroll
        for (int q = 0; q < QB; ++q)
          if (q0 + q < nq)
#pragma unroll
            for (int i = 0; i < IB; ++i) acc[q0 + q] = fma_t(v[q][i], wv[i], acc[q0 + q]);
      }
    }
  }
  if (nq > 0) publish<T, SLOTS>(words, P, wid, lane, tag, acc, nq);
}

// part[wid][i] = sum over this wave's columns of h_c V[i, c]
template <typename T, int SLOTS, typename VF>
__device__ __forceinline__ void small_partial(T* part, const VF& V, const T (&h)[SLOTS], int rows, int j, int wid,
                                              int lane) {
  const int nq = wid <= j ? (j - wid) / SMALL_NW + 1 : 0;
  for (int i0 = lane; i0 < rows; i0 += IB * WAVE) {
    T s[IB];
    int at[IB];
#pragma unroll
    for (int i = 0; i < IB; ++i) {
      at[i] = i0 + WAVE * i < rows ? i0 + WAVE * i : lane;
      s[i] = T(0);
    }
#pragma unroll
    for (int q0 = 0; q0 < SLOTS; q0 += QB) {
      if (q0 < nq) {
        T v[QB][IB];
#pragma unroll
        for (int q = 0; q < QB; ++q)
#pragma unroll
          for (int i = 0; i < IB; ++i) v[q][i] = V(q0 + q < nq ? wid + SMALL_NW * (q0 + q) : 0, at[i]);
#pragma unroll
        for (int q = 0; q < QB; ++q) {
          const T hq = q0 + q < nq ? h[q0 + q] : T(0);
#pragma unroll
          for (int i = 0; i < IB; ++i) s[i] = fma_t(hq, v[q][i], s[i]);
        }
      }
    }
#pragma unroll
    for (int i = 0; i < IB; ++i)
      if (i0 + WAVE * i < rows) part[wid * rows + at[i]] = s[i];
  }
}

template <typename T>
__device__ __forceinline__ T small_updated(const T* part, T w, int rows, int i) {
  T s = part[i];
#pragma unroll
  for (int g = 1; g < SMALL_NW; ++g) s += part[g * rows + i];
  return w - s;
}

// Row r of A (shared-offset slices) times the next basis vector, gathered as
// words (tag `tag`) of the unnormalised vector; the products and their order
// are those of sell_row.  The norm's sum is polled behind the first round's
// gathers, which are in flight meanwhile.
template <typename T, typename S, int U>
__device__ __forceinline__ bool gather_row(const Csr& A, const word_t* x, unsigned int tag, const word_t* norm, int P,
                                           int r, int lane, int base, int K, bool& have_inv, T& inv, T& y) {
#pragma clang fp contract(off)
  constexpr int WV = small_words_per_value<T>();
  const T* vals = (const T*)A.svals + base + lane;
  const int* soff = A.scol + base / SELL_C;
  T sum = T(0);
  for (int k0 = 0; k0 < K; k0 += U) {
    int cc[U];
    T vv[U];
    word_t w[U][WV];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int k = k0 + u < K ? k0 + u : K - 1;
      cc[u] = min(max(r + soff[k], 0), A.n - 1);
      vv[u] = vals[SELL_C * k];
    }
    auto load = [&] {
#pragma unroll
      for (int u = 0; u < U; ++u)
#pragma unroll
        for (int h = 0; h < WV; ++h) w[u][h] = get_word(x + (size_t)cc[u] * WV + h);
    };
    auto right = [&] {
      unsigned int off = 0;
#pragma unroll
      for (int u = 0; u < U; ++u)
#pragma unroll
        for (int h = 0; h < WV; ++h) off |= (unsigned int)w[u][h] ^ tag;
      return off == 0;
    };
    load();
    if (!have_inv) {
      T n2;
      if (!collect_one(norm, P, lane, tag, n2)) return false;
      inv = T(1) / sqrt(n2);
      have_inv = true;
    }
    if (!__all(right()) && !poll([&] {
          load();
          return right();
        }))
      return false;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const T p = vv[u] * Basis<S, T>::round(word_value(w[u], T(0)) * inv);
      if (k0 + u < K) sum = sum + p;
    }
  }
  y = sum;
  return true;
}

// ---------------------------------------------------------------------------
// the whole cycle
// ---------------------------------------------------------------------------

// The window (see window.hpp) with its rows.
template <typename T>
constexpr int win_chunks() {
  return sizeof(T) == 8 ? 96 : 128;
}
template <typename T>
struct Window : WindowMap<win_chunks<T>(), 512, SMALL_MAX_RL> {
  T x[win_chunks<T>() * SELL_C];
};

// Loads the window's rows (words with tag `tag`), scaled and rounded to the
// next basis vector, by the worker waves; the norm is polled behind the first
// batch of loads.
template <typename T, typename S>
__device__ __forceinline__ bool window_load(Window<T>& W, const word_t* x, int n, unsigned int tag, const word_t* norm,
                                            int P, int wid, int lane, bool have_inv, T& inv) {
  constexpr int WV = small_words_per_value<T>();
  constexpr int G = 4;
  for (int c0 = wid; c0 < W.chunks; c0 += G * SMALL_NW) {
    int row[G];
    word_t w[G][WV];
#pragma unroll
    for (int g = 0; g < G; ++g) {
      const int c = c0 + SMALL_NW * g;
      const int r = c < W.chunks ? W.chunk[c] * SELL_C + lane : -1;
      row[g] = r >= 0 && r < n ? r : -1;
    }
    auto load = [&] {
#pragma unroll
      for (int g = 0; g < G; ++g)
#pragma unroll
        for (int h = 0; h < WV; ++h) w[g][h] = get_word(x + (size_t)(row[g] < 0 ? 0 : row[g]) * WV + h);
    };
    auto right = [&] {
      unsigned int off = 0;
#pragma unroll
      for (int g = 0; g < G; ++g)
#pragma unroll
        for (int h = 0; h < WV; ++h) off |= row[g] < 0 ? 0u : (unsigned int)w[g][h] ^ tag;
      return off == 0;
    };
    load();
    if (!have_inv) {
      T n2;
      if (!collect_one(norm, P, lane, tag, n2)) return false;
      inv = T(1) / sqrt(n2);
      have_inv = true;
    }
    if (!__all(right()) && !poll([&] {
          load();
          return right();
        }))
      return false;
#pragma unroll
    for (int g = 0; g < G; ++g) {
      const int c = c0 + SMALL_NW * g;
      if (c < W.chunks) W.x[c * SELL_C + lane] = row[g] < 0 ? T(0) : Basis<S, T>::round(word_value(w[g], T(0)) * inv);
    }
  }
  return true;
}

// Wave w keeps the columns c = w + 7 q of the block's 64 RL rows in registers
// (lane l: rows l + 64 i), the newest by way of LDS; so a sweep is SLOTS x RL
// multiply-adds a lane and reads no V (kept in LDS, the sweeps took half of an
// iteration: 64^2, fp32: 6.8 instead of 4.5 ms a solve).
//
// Bound by the latency of the three exchanges, about 1.1 us each at 32 blocks.
// GMRES(50) to 1e-12, whole solves, against one kernel per operation: 64^2
// fp32 15.1 -> 4.5 ms, 171^2 fp64 26.1 -> 10.4, 27-point 45^3 with a bf16
// basis 11.9 -> 5.2, 500^2 68.3 -> 34.2; GMRES(100), 7-point 50^3 30.2 -> 16.5.
template <typename T, typename S, int SLOTS, int RL>
__global__ __launch_bounds__(SMALL_NT) void k_small_cycle(SmallArgs<T, S> a) {
  constexpr int WV = small_words_per_value<T>();
  constexpr int ROWS = WAVE * RL;
  __shared__ SmallShared<T> sh;
  __shared__ Window<T> win;
  __shared__ T s_w[ROWS];               // the working vector's rows
  __shared__ T s_part[SMALL_NW][ROWS];  // the waves' parts of V h
  T* s_vals = dyn_lds<T>();             // the rows' values of A, if they fit
  const int P = a.blocks, n = a.A.n;
  const int lane = threadIdx.x & (WAVE - 1);
  const int wid = __builtin_amdgcn_readfirstlane(threadIdx.x / WAVE);
  const bool worker = wid < SMALL_NW;
  const int r0 = blockIdx.x * ROWS;
  const StateHdr* hd = a.st.hdr;
  const int flags0 = hd->flags;
  const T gin = (T)hd->gamma_in;
  const bool check_stop = hd->stop_abs >= 0.0;
  const T stop_abs = (T)hd->stop_abs;
  T inv = (T)hd->inv_h;
  if (flags0 & F_DONE) return;
  if (threadIdx.x == 0) {
    sh.flags = 0;
    sh.lost = 0;
    sh.g = (T)a.st.g[0];
  }
  word_t* const h1w = a.words;
  word_t* const h2w = h1w + (size_t)SMALL_NW * P * LINE * WV;
  word_t* const nw = h2w + (size_t)SMALL_NW * P * LINE * WV;
  if (worker)
    for (int i = wid * WAVE + lane; i < ROWS; i += SMALL_NW * WAVE) {
      s_w[i] = T(0);
      if (r0 + i < n) {
        s_w[i] = a.wtmp[r0 + i];
        put_value(a.x + (size_t)(r0 + i) * WV, s_w[i], a.tag - 1);
      }
    }
  T V[SLOTS][RL];
#pragma unroll
  for (int q = 0; q < SLOTS; ++q)
#pragma unroll
    for (int i = 0; i < RL; ++i) V[q][i] = T(0);
  const bool writer = blockIdx.x == 0;
  // V[:, c]^T w of the wave's columns, summed over the blocks; then their part of V h
  auto project = [&](word_t* words, unsigned int tag, int nq, T* all, T (&h)[SLOTS]) {
    T wv[RL], acc[SLOTS];
#pragma unroll
    for (int i = 0; i < RL; ++i) wv[i] = s_w[lane + WAVE * i];
#pragma unroll
    for (int q = 0; q < SLOTS; ++q) {
      acc[q] = T(0);
#pragma unroll
      for (int i = 0; i < RL; ++i) acc[q] = fma_t(V[q][i], wv[i], acc[q]);
    }
#pragma unroll
    for (int q = 0; q < SLOTS; ++q) h[q] = T(0);
    bool ok = true;
    if (nq > 0) {
      publish<T, SLOTS>(words, P, wid, lane, tag, acc, nq);
      __builtin_amdgcn_s_sleep(POLL_WAIT);
      ok = collect<T, SLOTS>(words, P, wid, lane, tag, h, all, nq);
    }
#pragma unroll
    for (int i = 0; i < RL; ++i) {
      T s = T(0);
#pragma unroll
      for (int q = 0; q < SLOTS; ++q) s = fma_t(h[q], V[q][i], s);
      s_part[wid][lane + WAVE * i] = s;
    }
    return ok;
  };
  window_build<SMALL_NT>(win, a.A, r0 / SELL_C, min(RL, a.A.nslices - r0 / SELL_C), win_chunks<T>());
  const T* const vals = (const T*)a.A.svals + a.A.sptr[min(r0 / SELL_C, a.A.nslices)];
  const bool in_lds = win.chunks > 0 && (size_t)win.pair[RL] * SELL_C * sizeof(T) <= a.vals_lds;
  if (in_lds)
    for (int i = threadIdx.x; i < win.pair[RL] * SELL_C; i += SMALL_NT) s_vals[i] = vals[i];
  const int own = win.chunks > 0 ? win.own * SELL_C : 0;  // the block's rows in win.x
  __syncthreads();
  int j = 0;
  for (;; ++j) {
    const unsigned int tag = a.tag + (unsigned int)j;
    const int nq = wid <= j ? (j - wid) / SMALL_NW + 1 : 0;
    T h[SLOTS];
    bool lost = false;
    // v_j = round(w'' / ||w''||) and w = A v_j
    __builtin_amdgcn_s_sleep(POLL_WAIT);
    if (worker) {
      if (win.chunks > 0)
        lost = !window_load<T, S>(win, a.x, n, tag - 1, nw, P, wid, lane, j == 0, inv);
    } else if (j > 0) {
      T n2 = T(0);
      lost = !collect_one(nw, P, lane, tag - 1, n2);
      if (lane == 0) sh.nrm2 = n2;
    }
    __syncthreads();
    if (worker) {
      bool have_inv = j == 0;
      for (int s = wid; s < RL; s += SMALL_NW) {
        const int i = s * SELL_C + lane, r = r0 + i, sl = r0 / SELL_C + s;
        T y = T(0);
        if (sl < a.A.nslices && !lost) {
          if (win.chunks > 0) {
            y = in_lds ? window_row(win, win.x, s_vals + win.pair[s] * SELL_C, s, lane)
                       : window_row(win, win.x, vals + win.pair[s] * SELL_C, s, lane);
          } else {
            const int base = a.A.sptr[sl];
            const int K = (a.A.sptr[sl + 1] - base) / SELL_C;
            lost = !gather_row<T, S, 5>(a.A, a.x, tag - 1, nw, P, r, lane, base, K, have_inv, inv, y);
            if (!have_inv && !lost) {  // a slice without entries
              T n2 = T(0);
              lost = !collect_one(nw, P, lane, tag - 1, n2);
              inv = T(1) / sqrt(n2);
              have_inv = true;
            }
            win.x[i] = r < n ? Basis<S, T>::round(s_w[i] * inv) : T(0);
          }
          if (r < n) Basis<S, T>::store(a.V + (size_t)j * a.ldv + r, win.x[own + i]);
          else y = T(0);
        }
        s_w[i] = y;
      }
    }
    __syncthreads();
    if (worker) {
      if (wid == j % SMALL_NW) {
#pragma unroll
        for (int q = 0; q < SLOTS; ++q)
          if (q == j / SMALL_NW)
#pragma unroll
            for (int i = 0; i < RL; ++i) V[q][i] = r0 / SELL_C + i < a.A.nslices ? win.x[own + lane + WAVE * i] : T(0);
      }
      lost = !project(h1w, tag, nq, sh.h1[j & 1], h) || lost;
    } else if (j > 0) {
      small_givens<T>(a.st, sh, j - 1, a.kmax, gin, stop_abs, check_stop, writer);
    }
    if (lost && lane == 0) sh.lost = 1;
    __syncthreads();
    if ((sh.flags & F_DONE) || sh.lost) break;
    // w' = w - V h1, h2 = V^T w'
    if (worker)
      for (int i = wid * WAVE + lane; i < ROWS; i += SMALL_NW * WAVE) s_w[i] = small_updated(&s_part[0][0], s_w[i], ROWS, i);
    __syncthreads();
    if (worker) lost = !project(h2w, tag, nq, sh.h2, h);
    if (lost && lane == 0) sh.lost = 1;
    __syncthreads();
    if (sh.lost) break;
    // w'' = w' - V h2 for the other blocks, and its norm
    if (worker) {
      T nrm = T(0);
      for (int i = wid * WAVE + lane; i < ROWS; i += SMALL_NW * WAVE) {
        const T v = small_updated(&s_part[0][0], s_w[i], ROWS, i);
        s_w[i] = v;
        if (r0 + i < n) {
          put_value(a.x + (size_t)(r0 + i) * WV, v, tag);
          nrm = fma_t(v, v, nrm);
        }
      }
      nrm = lane_sum<1>(nrm);
      if (lane == 0) sh.red[wid] = nrm;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
      T s = sh.red[0];
#pragma unroll
      for (int g = 1; g < SMALL_NW; ++g) s += sh.red[g];
      put_value(nw + (size_t)blockIdx.x * LINE, s, tag);
    }
    if (j + 1 >= a.kmax) {
      if (!worker) {
        T n2 = T(0);
        lost = !collect_one(nw, P, lane, tag, n2);
        if (lane == 0) {
          sh.nrm2 = n2;
          if (lost) sh.lost = 1;
        }
        if (!lost) small_givens<T>(a.st, sh, j, a.kmax, gin, stop_abs, check_stop, writer);
      }
      break;
    }
  }
  __syncthreads();
  if (sh.lost && threadIdx.x == 0) {
    // every block gives up: the solve ends with an error
    StateHdr* o = a.st.hdr;
    o->lost = 1;
    o->flags = F_DONE | F_NUMERIC;
  }
}

// ---------------------------------------------------------------------------
// the phases one by one
// ---------------------------------------------------------------------------

// Words summed after a kernel boundary: every tag is right.
template <typename T, typename S, int SLOTS, int PH>
__global__ __launch_bounds__(SMALL_NT) void k_small_phase(SmallArgs<T, S> a) {
  constexpr int WV = small_words_per_value<T>();
  __shared__ SmallShared<T> sh;
  const int flags0 = load_flags(a.st.hdr);
  if (flags0 & F_DONE) return;
  const int rows = a.rows, P = a.blocks, j = a.j, n = a.A.n;
  T* w = dyn_lds<T>();
  T* part = w + rows;
  const int lane = threadIdx.x & (WAVE - 1);
  const int wid = __builtin_amdgcn_readfirstlane(threadIdx.x / WAVE);
  const bool worker = wid < SMALL_NW;
  const int r0 = blockIdx.x * rows;
  word_t* const h1w = a.words;
  word_t* const h2w = h1w + (size_t)SMALL_NW * P * LINE * WV;
  word_t* const nw = h2w + (size_t)SMALL_NW * P * LINE * WV;
  const unsigned int tag = a.tag + (unsigned int)j;
  const int nq = worker && wid <= j ? (j - wid) / SMALL_NW + 1 : 0;
  const VGlobal<T, S> V{a.V + r0, a.ldv, n - r0};
  T h[SLOTS];
  bool lost = false;
  if constexpr (PH == SMALL_GIVENS) {
    // one block: the sums of step j, the earlier rotations, the Givens step
    const StateHdr* hd = a.st.hdr;
    if (worker) {
      if (nq > 0) {
        lost = !collect<T, SLOTS>(h1w, P, wid, lane, tag, h, sh.h1[j & 1], nq);
        lost = !collect<T, SLOTS>(h2w, P, wid, lane, tag, h, sh.h2, nq) || lost;
      }
    } else {
      T n2 = T(0);
      lost = !collect_one(nw, P, lane, tag, n2);
      for (int i = lane; i < j; i += WAVE) {
        sh.cs[i] = (T)a.st.cs[i];
        sh.sn[i] = (T)a.st.sn[i];
      }
      if (lane == 0) {
        sh.nrm2 = n2;
        sh.g = (T)a.st.g[j];
      }
    }
    __syncthreads();
    if (!worker)
      small_givens<T>(a.st, sh, j, a.kmax, (T)hd->gamma_in, (T)hd->stop_abs, hd->stop_abs >= 0.0, true);
    __syncthreads();
  } else if constexpr (PH == SMALL_SPMV) {
    T inv = (T)a.st.hdr->inv_h;
    if (j > 0) {
      T n2 = T(0);
      lost = !collect_one(nw, P, lane, tag - 1, n2);
      inv = T(1) / sqrt(n2);
    }
    const XScaled<T, S> xs{a.wtmp, inv};
    if (worker)
      for (int s = wid; s * SELL_C < rows; s += SMALL_NW) {
        const int i = s * SELL_C + lane, r = r0 + i, sl = r0 / SELL_C + s;
        T y = T(0);
        if (sl < a.A.nslices) {
          y = sell_row<T>(a.A, xs, sl, r, lane);
          if (r < n) {
            Basis<S, T>::store(a.V + (size_t)j * a.ldv + r, xs(r));
            a.w1[r] = y;
          } else {
            y = T(0);
          }
        }
        w[i] = y;
      }
    // v_j's rows are read back by other waves of the block
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (worker) small_dots<T, SLOTS>(h1w, P, tag, V, w, rows, j, wid, lane);
  } else {
    // w' = w - V h1 and the partial sums of h2, or w'' = w' - V h2 and of its norm
    constexpr bool FIRST = PH == SMALL_UPDATE;
    const T* in = FIRST ? a.w1 : a.w2;
    T* out = FIRST ? a.w2 : a.wtmp;
    if (nq > 0) lost = !collect<T, SLOTS>(FIRST ? h1w : h2w, P, wid, lane, tag, h, sh.h2, nq);
    if (worker) small_partial<T, SLOTS>(part, V, h, rows, j, wid, lane);
    __syncthreads();
    T nrm = T(0);
    if (worker) {
      for (int i = wid * WAVE + lane; i < rows; i += SMALL_NW * WAVE) {
        w[i] = T(0);
        if (r0 + i < n) {
          const T v = small_updated(part, in[r0 + i], rows, i);
          w[i] = v;
          out[r0 + i] = v;
          if constexpr (!FIRST) nrm = fma_t(v, v, nrm);
        }
      }
      nrm = lane_sum<1>(nrm);
      if (lane == 0) sh.red[wid] = nrm;
    }
    __syncthreads();
    if constexpr (FIRST) {
      if (worker) small_dots<T, SLOTS>(h2w, P, tag, V, w, rows, j, wid, lane);
    } else if (threadIdx.x == 0) {
      T s = sh.red[0];
#pragma unroll
      for (int g = 1; g < SMALL_NW; ++g) s += sh.red[g];
      put_value(nw + (size_t)blockIdx.x * LINE, s, tag);
    }
  }
  if (lost && lane == 0) {
    a.st.hdr->lost = 1;
    a.st.hdr->flags = F_DONE | F_NUMERIC;
  }
}

__global__ void k_small_clear(unsigned long long* words, size_t count) {
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < count; i += (size_t)gridDim.x * blockDim.x)
    words[i] = 0;
}

template <typename T, typename S, int SLOTS>
SmallKernel<T, S> phase_of(SmallPhase ph) {
  switch (ph) {
    case SMALL_SPMV: return k_small_phase<T, S, SLOTS, SMALL_SPMV>;
    case SMALL_GIVENS: return k_small_phase<T, S, SLOTS, SMALL_GIVENS>;
    case SMALL_UPDATE: return k_small_phase<T, S, SLOTS, SMALL_UPDATE>;
    default: return k_small_phase<T, S, SLOTS, SMALL_NORM>;
  }
}

// Rows per lane of the instances: SLOTS x RL values of T take at most 128 of
// the 256 registers a lane has.
template <typename T, typename S, int SLOTS, int RL>
SmallKernel<T, S> cycle_of(int rl) {
  if constexpr (SLOTS * RL * (int)sizeof(T) > 128 * 4) {
    return nullptr;
  } else {
    if (rl == RL) return k_small_cycle<T, S, SLOTS, RL>;
    constexpr int NEXT = RL == 1 ? 2 : RL == 2 ? 3 : RL == 3 ? 4 : RL == 4 ? 6 : RL == 6 ? 8 : RL == 8 ? 12 : 16;
    if constexpr (RL == 16) return nullptr;
    else return cycle_of<T, S, SLOTS, NEXT>(rl);
  }
}

constexpr int RLS[] = {1, 2, 3, 4, 6, 8, 12, SMALL_MAX_RL};

int slots_of(int m) { return m <= 4 * SMALL_NW ? 4 : m <= 8 * SMALL_NW ? 8 : 16; }

}  // namespace

template <typename T, typename S>
SmallKernel<T, S> small_kernel(SmallPhase ph, int m, int rows) {
  const int sl = slots_of(m);
  if (ph == SMALL_CYCLE)
    return sl == 4   ? cycle_of<T, S, 4, 1>(rows / WAVE)
           : sl == 8 ? cycle_of<T, S, 8, 1>(rows / WAVE)
                     : cycle_of<T, S, 16, 1>(rows / WAVE);
  return sl == 4 ? phase_of<T, S, 4>(ph) : sl == 8 ? phase_of<T, S, 8>(ph) : phase_of<T, S, 16>(ph);
}
template SmallKernel<float, float> small_kernel<float, float>(SmallPhase, int, int);
template SmallKernel<float, bf16_t> small_kernel<float, bf16_t>(SmallPhase, int, int);
template SmallKernel<double, double> small_kernel<double, double>(SmallPhase, int, int);

// An exchange's time grows with the lines a wave reads: 1.1 us at 16 blocks,
// 1.6 us at 64, 2.4 us at 128, 5 us at 256 (one 128-byte line per block in
// fp32, two in fp64); more rows per block cost registers and time in between.
// So: at least 128 rows (4096 rows, fp32: 32 blocks 4.5 ms a solve, 16 blocks
// 4.6, 8 blocks 5.5), and as many as bring the blocks' lines to 128 (29241
// rows, fp64: 153 blocks 13.5 ms, 115 11.7, 77 10.5, 58 10.4; 91125 rows,
// bf16 basis: 238 blocks 5.8 ms, 178 5.6, 119 5.2, 89 6.0), or as many as the
// registers hold.
int small_rows(int64_t n, int m, int sT, int cus) {
  if (m > SMALL_MAX_M) return 0;
  const int64_t blocks = std::min(SMALL_MAX_P, cus);
  int rows = 0;
  for (int rl : RLS) {
    if (slots_of(m) * rl * sT > 128 * 4) break;
    rows = WAVE * rl;
    if (rl >= 2 && n * (sT / 4) <= 128 * (int64_t)rows) break;
  }
  return n <= rows * blocks ? rows : 0;
}

size_t small_cycle_lds(int rows, int sT) {
  const size_t fixed = sT == 8 ? sizeof(Window<double>) + sizeof(SmallShared<double>)
                               : sizeof(Window<float>) + sizeof(SmallShared<float>);
  const size_t used = fixed + (size_t)rows * (SMALL_NW + 1) * sT + 256;
  return used < SMALL_LDS ? (SMALL_LDS - used) / 256 * 256 : 0;
}

size_t small_phase_lds(int rows, int sT) { return (size_t)rows * (SMALL_NW + 1) * sT; }

size_t small_words(int blocks, int sT) {
  const size_t WV = sT / 4;
  return (2 * SMALL_NW * WV + 1) * (size_t)blocks * LINE;
}

void small_clear(unsigned long long* words, size_t count, hipStream_t s) {
  hipLaunchKernelGGL(k_small_clear, dim3((unsigned)std::min<size_t>(512, (count + 255) / 256)), dim3(256), 0, s, words,
                     count);
}

}  // namespace gir
