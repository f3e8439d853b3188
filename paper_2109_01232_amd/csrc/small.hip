// Kernels of the register-resident inner cycle (see small.hpp).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

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
// others' stores have arrived (1.8 -> 1.1 us).  WAIT_ONE, WAIT_TWO: the same in
// two stages, for the blocks that sum a group and for those that wait for them.
constexpr int POLL_WAIT = 12, WAIT_ONE = 8, WAIT_TWO = 16;
constexpr int LINE = 16;

template <typename T>
__device__ __forceinline__ word_t* line_of(word_t* words, int P, int wid, int b) {
  return words + ((size_t)wid * (P + SMALL_GROUPS) + b) * (LINE * small_words_per_value<T>());
}

// Past 64 blocks the lines are summed in two stages, first those of up to 16
// blocks of a die (block b runs on die b % 8) by one of them, which writes the
// group's line behind the blocks' (1.8 us at 256 blocks, where reading every
// line takes 5 us; 2.4 us at 128).
__host__ __device__ constexpr bool small_staged(int P) { return P > WAVE; }
constexpr int SMALL_STAGED_RL = 4;  // rows per lane from which on there are more than 64 blocks
struct Group {
  int g, first, count;  // its line, its first block (then every eighth), its blocks
  __device__ __forceinline__ Group(int g_, int P)
      : g(g_), first(g_ % 8 + 128 * (g_ / 8)), count(min(16, (P - first + 7) / 8)) {}
};
__device__ __forceinline__ int group_of(int b) { return b % 8 + 8 * (b / 128); }
__device__ __forceinline__ bool leads_group(int b) { return b / 8 % 16 == 0; }
__device__ __forceinline__ int groups_of(int P) { return 8 + max(0, min(8, P - 128)); }

// The single phases read what an earlier launch has written: every word is
// there, and the loads go through the caches (past them every block fetches
// every line from memory: an iteration of 62500 rows 27.5 instead of 25.6 us, of
// 22500 26.7 instead of 21.7).
template <bool ALONE>
__device__ __forceinline__ word_t look_at(const word_t* p) {
  if constexpr (ALONE) return *p;
  else return get_word(p);
}
template <bool ALONE, typename F>
__device__ __forceinline__ bool wait_for(const Wait& wt, F load) {
  if constexpr (ALONE) return __all(load());
  else return poll(wt, load);
}

// The words of `count` <= 16 lines, `stride` words apart, as a lane sees them:
// value lane % W of the lines lane / W + NB g.
template <typename T, int W, bool ALONE = false>
struct Lines {
  static constexpr int WV = small_words_per_value<T>();
  static constexpr int NB = WAVE / W < 16 ? WAVE / W : 16, G = 16 / NB;
  word_t w[G][WV];
  __device__ __forceinline__ void load(const word_t* lines, int stride, int count, int lane) {
#pragma unroll
    for (int g = 0; g < G; ++g) {
      const int b = NB * g + lane / W;
#pragma unroll
      for (int h = 0; h < WV; ++h) w[g][h] = look_at<ALONE>(lines + (unsigned)((b < count ? b : 0) * stride + WV * (lane % W) + h));
    }
  }
  // the tags are right; values from nq on are not there
  __device__ __forceinline__ bool right(int count, int nq, unsigned int tag, int lane) const {
    bool ok = true;
#pragma unroll
    for (int g = 0; g < G; ++g)
#pragma unroll
      for (int h = 0; h < WV; ++h)
        ok = ok && ((unsigned int)w[g][h] == tag || lane % W >= nq || NB * g + lane / W >= count);
    return ok;
  }
  // lane l: the sum of value l % W
  __device__ __forceinline__ T sum(int count, int nq, int lane) const {
    const int bl = lane / W;
    T s = T(0);
#pragma unroll
    for (int g = 0; g < G; ++g) s += NB * g + bl < count && bl < NB && lane % W < nq ? word_value(w[g], T(0)) : T(0);
    return lane_sum<W>(s);
  }
};

// out, lane l: the sum of value l % W over the lines.  False on giving up.
template <typename T, int W>
__device__ __forceinline__ bool take(const Wait& wt, const word_t* lines, int stride, int count, int nq,
                                     unsigned int tag, int lane, T& out) {
  Lines<T, W> k;
  const bool ok = poll(wt, [&] {
    k.load(lines, stride, count, lane);
    return k.right(count, nq, tag, lane);
  });
  if (!ok) return false;
  out = k.sum(count, nq, lane);
  return true;
}

// The two stages over P lines from `lines`, `line` words each, the groups'
// behind them.  The cycle kernel's blocks share the first one; ALONE (the single
// phases) a wave does all of it in the same order, eight groups' loads in flight
// together (group after group an iteration of 62500 rows launched phase by phase
// took 60 us instead of 30; the general kernels' 31).
template <typename T, int W, bool ALONE>
__device__ __forceinline__ bool take_staged(const Wait& wt, word_t* lines, int line, int P, bool leader, int nq,
                                            unsigned int tag, int lane, T& out) {
  if constexpr (ALONE) {
    typedef Lines<T, W, true> Group_;
    constexpr int NB = Group_::NB, AT = 32 / (Group_::G * Group_::WV) < 8 ? 32 / (Group_::G * Group_::WV) : 8;
    const int groups = groups_of(P);
    bool right = true;
    T sum = T(0);
    for (int g0 = 0; g0 < groups; g0 += AT) {
      Group_ k[AT];
      int count[AT];
#pragma unroll
      for (int i = 0; i < AT; ++i) {
        const Group G(g0 + i < groups ? g0 + i : 0, P);
        count[i] = g0 + i < groups ? G.count : 0;
        k[i].load(lines + (size_t)G.first * line, 8 * line, G.count, lane);
      }
#pragma unroll
      for (int i = 0; i < AT; ++i) {
        right = right && k[i].right(count[i], nq, tag, lane);
        const T s = k[i].sum(count[i], nq, lane);
        if (g0 + i < groups) sum += lane / W == (g0 + i) % NB && lane % W < nq ? s : T(0);
      }
    }
    out = lane_sum<W>(sum);
    return __all(right);
  }
  if (leader) {
    const Group G(group_of(blockIdx.x), P);
    T s;
    if (!take<T, W>(wt, lines + (size_t)G.first * line, 8 * line, G.count, nq, tag, lane, s)) return false;
    if (lane < nq) put_value(lines + (size_t)(P + G.g) * line + small_words_per_value<T>() * lane, s, tag);
    __builtin_amdgcn_s_sleep(WAIT_ONE);
  } else {
    __builtin_amdgcn_s_sleep(WAIT_TWO);
  }
  return take<T, W>(wt, lines + (size_t)P * line, line, groups_of(P), nq, tag, lane, out);
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
template <typename T, int SLOTS, bool STAGED, bool ALONE = false>
__device__ __forceinline__ bool collect(const Wait& wt, word_t* words, int P, int wid, int lane, unsigned int tag,
                                        T (&out)[SLOTS], T* all, int nq) {
  constexpr int WV = small_words_per_value<T>();
  constexpr int W = SLOTS, NB = WAVE / W;
  constexpr int G = 8 / WV;
  const int q = lane % W, bl = lane / W;
  const word_t* p = line_of<T>(words, P, wid, 0) + WV * q;
  T sum = T(0);
  if constexpr (STAGED) {
    if (!take_staged<T, W, ALONE>(wt, line_of<T>(words, P, wid, 0), LINE * WV, P, leads_group(blockIdx.x), nq, tag, lane,
                                  sum))
      return false;
  } else {
    // GN loads of NB blocks each from block b0; past the last block its line
    // again: a load under a condition has its result copied, and waited for, before
    // the next goes out (fp64, 15625 rows, 36.1 instead of 28.7 us an iteration)
    auto pass = [&](auto gn, int b0) {
      constexpr int GN = decltype(gn)::value;
      word_t w[GN][WV];
      const bool ok = wait_for<ALONE>(wt, [&] {
        bool right = true;
#pragma unroll
        for (int g = 0; g < GN; ++g) {
          const int b = b0 + NB * g + bl;
#pragma unroll
          for (int h = 0; h < WV; ++h) w[g][h] = look_at<ALONE>(p + (unsigned)((b < P ? b : P - 1) * LINE * WV + h));
        }
#pragma unroll
        for (int g = 0; g < GN; ++g)
#pragma unroll
          for (int h = 0; h < WV; ++h) right = right && ((unsigned int)w[g][h] == tag || q >= nq);
        return right;
      });
#pragma unroll
      for (int g = 0; g < GN; ++g)
        if (NB * g + b0 + bl < P && q < nq) sum += word_value(w[g], T(0));
      return ok;
    };
    if (WV == 1 && P <= NB * G / 4) {  // (fp64: the second copy of the code costs what it gives)
      if (!pass(std::integral_constant<int, G / 4>{}, 0)) return false;
    } else {
      for (int b0 = 0; b0 < P; b0 += NB * G)
        if (!pass(std::integral_constant<int, G>{}, b0)) return false;
    }
    sum = lane_sum<W>(sum);
  }
  // lane q holds the sum of value q; hand each to every lane
  if (lane < nq) all[wid + SMALL_NW * lane] = sum;
#pragma unroll
  for (int i = 0; i < SLOTS; ++i) out[i] = read_lane(sum, i);
  return true;
}

// one value a block, in a line of its own: the sum over the blocks
// (past 64 blocks `leader`: this wave sums its group's for the others).
template <typename T, bool STAGED, bool ALONE = false>
__device__ __forceinline__ bool collect_one(const Wait& wt, word_t* words, int P, int lane, unsigned int tag, T& out,
                                            bool leader = false) {
  constexpr int WV = small_words_per_value<T>();
  if constexpr (STAGED) {
    T s;
    if (!take_staged<T, 1, ALONE>(wt, words, LINE, P, leader, 1, tag, lane, s)) return false;
    out = read_lane(s, 0);
  } else {
    word_t w[WV];
    const bool ok = wait_for<ALONE>(wt, [&] {
      bool all = true;
#pragma unroll
      for (int h = 0; h < WV; ++h) w[h] = look_at<ALONE>(words + (unsigned)((lane < P ? lane : P - 1) * LINE + h));
#pragma unroll
      for (int h = 0; h < WV; ++h) all = all && (unsigned int)w[h] == tag;
      return all;
    });
    if (!ok) return false;
    out = lane_sum<1>(lane < P ? T(0) + word_value(w, T(0)) : T(0));
  }
  return true;
}

// the same in the single phases
template <typename T, int SLOTS>
__device__ __forceinline__ bool collect_alone(const Wait& wt, word_t* words, int P, int wid, int lane, unsigned int tag,
                                              T (&out)[SLOTS], T* all, int nq) {
  return small_staged(P) ? collect<T, SLOTS, true, true>(wt, words, P, wid, lane, tag, out, all, nq)
                         : collect<T, SLOTS, false, true>(wt, words, P, wid, lane, tag, out, all, nq);
}
template <typename T>
__device__ __forceinline__ bool collect_one_alone(const Wait& wt, word_t* words, int P, int lane, unsigned int tag,
                                                  T& out) {
  return small_staged(P) ? collect_one<T, true, true>(wt, words, P, lane, tag, out)
                         : collect_one<T, false, true>(wt, words, P, lane, tag, out);
}

// A block's rows of V in memory (the single phases): column c, local row i, 0 past n.
template <typename T, typename S>
struct VGlobal {
  const S* v;  // column 0 at the block's first row
  long ldv;
  int left;    // rows of the block below n
  // (not a load under a condition, which is waited for where that ends: an
  // iteration of 250000 rows 46.8 instead of 41.5 us, with a bf16 basis 80 instead of 39.6)
  __device__ __forceinline__ T operator()(int c, int i) const {
    const T x = Basis<S, T>::load(v + (size_t)c * ldv + (i < left ? i : 0));
    return i < left ? x : T(0);
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
template <typename T, typename S, int U, bool STAGED>
__device__ __forceinline__ bool gather_row(const Wait& wt, const Csr& A, const word_t* x, unsigned int tag,
                                           word_t* norm, int P, int r, int lane, int base, int K, bool& have_inv, T& inv, T& y) {
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
      if (!collect_one<T, STAGED>(wt, norm, P, lane, tag, n2)) return false;
      inv = T(1) / sqrt(n2);
      have_inv = true;
    }
    if (!__all(right()) && !poll(wt, [&] {
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
// PLAIN: the words' values as they are.
template <typename T, typename S, bool STAGED, bool PLAIN = false>
__device__ __forceinline__ bool window_load(const Wait& wt, Window<T>& W, const word_t* x, int n, unsigned int tag,
                                            word_t* norm, int P, int wid, int lane, bool have_inv, T& inv) {
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
    if (!PLAIN && !have_inv) {
      T n2;
      if (!collect_one<T, STAGED>(wt, norm, P, lane, tag, n2)) return false;
      inv = T(1) / sqrt(n2);
      have_inv = true;
    }
    if (!__all(right()) && !poll(wt, [&] {
          load();
          return right();
        }))
      return false;
#pragma unroll
    for (int g = 0; g < G; ++g) {
      const int c = c0 + SMALL_NW * g;
      const T v = word_value(w[g], T(0));
      if (c < W.chunks) W.x[c * SELL_C + lane] = row[g] < 0 ? T(0) : PLAIN ? v : Basis<S, T>::round(v * inv);
    }
  }
  return true;
}

// Wave w keeps the columns c = w + 7 q of the block's 64 RL rows in registers
// (lane l: rows l + 64 i), the newest by way of LDS; so a sweep is SLOTS x RL
// multiply-adds a lane and reads no V (kept in LDS, the sweeps took half of an
// iteration: 64^2, fp32: 6.8 instead of 4.5 ms a solve).
//
// Bound by the latency of the three exchanges, 1.1 us each at 32 blocks, 1.8 us
// in two stages.  GMRES(50) to 1e-12, whole solves, against one kernel per
// operation: 64^2 fp32 13.3 -> 3.7 ms, 171^2 fp64 29.3 -> 11.2, 27-point 45^3
// with a bf16 basis 11.6 -> 4.0, 500^2 68.3 -> 26.0; GMRES(100), 7-point 50^3
// 30.2 -> 9.6 (the two stages alone, against every block reading every line:
// 45^3 5.1 -> 4.0, 500^2 33.8 -> 26.0, 50^3 16.4 -> 9.6).
//
// PRE: z = M v_j first, exchanged block to block as the vector is.  Block
// Jacobi: one exchange more.  Polynomial: one per SpMV; the vectors alternate
// between two places, and no block writes a place again before every block
// within `near` of it (which holds all that read from it) has published the
// vector after, and so read this one.  2 us an exchange and SpMV, against
// 5-6 us a launch: 10000 rows, fp32, degree 10 6.6 -> 2.1 ms a solve, block
// Jacobi 12.9 -> 4.3; 27000 rows, fp64, degree 5 6.4 -> 2.5, block Jacobi 11.2
// -> 4.6; 125000 27-point rows, degree 20 13.2 -> 4.0, block Jacobi 11.1 -> 5.5;
// 216000 7-point rows, degree 10 12.4 -> 8.5, block Jacobi 18.7 -> 16.4.
template <typename T, typename S, int SLOTS, int RL, bool STAGED, bool PRE>
__global__ __launch_bounds__(SMALL_NT) void k_small_cycle(SmallArgs<T, S> a) {
  constexpr int WV = small_words_per_value<T>();
  constexpr int ROWS = WAVE * RL;
  __shared__ SmallShared<T> sh;
  __shared__ Window<T> win;
  __shared__ T s_w[ROWS];               // the working vector's rows
  __shared__ T s_part[SMALL_NW][ROWS];  // the waves' parts of V h
  T* s_vals = dyn_lds<T>();             // the rows' values of A, if they fit
  T* const s_pre = s_vals;              // PRE: rows of v_j, the program's vectors and y
  if constexpr (PRE) s_vals += SMALL_PRE_ROWS * ROWS;
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
  word_t* const h2w = h1w + (size_t)SMALL_NW * (P + SMALL_GROUPS) * LINE * WV;
  word_t* const nw = h2w + (size_t)SMALL_NW * (P + SMALL_GROUPS) * LINE * WV;
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
  auto project = [&](const Wait& wt, word_t* words, unsigned int tag, int nq, T* all, T (&h)[SLOTS]) {
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
      ok = collect<T, SLOTS, STAGED>(wt, words, P, wid, lane, tag, h, all, nq);
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
  // Rows too wide for the window's own table (their values do not fit LDS
  // either) have it in the values' place: 40 entries either side, 200000 rows,
  // 77 -> 29 us an iteration, against rows gathered one by one.
  window_build<SMALL_NT>(win, a.A, r0 / SELL_C, min(RL, a.A.nslices - r0 / SELL_C), win_chunks<T>(), (int*)s_vals,
                         PRE ? win.PAIRS : a.vals_lds / sizeof(int));
  const int* const off = win.wide() ? (const int*)s_vals : win.off;
  const T* const vals = (const T*)a.A.svals + a.A.sptr[min(r0 / SELL_C, a.A.nslices)];
  const bool in_lds = win.chunks > 0 && !win.wide() && (size_t)win.pair[RL] * SELL_C * sizeof(T) <= a.vals_lds;
  if (in_lds)
    for (int i = threadIdx.x; i < win.pair[RL] * SELL_C; i += SMALL_NT) s_vals[i] = vals[i];
  const int own = win.chunks > 0 ? win.own * SELL_C : 0;  // the block's rows in win.x
  __syncthreads();
  // the vector with `tag` at x into the window; every other wave's done too.
  // A wave that has given up waits no more.
  auto exchange_window = [&](const Wait& wt, word_t* x, unsigned int tag, int near, bool lost) {
    bool ok = !lost;
    if (lost) {
    } else if (worker) {
      ok = window_load<T, S, STAGED, true>(wt, win, x, n, tag, nullptr, P, wid, lane, true, inv);
    } else if (near > 0) {
      const int b = (int)blockIdx.x - near + lane;
      const bool there = lane <= 2 * near && b >= 0 && b < P;
      ok = poll(wt, [&] { return !there || (unsigned int)get_word(x + (size_t)(there ? b : 0) * ROWS * WV) == tag; });
    }
    __syncthreads();
    return ok;
  };
  int j = 0;
  for (;; ++j) {
    const unsigned int tag = a.tag + (unsigned int)j;
    const int nq = wid <= j ? (j - wid) / SMALL_NW + 1 : 0;
    // until every block's sums of the first projection are in, some may not be there
    const Wait wt{&a.st.hdr->lost, j == 0 ? ARRIVE_LOOKS : SILENT_LOOKS};
    T h[SLOTS];
    bool lost = false;
    // v_j = round(w'' / ||w''||) and w = A v_j
    __builtin_amdgcn_s_sleep(POLL_WAIT);
    if (worker) {
      if (win.chunks > 0)
        lost = !window_load<T, S, STAGED>(wt, win, a.x, n, tag - 1, nw, P, wid, lane, j == 0, inv);
    } else if (j > 0) {
      T n2 = T(0);
      lost = !collect_one<T, STAGED>(wt, nw, P, lane, tag - 1, n2, leads_group(blockIdx.x));
      if (lane == 0) sh.nrm2 = n2;
    }
    __syncthreads();
    if constexpr (PRE) {
      if (worker) {
        if (wid == j % SMALL_NW) {
#pragma unroll
          for (int q = 0; q < SLOTS; ++q)
            if (q == j / SMALL_NW)
#pragma unroll
              for (int i = 0; i < RL; ++i) V[q][i] = r0 / SELL_C + i < a.A.nslices ? win.x[own + lane + WAVE * i] : T(0);
        }
        for (int s = wid; s < RL; s += SMALL_NW) {
          const int i = s * SELL_C + lane, r = r0 + i;
          const T v = r < n ? win.x[own + i] : T(0);
          if (r < n) Basis<S, T>::store(a.V + (size_t)j * a.ldv + r, v);
          if (a.bj > 0) {
            // as k_bj_apply: the slice is a wave group of 64 / bj blocks
            const int g = lane / a.bj, m = min(a.bj, n - (r0 + s * SELL_C + g * a.bj));
            const T* Mg = a.minv + (size_t)(r0 / SELL_C + s) * a.bj * WAVE + lane;
            const T* xs = &win.x[own + s * SELL_C + g * a.bj];
            T acc = T(0);
            if (r < n) {
              for (int c = 0; c < m; ++c) acc += Mg[(size_t)c * WAVE] * xs[c];
              put_value(a.z + (size_t)r * WV, acc, tag);
            }
          } else {
            s_pre[i] = v;
          }
        }
      }
      if (a.bj > 0) {
        __syncthreads();
        lost = !exchange_window(wt, a.z, tag, 0, lost);
      }
      for (int k = 0; k < a.steps; ++k) {
        const SmallStep& ps = a.prog[k];
        word_t* const to = k & 1 ? a.z1 : a.z;
        const unsigned int ptag = tag * 256u + (unsigned int)k;
        const PolyCoef<T> cf = poly_coef<T>(ps.c, ps.has_y, ps.y_read, ps.d, ps.w);
        T* const Y = s_pre + 4 * ROWS;
        if (worker)
          for (int s = wid; s < RL; s += SMALL_NW) {
            const int i = s * SELL_C + lane, r = r0 + i;
            if (r0 / SELL_C + s >= a.A.nslices) break;
            const T t = in_lds ? window_row(win, win.x, s_vals + win.pair[s] * SELL_C, s, lane)
                               : window_row(win, win.x, vals + win.pair[s] * SELL_C, s, lane);
            const T xr = win.x[own + i], wr = cf.has_w ? s_pre[ps.w * ROWS + i] : T(0);
            T out = T(0);
            if (cf.has_y) {
              out = poly_y(cf, wr, xr, t, cf.y_read ? Y[i] : T(0));
              Y[i] = out;
            }
            if (cf.has_d) {
              out = poly_d(cf, wr, xr, t);
              s_pre[ps.d * ROWS + i] = out;
            }
            if (r < n) put_value(to + (size_t)r * WV, out, ptag);
          }
        __syncthreads();
        lost = !exchange_window(wt, to, ptag, a.near, lost);
      }
    }
    if (worker) {
      bool have_inv = j == 0;
      for (int s = wid; s < RL; s += SMALL_NW) {
        const int i = s * SELL_C + lane, r = r0 + i, sl = r0 / SELL_C + s;
        T y = T(0);
        if (sl < a.A.nslices && !lost) {
          if (PRE || win.chunks > 0) {
            y = in_lds ? window_row(win, win.x, s_vals + win.pair[s] * SELL_C, s, lane)
                       : window_row(win, off, win.x, vals + win.pair[s] * SELL_C, s, lane);
          } else {
            const int base = a.A.sptr[sl];
            const int K = (a.A.sptr[sl + 1] - base) / SELL_C;
            lost = !gather_row<T, S, 5, STAGED>(wt, a.A, a.x, tag - 1, nw, P, r, lane, base, K, have_inv, inv, y);
            if (!have_inv && !lost) {  // a slice without entries
              T n2 = T(0);
              lost = !collect_one<T, STAGED>(wt, nw, P, lane, tag - 1, n2);
              inv = T(1) / sqrt(n2);
              have_inv = true;
            }
            win.x[i] = r < n ? Basis<S, T>::round(s_w[i] * inv) : T(0);
          }
          if (r >= n) y = T(0);
          else if (!PRE) Basis<S, T>::store(a.V + (size_t)j * a.ldv + r, win.x[own + i]);
        }
        s_w[i] = y;
      }
    }
    __syncthreads();
    if (worker) {
      if (!PRE && wid == j % SMALL_NW) {
#pragma unroll
        for (int q = 0; q < SLOTS; ++q)
          if (q == j / SMALL_NW)
#pragma unroll
            for (int i = 0; i < RL; ++i) V[q][i] = r0 / SELL_C + i < a.A.nslices ? win.x[own + lane + WAVE * i] : T(0);
      }
      lost = !project(wt, h1w, tag, nq, sh.h1[j & 1], h) || lost;
    } else if (j > 0) {
      small_givens<T>(a.st, sh, j - 1, a.kmax, gin, stop_abs, check_stop, writer);
    }
    if (lost && lane == 0) sh.lost = j == 0 ? LOST_ABSENT : LOST_SILENT;
    __syncthreads();
    if ((sh.flags & F_DONE) || sh.lost) break;
    // w' = w - V h1, h2 = V^T w'
    if (worker)
      for (int i = wid * WAVE + lane; i < ROWS; i += SMALL_NW * WAVE) s_w[i] = small_updated(&s_part[0][0], s_w[i], ROWS, i);
    __syncthreads();
    if (worker) lost = !project(Wait{wt.lost, SILENT_LOOKS}, h2w, tag, nq, sh.h2, h);
    if (lost && lane == 0) sh.lost = LOST_SILENT;
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
        lost = !collect_one<T, STAGED>(Wait{wt.lost, SILENT_LOOKS}, nw, P, lane, tag, n2, leads_group(blockIdx.x));
        if (lane == 0) {
          sh.nrm2 = n2;
          if (lost) sh.lost = LOST_SILENT;
        }
        if (!lost) small_givens<T>(a.st, sh, j, a.kmax, gin, stop_abs, check_stop, writer);
      }
      break;
    }
  }
  __syncthreads();
  if (sh.lost && threadIdx.x == 0) give_up(a.st.hdr, sh.lost);
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
  word_t* const h2w = h1w + (size_t)SMALL_NW * (P + SMALL_GROUPS) * LINE * WV;
  word_t* const nw = h2w + (size_t)SMALL_NW * (P + SMALL_GROUPS) * LINE * WV;
  const unsigned int tag = a.tag + (unsigned int)j;
  const int nq = worker && wid <= j ? (j - wid) / SMALL_NW + 1 : 0;
  const VGlobal<T, S> V{a.V + r0, a.ldv, n - r0};
  const Wait wt{&a.st.hdr->lost, SILENT_LOOKS};
  T h[SLOTS];
  bool lost = false;
  // The Givens step of step jg by one block: sums and earlier rotations from the
  // state.  Beside the SpMV of the next step, whose blocks read none of it (an
  // iteration of three launches instead of four: 4096 rows 25.9 -> 19.5 us).
  auto givens = [&](int jg, unsigned int gtag) {
    const StateHdr* hd = a.st.hdr;
    for (int i = threadIdx.x; i <= jg; i += SMALL_NT) {
      sh.h1[jg & 1][i] = (T)a.st.h1_of(jg)[i];
      sh.h2[i] = (T)a.st.h2[i];
      if (i < jg) {
        sh.cs[i] = (T)a.st.cs[i];
        sh.sn[i] = (T)a.st.sn[i];
      }
    }
    if (!worker) {
      T n2 = T(0);
      lost = !collect_one_alone(wt, nw, P, lane, gtag, n2);
      if (lane == 0) {
        sh.nrm2 = n2;
        sh.g = (T)a.st.g[jg];
      }
    }
    __syncthreads();
    if (!worker)
      small_givens<T>(a.st, sh, jg, a.kmax, (T)hd->gamma_in, (T)hd->stop_abs, hd->stop_abs >= 0.0, true);
  };
  if constexpr (PH == SMALL_GIVENS) {
    givens(j, tag);
  } else if (PH == SMALL_SPMV && (int)blockIdx.x == P) {
    givens(j - 1, tag - 1);
  } else if constexpr (PH == SMALL_SPMV) {
    T inv = (T)a.st.hdr->inv_h;
    if (j > 0) {
      T n2 = T(0);
      lost = !collect_one_alone(wt, nw, P, lane, tag - 1, n2);
      inv = T(1) / sqrt(n2);
    }
    const XScaled<T, S> xs{a.wtmp, inv};
    for (int s = wid; s * SELL_C < rows; s += SMALL_NW + 1) {
      const int i = s * SELL_C + lane, r = r0 + i, sl = r0 / SELL_C + s;
      T y = T(0);
      if (sl < a.A.nslices) {
        y = sell_row<T, true>(a.A, xs, sl, r, lane);
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
    if (nq > 0) lost = !collect_alone<T, SLOTS>(wt, FIRST ? h1w : h2w, P, wid, lane, tag, h, sh.h2, nq);
    if (worker) small_partial<T, SLOTS>(part, V, h, rows, j, wid, lane);
    __syncthreads();
    if (blockIdx.x == 0)  // for the Givens step
      for (int i = threadIdx.x; i <= j; i += SMALL_NT) (FIRST ? a.st.h1_of(j) : a.st.h2)[i] = (double)sh.h2[i];
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
    a.st.hdr->lost = LOST_SILENT;
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
// a lane's registers.
constexpr int RLS[] = {2, 3, 4, 6, 8, 12, SMALL_MAX_RL};
template <typename T, typename S, int SLOTS, int I, bool PRE>
SmallKernel<T, S> cycle_of(int rl, bool staged) {
  if constexpr (I == sizeof(RLS) / sizeof(int)) {
    return nullptr;
  } else if constexpr (SLOTS * RLS[I] * (int)sizeof(T) > 128 * 4) {
    return nullptr;
  } else {
    if (rl != RLS[I]) return cycle_of<T, S, SLOTS, I + 1, PRE>(rl, staged);
    if constexpr (RLS[I] >= SMALL_STAGED_RL)
      if (staged) return k_small_cycle<T, S, SLOTS, RLS[I], true, PRE>;
    if constexpr (RLS[I] <= SMALL_STAGED_RL)
      if (!staged) return k_small_cycle<T, S, SLOTS, RLS[I], false, PRE>;
    return nullptr;
  }
}

int slots_of(int m) { return m <= 4 * SMALL_NW ? 4 : m <= 8 * SMALL_NW ? 8 : 16; }

}  // namespace

template <typename T, typename S, bool PRE>
SmallKernel<T, S> cycle_for(int sl, int rl, bool staged) {
  return sl == 4   ? cycle_of<T, S, 4, 0, PRE>(rl, staged)
         : sl == 8 ? cycle_of<T, S, 8, 0, PRE>(rl, staged)
                   : cycle_of<T, S, 16, 0, PRE>(rl, staged);
}

// How far apart the blocks are that exchange rows (blocks of `rows`), or more
// than any if a window does not fit.
template <typename T>
__global__ __launch_bounds__(SMALL_NT) void k_small_near(Csr A, int rows, int room, int* far) {
  __shared__ Window<T> win;
  const int s0 = blockIdx.x * (rows / SELL_C);
  window_build<SMALL_NT>(win, A, s0, min(rows / SELL_C, A.nslices - s0), win_chunks<T>(), dyn_lds<int>(), room);
  int d = win.chunks > 0 ? 1 : SMALL_MAX_P;
  for (int i = threadIdx.x; i < win.chunks; i += SMALL_NT) {
    const int c = min(max(win.chunk[i], 0), A.nslices - 1);
    d = max(d, abs(c / (rows / SELL_C) - (int)blockIdx.x));
  }
  atomicMax(far, d);
}

void small_near(const Csr& A, int sT, int rows, int blocks, bool pre, int* far, hipStream_t s) {
  const size_t lds = pre ? 0 : small_cycle_lds(rows, sT);
  const int room = pre ? Window<float>::PAIRS : (int)(lds / sizeof(int));
  if (sT == 8) hipLaunchKernelGGL(k_small_near<double>, dim3(blocks), dim3(SMALL_NT), lds, s, A, rows, room, far);
  else hipLaunchKernelGGL(k_small_near<float>, dim3(blocks), dim3(SMALL_NT), lds, s, A, rows, room, far);
}

template <typename T, typename S>
SmallKernel<T, S> small_kernel(SmallPhase ph, int m, int rows, int blocks) {
  const int sl = slots_of(m);
  if (ph == SMALL_CYCLE) return cycle_for<T, S, false>(sl, rows / WAVE, small_staged(blocks));
  if (ph == SMALL_CYCLE_PRE) return cycle_for<T, S, true>(sl, rows / WAVE, small_staged(blocks));
  return sl == 4 ? phase_of<T, S, 4>(ph) : sl == 8 ? phase_of<T, S, 8>(ph) : phase_of<T, S, 16>(ph);
}
template SmallKernel<float, float> small_kernel<float, float>(SmallPhase, int, int, int);
template SmallKernel<float, bf16_t> small_kernel<float, bf16_t>(SmallPhase, int, int, int);
template SmallKernel<double, double> small_kernel<double, double>(SmallPhase, int, int, int);

// An exchange of every block with every other grows with the lines a wave
// reads (1.1 us at 16 blocks, 1.6 at 64, 2.4 at 128, 5 at 256); in two stages
// it takes 1.8 us for all 256.  More rows per block cost registers and time in
// between.  So: at least 128 rows and at most 64 blocks as long as that takes
// no more than 256 rows a block (4096 rows, fp32: 64 blocks 4.8 ms a solve, 32
// 4.7, 16 4.9; 10000: 53 blocks 5.5, 40 5.4, 20 6.0), past that 256 rows or as
// many more as up to 256 blocks ask for (40000: 157 blocks 10.1, 105 10.1, 53
// 10.6; 160000: 209 blocks 18.2, 157 22.6; fp64 29241: 153 blocks 10.3, 115
// 10.2, 58 10.6; 62500: 245 blocks 17.4, 163 17.0, 123 18.4).
int small_rows(int64_t n, int m, int sT, int cus) {
  if (m > SMALL_MAX_M) return 0;
  const int64_t blocks = std::min(SMALL_MAX_P, cus);
  for (int rl : RLS) {
    if (slots_of(m) * rl * sT > 128 * 4) break;
    const int64_t rows = WAVE * rl, most = rl < SMALL_STAGED_RL ? std::min<int64_t>(blocks, WAVE) : blocks;
    if (n <= rows * most) return rl > SMALL_STAGED_RL && n <= rows * WAVE ? 0 : (int)rows;  // 0: fewer compute units
  }
  return 0;
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
  return (2 * SMALL_NW * WV + 1) * (size_t)(blocks + SMALL_GROUPS) * LINE;
}

void small_clear(unsigned long long* words, size_t count, hipStream_t s) {
  hipLaunchKernelGGL(k_small_clear, dim3((unsigned)std::min<size_t>(512, (count + 255) / 256)), dim3(256), 0, s, words,
                     count);
}

}  // namespace gir
