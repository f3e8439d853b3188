// Kernels of the LDS-resident inner cycle (see small.hpp).
#include <hip/hip_runtime.h>

#include <algorithm>

#include "small.hpp"
#include "spmv.hpp"

namespace gir {

namespace {

// a poll gives up after this many ticks of the 100 MHz clock (60 s: longer than
// other work on the GPU keeps a block waiting): every block then leaves the
// kernel and the solve reports an error
constexpr long long POLL_TICKS = 6000000000ll;

__device__ __forceinline__ float fma_t(float a, float b, float c) { return __builtin_fmaf(a, b, c); }
__device__ __forceinline__ double fma_t(double a, double b, double c) { return __builtin_fma(a, b, c); }

// ---------------------------------------------------------------------------
// sums over lanes without LDS: v + v of lane ^ M
// ---------------------------------------------------------------------------

typedef unsigned int uint2v __attribute__((ext_vector_type(2)));

// (a of lanes with bit M clear, with M set: b) and the same of lane ^ M; for
// M >= 16 one instruction swaps the halves of two registers
template <int M>
__device__ __forceinline__ uint2v lane_pair(unsigned int a, unsigned int b) {
  if constexpr (M == 32) {
    const auto r = __builtin_amdgcn_permlane32_swap(a, b, false, false);
    return uint2v{r[0], r[1]};
  } else if constexpr (M == 16) {
    const auto r = __builtin_amdgcn_permlane16_swap(a, b, false, false);
    return uint2v{r[0], r[1]};
  } else {
    const bool hi = threadIdx.x & M;
    const unsigned int keep = hi ? b : a, send = hi ? a : b;
    unsigned int got;
    if constexpr (M == 8) {
      got = __builtin_amdgcn_update_dpp(0, send, 0x128, 0xf, 0xf, false);  // row_ror:8
    } else if constexpr (M == 4) {
      got = __builtin_amdgcn_update_dpp(0, send, 0x104, 0xf, 0x5, false);   // row_shl:4, even banks
      got = __builtin_amdgcn_update_dpp(got, send, 0x114, 0xf, 0xa, false);  // row_shr:4, odd banks
    } else if constexpr (M == 2) {
      got = __builtin_amdgcn_update_dpp(0, send, 0x4e, 0xf, 0xf, false);  // quad_perm:[2,3,0,1]
    } else {
      got = __builtin_amdgcn_update_dpp(0, send, 0xb1, 0xf, 0xf, false);  // quad_perm:[1,0,3,2]
    }
    return uint2v{keep, got};
  }
}
// a + (a of lane ^ M) in lanes with bit M clear, b + (b of lane ^ M) where it is set
template <int M>
__device__ __forceinline__ float pair_sum(float a, float b) {
  const uint2v r = lane_pair<M>(__float_as_uint(a), __float_as_uint(b));
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
template <int M>
__device__ __forceinline__ double pair_sum(double a, double b) {
  const unsigned long long ua = (unsigned long long)__double_as_longlong(a);
  const unsigned long long ub = (unsigned long long)__double_as_longlong(b);
  const uint2v lo = lane_pair<M>((unsigned int)ua, (unsigned int)ub);
  const uint2v hi = lane_pair<M>((unsigned int)(ua >> 32), (unsigned int)(ub >> 32));
  return __longlong_as_double((long long)((unsigned long long)hi[0] << 32 | lo[0])) +
         __longlong_as_double((long long)((unsigned long long)hi[1] << 32 | lo[1]));
}
// sum over the lanes equal modulo W, in each of them
template <int W, typename T>
__device__ __forceinline__ T lane_sum(T v) {
  if constexpr (W <= 32) v = pair_sum<32>(v, v);
  if constexpr (W <= 16) v = pair_sum<16>(v, v);
  if constexpr (W <= 8) v = pair_sum<8>(v, v);
  if constexpr (W <= 4) v = pair_sum<4>(v, v);
  if constexpr (W <= 2) v = pair_sum<2>(v, v);
  if constexpr (W <= 1) v = pair_sum<1>(v, v);
  return v;
}
// The wave's sums of N = 4, 8 or 16 values at once: value l / (64 / N) in lane
// l.  Each step halves the values a lane still carries, so N values cost N - 1
// + log2(64 / N) additions where one after the other costs 6 N.
template <int N, int M, typename T>
__device__ __forceinline__ T lane_sums_step(T (&v)[N]) {
  T u[N / 2];
#pragma unroll
  for (int i = 0; i < N / 2; ++i) u[i] = pair_sum<M>(v[i], v[i + N / 2]);
  if constexpr (N == 2) {
    T x = u[0];
    if constexpr (M > 8) x = pair_sum<8>(x, x);
    if constexpr (M > 4) x = pair_sum<4>(x, x);
    if constexpr (M > 2) x = pair_sum<2>(x, x);
    if constexpr (M > 1) x = pair_sum<1>(x, x);
    return x;
  } else {
    return lane_sums_step<N / 2, M / 2>(u);
  }
}
template <int N, typename T>
__device__ __forceinline__ T lane_sums(T (&v)[N]) {
  static_assert(N == 4 || N == 8 || N == 16, "values");
  return lane_sums_step<N, 32>(v);
}

__device__ __forceinline__ float read_lane(float v, int l) {
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), l));
}
__device__ __forceinline__ double read_lane(double v, int l) {
  const unsigned long long u = (unsigned long long)__double_as_longlong(v);
  const unsigned int hi = __builtin_amdgcn_readlane((int)(u >> 32), l), lo = __builtin_amdgcn_readlane((int)u, l);
  return __longlong_as_double((long long)((unsigned long long)hi << 32 | lo));
}

// ---------------------------------------------------------------------------
// words: value and tag in 64 bits, written and read whole past the caches that
// the chip's dies do not share (relaxed, device scope); an fp64 value is two
// ---------------------------------------------------------------------------

typedef unsigned long long word_t;

__device__ __forceinline__ void put_word(word_t* p, unsigned int v, unsigned int tag) {
  __hip_atomic_store(p, (word_t)v << 32 | tag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ word_t get_word(const word_t* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void put_value(word_t* p, float v, unsigned int tag) { put_word(p, __float_as_uint(v), tag); }
__device__ __forceinline__ void put_value(word_t* p, double v, unsigned int tag) {
  const word_t u = (word_t)__double_as_longlong(v);
  put_word(p, (unsigned int)(u >> 32), tag);
  put_word(p + 1, (unsigned int)u, tag);
}
__device__ __forceinline__ float word_value(const word_t* w, float) { return __uint_as_float((unsigned int)(w[0] >> 32)); }
__device__ __forceinline__ double word_value(const word_t* w, double) {
  return __longlong_as_double((long long)((w[0] & 0xffffffff00000000ull) | w[1] >> 32));
}

// Repeats load() (which loads and says whether this lane's tags are right)
// until every lane's are; wave-uniform, false on time-out.
template <typename F>
__device__ __forceinline__ bool poll(F load) {
  long long t0 = 0;
  for (int tries = 0;; ++tries) {
    if (__all(load())) return true;
    if ((tries & 255) == 255) {
      const long long now = wall_clock64();
      if (t0 == 0) t0 = now;
      else if (now - t0 > POLL_TICKS) return false;
    }
  }
}

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

// ---------------------------------------------------------------------------
// state of a block
// ---------------------------------------------------------------------------

template <typename T>
struct SmallShared {
  T h1[2][SMALL_MAX_M];  // by the parity of j (the Givens step of j - 1 runs beside the first phase of j)
  T h2[SMALL_MAX_M];
  T col[SMALL_MAX_M + 2];
  T cs[SMALL_MAX_M], sn[SMALL_MAX_M];
  T red[SMALL_NW];
  T g;       // rotated right-hand side, entry j
  T nrm2;    // ||w''||^2 of the step the Givens wave works on
  int flags;
  int lost;  // a poll timed out
};

// Least-squares update of step j by one wave (see givens_tail): the column
// h1 + h2 rotated by the earlier rotations, the new one, the implicit
// residual, the stop tests.  Every block computes the same values; the one
// with `write` stores them.  cs, sn: LDS (cycle kernel) or staged from the state.
template <typename T>
__device__ __forceinline__ int small_givens(const State& st, SmallShared<T>& S, int j, int kmax, T gin, T stop_abs,
                                            bool check_stop, bool write) {
#pragma clang fp contract(off)
  const int lane = threadIdx.x & (WAVE - 1);
  const int ld = st.ld;
  double* Hc = st.Hbar + (size_t)j * ld;
  double* Rc = st.R + (size_t)j * ld;
  const T* h1 = S.h1[j & 1];
  T sq = T(0);
  for (int i = lane; i <= j; i += WAVE) {
    const T v = h1[i] + S.h2[i];
    S.col[i] = v;
    sq += v * v;
    if (write) {
      Hc[i] = (double)v;
      st.h1_of(j)[i] = (double)h1[i];
      st.h2[i] = (double)S.h2[i];
    }
  }
  sq = lane_sum<1>(sq);
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  int flags = 0;
  if (lane == 0) {
    StateHdr* hd = st.hdr;
    const T hn = sqrt(S.nrm2);
    const T colnorm = sqrt(sq + hn * hn);
    if (write) Hc[j + 1] = (double)hn;
    if (!isfinite(hn) || !isfinite(colnorm)) {
      flags = F_DONE | F_NUMERIC;
      if (write) hd->k = j;
    } else {
      T cur = S.col[0];
#pragma unroll 8
      for (int i = 0; i < j; ++i) {
        const T nxt = S.col[i + 1];
        const T c = S.cs[i], s = S.sn[i];
        S.col[i] = c * cur + s * nxt;
        cur = c * nxt - s * cur;
      }
      const T rho = hypot(cur, hn);
      const T c = rho == T(0) ? T(1) : cur / rho;
      const T s = rho == T(0) ? T(0) : hn / rho;
      S.col[j] = rho;
      S.col[j + 1] = T(0);
      S.cs[j] = c;
      S.sn[j] = s;
      const T gj = S.g;
      const T gj1 = -s * gj;
      S.g = gj1;
      const bool breakdown = hn <= (T)(100.0 * Unit<T>::roundoff) * colnorm;
      const bool stopped = check_stop && fabs(gj1) <= stop_abs;
      flags = (breakdown ? F_BREAKDOWN : 0) | (stopped ? F_STOPPED : 0);
      if (breakdown || stopped || j + 1 >= kmax) flags |= F_DONE;
      if (write) {
        st.cs[j] = (double)c;
        st.sn[j] = (double)s;
        st.g[j] = (double)(c * gj);
        st.g[j + 1] = (double)gj1;
        st.hist[j] = (double)(fabs(gj1) / gin);
        hd->k = j + 1;
        hd->implicit = (double)fabs(gj1);
        hd->inv_h = (double)(T(1) / hn);
      }
    }
    S.flags = flags;
    if (write) hd->flags = flags;
  }
  flags = __builtin_amdgcn_readfirstlane(flags);
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  if (write) {
    if (!(flags & F_NUMERIC))
      for (int i = lane; i <= j + 1; i += WAVE) Rc[i] = (double)S.col[i];
    for (int i = j + 2 + lane; i < ld; i += WAVE) {
      Hc[i] = 0.0;
      Rc[i] = 0.0;
    }
  }
  return flags;
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

// The rows of x a block's SpMV reads, in LDS: the set of 64-row chunks its
// slices' offsets reach, in ascending order, so that neighbouring chunks lie
// side by side and entry (slice, k) of lane l is at off[pair] + l.  Chunks
// outside the matrix are zeros (their values are zeros too).  Every row is
// then loaded once a block and iteration, all loads in flight together,
// instead of once per entry in dependent rounds (27-point rows: three rounds
// of nine).
constexpr int WIN_BITS = 8192;  // chunks between the first and the last
constexpr int WIN_PAIRS = 512;  // (slice, offset) pairs of a block
template <typename T>
constexpr int win_chunks() {
  return sizeof(T) == 8 ? 96 : 128;
}

template <typename T>
struct Window {
  T x[win_chunks<T>() * SELL_C];
  int off[WIN_PAIRS];
  int chunk[win_chunks<T>()];
  unsigned int bits[WIN_BITS / 32];
  int before[WIN_BITS / 32];  // set bits of the words before
  int pair[SMALL_MAX_RL + 1]; // first pair of each slice
  int first;                  // chunk of bit 0
  int chunks;                 // 0: the block does not fit, the rows are gathered one by one
  int own;                    // place of the block's own first chunk
};

// Built once per cycle by the whole block (all threads call it).
template <typename T, int RL>
__device__ __forceinline__ void window_build(Window<T>& W, const Csr& A, int r0) {
  const int s0 = r0 / SELL_C, ns = min(RL, A.nslices - s0);
  for (int i = threadIdx.x; i < WIN_BITS / 32; i += SMALL_NT) W.bits[i] = 0;
  if (threadIdx.x == 0) {
    W.first = s0;
    int p = 0;
    for (int s = 0; s <= RL; ++s) {
      W.pair[s] = p;
      if (s < ns) p += (A.sptr[s0 + s + 1] - A.sptr[s0 + s]) / SELL_C;
    }
    W.chunks = p <= WIN_PAIRS;
  }
  __syncthreads();
  if (!W.chunks) return;
  // offset of pair p of slice s
  auto offset = [&](int s, int p) { return A.scol[A.sptr[s0 + s] / SELL_C + p - W.pair[s]]; };
  for (int s = threadIdx.x; s < ns; s += SMALL_NT)
    if (W.pair[s + 1] > W.pair[s]) atomicMin(&W.first, s0 + s + (offset(s, W.pair[s]) >> 6));  // ascending offsets
  __syncthreads();
  bool fits = true;
  auto mark = [&](int c) {
    const int b = c - W.first;
    if (b < WIN_BITS) atomicOr(&W.bits[b >> 5], 1u << (b & 31));
    else fits = false;
  };
  for (int s = 0; s < ns; ++s) {
    if (threadIdx.x == 0) mark(s0 + s);
    for (int p = W.pair[s] + threadIdx.x; p < W.pair[s + 1]; p += SMALL_NT) {
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
    if (threadIdx.x == WAVE - 1) W.chunks = fits && incl <= win_chunks<T>() ? incl : 0;
  }
  __syncthreads();
  if (!W.chunks) return;
  auto place = [&](int c) {
    const int b = c - W.first;
    return W.before[b >> 5] + __popc(W.bits[b >> 5] & ((1u << (b & 31)) - 1));
  };
  for (int i = threadIdx.x; i < WIN_BITS / 32; i += SMALL_NT)
    for (unsigned int m = W.bits[i], k = 0; m; m &= m - 1, ++k) W.chunk[W.before[i] + k] = W.first + 32 * i + __ffs(m) - 1;
  for (int s = 0; s < ns; ++s)
    for (int p = W.pair[s] + threadIdx.x; p < W.pair[s + 1]; p += SMALL_NT) {
      const int o = offset(s, p);
      W.off[p] = place(s0 + s + (o >> 6)) * SELL_C + (o & 63);
    }
  if (threadIdx.x == 0) W.own = place(s0);
  __syncthreads();
}

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

// Row sums of slice s from the window, in the order of sell_row; vals: the
// slice's values (LDS or memory), 64 per entry.
template <typename T>
__device__ __forceinline__ T window_row(const Window<T>& W, const T* vals, int s, int lane) {
#pragma clang fp contract(off)
  constexpr int U = 9;
  const int p0 = W.pair[s], K = W.pair[s + 1] - p0;
  T sum = T(0);
  for (int k0 = 0; k0 < K; k0 += U) {
    T vv[U], xv[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int k = k0 + u < K ? k0 + u : K - 1;
      vv[u] = vals[SELL_C * k + lane];
      xv[u] = W.x[W.off[p0 + k] + lane];
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const T p = vv[u] * xv[u];
      if (k0 + u < K) sum = sum + p;
    }
  }
  return sum;
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
  window_build<T, RL>(win, a.A, r0);
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
            y = in_lds ? window_row(win, s_vals + win.pair[s] * SELL_C, s, lane)
                       : window_row(win, vals + win.pair[s] * SELL_C, s, lane);
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
