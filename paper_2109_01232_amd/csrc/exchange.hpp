// What the cycle kernels share (small.hip, mid.hip): sums over lanes without
// LDS, the tagged words by which blocks exchange values inside a kernel, and
// the Givens step of one wave.
#pragma once

#include "small.hpp"

namespace gir {

// A wait gives up after this many looks, of 0.5 to 1 us each.  Until every block
// has taken part in one exchange some may not be on the GPU at all: other work
// holds their compute units, or another process's cycle kernel that waits for
// its own blocks.  That wait is short (0.1 s), and the host then has the cycle
// made by kernels whose blocks need not run together.  A block that was there
// and falls silent for a minute is an error.  (Looks, not the clock: read
// as well, it cost the small cycles 3-5 %.)
constexpr int ARRIVE_LOOKS = 1 << 17, SILENT_LOOKS = 1 << 26;

// What a wave needs to wait: the word by which a block that has given up tells
// all others, and how many looks it takes.
struct Wait {
  const int32_t* lost;
  int looks;
};

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
// until every lane's are; wave-uniform, false on giving up.
template <typename F>
__device__ __forceinline__ bool poll(const Wait& wt, F load) {
  for (int looks = 1;; ++looks) {
    if (__all(load())) return true;
    if ((looks & 255) == 0 &&
        (looks >= wt.looks || __builtin_amdgcn_readfirstlane(
                                  __hip_atomic_load(wt.lost, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))))
      return false;
  }
}

// By one thread of a block that has given up, at the kernel's end.  A cycle that
// cannot be made again is over.
__device__ __forceinline__ void give_up(StateHdr* hd, int32_t why) {
  const int32_t first = __hip_atomic_load(&hd->lost, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  if (first == 0) (void)__hip_atomic_fetch_or(&hd->lost, why, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  if ((first ? first : why) & LOST_SILENT) hd->flags = F_DONE | F_NUMERIC;
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
  T red[8];  // by wave
  T g;       // rotated right-hand side, entry j
  T nrm2;    // ||w''||^2 of the step the Givens wave works on
  int flags;
  int lost;  // LOST_*: a wait of this block was given up
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

}  // namespace gir
