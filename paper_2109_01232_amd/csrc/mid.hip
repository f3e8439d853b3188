// Inner cycles of systems whose Krylov basis fits the registers of the GPU's
// compute units in part: one cooperative launch of one block per compute unit.
//
// The chip's 256 compute units have 128 MB of vector registers, half of the
// basis of GMRES(50) on 10^6 rows.  A block keeps its rows of the first
// columns there for the whole cycle (64 MB: half of the registers) and reads
// only the later ones from memory (10^6 rows in fp32: 16 resident columns, on
// average 12 instead of 25 are read per sweep); the work vectors w, w', w''
// and the rows of x the SpMV gathers never leave LDS.
//
// Waves split the columns (wave w: c = w + 8 q), a lane has 16 bytes of
// consecutive rows per step and column.  The loads of two steps are in flight,
// across the barriers and the exchanges too.  The reductions are exchanges
// inside the kernel (tagged words, see exchange.hpp) in two stages of 16
// blocks: 1.8 us for all 256, where every block reading every other's line
// takes 5 us.
//
// Bound by memory where most columns are read (27-point 128^3 in fp32: 705 MB
// an iteration at 4.6 TB/s), by the vector units and LDS barriers where most are
// resident; with few columns to read the general kernels are faster (see
// mid_min_steps).  Whole solves to 1e-12, GMRES(50), against one kernel per
// operation: fp32 5-point 513^2 88.5 -> 41.8 ms, 600^2 98.8 -> 53.2, 27-point
// 80^3 15.8 -> 10.3, 101^3 24.8 -> 18.7, 128^3 50.3 -> 42.9; bf16 basis 80^3 17.3
// -> 11.9, 128^3 42.5 -> 37.2; fp64 7-point 52^3 28.6 -> 16.1, 27-point 101^3
// 50.7 -> 40.0.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

#include "exchange.hpp"
#include "spmv.hpp"
#include "window.hpp"

namespace gir {

namespace {

constexpr int MID_P = MID_BLOCKS;   // logical: 32 neighbours per die
constexpr int MID_GROUP = 16;       // blocks of an exchange's first stage
constexpr int MID_NW = 8;
constexpr int MID_NT = MID_NW * WAVE;
static_assert(MID_NT == MID_THREADS, "threads");
static_assert(sizeof(SmallShared<float>::red) >= MID_NW * sizeof(float), "one sum per wave");
constexpr int MID_SLOTS = 8;        // columns of a wave: restart <= 64
constexpr int LINE = 16;            // words of a line: 8 values of fp64, 128 bytes
// first looks, in 64 clocks after the own store: the leaders of a stage, and
// the blocks that wait for both stages
constexpr int WAIT_ONE = 8, WAIT_TWO = 24;

// words of one exchange of column sums: [wave][block], then [wave][group]
constexpr size_t MID_SUMS = (size_t)MID_NW * (MID_P + MID_P / MID_GROUP) * LINE;
constexpr size_t MID_NORM = (size_t)(MID_P + MID_P / MID_GROUP) * LINE;
static_assert(SMALL_WORDS_AT + (2 * MID_SUMS + MID_NORM) * sizeof(word_t) <= (size_t)MAX_BLOCKS * PART_COLS * 8,
              "the words fit the workspace's partials");

// The vector other blocks gather from: written and read past the caches that
// the chip's dies do not share.
__device__ __forceinline__ float load_shared(const float* p) {
  return __uint_as_float(__hip_atomic_load((const unsigned int*)p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
}
__device__ __forceinline__ double load_shared(const double* p) {
  return __longlong_as_double((long long)__hip_atomic_load((const word_t*)p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
}
__device__ __forceinline__ void store_shared(float* p, float v) {
  __hip_atomic_store((unsigned int*)p, __float_as_uint(v), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void store_shared(double* p, double v) {
  __hip_atomic_store((word_t*)p, (word_t)__double_as_longlong(v), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// What a lane has of a column's step: 16 bytes of consecutive rows as stored.
template <typename S>
struct V4 {
  static constexpr int RPL = 16 / sizeof(S);  // rows
  unsigned int u[4];
  __device__ __forceinline__ void keep(int k) {  // the first k rows, 0 after them
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      if constexpr (sizeof(S) == 2) u[w] = k > 2 * w + 1 ? u[w] : k > 2 * w ? u[w] & 0xffffu : 0u;
      else u[w] = w / (int)(sizeof(S) / 4) < k ? u[w] : 0u;
    }
  }
  __device__ __forceinline__ float get(int i, float) const {
    if constexpr (sizeof(S) == 2) return __uint_as_float((i & 1) ? (u[i / 2] & 0xffff0000u) : (u[i / 2] << 16));
    else return __uint_as_float(u[i]);
  }
  __device__ __forceinline__ double get(int i, double) const {
    return __longlong_as_double((long long)((word_t)u[2 * i + 1] << 32 | u[2 * i]));
  }
  __device__ __forceinline__ void set(const float* x) {  // values already rounded to S
#pragma unroll
    for (int w = 0; w < 4; ++w)
      if constexpr (sizeof(S) == 2) u[w] = __float_as_uint(x[2 * w]) >> 16 | (__float_as_uint(x[2 * w + 1]) & 0xffff0000u);
      else u[w] = __float_as_uint(x[w]);
  }
  __device__ __forceinline__ void set(const double* x) {
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const word_t b = (word_t)__double_as_longlong(x[i]);
      u[2 * i] = (unsigned int)b, u[2 * i + 1] = (unsigned int)(b >> 32);
    }
  }
};

// Barrier for LDS alone: loads from memory stay in flight across it.
__device__ __forceinline__ void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// Sum over the 16 lines from `lines` of their first nq values: lane l has
// value l % 8.  False on time-out.
template <typename T>
__device__ __forceinline__ bool take(const Wait& wt, const word_t* lines, int nq, unsigned int tag, int lane, T& out) {
  constexpr int WV = small_words_per_value<T>();
  const int q = lane & 7;
  const word_t* p = lines + (lane >> 3) * LINE + WV * q;
  word_t w[2][WV];
  const bool ok = poll(wt, [&] {
#pragma unroll
    for (int g = 0; g < 2; ++g)
#pragma unroll
      for (int h = 0; h < WV; ++h) w[g][h] = get_word(p + 8 * LINE * g + h);
    bool right = true;
#pragma unroll
    for (int g = 0; g < 2; ++g)
#pragma unroll
      for (int h = 0; h < WV; ++h) right = right && ((unsigned int)w[g][h] == tag || q >= nq);
    return right;
  });
  if (!ok) return false;
  const T s = word_value(w[0], T(0)) + word_value(w[1], T(0));
  out = lane_sum<8>(q < nq ? s : T(0));
  return true;
}

// Second half of an exchange whose blocks have written their line in `first`
// ([256] lines): block 0 of every 16 sums its group's into `second` ([16]),
// everyone sums those.
template <typename T>
__device__ __forceinline__ bool combine(const Wait& wt, word_t* first, word_t* second, int lb, bool leads, int nq,
                                        unsigned int tag, int lane, T& out) {
  constexpr int WV = small_words_per_value<T>();
  if (leads) {
    __builtin_amdgcn_s_sleep(WAIT_ONE);
    T s;
    if (!take(wt, first + (size_t)lb * LINE, nq, tag, lane, s)) return false;
    if (lane < nq) put_value(second + (size_t)(lb / MID_GROUP) * LINE + WV * lane, s, tag);
    __builtin_amdgcn_s_sleep(WAIT_ONE);
  } else {
    __builtin_amdgcn_s_sleep(WAIT_TWO);
  }
  return take(wt, second, nq, tag, lane, out);
}

// Slices of a block, and the map of its window of x (see window.hpp)
constexpr int MID_SLICES = 128, MID_PAIRS = 27 * MID_SLICES, MID_CHUNKS = 448;
typedef WindowMap<MID_CHUNKS, MID_PAIRS, MID_SLICES> MidWindow;

// QR columns of a wave stay in registers, indexed by step (a wave-uniform
// register index: unrolled, the sweeps' code outgrew the instruction cache
// and their registers spilled; vectors of 32 because the compiler keeps ones
// of 8 and 10 in scratch memory, 3x slower).  At most STEPS steps per block.
template <typename T, typename S, int QR, int STEPS, int U>
__global__ __launch_bounds__(MID_NT) void k_mid_cycle(SmallArgs<T, S> a) {
  constexpr int WV = small_words_per_value<T>();
  constexpr int NS = MID_SLOTS - QR;  // columns of a wave read from memory at most
  constexpr int NB = NS > 0 ? NS : 1;
  constexpr int RPL = V4<S>::RPL, STEP = WAVE * RPL;
  static_assert(QR * STEPS <= 32, "registers");
  typedef unsigned int res_t __attribute__((ext_vector_type(32)));
  __shared__ SmallShared<T> sh;
  __shared__ MidWindow win;
  __shared__ __align__(16) T s_y[STEPS * STEP];        // the working vector's rows
  __shared__ int s_next;                               // next slice of the SpMV
  // the window of x, and after the SpMV the waves' parts of V h, [2][wave][STEP]
  T* const s_x = dyn_lds<T>();
  T* const s_part = s_x;
  const int lane = threadIdx.x & (WAVE - 1);
  const int wid = __builtin_amdgcn_readfirstlane(threadIdx.x / WAVE);
  const int lb = (int)(blockIdx.x % 8) * (MID_P / 8) + (int)blockIdx.x / 8;
  const bool leads = lb % MID_GROUP == 0;
  const int sl0 = (int)((long)a.A.nslices * lb / MID_P), sl1 = (int)((long)a.A.nslices * (lb + 1) / MID_P);
  const int n = a.A.n, r0 = sl0 * SELL_C;
  const int rows = min(sl1 * SELL_C, n) - r0;  // > 0: at least 256 slices
  const int steps = (rows + STEP - 1) / STEP;
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
    s_next = 0;
  }
  for (int i = threadIdx.x; i < STEPS * STEP; i += MID_NT) s_y[i] = i < rows ? a.wtmp[r0 + i] : T(0);
  window_build<MID_NT>(win, a.A, sl0, sl1 - sl0, a.rows);
  const T* const own = s_x + win.own * SELL_C;  // the block's rows of x
  word_t* const h1w = a.words;
  word_t* const h2w = h1w + MID_SUMS;
  word_t* const nw = h2w + MID_SUMS;
  const bool writer = lb == 0;
  res_t res[4];  // word k of the lane's 16 bytes of step s, column wid + 8 q: [k][QR s + q]
#pragma unroll
  for (int k = 0; k < 4; ++k) res[k] = 0;
  // 16 bytes per lane of step s of the wave's columns in memory; 0 from column
  // `upto` on and past the last step, by an offset past the buffer's end, so
  // that the number of loads in flight is the same on every path
  const unsigned int col_bytes = (unsigned int)a.ldv * sizeof(S);
  const auto rsrc = __builtin_amdgcn_make_buffer_rsrc((void*)(a.V + r0), 0, (int)((MID_MAX_M + 1) * col_bytes), 0x00020000);
  auto load = [&](V4<S> (&v)[NB], int s, int upto) {
#pragma unroll
    for (int q = 0; q < NS; ++q) {
      const int c = wid + MID_NW * (QR + q);
      const unsigned int at = c < upto && s < steps ? c * col_bytes + s * (int)(STEP * sizeof(S)) : 0x80000000u;
      const auto w = __builtin_amdgcn_raw_buffer_load_b128(rsrc, at + 16 * lane, 0, 0);
#pragma unroll
      for (int k = 0; k < 4; ++k) v[q].u[k] = w[k];
    }
  };
  // One step of a pass over V.  MODE 0: acc = V^T y.  1: y -= V h and
  // acc = V^T y.  2: y -= V h, the squares summed into acc[0].  Columns not
  // formed yet are zeros: no branches, the vector units are what bounds the
  // steps whose columns are resident
  auto step = [&](auto mode, int s, V4<S> (&vs)[NB], const T (&h)[MID_SLOTS], T (&acc)[MID_SLOTS]) {
    constexpr int MODE = decltype(mode)::value;
    const int row0 = s * STEP + RPL * lane;
    if ((s + 1) * STEP > rows)
#pragma unroll
      for (int q = 0; q < NS; ++q) vs[q].keep(rows - row0);
    V4<S> vr[QR];
#pragma unroll
    for (int q = 0; q < QR; ++q)
#pragma unroll
      for (int k = 0; k < 4; ++k) vr[q].u[k] = res[k][QR * s + q];
    if constexpr (MODE != 0) {
      T p[RPL];
#pragma unroll
      for (int i = 0; i < RPL; ++i) {
        p[i] = T(0);
#pragma unroll
        for (int q = 0; q < QR; ++q) p[i] = fma_t(h[q], vr[q].get(i, T(0)), p[i]);
      }
#pragma unroll
      for (int q = 0; q < NS; ++q)
#pragma unroll
        for (int i = 0; i < RPL; ++i) p[i] = fma_t(h[QR + q], vs[q].get(i, T(0)), p[i]);
      T* part = s_part + (s & 1) * (MID_NW * STEP);
      T* out = part + wid * STEP + RPL * lane;
#pragma unroll
      for (int i = 0; i < RPL; ++i) out[i] = p[i];
      lds_barrier();
      for (int at = threadIdx.x; at < STEP; at += MID_NT) {
        const int row = s * STEP + at;
        T v[MID_NW + 1];
#pragma unroll
        for (int w = 0; w < MID_NW; ++w) v[w] = part[w * STEP + at];
        v[MID_NW] = s_y[row];
        // all reads are out before the first is used
        asm volatile("" : "+v"(v[0]), "+v"(v[1]), "+v"(v[2]), "+v"(v[3]), "+v"(v[4]), "+v"(v[5]), "+v"(v[6]), "+v"(v[7]), "+v"(v[8]));
        T t = v[0];
#pragma unroll
        for (int w = 1; w < MID_NW; ++w) t += v[w];
        const T y = row < rows ? v[MID_NW] - t : T(0);
        s_y[row] = y;
        if constexpr (MODE == 2) acc[0] = fma_t(y, y, acc[0]);
      }
      if constexpr (MODE == 1) lds_barrier();
    }
    if constexpr (MODE != 2) {
      T y[RPL];
#pragma unroll
      for (int i = 0; i < RPL; ++i) y[i] = s_y[row0 + i];
#pragma unroll
      for (int q = 0; q < QR; ++q)
#pragma unroll
        for (int i = 0; i < RPL; ++i) acc[q] = fma_t(vr[q].get(i, T(0)), y[i], acc[q]);
#pragma unroll
      for (int q = 0; q < NS; ++q)
#pragma unroll
        for (int i = 0; i < RPL; ++i) acc[QR + q] = fma_t(vs[q].get(i, T(0)), y[i], acc[QR + q]);
    }
  };
  // A pass: two steps' loads are in flight, the first of the next pass's too
  V4<S> va[NB], vb[NB];
  auto sweep = [&](auto mode, int upto, const T (&h)[MID_SLOTS], T (&acc)[MID_SLOTS]) {
#pragma unroll
    for (int q = 0; q < MID_SLOTS; ++q) acc[q] = T(0);
#pragma unroll 1
    for (int s = 0; s < steps; s += 2) {
      load(vb, s + 1, upto);
      step(mode, s, va, h, acc);
      load(va, s + 2 < steps ? s + 2 : 0, upto);
      if (s + 1 < steps) step(mode, s + 1, vb, h, acc);
    }
  };
  // the wave's column sums over all blocks: into h (every lane) and all[]
  auto exchange = [&](int looks, word_t* words, unsigned int tag, int nq, T (&acc)[MID_SLOTS], T* all,
                      T (&h)[MID_SLOTS]) {
    word_t* first = words + (size_t)wid * MID_P * LINE;
    word_t* second = words + (size_t)MID_NW * MID_P * LINE + (size_t)wid * (MID_P / MID_GROUP) * LINE;
    const T v = lane_sums<MID_SLOTS>(acc);
    if (lane % (WAVE / MID_SLOTS) == 0 && lane / (WAVE / MID_SLOTS) < nq)
      put_value(first + (size_t)lb * LINE + WV * (lane / (WAVE / MID_SLOTS)), v, tag);
    T s = T(0);
    const bool ok = nq == 0 || combine(Wait{&a.st.hdr->lost, looks}, first, second, lb, leads, nq, tag, lane, s);
    if (lane < nq) all[wid + MID_NW * lane] = s;
#pragma unroll
    for (int q = 0; q < MID_SLOTS; ++q) h[q] = q < nq ? read_lane(s, q) : T(0);
    return ok;
  };
  load(va, 0, 0);
  __syncthreads();
  int j = 0;
  for (;; ++j) {
    const unsigned int tag = a.tag + (unsigned int)j;
    const int nq = wid <= j ? (j - wid) / MID_NW + 1 : 0;
    T h[MID_SLOTS], acc[MID_SLOTS];
    bool lost = false;
    // x = v_j = round(w'' / ||w''||) into the window, then w = A x slice by
    // slice; the last wave makes the Givens step of j - 1 first
    constexpr int LOADS = 8;
    for (int c0 = wid; c0 < win.chunks; c0 += LOADS * MID_NW) {
      T x[LOADS];
#pragma unroll
      for (int u = 0; u < LOADS; ++u) {
        const int c = c0 + MID_NW * u;
        const int r = win.chunk[c < win.chunks ? c : c0] * SELL_C + lane;
        x[u] = load_shared(a.wtmp + (r >= 0 && r < n ? r : r0));
        if (r < 0 || r >= n) x[u] = T(0);
      }
#pragma unroll
      for (int u = 0; u < LOADS; ++u)
        if (c0 + MID_NW * u < win.chunks) s_x[(c0 + MID_NW * u) * SELL_C + lane] = Basis<S, T>::round(x[u] * inv);
    }
    lds_barrier();
    if (j > 0 && wid == MID_NW - 1) small_givens<T>(a.st, sh, j - 1, a.kmax, gin, stop_abs, check_stop, writer);
    const T* const vals = (const T*)a.A.svals + a.A.sptr[sl0];
    for (;;) {
      int s = 0;
      if (lane == 0) s = atomicAdd(&s_next, 1);
      s = __builtin_amdgcn_readfirstlane(s);
      if (s >= sl1 - sl0) break;
      const int i = s * SELL_C + lane, r = r0 + i;
      const T y = window_row<T, U>(win, s_x, vals + win.pair[s] * SELL_C, s, lane);
      if (r < n) Basis<S, T>::store(a.V + (size_t)j * a.ldv + r, own[i]);
      s_y[i] = r < n ? y : T(0);
    }
    // column j is read back by other waves of the block
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if ((sh.flags & F_DONE) | sh.lost) break;  // one test: with a branch for each the compiler spills res
    if (threadIdx.x == 0) s_next = 0;
#pragma unroll
    for (int q = 0; q < MID_SLOTS; ++q) h[q] = T(0);
    // the newest column: its wave takes it from LDS, all of it into registers
    // or its first step (requested before it was there)
    if (wid == j % MID_NW) {
      auto take_newest = [&](int s) {
        V4<S> v;
        T x[RPL];
        const int row0 = s * STEP + RPL * lane;
#pragma unroll
        for (int i = 0; i < RPL; ++i) x[i] = row0 + i < rows ? own[row0 + i] : T(0);
        v.set(x);
        return v;
      };
#pragma unroll
      for (int q = 0; q < QR; ++q)
        if (q == j / MID_NW)
#pragma unroll 1
          for (int s = 0; s < steps; ++s) {
            const V4<S> v = take_newest(s);
#pragma unroll
            for (int k = 0; k < 4; ++k) res[k][QR * s + q] = v.u[k];
          }
#pragma unroll
      for (int q = 0; q < NS; ++q)
        if (QR + q == j / MID_NW) va[q] = take_newest(0);
    }
    sweep(std::integral_constant<int, 0>{}, j + 1, h, acc);
    lds_barrier();  // the window gives way to the parts
    lost = !exchange(j == 0 ? ARRIVE_LOOKS : SILENT_LOOKS, h1w, tag, nq, acc, sh.h1[j & 1], h);
    sweep(std::integral_constant<int, 1>{}, j + 1, h, acc);
    // a wave that has given up stays silent: no block passes this exchange then
    const bool absent = lost && j == 0;
    lost = !exchange(SILENT_LOOKS, h2w, tag, lost ? 0 : nq, acc, sh.h2, h) || lost;
    sweep(std::integral_constant<int, 2>{}, j + 1, h, acc);
    const T nrm = lane_sum<1>(acc[0]);
    if (lane == 0) {
      sh.red[wid] = nrm;
      if (lost) sh.lost = absent ? LOST_ABSENT : LOST_SILENT;
    }
    lds_barrier();
    if (sh.lost) break;  // wtmp stays as it was: the cycle may be made again
    for (int i = threadIdx.x; i < rows; i += MID_NT) store_shared(a.wtmp + r0 + i, s_y[i]);
    // the rows are out before the norm says so
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (threadIdx.x == 0) {
      T t = sh.red[0];
#pragma unroll
      for (int w = 1; w < MID_NW; ++w) t += sh.red[w];
      put_value(nw + (size_t)lb * LINE, t, tag);
    }
    T n2 = T(0);
    lost = !combine(Wait{&a.st.hdr->lost, SILENT_LOOKS}, nw, nw + (size_t)MID_P * LINE, lb, leads && wid == 0, 1, tag, lane, n2);
    n2 = read_lane(n2, 0);
    asm volatile("" ::: "memory");  // the gathers below stay behind the exchange
    inv = T(1) / sqrt(n2);
    if (lane == 0) {
      if (wid == MID_NW - 1) sh.nrm2 = n2;
      if (lost) sh.lost = LOST_SILENT;
    }
    if (j + 1 >= a.kmax) {
      if (wid == MID_NW - 1 && !lost) small_givens<T>(a.st, sh, j, a.kmax, gin, stop_abs, check_stop, writer);
      break;
    }
  }
  __syncthreads();
  if (sh.lost && threadIdx.x == 0) give_up(a.st.hdr, sh.lost);
}

// Tells in `wide` if a block's window needs more than `most` chunks.
__global__ __launch_bounds__(MID_NT) void k_mid_fits(Csr A, int most, int* wide) {
  __shared__ MidWindow win;
  const int lb = blockIdx.x;
  const int sl0 = (int)((long)A.nslices * lb / MID_P), sl1 = (int)((long)A.nslices * (lb + 1) / MID_P);
  window_build<MID_NT>(win, A, sl0, sl1 - sl0, most);
  if (threadIdx.x == 0 && win.chunks == 0) *wide = 1;
}

}  // namespace

void mid_fits(const Csr& A, int chunks, int* wide, hipStream_t s) {
  hipLaunchKernelGGL(k_mid_fits, dim3(MID_P), dim3(MID_NT), 0, s, A, chunks, wide);
}

size_t mid_words() { return 2 * MID_SUMS + MID_NORM; }

// 120 or 128 registers of a lane hold basis columns: 4 QR STEPS, so the fewer
// steps a block has the more columns stay.  A step has 4 slices of fp32, 8 of
// bf16, 2 of fp64.  U: entries of a row loaded together (27-point 128^3 44.5
// -> 43.2 ms with 14 instead of 9, bf16 basis 39.5 -> 37.8; 27 spills registers;
// both in one kernel, chosen per slice, 7-point 90^3 43.9 -> 52.0; fp64 equal).
template <typename T, typename S, int U>
static MidKernel<T, S> mid_of(int64_t nslices) {
  constexpr int PER = V4<S>::RPL;
  const int64_t s = (nslices + MID_P - 1) / MID_P;  // slices of a block
  // the window has what the rows of y leave of the LDS, at least the parts' place
  const auto of = [](SmallKernel<T, S> k, int steps) {
    const size_t used = sizeof(SmallShared<T>) + sizeof(MidWindow) + (size_t)steps * WAVE * PER * sizeof(T) + 256;
    const size_t part = 2 * MID_NW * WAVE * PER * sizeof(T), chunk = SELL_C * sizeof(T);
    const int chunks = (int)std::min((SMALL_LDS - used) / chunk, (size_t)MID_CHUNKS);
    return MidKernel<T, S>{k, chunks, (unsigned)std::max(part, chunks * chunk)};
  };
  if (s > MID_SLICES || s > 32 * PER) return {nullptr, 0, 0};
  if constexpr (PER > 2)  // fp64: the smallest system has nine slices a block
    if (s <= 4 * PER) return of(k_mid_cycle<T, S, 8, 4, U>, 4);
  if (s <= 5 * PER) return of(k_mid_cycle<T, S, 6, 5, U>, 5);
  if (s <= 6 * PER) return of(k_mid_cycle<T, S, 5, 6, U>, 6);
  if (s <= 8 * PER) return of(k_mid_cycle<T, S, 4, 8, U>, 8);
  if (s <= 10 * PER) return of(k_mid_cycle<T, S, 3, 10, U>, 10);
  if (s <= 16 * PER) return of(k_mid_cycle<T, S, 2, 16, U>, 16);
  if constexpr (PER < 8) return of(k_mid_cycle<T, S, 1, 32, U>, 32);
  return {nullptr, 0, 0};
}
template <>
MidKernel<float, float> mid_kernel<float, float>(int64_t nslices, bool wide) {
  return wide ? mid_of<float, float, 14>(nslices) : mid_of<float, float, 9>(nslices);
}
template <>
MidKernel<float, bf16_t> mid_kernel<float, bf16_t>(int64_t nslices, bool wide) {
  return wide ? mid_of<float, bf16_t, 14>(nslices) : mid_of<float, bf16_t, 9>(nslices);
}
template <>
MidKernel<double, double> mid_kernel<double, double>(int64_t nslices, bool) {
  return mid_of<double, double, 9>(nslices);
}

}  // namespace gir
