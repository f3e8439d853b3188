// Inner cycles of systems whose Krylov basis fits the registers of the GPU's
// compute units (declarations; kernels in small.hip).
//
// A cycle of such a system is bound by latency: as separate kernels an
// iteration is five dependent launches of a few microseconds each whatever the
// rows.  Here the rows are split over at most one block per compute unit, the
// waves of a block keep its rows of V in registers, and one cooperative launch
// runs the whole cycle.  The three reductions of an iteration (h1, h2, ||w''||^2)
// are exchanges between the blocks: a block stores its partial sums as 64-bit
// words of value and tag, and every block adds all of them in the same order,
// past 64 blocks in two stages.  A word is complete when its tag is the
// iteration's, so an exchange is one store and one load in flight, without
// flags, fences or a second trip.
//
// The same phases can be launched one by one (profiling, the allocation-free
// entry point, a cooperative launch that is refused or whose blocks are not all
// on the GPU): the same partition, order of operations and words, so the same bits.
#pragma once

#include "device.hpp"

namespace gir {

// Waves of a block: seven share the columns (wave w has c = w + 7 q), one makes
// the Givens steps; with eight a lane has 256 registers (with a ninth 168).
constexpr int SMALL_NW = 7;
constexpr int SMALL_NT = (SMALL_NW + 1) * WAVE;
constexpr int SMALL_MAX_M = 16 * SMALL_NW;           // restart lengths of this path
constexpr int SMALL_MAX_RL = 16;                     // rows per lane (64 RL rows per block)
constexpr size_t SMALL_LDS = 160 << 10;              // of a compute unit
constexpr int SMALL_MAX_P = 256;                     // blocks
constexpr int SMALL_GROUPS = 16;                     // of up to 16 blocks: an exchange's second stage
constexpr size_t SMALL_WORDS_AT = (size_t)MAX_BLOCKS * 8;  // the words follow the partials of the cycle's set-up

enum SmallPhase { SMALL_SPMV = 0, SMALL_GIVENS, SMALL_UPDATE, SMALL_NORM, SMALL_CYCLE, SMALL_CYCLE_PRE };

// One SpMV step of a polynomial preconditioner's product form, in the inner
// precision: vectors 0 (v_j) to 3, 4 none.
template <typename T>
struct PolyCoef {
  T ay, aw, ax, at;  // y = ay*y + aw*W + ax*X + at*(A X)
  T bw, bx, bt;      // d = bw*W + bx*X + bt*(A X)
  int has_y, y_read, has_d, has_w;
};
template <typename T>
__device__ __forceinline__ T poly_y(const PolyCoef<T>& cf, T wr, T xr, T t, T y) {
  T yv = cf.aw * wr + cf.ax * xr + cf.at * t;
  if (cf.y_read) yv += cf.ay * y;
  return yv;
}
template <typename T>
__device__ __forceinline__ T poly_d(const PolyCoef<T>& cf, T wr, T xr, T t) {
  return cf.bw * wr + cf.bx * xr + cf.bt * t;
}
struct SmallStep {
  double c[7];  // ay, aw, ax, at, bw, bx, bt
  int w, d, has_y, y_read;
};
template <typename T>
__host__ __device__ inline PolyCoef<T> poly_coef(const double* c, int has_y, int y_read, int d, int w) {
  return {(T)c[0], (T)c[1], (T)c[2], (T)c[3], (T)c[4], (T)c[5], (T)c[6], has_y, y_read, d < 4, w < 4};
}
constexpr int SMALL_PRE_ROWS = 5;    // vectors of a block's rows a preconditioner's steps keep in LDS
constexpr int SMALL_MAX_NEAR = 31;   // a wave looks at 63 neighbours
constexpr size_t SMALL_PROG_AT = (size_t)MAX_BLOCKS * PART_COLS * 8 - 256 * sizeof(SmallStep);  // in the partials' place

template <typename T, typename S>
struct SmallArgs {
  Csr A;
  T* wtmp;  // unnormalised next basis vector
  T* w1;    // phases launched one by one: A v_j and w'
  T* w2;
  S* V;
  long ldv;
  State st;
  unsigned long long* words;  // partial sums: h1, h2 (a line per wave and block, then per group), norm (a line per block, group)
  unsigned long long* x;      // the unnormalised vector as words (the cycle kernel's gathers)
  unsigned int tag;           // of the cycle, > 1; iteration j uses tag + j, the gathers of j = 0 tag - 1
  unsigned int vals_lds;  // dynamic LDS of the cycle kernel: the block's rows of A, if they fit
  int rows, blocks;           // partition: rows per block (multiple of 64), blocks
  int j, kmax;
  // SMALL_CYCLE_PRE: block Jacobi of block size bj (inverses as k_bj_apply's) or a polynomial of `steps` steps
  int bj, steps, near;
  const T* minv;
  const SmallStep* prog;
  unsigned long long *z, *z1;  // vectors as words
};

template <typename T>
constexpr int small_words_per_value() {
  return sizeof(T) / 4;
}

// Rows per block of an n-row system at restart m, or 0 if it does not fit.
int small_rows(int64_t n, int m, int sT, int cus);
size_t small_cycle_lds(int rows, int sT);  // dynamic LDS: of the cycle kernel, of a phase
size_t small_phase_lds(int rows, int sT);

template <typename T, typename S>
using SmallKernel = void (*)(SmallArgs<T, S>);
template <typename T, typename S>
SmallKernel<T, S> small_kernel(SmallPhase ph, int m, int rows, int blocks);

// far: at least the distance of blocks that exchange rows, SMALL_MAX_P if a
// window does not fit (of the cycle kernel with a preconditioner, or without)
void small_near(const Csr& A, int sT, int rows, int blocks, bool pre, int* far, hipStream_t s);

// words of the partial sums
size_t small_words(int blocks, int sT);

// sets every word's tag to 0 (never an iteration's)
void small_clear(unsigned long long* words, size_t count, hipStream_t s);

// mid.hip: cycles of larger systems, the first columns of the basis in
// registers; one block per compute unit (MID_BLOCKS of MID_THREADS threads),
// or nullptr where the system is too large.  Uses SmallArgs' A, wtmp, V, ldv,
// st, words, tag and kmax.
constexpr int MID_BLOCKS = 256, MID_THREADS = 512, MID_MAX_M = 64;
template <typename T, typename S>
struct MidKernel {
  SmallKernel<T, S> k;
  int chunks;    // capacity of its window of x (SmallArgs' rows)
  unsigned lds;  // dynamic LDS
};
// sets *wide if a block's window does not fit
void mid_fits(const Csr& A, int chunks, int* wide, hipStream_t s);
template <typename T, typename S>
MidKernel<T, S> mid_kernel(int64_t nslices, bool wide);  // wide: slices of more than 9 entries a row
template <>
MidKernel<float, float> mid_kernel<float, float>(int64_t nslices, bool wide);
template <>
MidKernel<float, bf16_t> mid_kernel<float, bf16_t>(int64_t nslices, bool wide);
template <>
MidKernel<double, double> mid_kernel<double, double>(int64_t nslices, bool wide);
size_t mid_words();

}  // namespace gir
