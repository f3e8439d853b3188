// Matrix set-up on the GPU (gfx950): the row-tile table, the choice of the
// SpMV layout and the sliced copies, from the caller's CSR arrays.
//
// Three launches and one read of a 64-byte decision by the host (rows of more than
// SELL_MAX_ROW entries on average: one, k_setup_values, and the row pointers read):
//   k_setup_scan    per 64-row slice: longest row, size of the sorted union
//                   of its rows' column offsets, order and distance checks;
//                   per tile segment: where a tile chain entering it leaves it
//   k_setup_decide  (one block) sums over the slices, layout choice, entry
//                   point of every tile segment
//   k_setup_build   slice pointers, offset lists or column indices, fp32 and
//                   fp64 values, the fp32 copy of the CSR values, tile table
//
// Bound by memory: the CSR arrays are read once (the column indices twice) and
// every copy is written once.  7-point 150^3 (23.5 M nonzeros), set-up and
// one product in each precision: 0.34 ms (scan 76 us, decide 30, build 135),
// where copying the row pointers and column indices to the host and walking them
// there took 38.0 ms.
#pragma once

#include "device.hpp"

namespace gir {

constexpr int SETUP_MAX_BLOCKS = 1024;  // = threads of k_setup_decide
constexpr int SETUP_MIN_BLOCKS = 256;   // where there are as many slices
constexpr int SETUP_CHUNK = 256;        // slices whose pointers a block scans at once
// Tiles start on multiples of 8 rows ("units") as long as 8 rows fit a tile,
// i.e. no row is longer than TILE_NNZ / 8; longer rows go through the host.
constexpr int TILE_UNIT = 8;
constexpr int TILE_SPAN = TILE_ROWS / TILE_UNIT;  // units of a tile at most
constexpr int TILE_SEG = 1024;                    // units per segment of the tile chain
constexpr int TILE_MAX_ROW = TILE_NNZ / TILE_UNIT;

// Offsets of a slice's rows seen so far, a hash table in LDS: SELL_MAX_ROW and a
// step's 64 more are the most it holds.
constexpr int UNION_SLOTS = 1024;
static_assert(SELL_MAX_ROW + WAVE < UNION_SLOTS, "the table never fills");

enum : int32_t { SETUP_LONG = 1, SETUP_UNORDERED = 2, SETUP_FAR = 4 };

// Sums over the slices of one block of k_setup_scan; k_setup_decide replaces
// the two sums by those of the blocks before it.
struct SetupInfo {
  long long sumK, sumU;
  int32_t bad_row;  // first row whose pointer decreases (INT_MAX: none)
  int32_t max_len, max_u;
  int32_t flags;
};
static_assert(sizeof(SetupInfo) == 32, "SetupInfo");

struct SetupDecision {
  int32_t first, last;  // rowptr[0], rowptr[n]
  int32_t bad_row;
  int32_t max_len;
  int32_t sell, shared, d16, wide;
  int32_t ntiles, lds_nnz;
  int32_t pad[6];
};
static_assert(sizeof(SetupDecision) == 64, "SetupDecision");

// What the set-up kernels read and write.  The scratch (decision, infos, tile
// chain tables) lies in the tile table's region behind its largest possible
// number of tiles, n / 8 + 2 (of the max_tiles + 1 = n + 1 that
// the region has room for).
struct Setup {
  int n;
  long long nnz;
  const int* rowptr;
  const int* col;
  const double* vals;
  int ns;        // slices
  int nblocks;   // blocks over the slices
  int nseg;      // tile segments
  int cap;       // entries of a slice staged in LDS per wave
  long long max_entries;
  float* v32;       // fp32 copy of the CSR values
  int* tile_row;    // tile table
  int* chain;       // [nseg][TILE_SPAN] (tiles << 8 | exit unit past the segment)
  int2* entry;      // [nseg] entry unit, number of the first tile
  SetupInfo* info;  // [nblocks]
  SetupDecision* dec;
  int* sptr;   // ns + 1 slice pointers; between scan and build (K << 16 | U) of each slice
  int* scol;
  float* sv32;
  double* sv64;
};

// The offsets c - r of one slice's rows in ascending order, each lane walking
// its own row (strictly increasing): next() gives the smallest offset not yet
// taken, the lanes that hold it, and moves those on.  The lanes' current
// offsets are mostly equal, so the smallest is found by asking whether any
// lane holds less than the first one's.
struct SliceCursor {
  const int* c;  // columns of the slice's entries
  int r, p, end, cur;
  __device__ __forceinline__ void start(const int* cols, int row, int p0, int p1) {
    c = cols;
    r = row;
    p = p0;
    end = p1;
    cur = p < end ? c[p] - r : 0;
  }
  // false when every row is used up; m: the offset (wave-uniform), hit: this
  // lane holds it, at: its entry
  __device__ __forceinline__ bool next(int& m, bool& hit, int& at) {
    const unsigned long long alive = __ballot(p < end);
    if (!alive) return false;
    m = __builtin_amdgcn_readlane(cur, __ffsll(alive) - 1);
    for (;;) {
      const unsigned long long less = __ballot(p < end && cur < m);
      if (!less) break;
      m = __builtin_amdgcn_readlane(cur, __ffsll(less) - 1);
    }
    hit = p < end && cur == m;
    at = p;
    if (hit) {
      ++p;
      if (p < end) cur = c[p] - r;
    }
    return true;
  }
};

// Orders a wave's LDS writes before its own lanes' later reads.
__device__ __forceinline__ void wave_lds_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Adds the offset d of each lane that has one; the number that were new.
__device__ __forceinline__ int union_add(int* table, int d, bool has) {
  bool added = false;
  for (unsigned at = (unsigned)d * 2654435761u >> 22; __any(has); at = (at + 1) % UNION_SLOTS) {
    if (!has) continue;
    int old = table[at];
    if (old == INT32_MIN) old = atomicCAS(&table[at], INT32_MIN, d);
    added = added || old == INT32_MIN;
    has = old != INT32_MIN && old != d;
  }
  return __popcll(__ballot(added));
}

__device__ __forceinline__ int wave_max_int(int v) {
#pragma unroll
  for (int o = WAVE / 2; o > 0; o >>= 1) v = max(v, __shfl_xor(v, o, WAVE));
  return v;
}

// rowptr at the units seg0 .. seg0 + TILE_SEG + TILE_SPAN, in LDS.
__device__ __forceinline__ void tile_stage(const Setup& S, int seg, int* cum) {
  const long long u0 = (long long)seg * TILE_SEG;
  for (int i = threadIdx.x; i <= TILE_SEG + TILE_SPAN; i += blockDim.x) {
    const long long r = (u0 + i) * TILE_UNIT;
    cum[i] = S.rowptr[r < S.n ? r : S.n];
  }
  __syncthreads();
}

// For each of the TILE_SPAN units a tile chain can enter segment `seg` at: how
// many tiles start in it and where the chain enters the next one.
__device__ __forceinline__ void tile_chains(const Setup& S, int seg, int* cum) {
  tile_stage(S, seg, cum);
  if (threadIdx.x >= TILE_SPAN) return;
  const long long left = ((long long)S.n + TILE_UNIT - 1) / TILE_UNIT - (long long)seg * TILE_SEG;
  const int nu = left < TILE_SEG + TILE_SPAN ? (int)left : TILE_SEG + TILE_SPAN;  // last boundary, in units
  // a unit that fills more than a tile has a row too long for units: the host cuts
  bool fits = true;
  for (int i = threadIdx.x; i < nu; i += TILE_SPAN) fits = fits && cum[i + 1] - cum[i] <= TILE_NNZ;
  fits = __all(fits);
  int u = threadIdx.x, tiles = 0, span = TILE_SPAN / 2;
  while (fits && u < TILE_SEG && u < nu) {
    // the last boundary of a tile from u: at most TILE_SPAN units, TILE_NNZ
    // nonzeros; looked for first where the tile before had its own
    int lo = u + 1, hi = min(u + TILE_SPAN, nu);
    const int guess = min(u + span, hi);
    if (cum[guess] - cum[u] > TILE_NNZ) hi = guess - 1;
    else lo = guess;
    if (lo < hi && cum[lo + 1] - cum[u] > TILE_NNZ) hi = lo;
    while (lo < hi) {
      const int mid = (lo + hi + 1) / 2;
      if (cum[mid] - cum[u] <= TILE_NNZ) lo = mid;
      else hi = mid - 1;
    }
    span = lo - u;
    u = lo;
    ++tiles;
  }
  S.chain[(size_t)seg * TILE_SPAN + threadIdx.x] = tiles << 8 | (u > TILE_SEG ? u - TILE_SEG : 0);
}

__global__ __launch_bounds__(BLOCK) void k_setup_scan(Setup S) {
  int* lds = dyn_lds<int>();
  if ((int)blockIdx.x >= S.nblocks) {
    tile_chains(S, blockIdx.x - S.nblocks, lds);
    return;
  }
  const int lane = threadIdx.x & (WAVE - 1);
  const int wid = __builtin_amdgcn_readfirstlane(threadIdx.x / WAVE);
  int* sc = lds + wid * S.cap;
  int* const table = lds + NWAVES * S.cap + wid * UNION_SLOTS;
  const int s0 = (int)((long long)S.ns * blockIdx.x / S.nblocks);
  const int s1 = (int)((long long)S.ns * (blockIdx.x + 1) / S.nblocks);
  long long sumK = 0, sumU = 0;
  int bad_row = INT32_MAX, max_len = 0, max_u = 0, flags = 0;
  for (int s = s0 + wid; s < s1; s += NWAVES) {
    const int r = s * SELL_C + lane;
    int p0 = 0, p1 = 0;
    if (r < S.n) {
      p0 = S.rowptr[r];
      p1 = S.rowptr[r + 1];
      if (p1 < p0) bad_row = min(bad_row, r);
    }
    // entries are touched only where all of the slice's pointers are in order and in range
    const bool valid = p0 >= 0 && p1 >= p0 && p1 <= S.nnz;
    const bool ok = __all(valid);
    const int len = valid ? p1 - p0 : 0;
    const int K = wave_max_int(len);
    max_len = max(max_len, K);
    int U = 0;
    if (K > SELL_MAX_ROW) flags |= SETUP_LONG;
    // (past the storage the matrix has no slices and its union is not asked for)
    if (ok && K > 0 && K <= SELL_MAX_ROW && SELL_C * (sumK + K) <= S.max_entries) {
      const int rows = min(SELL_C, S.n - s * SELL_C);
      const int q0 = __builtin_amdgcn_readlane(p0, 0);
      const int cnt = __builtin_amdgcn_readlane(p1, rows - 1) - q0;
      const int a = r < S.n ? p0 - q0 : 0, b = r < S.n ? p1 - q0 : 0;
      // Each lane walks its row beside the longest one's.  Rows that all begin
      // as that one does (the inside of a stencil's grid) have its offsets for
      // their union.  Where few do not (a grid's edge) the rows are merged,
      // smallest offset by smallest offset; else that takes as many steps as there
      // are entries, and the union is counted in the table (1000 random rows of 20
      // entries, whole set-up, 703 -> 55 us; 300000 836 -> 150).  Slices
      // too large to stage are not merged, each step would read memory.
      auto look = [&](const int* cols, bool staged) {
        constexpr int AHEAD = 8;  // entries loaded together
        const int longest = __ffsll(__ballot(len == K)) - 1;
        bool unordered = false, far = false, differ = false;
        int prev = 0;
        auto walk = [&](auto step) {
          for (int k0 = 0; k0 < K; k0 += AHEAD) {
            int d[AHEAD];
#pragma unroll
            for (int u = 0; u < AHEAD; ++u) d[u] = cols[min(a + k0 + u, cnt - 1)] - r;
#pragma unroll
            for (int u = 0; u < AHEAD; ++u)
              if (k0 + u < K) step(k0 + u, d[u], a + k0 + u < b);
          }
        };
        walk([&](int k, int d, bool has) {
          unordered = unordered || (has && k > 0 && d <= prev);
          far = far || (has && (d > 32767 || d < -32767));
          differ = differ || (has && d != __builtin_amdgcn_readlane(d, longest));
          prev = d;
        });
        if (__any(far)) flags |= SETUP_FAR;
        if (__any(unordered)) {
          flags |= SETUP_UNORDERED;
          return;
        }
        U = K;
        if (!__any(differ)) return;
        const bool merge = staged && __popcll(__ballot(differ)) <= WAVE / 4;
        if (merge) {
          SliceCursor cu;
          cu.start(cols, r, a, b);
          int m, at;
          bool hit;
          for (U = 0; U <= 2 * K; ++U)
            if (!cu.next(m, hit, at)) break;
        }
        if (!merge || U > 2 * K) {
          for (int i = lane; i < UNION_SLOTS; i += WAVE) table[i] = INT32_MIN;
          wave_lds_sync();
          U = 0;
          walk([&](int, int d, bool has) {
            if (U <= SELL_MAX_ROW) U += union_add(table, d, has);
          });
        }
        if (U > SELL_MAX_ROW) flags |= SETUP_UNORDERED;
      };
      if (cnt <= S.cap) {
        for (int i = lane; i < cnt; i += 4 * WAVE) {
          int c[4];
#pragma unroll
          for (int u = 0; u < 4; ++u) c[u] = S.col[q0 + min(i + u * WAVE, cnt - 1)];
#pragma unroll
          for (int u = 0; u < 4; ++u)
            if (i + u * WAVE < cnt) sc[i + u * WAVE] = c[u];
        }
        wave_lds_sync();
        look(sc, true);
        wave_lds_sync();  // sc is free for the next slice
      } else {
        look(S.col + q0, false);
      }
    }
    const int Kc = min(K, SELL_MAX_ROW + 1);
    sumK += Kc;
    sumU += U;
    max_u = max(max_u, U);
    if (lane == 0) S.sptr[s] = Kc << 16 | U;
  }
#pragma unroll
  for (int o = WAVE / 2; o > 0; o >>= 1) bad_row = min(bad_row, __shfl_xor(bad_row, o, WAVE));
  __shared__ SetupInfo s_info[NWAVES];
  if (lane == 0) s_info[wid] = SetupInfo{sumK, sumU, bad_row, max_len, max_u, flags};
  __syncthreads();
  if (threadIdx.x == 0) {
    SetupInfo t = s_info[0];
    for (int w = 1; w < NWAVES; ++w) {
      const SetupInfo& o = s_info[w];
      t.sumK += o.sumK;
      t.sumU += o.sumU;
      t.bad_row = min(t.bad_row, o.bad_row);
      t.max_len = max(t.max_len, o.max_len);
      t.max_u = max(t.max_u, o.max_u);
      t.flags |= o.flags;
    }
    S.info[blockIdx.x] = t;
  }
}

__global__ __launch_bounds__(SETUP_MAX_BLOCKS) void k_setup_decide(Setup S) {
  __shared__ long long s_k[SETUP_MAX_BLOCKS], s_u[SETUP_MAX_BLOCKS];
  __shared__ int s_bad, s_len, s_mu, s_flags;
  // Tile segments staged at once, in groups: every entry's way through a group
  // side by side, the groups one after the other, then each group's segments
  // (7-point 150^3, 412 segments: this kernel 37 -> 29 us, against the
  // segments one after the other)
  constexpr int GROUPS = SETUP_MAX_BLOCKS / TILE_SPAN, GROUP = 8, CHUNK = GROUPS * GROUP;
  __shared__ int s_chain[CHUNK * TILE_SPAN];
  __shared__ int s_way[GROUPS * TILE_SPAN];
  __shared__ int2 s_from[GROUPS];
  const int t = threadIdx.x;
  if (t == 0) {
    s_bad = INT32_MAX;
    s_len = s_mu = s_flags = 0;
  }
  __syncthreads();
  SetupInfo mine{0, 0, INT32_MAX, 0, 0, 0};
  if (t < S.nblocks) {
    mine = S.info[t];
    atomicMin(&s_bad, mine.bad_row);
    atomicMax(&s_len, mine.max_len);
    atomicMax(&s_mu, mine.max_u);
    atomicOr(&s_flags, mine.flags);
  }
  s_k[t] = mine.sumK;
  s_u[t] = mine.sumU;
  __syncthreads();
  for (int o = 1; o < SETUP_MAX_BLOCKS; o *= 2) {
    const long long k = t >= o ? s_k[t - o] : 0, u = t >= o ? s_u[t - o] : 0;
    __syncthreads();
    s_k[t] += k;
    s_u[t] += u;
    __syncthreads();
  }
  if (t < S.nblocks) {
    S.info[t].sumK = s_k[t] - mine.sumK;
    S.info[t].sumU = s_u[t] - mine.sumU;
  }
  // the tile chain over the segments, their tables staged in LDS
  int u = 0, tiles = 0;
  for (int g0 = 0; g0 < S.nseg && S.nseg > 1; g0 += CHUNK) {
    const int cnt = min(CHUNK, S.nseg - g0);
    __syncthreads();
    for (int i = t; i < cnt * TILE_SPAN; i += SETUP_MAX_BLOCKS) s_chain[i] = S.chain[(size_t)g0 * TILE_SPAN + i];
    __syncthreads();
    const int first = t / TILE_SPAN * GROUP;
    if (first < cnt) {
      int w = t % TILE_SPAN, made = 0;
      for (int g = first; g < min(first + GROUP, cnt); ++g) {
        const int c = s_chain[g * TILE_SPAN + w];
        w = c & 255;
        made += c >> 8;
      }
      s_way[t] = made << 8 | w;
    }
    __syncthreads();
    if (t == 0)
      for (int g = 0; g * GROUP < cnt; ++g) {
        s_from[g] = make_int2(u, tiles);
        const int c = s_way[g * TILE_SPAN + u];
        u = c & 255;
        tiles += c >> 8;
      }
    __syncthreads();
    if (t < GROUPS && t * GROUP < cnt) {
      int2 e = s_from[t];
      for (int g = t * GROUP; g < min((t + 1) * GROUP, cnt); ++g) {
        S.entry[g0 + g] = e;
        const int c = s_chain[g * TILE_SPAN + e.x];
        e = make_int2(c & 255, e.y + (c >> 8));
      }
    }
  }
  if (t == 0) {
    if (S.nseg == 1) S.entry[0] = make_int2(0, 0);
    SetupDecision d{};
    d.first = S.rowptr[0];
    d.last = S.rowptr[S.n];
    d.bad_row = s_bad;
    d.max_len = s_len;
    const long long slots = SELL_C * s_k[SETUP_MAX_BLOCKS - 1], shared = SELL_C * s_u[SETUP_MAX_BLOCKS - 1];
    d.sell = S.nnz > 0 && !(s_flags & SETUP_LONG) && slots <= S.max_entries && slots <= INT32_MAX;
    d.shared = d.sell && !(s_flags & SETUP_UNORDERED) && shared <= S.max_entries && shared <= INT32_MAX &&
               (double)shared <= SHARED_MAX_GROWTH * (double)slots;
    d.d16 = d.sell && !d.shared && !(s_flags & SETUP_FAR);
    d.wide = d.shared && s_mu > 9;
    d.ntiles = tiles;  // one segment: counted by k_setup_build
    d.lds_nnz = 1;
    *S.dec = d;
  }
}

// The tiles that start in segment `seg`, by one wave: lane l asks whether the
// tile from u reaches l + 1 units.
__device__ __forceinline__ void tile_emit(const Setup& S, int seg, int* cum) {
  tile_stage(S, seg, cum);
  if (threadIdx.x >= WAVE) return;
  const int lane = threadIdx.x;
  const long long total = ((long long)S.n + TILE_UNIT - 1) / TILE_UNIT, u0 = (long long)seg * TILE_SEG;
  const int nu = total - u0 < TILE_SEG + TILE_SPAN ? (int)(total - u0) : TILE_SEG + TILE_SPAN;
  const int2 e = S.entry[seg];
  int u = e.x, tile = e.y, most = 1;
  while (u < TILE_SEG && u < nu) {
    const int v = u + 1 + lane;
    const bool in = v <= nu && cum[min(v, TILE_SEG + TILE_SPAN)] - cum[u] <= TILE_NNZ;
    const int len = max(1, __popcll(__ballot(in)));  // row pointers rise: the lanes that fit come first
    if (lane == 0) S.tile_row[tile] = (int)((u0 + u) * TILE_UNIT);
    most = max(most, cum[u + len] - cum[u]);
    u += len;
    ++tile;
  }
  if (lane == 0) {
    if (u0 + u >= total) S.tile_row[tile] = S.n;
    if (S.nseg == 1) S.dec->ntiles = tile;
    atomicMax(&S.dec->lds_nnz, most);
  }
}

// The fp32 copy of the CSR values by block `block` of `blocks`.
__device__ __forceinline__ void cast_values(const Setup& S, int block, int blocks) {
  const long long stride = (long long)blocks * BLOCK;
  for (long long i = (long long)block * BLOCK + threadIdx.x; i < S.nnz; i += 4 * stride) {
    double v[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) v[u] = S.vals[i + u * stride < S.nnz ? i + u * stride : i];
#pragma unroll
    for (int u = 0; u < 4; ++u)
      if (i + u * stride < S.nnz) S.v32[i + u * stride] = (float)v[u];
  }
}
__global__ __launch_bounds__(BLOCK) void k_setup_values(Setup S) { cast_values(S, blockIdx.x, gridDim.x); }

__global__ __launch_bounds__(BLOCK) void k_setup_build(Setup S) {
  const SetupDecision* dec = S.dec;
  if (dec->bad_row != INT32_MAX || dec->first != 0 || dec->last != S.nnz) return;
  char* lds = dyn_lds<char>();
  const bool sell = dec->sell, shared = dec->shared, d16 = dec->d16;
  const int extra = (int)blockIdx.x - S.nblocks - S.nseg;  // blocks for the fp32 copy alone
  if ((int)blockIdx.x >= S.nblocks && extra < 0) {
    if (dec->max_len <= TILE_MAX_ROW) tile_emit(S, blockIdx.x - S.nblocks, (int*)lds);
    return;
  }
  if (!sell) {
    // no slices to fill: the values alone, over as many blocks as they need
    // (slice by slice, 3000 rows of 544 entries, which k_setup_values now takes, 750 us)
    cast_values(S, extra < 0 ? (int)blockIdx.x : S.nblocks + extra, gridDim.x - S.nseg);
    return;
  }
  if (extra >= 0) return;
  __shared__ int s_base[SETUP_CHUNK], s_wave[NWAVES];
  const int lane = threadIdx.x & (WAVE - 1);
  const int wid = __builtin_amdgcn_readfirstlane(threadIdx.x / WAVE);
  double* sv = (double*)lds + wid * S.cap;
  int* sc = (int*)(lds + (size_t)NWAVES * S.cap * sizeof(double)) + wid * S.cap;
  const int s0 = (int)((long long)S.ns * blockIdx.x / S.nblocks);
  const int s1 = (int)((long long)S.ns * (blockIdx.x + 1) / S.nblocks);
  int before = (int)(shared ? S.info[blockIdx.x].sumU : S.info[blockIdx.x].sumK);  // slots / 64 of the slices before
  for (int c0 = s0; c0 < s1; c0 += SETUP_CHUNK) {
    const int c1 = min(c0 + SETUP_CHUNK, s1);
    // slice pointers of the chunk: exclusive sums of the slices' widths
    const int mine = c0 + (int)threadIdx.x;
    const int w = mine < c1 ? S.sptr[mine] : 0;
    const int width = shared ? w & 0xffff : w >> 16;
    int x = width;
#pragma unroll
    for (int o = 1; o < WAVE; o *= 2) {
      const int y = __shfl_up(x, o, WAVE);
      if (lane >= o) x += y;
    }
    if (lane == WAVE - 1) s_wave[wid] = x;
    __syncthreads();
    int at = before, sum = 0;
    for (int q = 0; q < NWAVES; ++q) {
      if (q < wid) at += s_wave[q];
      sum += s_wave[q];
    }
    s_base[threadIdx.x] = at + x - width;
    if (mine < c1) S.sptr[mine] = SELL_C * (at + x - width);
    before += sum;
    __syncthreads();
    if (c1 == S.ns && threadIdx.x == 0) S.sptr[S.ns] = SELL_C * before;
    for (int s = c0 + wid; s < c1; s += NWAVES) {
      const int r = s * SELL_C + lane;
      const int rows = min(SELL_C, S.n - s * SELL_C);
      const int p0 = r < S.n ? S.rowptr[r] : 0, p1 = r < S.n ? S.rowptr[r + 1] : 0;
      const int q0 = __builtin_amdgcn_readlane(p0, 0);
      const int cnt = __builtin_amdgcn_readlane(p1, rows - 1) - q0;
      const bool staged = cnt <= S.cap;
      // (four entries' loads together: 7-point 150^3, this kernel 190 -> 135 us)
      for (int i = lane; i < cnt; i += 4 * WAVE) {
        double v[4];
        int c[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const int at = q0 + min(i + u * WAVE, cnt - 1);
          v[u] = S.vals[at];
          if (staged) c[u] = S.col[at];
        }
#pragma unroll
        for (int u = 0; u < 4; ++u)
          if (i + u * WAVE < cnt) {
            S.v32[q0 + i + u * WAVE] = (float)v[u];
            if (staged) {
              sv[i + u * WAVE] = v[u];
              sc[i + u * WAVE] = c[u];
            }
          }
      }
      const int a = r < S.n ? p0 - q0 : 0, b = r < S.n ? p1 - q0 : 0;
      const int base = s_base[s - c0];
      const int K = (s + 1 < c1 ? s_base[s + 1 - c0] : before) - base;
      auto fill = [&](const int* cols, const double* vals) {
        size_t e = (size_t)SELL_C * base + lane;
        if (shared) {
          SliceCursor cu;
          cu.start(cols, r, a, b);
          for (int k = 0; k < K; ++k, e += SELL_C) {
            int m = 0, at = 0;
            bool hit = false;
            (void)cu.next(m, hit, at);
            const double v = hit ? vals[at] : 0.0;
            if (lane == 0) S.scol[base + k] = m;
            S.sv64[e] = v;
            S.sv32[e] = (float)v;
          }
        } else {
          // columns, or (d16) 16-bit offsets from the row; padding entries
          // point at the row itself (offset 0), rows past n at row 0
          // (four entries' loads go out before their stores)
          const int rr = r < S.n ? r : 0;
          for (int k0 = 0; k0 < K; k0 += 4) {
            int c[4];
            double v[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
              const int p = min(a + k0 + u, cnt - 1);
              c[u] = cols[p];
              v[u] = vals[p];
            }
#pragma unroll
            for (int u = 0; u < 4; ++u)
              if (k0 + u < K) {
                const bool in = a + k0 + u < b;
                const int col = in ? c[u] : rr;
                const double val = in ? v[u] : 0.0;
                if (d16) ((short*)S.scol)[e] = (short)(col - rr);
                else S.scol[e] = col;
                S.sv64[e] = val;
                S.sv32[e] = (float)val;
                e += SELL_C;
              }
          }
        }
      };
      if (staged) {
        wave_lds_sync();
        fill(sc, sv);
        wave_lds_sync();  // the staging area is free for the next slice
      } else {
        fill(S.col + q0, S.vals + q0);
      }
    }
    __syncthreads();  // s_base is free for the next chunk
  }
}

}  // namespace gir
