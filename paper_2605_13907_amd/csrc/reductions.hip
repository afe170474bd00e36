// Per-row scalar work and the batch-wide reductions of the path.
//
// The batch is a set of variable-length segments (responses) of rows, some rows masked out.  Every response is cut into
// tiles of 256 rows or a power of two times that (each workgroup works the tiling out for itself, for up to
// kSelfPlanResponses responses; beyond that a small plan kernel does it once); level 1 reduces a tile per wavefront to a
// partial, without a barrier; level 2, run by whichever workgroup of the same launch finishes last, folds the partials of
// each response in order, forms the group-relative advantages (Eq. 3) and the batch moments, and evaluates the three
// diagnostics and the mixing coefficient (Eq. 12-17).  Everything is accumulated in fp64 in a fixed order (no floating
// point atomics), so results are bit-reproducible from run to run; spreads are carried as (count, mean, squared
// deviations) triples, never as differences of power sums.
//
// These kernels move a few bytes per row (about a megabyte per batch) and are bound by the length of their dependent
// chains and, small as they are, by the instruction fetches of code that runs once.  Hence a tile per wavefront without
// barriers, 16 wavefronts to a workgroup that share one look at cu_rows, level 2 by 1,024 threads in one pass, partials as
// arrays of words (12,000 separate reads of 1,700 structures by one compute unit before), and code that is not unrolled.
// Diagnostics and row coefficients, us, a 256-thread workgroup per tile of 1,024 rows before and now: 512 rows in 8
// responses 12.9 and 7.1 -> 7.3 and 4.2; 8,192 in 16 12.8, 7.7 -> 9.6, 7.4; 41,643 in 16 13.3, 8.9 -> 11.1, 7.7; 200,000 in
// 512 19.8, 13.8 -> 14.1, 9.7; 1,200,000 in 1,024 (with stale policy and KL term) 38.0, 29.5 -> 21.8, 17.1; 4,000,000 in 8
// 50, 43 -> 33.5, 34.
#include "ais_internal.h"
#include "row_coeff.h"

#include <algorithm>
#include <cmath>
#include <type_traits>

namespace ais {
namespace {

using dev::CoeffRule;
using dev::RowTerm;
using dev::response_weight;
using dev::row_term;

// What a workgroup of one launch leaves for the workgroup that finishes last goes through device-scope accesses: they
// reach memory that every XCD sees, so no cache has to be written back or invalidated for them.
template <typename V>
__device__ __forceinline__ void put_device(V* p, V v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <typename V>
__device__ __forceinline__ V get_device(const V* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ long long clampll(long long v, long long lo, long long hi) {
  return v < lo ? lo : (v > hi ? hi : v);
}

// Row range of response i, forced into [0, n_rows] and non-negative length whatever cu_rows holds.
__device__ __forceinline__ void response_rows(const long long* cu_rows, int i, long long n_rows, long long& lo,
                                              long long& hi) {
  lo = clampll(cu_rows[i], 0, n_rows);
  hi = clampll(cu_rows[i + 1], lo, n_rows);
}

// ---- plan: tile_off[i] = first tile of response i, tile_off[n_resp] = number of tiles -------------------
// One workgroup.  Each thread owns a contiguous chunk of responses; thread 0 scans the 256 chunk totals.
__global__ __launch_bounds__(kPlanThreads) void plan_kernel(const long long* __restrict__ cu_rows, int n_resp,
                                                            long long n_rows, int* __restrict__ tile_off,
                                                            int max_tiles, int* __restrict__ status) {
  __shared__ long long chunk_sum[kPlanThreads];
  const int tid = threadIdx.x;
  const int per = (n_resp + kPlanThreads - 1) / kPlanThreads;
  const int i0 = min(n_resp, tid * per), i1 = min(n_resp, i0 + per);
  long long sum = 0;
  bool bad = false;
  for (int i = i0; i < i1; ++i) {
    long long lo, hi;
    response_rows(cu_rows, i, n_rows, lo, hi);
    bad |= (cu_rows[i] != lo) || (cu_rows[i + 1] != hi);
    sum += (hi - lo + kPlanTileRows - 1) / kPlanTileRows;
  }
  if (tid == 0 && n_resp > 0) bad |= (cu_rows[0] != 0) || (cu_rows[n_resp] != n_rows);
  chunk_sum[tid] = sum;
  __syncthreads();
  if (tid == 0) {
    long long run = 0;
    for (int t = 0; t < kPlanThreads; ++t) {
      long long s = chunk_sum[t];
      chunk_sum[t] = run;
      run += s;
    }
    if (run > max_tiles) bad = true;             // cannot happen when cu_rows is a partition of the rows
    tile_off[n_resp] = (int)clampll(run, 0, max_tiles);
  }
  __syncthreads();
  long long run = chunk_sum[tid];
  for (int i = i0; i < i1; ++i) {
    long long lo, hi;
    response_rows(cu_rows, i, n_rows, lo, hi);
    tile_off[i] = (int)clampll(run, 0, max_tiles);
    run += (hi - lo + kPlanTileRows - 1) / kPlanTileRows;
  }
  if (bad) atomicOr(status, AIS_STATUS_BAD_CU);
}

// Response that owns tile b: the last i with tile_off[i] <= b.
__device__ __forceinline__ int find_response(const int* __restrict__ tile_off, int n_resp, int b) {
  int lo = 0, hi = n_resp;          // invariant: tile_off[lo] <= b < tile_off[hi]
  while (hi - lo > 1) {
    int mid = (lo + hi) >> 1;
    if (tile_off[mid] <= b) lo = mid; else hi = mid;
  }
  return lo;
}

// Sum over each row of 16 lanes.
__device__ __forceinline__ int row_sum(int v) {
  v += __builtin_amdgcn_update_dpp(0, v, 0xB1, 0xf, 0xf, true);
  v += __builtin_amdgcn_update_dpp(0, v, 0x4E, 0xf, 0xf, true);
  v += __builtin_amdgcn_update_dpp(0, v, 0x141, 0xf, 0xf, true);
  return v + __builtin_amdgcn_update_dpp(0, v, 0x140, 0xf, 0xf, true);
}

constexpr int kThreads = 1024;
constexpr int kWaves = kThreads / 64;
constexpr int kLaneRows = 4;                     // rows of a lane whose inputs are loaded together
constexpr int kChunkRows = 64 * kLaneRows;       // rows of a wavefront that are

// Rows [row0, row0 + len) of response `resp`, the work of one wavefront.
struct Tile {
  int resp, row0, len;
};

// The tiling of the batch as a workgroup sees it: from the plan kernel's array in memory, or worked out by the workgroup
// itself into LDS, a thread per response.  The latter costs one read of cu_rows (8 KiB at most) and a scan where the
// former costs a launch and a chain of log2(n_resp) dependent reads in every wavefront.
// Both are used the same way: init, then open() for every window of kWaves tiles, whose tiles the wavefronts take in turn.
template <bool SELF>
struct Tiling;

template <>
struct Tiling<false> {
  const int* tile_off;
  const long long* cu_rows;
  int n_resp, n_rows;
  __device__ __forceinline__ void init(const int* off, const long long* cu, int resp, long long rows, int, int, int*) {
    tile_off = off;
    cu_rows = cu;
    n_resp = resp;
    n_rows = (int)rows;
  }
  __device__ __forceinline__ int tiles() const { return tile_off[n_resp]; }
  __device__ __forceinline__ int first(int i) const { return tile_off[i]; }
  __device__ __forceinline__ void open(int) const {}
  __device__ __forceinline__ Tile tile(int b, int) const {
    const int i = find_response(tile_off, n_resp, b);
    long long lo, hi;
    response_rows(cu_rows, i, n_rows, lo, hi);
    const long long r0 = lo + (long long)(b - tile_off[i]) * kPlanTileRows;
    const int len = (int)min(hi - r0, (long long)kPlanTileRows);
    return Tile{__builtin_amdgcn_readfirstlane(i), __builtin_amdgcn_readfirstlane((int)r0),
                __builtin_amdgcn_readfirstlane(len)};
  }
};

template <>
struct Tiling<true> {
  struct Shared {
    int off[kSelfPlanResponses + 1];
    int wave_tiles[kWaves];
    Tile window[kWaves];
  };
  __device__ static Shared& shared() {
    __shared__ Shared sh;
    return sh;
  }
  static_assert(kSelfPlanResponses <= kThreads, "a thread per response");
  int shift, n_tiles;
  int lo, hi, tile0, tile1;          // of the thread's response: its rows and its tiles
  // Must be called by all threads of the workgroup.  Workgroup 0 reports a cu_rows that is no partition of the rows.
  __device__ __forceinline__ void init(const int*, const long long* __restrict__ cu, int n_resp, long long n_rows,
                                       int tile_shift, int max_tiles, int* status) {
    Shared& sh = shared();
    shift = tile_shift;
    const int i = threadIdx.x, lane = i & 63, wave = i >> 6;
    bool bad = false;
    lo = hi = 0;
    if (i < n_resp) {
      const long long c0 = cu[i], c1 = cu[i + 1];
      const long long l = clampll(c0, 0, n_rows), h = clampll(c1, l, n_rows);
      bad = c0 != l || c1 != h || (i == 0 && c0 != 0) || (i == n_resp - 1 && c1 != n_rows);
      lo = (int)l;
      hi = (int)h;
    }
    const int mine = (int)(((long long)(hi - lo) + (1 << shift) - 1) >> shift);
    int incl = mine;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
      const int o = __shfl_up(incl, off);
      incl += lane >= off ? o : 0;
    }
    if (lane == 63) sh.wave_tiles[wave] = incl;
    __syncthreads();
    static_assert(kWaves == 16, "a row of lanes");
    const int t = sh.wave_tiles[lane & 15];
    const int before = incl - mine + row_sum((lane & 15) < wave ? t : 0), total = row_sum(t);
    bad |= total > max_tiles;                    // cannot happen when cu_rows is a partition of the rows
    n_tiles = min(total, max_tiles);
    tile0 = min(before, max_tiles);
    tile1 = min(before + mine, max_tiles);
    if (i < n_resp) sh.off[i] = tile0;
    if (i == 0) sh.off[n_resp] = n_tiles;
    if (bad && blockIdx.x == 0) atomicOr(status, AIS_STATUS_BAD_CU);
  }
  __device__ __forceinline__ int tiles() const { return n_tiles; }
  __device__ __forceinline__ int first(int i) const { return shared().off[i]; }
  // Publishes tiles w0 .. w0 + kWaves - 1.  Must be called by all threads of the workgroup.
  __device__ __forceinline__ void open(int w0) const {
    Shared& sh = shared();
    __syncthreads();                             // the window before has been read
    for (int b = max(tile0, w0); b < min(tile1, w0 + kWaves); ++b) {
      const int r0 = lo + ((b - tile0) << shift);
      sh.window[b - w0] = Tile{(int)threadIdx.x, r0, min(hi - r0, 1 << shift)};
    }
    __syncthreads();
  }
  __device__ __forceinline__ Tile tile(int b, int w0) const {
    const Tile t = shared().window[b - w0];
    return Tile{__builtin_amdgcn_readfirstlane(t.resp), __builtin_amdgcn_readfirstlane(t.row0),
                __builtin_amdgcn_readfirstlane(t.len)};
  }
};

// The value of the lane that level LEVEL (0..5) of a butterfly pairs with this one: after level k the 2^(k + 1) lanes of
// an aligned group hold the same set.  The first four levels stay inside a row of 16 lanes and go through the vector ALU
// (DPP: quad_perm xor 1, xor 2, row_half_mirror, row_mirror); all lanes must be active.
template <int LEVEL, typename V>
__device__ __forceinline__ V butterfly(V v) {
  static_assert(sizeof(V) == 8, "two registers");
  if (LEVEL >= 4) return __shfl_xor(v, 1 << LEVEL);
  constexpr int kCtrl = LEVEL == 0 ? 0xB1 : LEVEL == 1 ? 0x4E : LEVEL == 2 ? 0x141 : 0x140;
  struct Words { int lo, hi; } w = __builtin_bit_cast(Words, v);
  w.lo = __builtin_amdgcn_update_dpp(0, w.lo, kCtrl, 0xf, 0xf, true);
  w.hi = __builtin_amdgcn_update_dpp(0, w.hi, kCtrl, 0xf, 0xf, true);
  return __builtin_bit_cast(V, w);
}

// Sum over a wavefront, in a fixed order.  No barrier is involved: these kernels are latency-bound and a workgroup
// barrier per tree level was most of their time.
template <typename V>
__device__ __forceinline__ V wave_sum(V v) {
  v += butterfly<0>(v);
  v += butterfly<1>(v);
  v += butterfly<2>(v);
  v += butterfly<3>(v);
  v += butterfly<4>(v);
  v += butterfly<5>(v);
  return v;
}

// Count, mean and sum of squared deviations from the mean of a set of values; all zero for the empty set.  Sets are
// merged pairwise (the update of Chan, Golub and LeVeque): the error of the spread scales with the spread itself, not
// with the mean, and a set of equal values has spread exactly 0 however it was split.
struct Moments {
  double n, mean, m2;
};

// 1 / n to the last bit or the one beside it, for n a count: no scaling for extreme exponents.
__device__ __forceinline__ double reciprocal(double n) {
  double r = __builtin_amdgcn_rcp(n);
  r = __builtin_fma(__builtin_fma(-n, r, 1.0), r, r);
  return __builtin_fma(__builtin_fma(-n, r, 1.0), r, r);
}

// Free of branches: an empty set is merged like any other (its share is 0, or the other's is 1).
__device__ __forceinline__ Moments merge(const Moments& a, const Moments& b) {
  const double n = a.n + b.n, delta = b.mean - a.mean;
  const double share = a.n == 0.0 ? 1.0 : b.n * reciprocal(fmax(n, 1.0));
  Moments r;
  r.n = n;
  r.mean = a.mean + delta * share;
  r.m2 = a.m2 + b.m2 + delta * delta * (a.n * share);
  return r;
}

template <int LEVEL>
__device__ __forceinline__ Moments merge_level(const Moments& m) {
  return merge(m, Moments{butterfly<LEVEL>(m.n), butterfly<LEVEL>(m.mean), butterfly<LEVEL>(m.m2)});
}

// The value of lane `src` (uniform), in all lanes.
__device__ __forceinline__ double lane_value(double v, int src) {
  struct Words { int lo, hi; } w = __builtin_bit_cast(Words, v);
  w.lo = __builtin_amdgcn_readlane(w.lo, src);
  w.hi = __builtin_amdgcn_readlane(w.hi, src);
  return __builtin_bit_cast(double, w);
}

// True in exactly one workgroup of the grid: the one that finishes last.  Every workgroup calls this once, after its own
// results have been written with put_device.  They have reached memory when every wavefront has waited for its stores, and
// only then is the ticket taken; the last workgroup reads them with get_device.  (A device-wide fence here instead, which
// writes a whole L2 back for the few bytes of a partial, makes the two calls of 1.2 million rows 79 instead of 62 us.)
// Level 2 of each reduction runs in that workgroup, which saves a kernel launch per reduction; the order in which level
// 2 folds the partials does not depend on which workgroup happens to be last, so results stay bit-reproducible.
struct Tickets {
  int* own;      // 0 when the launch begins and when it ends
  int* next;     // the launch's that comes after it
};

__device__ __forceinline__ bool last_workgroup(Tickets t) {
  __shared__ int s_last;
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  if (gridDim.x == 1) return true;             // uniform; nobody to wait for, the tickets stay as they are
  if (threadIdx.x == 0) {
    s_last = __hip_atomic_fetch_add(t.own, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == (int)gridDim.x - 1;
    if (s_last) {
      put_device(t.own, 0);                  // every other workgroup has taken its ticket: ready for a later launch
      // Launches take turns with two tickets, and each clears the other's: should launches of one context ever have
      // overlapped, which leaves a count behind, the results of one call are lost and the calls after it are sound.
      put_device(t.next, 0);
    }
  }
  __syncthreads();
  return s_last != 0;
}

// The partials of the tiles, NW words each: in memory, or in LDS where one workgroup does it all.
constexpr int kOwnTiles = kWaves;                // most tiles that a single workgroup takes on
template <int NW>
struct Partials {
  double* global;
  double* local;                                 // [word][kOwnTiles]
  int stride;
  bool own;                                      // uniform for the launch
  struct Words { double v[NW]; };
  __device__ __forceinline__ void put(int tile, const Words& q) const {
    if (own) {
#pragma unroll
      for (int k = 0; k < NW; ++k) local[k * kOwnTiles + tile] = q.v[k];
    } else {
      double* to = global + tile;
#pragma unroll
      for (int k = 0; k < NW; ++k) put_device(to + (size_t)k * stride, q.v[k]);
    }
  }
  __device__ __forceinline__ Words get(int tile) const {
    Words q;
    if (own) {
#pragma unroll
      for (int k = 0; k < NW; ++k) q.v[k] = local[k * kOwnTiles + tile];
    } else {
      const double* from = global + tile;
#pragma unroll
      for (int k = 0; k < NW; ++k) q.v[k] = get_device(from + (size_t)k * stride);
    }
    return q;
  }
};

// Group-relative advantage of response i (Eq. 3): reward minus the mean over the G responses of the prompt, as stored.
__device__ __forceinline__ float advantage(const float* rewards, int i, int group_size, const ais_params& p) {
  const int g0 = (i / group_size) * group_size;
  double mean = 0;
  for (int j = 0; j < group_size; ++j) mean += (double)rewards[g0 + j];
  mean /= group_size;
  double a = (double)rewards[i] - mean;
  if (p.adv_mode == 1) {
    double var = 0;
    for (int j = 0; j < group_size; ++j) {
      const double e = (double)rewards[g0 + j] - mean;
      var += e * e;
    }
    const double den = sqrt(var / group_size) + (double)p.eps_std;
    a = den > 0.0 ? a / den : 0.0;     // eps_std = 0 and equal rewards: 0 / 0, read as 0
  }
  return (float)a;
}

// ---- level 2: responses -> batch moments, diagnostics, alpha ---------------------------------------------------------
// Runs in the last workgroup of diag_reduce_kernel.  A response's tiles are folded by a group of L lanes, L (a power of
// two) as large as the responses leave threads for and no larger than their tiles need on average: lane l folds
// tiles l, l + L, ... in order, then the lanes are merged in a fixed tree.  With one thread per response a batch of 4
// responses of 1,000 tiles was a chain of 1,000 dependent reads.  A second wavefront for a response and more come only
// where each lane has more than five tiles without it: a step of the chain is 0.3 us, a wavefront more at work 0.2 (300,000
// rows in 1, 2 and 8 responses, 64 lanes each: 20.3, 17.5, 15.9 us; as many as there are threads: 17.6, 17.5, 17.4).
int fold_lanes(int n_resp, long long most_tiles) {
  int lanes = 1;
  while ((lanes < 64 ? 1 : 5) * (long long)lanes * n_resp < most_tiles && 2LL * lanes * n_resp <= kThreads) lanes <<= 1;
  return lanes;
}
// The code runs once per launch, cold: its size is part of its time (a kilobyte of straight code costs 0.3 us of
// instruction fetches), so what is the same for several quantities is done once, by lanes that hold one each.
// WIDE: more than 64 lanes for a response (in a kernel of its own: in the others the code for it, which they do not run, was
// 0.2 us of 1,200,000 rows in 1,024 responses).
template <bool SELF, bool WIDE>
__device__ void diag_final(const Partials<kDiagWords>& partials, const Tiling<SELF>& tiling, int n_resp, int lanes,
                           int group_size, const float* rewards, const float* s_adv, const ais_params& p,
                           float* __restrict__ adv_out, int* __restrict__ count_out, ais_diag* __restrict__ diag_out,
                           const int* status, double* lds) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  Moments m[3] = {};                                  // of w_bar, of A and of A w_bar over the thread's valid rows
  double d[4] = {};                                   // sums: |d|, d, |dp|, rows with rho > C (exact in fp64)
  const int l = threadIdx.x & (lanes - 1);
  const int per_pass = kThreads / lanes;
  for (int i0 = 0; i0 < n_resp; i0 += per_pass) {     // uniform: the lanes of a wavefront merge across groups below
    const int i = i0 + threadIdx.x / lanes;
    Moments r{0, 0, 0};
    double a = 0.0;
    if (i < n_resp) {
      const int t1 = tiling.first(i + 1);
      int t = tiling.first(i) + l;
      Partials<kDiagWords>::Words q{};
      if (t < t1) q = partials.get(t);
      a = SELF ? (double)s_adv[i] : (double)advantage(rewards, i, group_size, p);
      while (t < t1) {
        const auto next = partials.get(min(t + lanes, t1 - 1));    // in flight while this one is folded
        const unsigned long long counts = __builtin_bit_cast(unsigned long long, q.v[kCounts]);
        r = merge(r, Moments{(double)(unsigned)counts, q.v[kMeanW], q.v[kM2W]});
        d[0] += q.v[kSumAbs];
        d[1] += q.v[kSumD];
        d[2] += q.v[kSumDp];
        d[3] += (double)(unsigned)(counts >> 32);
        q = next;
        t += lanes;
      }
    }
    for (int off = 1; off < (WIDE ? 64 : lanes); off <<= 1)   // uniform: every lane of the wavefront takes part
      r = merge(r, Moments{__shfl_xor(r.n, off), __shfl_xor(r.mean, off), __shfl_xor(r.m2, off)});
    if ((WIDE ? lane : l) != 0 || i >= n_resp) continue;   // lane 0 of the group goes on (WIDE: of each of its wavefronts)
    if (!WIDE || l == 0) adv_out[i] = (float)a;
    if (!WIDE) count_out[i] = (int)r.n;
    // token-level moments of A and A w_bar: A (the stored fp32 value) is constant over the response's rows, so these
    // have mean A mean(w_bar) and squared deviations A^2 m2(w_bar)
    const Moments of[3] = {r, Moments{r.n, a, 0.0}, Moments{r.n, a * r.mean, a * a * r.m2}};
    if (r.n == 0.0) continue;
#pragma unroll
    for (int k = 0; k < 3; ++k) m[k] = m[0].n == 0.0 || n_resp <= per_pass ? of[k] : merge(m[k], of[k]);
  }
  // over the wavefront, in two passes as in level 1: the mean as a difference from one lane's, then the deviations from it
  const unsigned long long some = __ballot(m[0].n != 0.0);
  if (some != 0) {                                     // uniform
    const int src = __builtin_ctzll(some);
    const double n = wave_sum(m[0].n), inv = reciprocal(n);
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      const double x0 = lane_value(m[k].mean, src);
      const double mean = x0 + wave_sum(m[k].n * (m[k].mean - x0)) * inv;
      const double e = m[k].mean - mean;
      m[k].m2 = wave_sum(m[k].m2 + m[k].n * (e * e));
      m[k].mean = mean;
    }
#pragma unroll
    for (int k = 0; k < 3; ++k) m[k].n = n;
  }
#pragma unroll
  for (int k = 0; k < 4; ++k) d[k] = wave_sum(d[k]);
  if (lane == 0) {
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      lds[(4 * k + 0) * kWaves + wave] = m[k].n;
      lds[(4 * k + 1) * kWaves + wave] = m[k].mean;
      lds[(4 * k + 2) * kWaves + wave] = m[k].m2;
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) lds[(4 * k + 3) * kWaves + wave] = d[k];
  }
  __syncthreads();
  if (wave != 0) return;
  if (WIDE && lane < n_resp) {                         // responses of several wavefronts, one pass: their parts' counts
    double n = 0.0;
    for (int w = 0; w < lanes >> 6; ++w) n += lds[lane * (lanes >> 6) + w];
    count_out[lane] = (int)n;
  }
  // over the workgroup: 16 lanes for each of w_bar, A, A w_bar (and nothing), one for each wavefront; the sums likewise
  static_assert(kWaves == 16, "four groups of 16 lanes");
  const int v = lane & 15, set = lane >> 4, mine = 4 * min(set, 2) * kWaves + v;
  Moments b{lds[mine], lds[mine + kWaves], lds[mine + 2 * kWaves]};
  double sum = lds[(4 * set + 3) * kWaves + v];
  b = merge_level<0>(b);
  b = merge_level<1>(b);
  b = merge_level<2>(b);
  b = merge_level<3>(b);
  sum += butterfly<0>(sum);
  sum += butterfly<1>(sum);
  sum += butterfly<2>(sum);
  sum += butterfly<3>(sum);

  ais_diag out;
  const double N = b.n;
  out.n_valid = (long long)N;
  out.status = get_device(status);
  out.reserved = 0;
  if (N == 0.0) {
    out.mean_w = out.var_w = out.cv2 = out.dbar = out.std_a = out.std_aw = out.dsigma = 0.0;
    out.ess_ratio = 1.0; out.alpha_ess = 1.0; out.alpha_mis = 0.0; out.alpha_var = 0.0; out.clip_frac = 0.0;
    out.alpha = 0.0; out.kl_roll_train = 0.0; out.mean_abs_dp = 0.0;
  } else {
    const double var = b.m2 / N, std = sqrt(var), mean_sum = sum / N;
    out.mean_w = lane_value(b.mean, 0);
    out.var_w = lane_value(var, 0);
    out.std_a = lane_value(std, 16);
    out.std_aw = lane_value(std, 32);
    out.dbar = lane_value(mean_sum, 0);                             // Eq. 13
    out.kl_roll_train = -lane_value(mean_sum, 16);   // tokens were drawn from pi_roll: mean of log pi_roll - log pi_train
    out.mean_abs_dp = lane_value(mean_sum, 32);
    out.clip_frac = lane_value(mean_sum, 48);
    // three quotients: std / mean of w_bar (mean^2 alone may underflow); Eq. 14; Eq. 15.  Where every truncated ratio
    // underflowed to 0, CV^2 is 0 / 0 and read as 0 (equal weights), like the empty batch; with eps_std = 0 and all
    // advantages equal the ratio of Eq. 15 is 0 / 0: nothing to amplify, read as 0.
    const double num = lane == 0 ? lane_value(std, 0) : lane == 1 ? out.dbar : out.std_aw;
    const double den = lane == 0 ? out.mean_w : lane == 1 ? (double)p.delta : out.std_a + (double)p.eps_std;
    const double q = den > 0.0 ? num / den : 0.0;
    const double cv = lane_value(q, 0);
    out.cv2 = cv * cv;
    out.alpha_mis = fmin(1.0, lane_value(q, 1));
    out.dsigma = lane_value(q, 2);
    const double gamma = (double)p.gamma;
    const double q2 = (lane == 0 ? 1.0 : out.dsigma - gamma) / (lane == 0 ? 1.0 + out.cv2 : gamma);
    out.ess_ratio = lane_value(q2, 0);
    out.alpha_ess = sqrt(out.ess_ratio);                            // Eq. 12
    out.alpha_var = fmax(0.0, lane_value(q2, 1));                   // Eq. 16
    const double rel = fmin(1.0, fmax(0.0, out.alpha_ess - (double)p.beta_var * out.alpha_var));
    out.alpha = rel * out.alpha_mis;                                // Eq. 17
  }
  if (p.alpha_override >= 0.f) out.alpha = (double)p.alpha_override;
  if (lane == 0) *diag_out = out;
}

// ---- level 1: a tile of one response per wavefront; level 2 in the last workgroup ------------------------------------
// A chunk of 256 rows (four per lane) is reduced in two passes over its registers: the sum of w_bar - x0, x0 being some
// row's w_bar, gives the mean, the squared deviations from it the spread.  Equal values have spread exactly 0, and each pass
// is six dependent additions where merging (count, mean, spread) triples lane by lane was six times ten.
// The four rows of a lane take turns in one copy of the code (three exponentials each): see diag_final for why.
template <bool SELF, bool WIDE>
__global__ __launch_bounds__(kThreads, 4) void diag_reduce_kernel(
    const float* __restrict__ logp_train, const float* __restrict__ logp_roll,
    const unsigned char* __restrict__ valid, long long n_rows, const long long* __restrict__ cu_rows, int n_resp,
    const int* __restrict__ tile_off, TileRule rule, double* partial, int lanes, int group_size,
    const float* __restrict__ rewards, ais_params p, double lnC, float* __restrict__ adv_out, int* __restrict__ count_out,
    ais_diag* __restrict__ diag_out, int* status, Tickets tickets) {
  __shared__ double lds[16 * kWaves];                // three sets of moments and four sums per wavefront
  __shared__ double own_partials[kDiagWords * kOwnTiles];
  __shared__ float s_rewards[SELF ? kSelfPlanResponses : 1], s_adv[SELF ? kSelfPlanResponses : 1];
  if (SELF && (int)threadIdx.x < n_resp) s_rewards[threadIdx.x] = rewards[threadIdx.x];
  Tiling<SELF> tiling;
  tiling.init(tile_off, cu_rows, n_resp, n_rows, rule.shift, rule.max_tiles, status);
  const int n_tiles = tiling.tiles();
  const Partials<kDiagWords> partials{partial, own_partials, rule.max_tiles, rule.max_tiles <= kOwnTiles};
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int per = (n_tiles + (int)gridDim.x - 1) / (int)gridDim.x;
  const int b0 = blockIdx.x * per, b1 = min(n_tiles, b0 + per);
  // the advantages, by the wavefronts that have no tile first
  auto advantages = [&] {
    const int i = kThreads - 1 - (int)threadIdx.x;
    if (SELF && i < n_resp) s_adv[i] = advantage(s_rewards, i, group_size, p);
  };
  if (b0 >= b1) {                                              // uniform: a workgroup without tiles
    __syncthreads();
    advantages();
  }
  for (int w0 = b0; w0 < b1; w0 += kWaves) {                   // uniform for the workgroup
    tiling.open(w0);
    const int b = w0 + wave;
    if (b >= b1) {
      if (w0 == b0) advantages();
      continue;
    }
    const Tile tile = tiling.tile(b, w0);
    float ltf[kLaneRows], lrf[kLaneRows];
    unsigned char live[kLaneRows] = {1, 1, 1, 1};
    auto load = [&](int c0) {                    // the chunk that begins at row c0 of the tile (rows past its end: its last)
#pragma unroll
      for (int k = 0; k < kLaneRows; ++k) {
        const unsigned r = min(c0 + 64 * k + lane, tile.len - 1);
        ltf[k] = logp_train[tile.row0 + r];
        lrf[k] = logp_roll[tile.row0 + r];
      }
      if (valid != nullptr) {
#pragma unroll
        for (int k = 0; k < kLaneRows; ++k) live[k] = valid[tile.row0 + (unsigned)min(c0 + 64 * k + lane, tile.len - 1)];
      }
    };
    Moments mw{0, 0, 0};
    double sabs = 0, sd = 0, sdp = 0;
    int nclip = 0;
    if (tile.len > 0) load(0);
    if (w0 == b0) advantages();                                // while the rows are on their way
    for (int c0 = 0; c0 < tile.len; c0 += kChunkRows) {        // uniform for the wavefront
      double w[kLaneRows] = {}, some = 0;
      bool was[kLaneRows] = {}, any = false;
      int cnt = 0;
      const int n_k = min(kLaneRows, (tile.len - c0 + 63) >> 6);
#pragma unroll 1
      for (int k = 0; k < n_k; ++k) {
        const double lt = (double)ltf[0], lr = (double)lrf[0];
        const double d = lt - lr;                              // log rho (Alg. 1, sampler-trainer ratio)
        const double wk = exp(fmin(d, lnC));                   // w_bar = min(rho, C) (Eq. 10)
        const double dp = fabs(exp(lt) - exp(lr));
        const bool o = c0 + 64 * k + lane < tile.len && live[0] != 0;
        cnt += (int)__popcll(__ballot(o));
        sabs += o ? fabs(d) : 0.0;
        sd += o ? d : 0.0;
        sdp += o ? dp : 0.0;
        nclip += (int)__popcll(__ballot(o && d > lnC));
        some = o && !any ? wk : some;
        any |= o;
#pragma unroll
        for (int j = 0; j < kLaneRows - 1; ++j) {              // the lane's next row, and room for the one after this
          ltf[j] = ltf[j + 1];
          lrf[j] = lrf[j + 1];
          live[j] = live[j + 1];
          w[kLaneRows - 1 - j] = w[kLaneRows - 2 - j];
          was[kLaneRows - 1 - j] = was[kLaneRows - 2 - j];
        }
        w[0] = wk;
        was[0] = o;
      }
      if (c0 + kChunkRows < tile.len) load(c0 + kChunkRows);   // on its way while this chunk is folded
      const unsigned long long some_mask = __ballot(any);
      if (some_mask == 0) continue;                            // uniform
      const double x0 = lane_value(some, __builtin_ctzll(some_mask));
      double dev = 0;
#pragma unroll
      for (int k = 0; k < kLaneRows; ++k) {
        w[k] = was[k] ? w[k] - x0 : 0.0;
        dev += w[k];
      }
      const double mean = wave_sum(dev) * reciprocal((double)cnt);
      double m2 = 0;
#pragma unroll
      for (int k = 0; k < kLaneRows; ++k) {
        const double e = was[k] ? w[k] - mean : 0.0;
        m2 += e * e;
      }
      mw = merge(mw, Moments{(double)cnt, x0 + mean, wave_sum(m2)});
    }
    sabs = wave_sum(sabs);
    sd = wave_sum(sd);
    sdp = wave_sum(sdp);
    if (lane == 0) {
      const unsigned long long counts = (unsigned long long)(unsigned)nclip << 32 | (unsigned)mw.n;
      partials.put(b, {mw.mean, mw.m2, sabs, sd, sdp, __builtin_bit_cast(double, counts)});
    }
  }
  // ---- level 2, in the workgroup that finishes last ----
  if (last_workgroup(tickets))
    diag_final<SELF, WIDE>(partials, tiling, n_resp, lanes, group_size, rewards, s_adv, p, adv_out, count_out, diag_out, status,
                     lds);
}

// ---- per-row coefficient of the gradient, rectification weight, loss ------------------------------------------------
template <bool SELF>
__global__ __launch_bounds__(kThreads, 4) void row_coeff_kernel(
    CoeffInputs in, long long n_rows, const int* __restrict__ tile_off, TileRule rule, double* partial,
    float* __restrict__ g_out, float* __restrict__ wtilde_out, float g_scale, double* __restrict__ loss_out, int* status,
    Tickets tickets) {
  __shared__ double lds[kWaves];
  __shared__ double own_partials[kOwnTiles];
  const CoeffRule coeff(in.p, in.diag->alpha, in.lnC, in.logp_old != nullptr, in.logp_ref != nullptr);
  Tiling<SELF> tiling;
  tiling.init(tile_off, in.cu_rows, in.n_resp, n_rows, rule.shift, rule.max_tiles, status);
  const int n_tiles = tiling.tiles();
  const Partials<1> partials{partial, own_partials, rule.max_tiles, rule.max_tiles <= kOwnTiles};
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int per = (n_tiles + (int)gridDim.x - 1) / (int)gridDim.x;
  const int b0 = blockIdx.x * per, b1 = min(n_tiles, b0 + per);
  for (int w0 = b0; w0 < b1; w0 += kWaves) {                   // uniform for the workgroup
    tiling.open(w0);
    const int b = w0 + wave;
    if (b >= b1) continue;
    const Tile tile = tiling.tile(b, w0);
    const float a32 = in.adv[tile.resp];
    const int cnt = in.count[tile.resp];
    float ltf[kLaneRows], rollf[kLaneRows], oldf[kLaneRows], reff[kLaneRows];
    unsigned char live[kLaneRows] = {1, 1, 1, 1};
    auto load = [&](int c0) {                    // the chunk that begins at row c0 of the tile (rows past its end: its last)
      unsigned r[kLaneRows];
#pragma unroll
      for (int k = 0; k < kLaneRows; ++k) {
        r[k] = tile.row0 + (unsigned)min(c0 + 64 * k + lane, tile.len - 1);
        ltf[k] = in.logp_train[r[k]];
        rollf[k] = in.logp_roll[r[k]];
      }
      if (coeff.has_old) {
#pragma unroll
        for (int k = 0; k < kLaneRows; ++k) oldf[k] = in.logp_old[r[k]];
      }
      if (coeff.kl) {
#pragma unroll
        for (int k = 0; k < kLaneRows; ++k) reff[k] = in.logp_ref[r[k]];
      }
      if (in.valid != nullptr) {
#pragma unroll
        for (int k = 0; k < kLaneRows; ++k) live[k] = in.valid[r[k]];
      }
    };
    if (tile.len > 0) load(0);
    const double a = (double)a32;
    const double wgt = response_weight(in.n_resp, cnt);
    double acc = 0;
    for (int c0 = 0; c0 < tile.len; c0 += kChunkRows) {        // uniform for the wavefront
      const int n_k = min(kLaneRows, (tile.len - c0 + 63) >> 6);
      // the four rows of a lane take turns in one copy of the code
#pragma unroll 1
      for (int k = 0; k < n_k; ++k) {
        float g = 0.f, wt = 0.f;
        const int r = c0 + 64 * k + lane;
        if (r < tile.len && live[0] != 0) {
          const RowTerm t = row_term(coeff, ltf[0], rollf[0], oldf[0], reff[0], a);
          acc -= wgt * t.obj;
          g = (float)(wgt * t.dobj * (double)g_scale);
          wt = (float)t.wtilde;
        }
        if (r < tile.len) {
          g_out[tile.row0 + (unsigned)r] = g;
          if (wtilde_out != nullptr) wtilde_out[tile.row0 + (unsigned)r] = wt;
        }
#pragma unroll
        for (int j = 0; j < kLaneRows - 1; ++j) {
          ltf[j] = ltf[j + 1];
          rollf[j] = rollf[j + 1];
          oldf[j] = oldf[j + 1];
          reff[j] = reff[j + 1];
          live[j] = live[j + 1];
        }
      }
      if (c0 + kChunkRows < tile.len) load(c0 + kChunkRows);
    }
    acc = wave_sum(acc);
    if (lane == 0) partials.put(b, {acc});
  }
  if (!last_workgroup(tickets)) return;
  double acc = 0;
#pragma unroll 4
  for (int t = threadIdx.x; t < n_tiles; t += kThreads) acc += partials.get(t).v[0];
  acc = wave_sum(acc);
  if (lane == 0) lds[wave] = acc;
  __syncthreads();
  if (wave != 0) return;
  acc = lds[lane & (kWaves - 1)];
  acc += butterfly<0>(acc);
  acc += butterfly<1>(acc);
  acc += butterfly<2>(acc);
  acc += butterfly<3>(acc);
  if (threadIdx.x == 0) *loss_out = acc;
}

// Workgroups of a reduction: a tile per wavefront, four or more wavefronts at work in each, on as many compute units as
// that gives; one workgroup alone where it has a wavefront for every tile: its partials stay in LDS and it takes no ticket,
// 2 to 3 us less.  (Alone up to 64 tiles, four rounds: 4,096 rows in 16 responses 11.4 and 8.0 us instead of 10.5 and 7.2.)
int reduction_grid(const ais_ctx* ctx, int max_tiles) {
  if (max_tiles <= kOwnTiles) return 1;
  const int per = std::max(4, (max_tiles + ctx->n_cus - 1) / ctx->n_cus);
  return (max_tiles + per - 1) / per;
}

// A launch of one workgroup neither takes a ticket nor clears the other's, so it is not counted as a turn: launches of many
// workgroups would otherwise, with such ones between them, come to the same ticket every time.
Tickets take_tickets(ais_ctx* ctx, bool in_static, int grid) {
  int* pair = ctx->status_dev + (in_static ? kStaticTicketWord : kTicketWord);
  unsigned& turns = in_static ? ctx->static_turns : ctx->turns;
  const unsigned turn = (grid > 1 ? turns++ : turns) & 1u;
  return Tickets{pair + turn, pair + (turn ^ 1u)};
}

}  // namespace

// Tiles of 256 rows, or twice, four times, ... as many where that would be more than kMaxTiles; of kPlanTileRows where
// the plan kernel lays them out.  With kMaxTiles and 1,024 responses every tile has a wavefront at one workgroup per compute
// unit.  (8,192: 1,200,000 rows in 1,024 responses 25.7 and 18.4 instead of 21.9 and 17.2 us; 1,536: 25.3 and 23.0.  Tiles of
// 64 rows while they are few: 41,643 rows in 16 responses 14.1 and 7.9 instead of 13.7 and 7.7, both with a longer level 2 than
// the present one, which makes the latter 11.1.)
constexpr int kMaxTiles = 3072;
TileRule tile_rule(long long n_rows, int n_resp) {
  int shift = 8;
  if (n_resp > kSelfPlanResponses) {
    static_assert(kPlanTileRows == 1 << 10, "shift below");
    shift = 10;
  } else {
    while (((n_rows + (1LL << shift) - 1) >> shift) > kMaxTiles) ++shift;
  }
  return TileRule{shift, (int)((n_rows + (1LL << shift) - 1) >> shift) + n_resp};
}

// Monotone in both arguments, so that a call at the largest batch sizes the workspace for all others: the partials have
// room for kMaxTiles tiles of whole responses as soon as there are that many rows, whatever rule cuts them.
WorkspaceLayout workspace_layout(long long n_rows, int n_resp) {
  auto up = [](size_t v) { return (v + 255) & ~size_t(255); };
  const long long fine = std::min<long long>((n_rows + kChunkRows - 1) / kChunkRows, kMaxTiles);
  const long long planned = (n_rows + kPlanTileRows - 1) / kPlanTileRows;
  const size_t tiles = (size_t)(std::max(fine, planned) + n_resp);
  WorkspaceLayout w;
  w.tile_off = 0;
  w.partial = up(w.tile_off + sizeof(int) * (size_t)(n_resp + 2));
  w.g = up(w.partial + sizeof(double) * kDiagWords * tiles);
  w.total = up(w.g + sizeof(float) * (size_t)n_rows);
  return w;
}

// The documented limit of ais_diagnostics_static, 56 bytes for each of the tiles of 1,024 rows that the batch may have
// beside 4 for each response: at least what tiling and partials take under either rule.
size_t static_scratch_bytes(long long n_rows, int n_resp) {
  auto up = [](size_t v) { return (v + 255) & ~size_t(255); };
  static_assert(sizeof(double) * kDiagWords <= 56, "partials of planned tiles fit what is documented");
  static_assert(sizeof(int) * (kSelfPlanResponses + 2) + 256 +
                        sizeof(double) * kDiagWords * (kMaxTiles + kSelfPlanResponses) <= AIS_STATIC_SCRATCH_BYTES,
                "those of other batches always fit");
  return up(up(sizeof(int) * (size_t)(n_resp + 2)) +
            56 * ((size_t)((n_rows + kPlanTileRows - 1) / kPlanTileRows) + (size_t)n_resp));
}

// Writes the tiling for batches of more responses than a workgroup works out for itself; nothing to do otherwise.
int launch_plan(ais_ctx* ctx, const long long* cu_rows, int n_resp, long long n_rows, int* tile_off) {
  if (n_resp <= kSelfPlanResponses) return AIS_OK;
  plan_kernel<<<1, kPlanThreads, 0, ctx->stream>>>(cu_rows, n_resp, n_rows, tile_off,
                                                   tile_rule(n_rows, n_resp).max_tiles, ctx->status_dev);
  return hip_fail(ctx, hipGetLastError());
}

int launch_diagnostics(ais_ctx* ctx, const float* logp_train, const float* logp_roll, const unsigned char* valid,
                       long long n_rows, const long long* cu_rows, int n_resp, int group_size,
                       const float* rewards, const ais_params& p, int* tile_off, double* partial, bool in_static,
                       float* adv_out, int* count_out, ais_diag* diag_out) {
  const TileRule rule = tile_rule(n_rows, n_resp);
  const int lanes = fold_lanes(n_resp, (n_rows + (1LL << rule.shift) - 1) >> rule.shift);
  auto kernel = n_resp > kSelfPlanResponses ? diag_reduce_kernel<false, false>
                : lanes > 64                ? diag_reduce_kernel<true, true>
                                            : diag_reduce_kernel<true, false>;
  const int grid = reduction_grid(ctx, rule.max_tiles);
  kernel<<<grid, kThreads, 0, ctx->stream>>>(
      logp_train, logp_roll, valid, n_rows, cu_rows, n_resp, tile_off, rule, partial, lanes, group_size, rewards, p,
      std::log((double)p.C), adv_out, count_out, diag_out, ctx->status_dev, take_tickets(ctx, in_static, grid));
  return hip_fail(ctx, hipGetLastError());
}

int launch_row_coeff(ais_ctx* ctx, const CoeffInputs& in, long long n_rows, int* tile_off, double* partial, float* g_out,
                     float* wtilde_out, double* loss_out, float g_scale) {
  auto kernel = in.n_resp <= kSelfPlanResponses ? row_coeff_kernel<true> : row_coeff_kernel<false>;
  const TileRule rule = tile_rule(n_rows, in.n_resp);
  const int grid = reduction_grid(ctx, rule.max_tiles);
  kernel<<<grid, kThreads, 0, ctx->stream>>>(
      in, n_rows, tile_off, rule, partial, g_out, wtilde_out, g_scale, loss_out, ctx->status_dev,
      take_tickets(ctx, false, grid));
  return hip_fail(ctx, hipGetLastError());
}

}  // namespace ais
