// Per-row scalar work and the batch-wide reductions of the path.
//
// The batch is a set of variable-length segments (responses) of rows, some rows masked out.  Up to kSelfPlanResponses responses
// the rows are dealt out evenly to at most one workgroup per compute unit, whatever responses they belong to: a row finds its
// response by its number, and everything that depends on the response alone is in LDS.  Beyond that a small plan kernel cuts
// every response into tiles of 1,024 rows and a wavefront takes a tile.  Level 1 reduces a workgroup's rows (or a tile) to a
// partial; level 2, run by whichever workgroup of the same launch finishes last, merges the partials in order and evaluates the
// three diagnostics and the mixing coefficient (Eq. 12-17).  Everything is accumulated in fp64 in a fixed order (no floating
// point atomics), so results are bit-reproducible from run to run.  Spreads are carried as sums of differences from a value of
// the set, and summed again about the mean where that value lies far from it (kFarSpread), or as (count, mean, squared
// deviations): 1,200,000 ratios near 1 whose first is truncated at 5 have a variance right to 1e-15 of itself (1.2e-10 about that
// first value alone).
//
// These kernels move a few bytes per row (about a megabyte per batch) and are bound by the length of their dependent chains, by
// the instruction fetches of code that runs once, and from some 500,000 rows on by fp64 instructions: 150 of them a row, 840
// cycles for 64 rows before and 550 now.  Hence rows asked for before anything else, one copy of the code for all rows of a
// thread, exponentials of 20 instructions (row_coeff.h) and two of them where there were three, sums over the workgroup through
// LDS (see MergeRoom).  Diagnostics and row coefficients, us a call in a graph of forty, tiles of responses dealt to wavefronts
// before and rows dealt out evenly now: 512 rows in 8 responses 7.8 and 4.4 -> 5.7 and 3.5; 2,048 in 8 9.5 and 5.5 -> 7.4 and 5.0;
// 2,432 masked in 128 8.5 and 5.4 -> 8.0 and 4.9; 19,968 masked in 128 9.6 and 6.5 -> 8.4 and 5.3; 41,643 in 16 10.8 and 6.7 -> 8.1
// and 5.6; 108,495 in 104 13.1 and 7.6 -> 9.1 and 6.6; 299,000 masked in 1,024 16.9 and 9.4 -> 12.8 and 9.8; 1,200,000 in 1,024 26.0
// and 13.5 -> 15.3 and 13.6; 4,000,000 in 8 33.6 and 26.2 -> 24.6 and 23.8.
#include "ais_internal.h"
#include "row_coeff.h"

#include <algorithm>
#include <cmath>
#include <type_traits>

namespace ais {
namespace {

using dev::CoeffRule;
using dev::RowTerm;
using dev::exp64;
using dev::exp64_finite;
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

constexpr int kThreads = 1024;
constexpr int kWaves = kThreads / 64;
constexpr int kLaneRows = 4;                     // rows of a lane whose inputs are loaded together
constexpr int kChunkRows = 64 * kLaneRows;       // rows of a wavefront that are
constexpr int kAtOnce = 8;                       // the same, where rows are dealt out evenly

// Rows [row0, row0 + len) of response `resp`, the work of one wavefront.
struct Tile {
  int resp, row0, len;
};

// The tiling of a batch of more than kSelfPlanResponses responses, from the plan kernel's array in memory.
struct Tiling {
  const int* tile_off;
  const long long* cu_rows;
  int n_resp, n_rows;
  __device__ __forceinline__ int tiles() const { return tile_off[n_resp]; }
  __device__ __forceinline__ int first(int i) const { return tile_off[i]; }
  __device__ __forceinline__ Tile tile(int b) const {
    const int i = find_response(tile_off, n_resp, b);
    long long lo, hi;
    response_rows(cu_rows, i, n_rows, lo, hi);
    const long long r0 = lo + (long long)(b - tile_off[i]) * kPlanTileRows;
    const int len = (int)min(hi - r0, (long long)kPlanTileRows);
    return Tile{__builtin_amdgcn_readfirstlane(i), __builtin_amdgcn_readfirstlane((int)r0),
                __builtin_amdgcn_readfirstlane(len)};
  }
};

// The responses of a batch of up to kSelfPlanResponses, a thread each: their rows, forced into [0, n_rows], in LDS, so that a row
// finds its own whatever way the rows are dealt out.
struct Responses {
  int lo[kSelfPlanResponses], hi[kSelfPlanResponses];
  // Must be called by all threads of the workgroup, and a barrier before search().  Workgroup 0 reports a cu_rows that is no
  // partition of the rows.
  __device__ __forceinline__ void init(const long long* __restrict__ cu, int n_resp, long long n_rows, int* status) {
    static_assert(kSelfPlanResponses <= kThreads, "a thread per response");
    const int i = threadIdx.x;
    int l = 0x7fffffff, h = 0;
    if (i < n_resp) {
      const long long c0 = cu[i], c1 = cu[i + 1];
      l = (int)clampll(c0, 0, n_rows);
      h = (int)clampll(c1, l, n_rows);
      const bool bad = c0 != l || c1 != h || (i == 0 && c0 != 0) || (i == n_resp - 1 && c1 != n_rows);
      if (bad && blockIdx.x == 0) {
        atomicOr(status, AIS_STATUS_BAD_CU);
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");       // a workgroup alone reads the word after no more than barriers
      }
    }
    if (i < kSelfPlanResponses) {
      lo[i] = l;
      hi[i] = h;
    }
  }
  // The last response that begins at row `first` or before it, and that of row `last` (both uniform): 32 lanes look for either, 32
  // responses at a step.
  __device__ __forceinline__ void of_both(int first, int last, int& i_first, int& i_last) const {
    const int lane = threadIdx.x & 63, in = lane & 31, row = lane < 32 ? first : last;
    auto count = [](unsigned long long below, int& f, int& l) {
      f = max(__popc((unsigned)below) - 1, 0);
      l = max(__popc((unsigned)(below >> 32)) - 1, 0);
    };
    int f, l, f2, l2;
    static_assert(kSelfPlanResponses == 32 * 32, "two steps");
    count(__ballot(lo[32 * in] <= row), f, l);
    count(__ballot(lo[32 * (lane < 32 ? f : l) + in] <= row), f2, l2);
    i_first = 32 * f + f2;
    i_last = 32 * l + l2;
  }
  // The same for a row of each lane, among the responses from `first` to `last` (uniform): those of the rows at either end.  Every step
  // waits for LDS, and there is one where the rows have two responses.  (Among all responses, row coefficients of 335,307 rows in
  // 1,024 10.12 us and diagnostics 12.11; now 9.83 and 11.88; diagnostics of 41,643 in 1,024 9.15 and 8.83.)
  __device__ __forceinline__ int search(int row, int first, int last) const {
    int i = first;
    for (int step = last > first ? 1 << (31 - __builtin_clz(last - first)) : 0; step > 0; step >>= 1)        // uniform
      if (i + step <= last && lo[i + step] <= row) i += step;
    return i;
  }
  // Whether response i, which has been found for the row, holds it: it does unless cu_rows is no partition.
  __device__ __forceinline__ bool holds(int i, int row) const { return lo[i] <= row && row < hi[i]; }
};

// The rows of a wavefront, one run of them, 64 at a time: while they stay inside a response it is looked for once.
struct WaveRows {
  int first, end;                                    // uniform, as all of this
  int i = 0, last = 0;                               // responses of the first and the last of the turn's 64
  int lo = 1, hi = 0;                                // rows of i, if it held the last 64
  __device__ __forceinline__ WaveRows(int r0, int r1, int rows_each) {
    const int run = ((rows_each + kWaves - 1) / kWaves + 63) / 64 * 64;
    const int at = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6) * run;
    first = at < r1 - r0 ? r0 + at : r1;
    end = run < r1 - first ? first + run : r1;
  }
  __device__ __forceinline__ int turns() const { return (end - first + 63) >> 6; }
  // Row of this lane in turn k (past the end: the last).
  __device__ __forceinline__ int row(int k) const {
    return (int)min((unsigned)first + 64 * k + (threadIdx.x & 63), (unsigned)(end - 1));
  }
  __device__ __forceinline__ bool in(int k) const { return (unsigned)first + 64 * k + (threadIdx.x & 63) < (unsigned)end; }
  // Whether the rows of turn k have a response in common, which is i then.
  __device__ __forceinline__ bool common(const Responses& resp, int k) {
    const int a = first + 64 * k, b = min(63, end - 1 - a) + a;
    if (lo <= a && b < hi) return true;
    resp.of_both(a, b, i, last);
    if (i == last) {
      lo = __builtin_amdgcn_readfirstlane(resp.lo[i]);
      hi = __builtin_amdgcn_readfirstlane(resp.hi[i]);
      if (lo <= a && b < hi) return true;
    }
    lo = 1;
    hi = 0;
    return false;
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

// The partials of the tiles or workgroups, NW words each, as arrays of words: lanes that read consecutive ones read consecutive
// words.
template <int NW>
struct Partials {
  double* global;
  int stride;
  struct Words { double v[NW]; };
  __device__ __forceinline__ void put(int tile, const Words& q) const {
    double* to = global + tile;
#pragma unroll
    for (int k = 0; k < NW; ++k) put_device(to + (size_t)k * stride, q.v[k]);
  }
  __device__ __forceinline__ Words get(int tile) const {
    Words q;
    const double* from = global + tile;
#pragma unroll
    for (int k = 0; k < NW; ++k) q.v[k] = get_device(from + (size_t)k * stride);
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

// What a row brings to the diagnostics: d = log rho (Alg. 1, sampler-trainer ratio), w_bar = min(rho, C) (Eq. 10) and
// |pi_train - pi_roll|.  Two exponentials for three quantities: e^-|d|, whose reciprocal the ratio is where it exceeds 1, and
// the larger probability, of which 1 - e^-|d| is the part that the smaller one lacks.
struct RowRatio {
  double d, w, dp;
};
__device__ __forceinline__ RowRatio row_ratio(float train, float roll, double lnC, double C) {
  const double t = (double)train, l = (double)roll;
  RowRatio r;
  r.d = t - l;
  // (of a NaN the sums tell: the ratio counts as truncated)
  const double less = exp64_finite(fmax(-fabs(r.d), -800.0));
  const double most = exp64(__builtin_isunordered(train, roll) ? __builtin_nan("") : fmax(t, l));
  const double rho = r.d <= 0.0 ? less : reciprocal(less);
  r.w = r.d <= lnC ? fmin(rho, C) : C;
  r.dp = most * (1.0 - less);
  return r;
}

// Sums of a set of values as differences from x0, one of them or their mean: sum (x - x0), sum (x - x0)^2.  Values that are all
// equal have both exactly 0, whatever parts they were summed in.
struct Shifted {
  double x0, s1, s2;
  __device__ __forceinline__ void add(double x) {
    const double e = x - x0;
    s1 += e;
    s2 = fma(e, e, s2);
  }
  __device__ __forceinline__ void rebase(double n, double to) {      // of n values; of none: stays 0
    const double e = x0 - to, ne = n * e;
    s2 = fma(e, s1 + s1 + ne, s2);
    s1 += ne;
    x0 = to;
  }
};

// The rows of a thread, a wavefront or a workgroup as the diagnostics see them: their number, w_bar, A and A w_bar over them, and
// the sums of |d|, d, |dp| and of rows with rho > C.
struct RowSums {
  double n;
  Shifted x[3];
  double d[4];
};
constexpr int kRowSums = 11, kRowWords = kRowSums + 3;      // n, s1 of the three sets, their s2, the four sums; and the three x0
// Sums of squares about x0 that are more than so many times the spread lose the digits by which they are: s2 = spread + n (x0 -
// mean)^2, and its rounding goes with the whole of it.
constexpr double kFarSpread = 16.0;
template <typename F>
__device__ __forceinline__ void each_sum(RowSums& r, F&& f) {
  f(0, r.n);
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    f(1 + k, r.x[k].s1);
    f(4 + k, r.x[k].s2);
  }
#pragma unroll
  for (int k = 0; k < 4; ++k) f(7 + k, r.d[k]);
}
// Over the workgroup, in all threads' words[]: a thread with rows gives its x0 to all, and the sums, eleven for each of 1,024
// threads, are added by a wavefront each from LDS, lane by lane over the wavefronts and then over the lanes.  (Six exchanges
// across the lanes of all sixteen wavefronts for every sum, and four more in one of them, were 4 us of 10 twice over.)
struct MergeRoom {
  double sum[kRowSums * kThreads], words[kRowWords];
  int first;
};
__device__ __forceinline__ void merge_workgroup(const RowSums& r, MergeRoom& room) {
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  if (tid == 0) room.first = kThreads;
  __syncthreads();
  const unsigned long long some = __ballot(r.n != 0.0);
  if (some != 0 && lane == 0) atomicMin(&room.first, (tid & ~63) + __builtin_ctzll(some));
  if (tid < 3) room.words[kRowSums + tid] = 0.0;
  __syncthreads();
  if (tid == room.first) {
#pragma unroll
    for (int k = 0; k < 3; ++k) room.words[kRowSums + k] = r.x[k].x0;
  }
  __syncthreads();
  RowSums about = r;
#pragma unroll
  for (int k = 0; k < 3; ++k) about.x[k].rebase(r.n, room.words[kRowSums + k]);
  each_sum(about, [&](int k, double& v) { room.sum[k * kThreads + tid] = v; });
  __syncthreads();
  auto add = [&](int sums) {                           // the first of them, a wavefront each
    if (wave < sums) {
      double v = 0;
#pragma unroll
      for (int w = 0; w < kWaves; ++w) v += room.sum[wave * kThreads + 64 * w + lane];
      v = wave_sum(v);
      if (lane == 0) room.words[wave] = v;
    }
    __syncthreads();
  };
  add(kRowSums);
  // A spread about x0 is the difference of its two sums.  Where x0 lies so far from the mean that this costs digits, the sums are
  // taken again, about the mean.
  const double n = room.words[0];
  bool far = false;
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    const double s1 = room.words[1 + k], s2 = room.words[4 + k];
    far |= kFarSpread * s1 * s1 > (kFarSpread - 1.0) * n * s2;
  }
  if (!far) return;                                    // uniform
  const double share = reciprocal(n);
  double mean[3];
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    mean[k] = fma(room.words[1 + k], share, room.words[kRowSums + k]);
    Shifted x = r.x[k];
    x.rebase(r.n, mean[k]);
    room.sum[(1 + k) * kThreads + tid] = x.s1;
    room.sum[(4 + k) * kThreads + tid] = x.s2;
  }
  __syncthreads();
  if (tid < 3) room.words[kRowSums + tid] = tid == 0 ? mean[0] : tid == 1 ? mean[1] : mean[2];
  add(7);                                              // (the first, the number of rows, is what it was)
}

// Over the workgroups, in words[] of the one that finishes last (a barrier before they are read): a set or a sum to each of seven
// wavefronts, four workgroups to a lane, nothing but the result through LDS.  (As merge_workgroup does it, over as many threads as
// there are workgroups, 1,024 rows to a workgroup: 2,432 masked rows 9.9 us and 8.6 so, 19,968 10.3 and 8.9, 1,200,000 16.3 and 15.3.)
constexpr int kMostWorkgroups = 256;
__device__ __forceinline__ void merge_workgroups(const double* partial, int n_wg, MergeRoom& room) {
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if (wave >= 7) return;
  const bool set = wave < 3;                           // w_bar, A, A w_bar; the four sums are s1 of sets of no rows
  constexpr int kEach = kMostWorkgroups / 64;
  double n[kEach], s1[kEach], s2[kEach], x0[kEach];
#pragma unroll
  for (int k = 0; k < kEach; ++k) {
    const int b = lane + 64 * k;
    n[k] = s1[k] = s2[k] = x0[k] = 0.0;
    if (b < n_wg) {
      s1[k] = get_device(partial + (size_t)(set ? 1 + wave : 4 + wave) * n_wg + b);
      if (set) {
        n[k] = get_device(partial + b);
        s2[k] = get_device(partial + (size_t)(4 + wave) * n_wg + b);
        x0[k] = get_device(partial + (size_t)(kRowSums + wave) * n_wg + b);
      }
    }
  }
  double to = 0.0, rows = 0.0, t1, t2;
#pragma unroll
  for (int k = 0; k < kEach; ++k) {
    const unsigned long long some = __ballot(n[k] != 0.0);
    if (some != 0 && rows == 0.0) to = lane_value(x0[k], __builtin_ctzll(some));
    rows = some != 0 ? 1.0 : rows;
  }
  auto about = [&](double at) {
    rows = t1 = t2 = 0.0;
#pragma unroll
    for (int k = 0; k < kEach; ++k) {
      Shifted x{x0[k], s1[k], s2[k]};
      x.rebase(n[k], at);
      rows += n[k];
      t1 += x.s1;
      t2 += x.s2;
    }
    rows = wave_sum(rows);
    t1 = wave_sum(t1);
    t2 = wave_sum(t2);
  };
  about(to);
  if (kFarSpread * t1 * t1 > (kFarSpread - 1.0) * rows * t2 && set) {            // uniform; see merge_workgroup
    to = fma(t1, reciprocal(rows), to);
    about(to);
  }
  if (lane == 0) {
    if (wave == 0) room.words[0] = rows;
    room.words[set ? 1 + wave : 4 + wave] = t1;
    if (set) {
      room.words[4 + wave] = t2;
      room.words[kRowSums + wave] = to;
    }
  }
}

// ---- level 2: batch moments, diagnostics, alpha -----------------------------------------------------------------------
// The code runs once per launch, cold: its size is part of its time (a kilobyte of straight code costs 0.3 us of
// instruction fetches), so what is the same for several quantities is done once, by lanes that hold one each.  By wavefront 0:
// lanes 16 s .. 16 s + 15 hold the moments of w_bar, A and A w_bar (s = 0 .. 2) in `b` and the sums of |d|, d, |dp| and of rows
// with rho > C (0 .. 3) in `sum`.
__device__ __forceinline__ void diag_formulas(const Moments& b, double sum, const ais_params& p,
                                              ais_diag* __restrict__ diag_out, const int* status) {
  const int lane = threadIdx.x & 63;
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

// ---- diagnostics of up to kSelfPlanResponses responses -----------------------------------------------------------------
// Every workgroup takes rows_each rows, a run for each of its wavefronts, whatever responses they belong to: a row's advantage is known as soon
// as the rewards are, so a thread sums w_bar, A and A w_bar over its rows (see Shifted), and threads, wavefronts and workgroups
// are merged by plain sums of differences from one value.  What is loaded for the rows is asked for before anything else.
// Where there is a mask, a workgroup's number of valid rows of response i goes to word i + blockIdx of `counts`: the pairs of a
// response and a workgroup that share rows, in order, have words of their own.
__global__ __launch_bounds__(kThreads, 4) void diag_rows_kernel(
    const float* __restrict__ logp_train, const float* __restrict__ logp_roll, const unsigned char* __restrict__ valid,
    int n_rows, int rows_each, const long long* __restrict__ cu_rows, int n_resp, double* partial, int* counts,
    int group_size, const float* __restrict__ rewards, ais_params p, double lnC, float* __restrict__ adv_out,
    int* __restrict__ count_out, ais_diag* __restrict__ diag_out, int* status, Tickets tickets) {
  __shared__ Responses resp;
  __shared__ float s_rewards[kSelfPlanResponses], s_adv[kSelfPlanResponses];
  __shared__ int s_count[kSelfPlanResponses];
  __shared__ MergeRoom room;
  const int tid = threadIdx.x, lane = tid & 63;
  const int r0 = blockIdx.x * rows_each, r1 = n_rows - r0 < rows_each ? n_rows : r0 + rows_each;
  float lt[kAtOnce], lr[kAtOnce];
  unsigned char live[kAtOnce] = {1, 1, 1, 1, 1, 1, 1, 1};
  WaveRows wave_rows(r0, r1, rows_each);
  const int turns = wave_rows.turns();
  auto load = [&](int k0) {                          // those of turns k0 .. k0 + 7 (rows past the end: the last)
    auto four = [&](auto from) __attribute__((always_inline)) {
#pragma unroll
      for (int k = from.value; k < from.value + 4; ++k) {
        const int r = wave_rows.row(k0 + k);
        lt[k] = logp_train[r];
        lr[k] = logp_roll[r];
        if (valid != nullptr) live[k] = valid[r];
      }
    };
    four(std::integral_constant<int, 0>{});
    if (turns - k0 > 4) four(std::integral_constant<int, 4>{});
  };
  if (turns > 0) load(0);                            // uniform
  if (tid < n_resp) s_rewards[tid] = rewards[tid];
  resp.init(cu_rows, n_resp, n_rows, status);
  s_count[tid] = 0;
  __syncthreads();
  if (tid < n_resp) {
    const float a = advantage(s_rewards, tid, group_size, p);
    s_adv[tid] = a;
    if (blockIdx.x == 0) adv_out[tid] = a;
    if (valid == nullptr && blockIdx.x == 0) count_out[tid] = resp.hi[tid] - resp.lo[tid];
  }
  __syncthreads();
  RowSums sums = {};
  int n = 0;
  for (int k0 = 0; k0 < turns; k0 += kAtOnce) {                          // uniform
    // the rows take turns in one copy of the code
    const int k1 = min(turns, k0 + kAtOnce);
#pragma unroll 1
    for (int k = k0; k < k1; ++k) {
      const bool one = wave_rows.common(resp, k);                        // uniform
      const int i = one ? wave_rows.i : resp.search(wave_rows.row(k), wave_rows.i, wave_rows.last);
      const bool on = wave_rows.in(k) && live[0] != 0 && (one || resp.holds(i, wave_rows.row(k)));
      if (valid != nullptr) {
        const unsigned long long mask = __ballot(on);
        if (one) {
          if (lane == 0) atomicAdd(&s_count[i], (int)__popcll(mask));
        } else if (on) {
          atomicAdd(&s_count[i], 1);
        }
      }
      const RowRatio q = row_ratio(lt[0], lr[0], lnC, (double)p.C);
      const double a = (double)s_adv[i];
      const double x[3] = {q.w, a, a * q.w};
      if (on) {
        if (n++ == 0) {
#pragma unroll
          for (int s = 0; s < 3; ++s) sums.x[s].x0 = x[s];
        }
#pragma unroll
        for (int s = 0; s < 3; ++s) sums.x[s].add(x[s]);
        sums.d[0] += fabs(q.d);
        sums.d[1] += q.d;
        sums.d[2] += q.dp;
        sums.d[3] += q.d > lnC ? 1.0 : 0.0;
      }
#pragma unroll
      for (int j = 0; j < kAtOnce - 1; ++j) {                  // the thread's next row
        lt[j] = lt[j + 1];
        lr[j] = lr[j + 1];
        live[j] = live[j + 1];
      }
    }
    if (k1 < turns) load(k1);
  }
  sums.n = (double)n;
  const int n_wg = gridDim.x;
  merge_workgroup(sums, room);
  if (n_wg > 1) {                                                        // uniform
    if (tid < kRowWords) put_device(partial + (size_t)tid * n_wg + blockIdx.x, room.words[tid]);
    if (valid != nullptr && tid < n_resp && resp.lo[tid] < r1 && resp.hi[tid] > r0)
      put_device(counts + tid + (int)blockIdx.x, s_count[tid]);
    if (!last_workgroup(tickets)) return;
    merge_workgroups(partial, n_wg, room);
    if (valid != nullptr) {
      // the parts of a response's count: by its thread, those of responses with many by its wavefront, to which neighbours are
      // not dealt: it takes one after the other.  (60,000 masked rows in 16 responses, all of them in one wavefront and so: 13.7 and
      // 10.7 us; 11,000 in 1,024, none with many parts, 11.2 and 11.5 for the scattered words.)
      const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), r = wave + kWaves * lane;
      int b0 = 0, parts = 0, sum = 0;
      if (r < n_resp && resp.hi[r] > resp.lo[r]) {
        b0 = resp.lo[r] / rows_each;
        parts = (resp.hi[r] - 1) / rows_each - b0 + 1;
      }
      const int* mine = counts + r + b0;
#pragma unroll
      for (int k = 0; k < 4; ++k)
        if (k < parts && parts <= 4) sum += get_device(mine + k);
      for (unsigned long long many = __ballot(parts > 4); many != 0; many &= many - 1) {         // uniform
        const int src = __builtin_ctzll(many);
        const int first = __builtin_amdgcn_readlane(b0, src) + wave + kWaves * src, len = __builtin_amdgcn_readlane(parts, src);
        int part = 0;
        for (int k = lane; k < len; k += 64) part += get_device(counts + first + k);
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) part += __shfl_xor(part, off);
        if (lane == src) sum = part;
      }
      if (r < n_resp) count_out[r] = sum;
    }
    __syncthreads();
  } else if (valid != nullptr && tid < n_resp) {
    count_out[tid] = s_count[tid];
  }
  if (tid >= 64) return;
  // lanes 16 s .. 16 s + 15 go on with the set s and the sum s
  const int set = min(lane >> 4, 2);
  const double n_rows_in = room.words[0], s1 = room.words[1 + set], s2 = room.words[4 + set];
  const double share = reciprocal(fmax(n_rows_in, 1.0));
  const double spread = fma(-s1, s1 * share, s2);                // (below 0 by rounding: 0; a NaN stays one)
  const Moments b{n_rows_in, fma(s1, share, room.words[kRowSums + set]), spread < 0.0 ? 0.0 : spread};
  diag_formulas(b, room.words[7 + (lane >> 4)], p, diag_out, status);
}

// ---- diagnostics of more responses: a tile of one response per wavefront; level 2 in the last workgroup ---------------------
// A chunk of 256 rows (four per lane) is reduced in two passes over its registers: the sum of w_bar - x0, x0 being some
// row's w_bar, gives the mean, the squared deviations from it the spread.  Equal values have spread exactly 0, and each pass
// is six dependent additions where merging (count, mean, spread) triples lane by lane was six times ten.
// The four rows of a lane take turns in one copy of the code (two exponentials each): see diag_formulas for why.
__global__ __launch_bounds__(kThreads, 4) void diag_reduce_kernel(
    const float* __restrict__ logp_train, const float* __restrict__ logp_roll,
    const unsigned char* __restrict__ valid, long long n_rows, const long long* __restrict__ cu_rows, int n_resp,
    const int* __restrict__ tile_off, TileRule rule, double* partial, int group_size,
    const float* __restrict__ rewards, ais_params p, double lnC, float* __restrict__ adv_out, int* __restrict__ count_out,
    ais_diag* __restrict__ diag_out, int* status, Tickets tickets) {
  __shared__ double lds[16 * kWaves];                // three sets of moments and four sums per wavefront
  const Tiling tiling{tile_off, cu_rows, n_resp, (int)n_rows};
  const int n_tiles = tiling.tiles();
  const Partials<kDiagWords> partials{partial, rule.max_tiles};
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int per = (n_tiles + (int)gridDim.x - 1) / (int)gridDim.x;
  const int b0 = blockIdx.x * per, b1 = min(n_tiles, b0 + per);
  for (int b = b0 + wave; b < b1; b += kWaves) {               // uniform for the wavefront
    const Tile tile = tiling.tile(b);
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
    for (int c0 = 0; c0 < tile.len; c0 += kChunkRows) {        // uniform for the wavefront
      double w[kLaneRows] = {}, some = 0;
      bool was[kLaneRows] = {}, any = false;
      int cnt = 0;
      const int n_k = min(kLaneRows, (tile.len - c0 + 63) >> 6);
#pragma unroll 1
      for (int k = 0; k < n_k; ++k) {
        const RowRatio q = row_ratio(ltf[0], lrf[0], lnC, (double)p.C);
        const bool o = c0 + 64 * k + lane < tile.len && live[0] != 0;
        cnt += (int)__popcll(__ballot(o));
        sabs += o ? fabs(q.d) : 0.0;
        sd += o ? q.d : 0.0;
        sdp += o ? q.dp : 0.0;
        nclip += (int)__popcll(__ballot(o && q.d > lnC));
        some = o && !any ? q.w : some;
        any |= o;
#pragma unroll
        for (int j = 0; j < kLaneRows - 1; ++j) {              // the lane's next row, and room for the one after this
          ltf[j] = ltf[j + 1];
          lrf[j] = lrf[j + 1];
          live[j] = live[j + 1];
          w[kLaneRows - 1 - j] = w[kLaneRows - 2 - j];
          was[kLaneRows - 1 - j] = was[kLaneRows - 2 - j];
        }
        w[0] = q.w;
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
  if (!last_workgroup(tickets)) return;
  // ---- level 2: a thread folds the tiles of a response in order, and takes the next 1,024 responses after these
  Moments m[3] = {};                                           // of w_bar, of A and of A w_bar over the thread's valid rows
  double d[4] = {};
  for (int i = threadIdx.x; i < n_resp; i += kThreads) {
    Moments r{0, 0, 0};
    const int t1 = tiling.first(i + 1);
    int t = tiling.first(i);
    Partials<kDiagWords>::Words q{};
    if (t < t1) q = partials.get(t);
    const double a = (double)advantage(rewards, i, group_size, p);
    while (t < t1) {
      const auto next = partials.get(min(t + 1, t1 - 1));      // in flight while this one is folded
      const unsigned long long counts = __builtin_bit_cast(unsigned long long, q.v[kCounts]);
      r = merge(r, Moments{(double)(unsigned)counts, q.v[kMeanW], q.v[kM2W]});
      d[0] += q.v[kSumAbs];
      d[1] += q.v[kSumD];
      d[2] += q.v[kSumDp];
      d[3] += (double)(unsigned)(counts >> 32);
      q = next;
      ++t;
    }
    adv_out[i] = (float)a;
    count_out[i] = (int)r.n;
    // token-level moments of A and A w_bar: A (the stored fp32 value) is constant over the response's rows, so these
    // have mean A mean(w_bar) and squared deviations A^2 m2(w_bar)
    if (r.n == 0.0) continue;
    const Moments of[3] = {r, Moments{r.n, a, 0.0}, Moments{r.n, a * r.mean, a * a * r.m2}};
    const bool none = m[0].n == 0.0;
#pragma unroll
    for (int k = 0; k < 3; ++k) m[k] = none ? of[k] : merge(m[k], of[k]);
  }
  // over the wavefront in two passes: the mean as a difference from one lane's, then the deviations from it
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
  // over the workgroup: 16 lanes for each of w_bar, A, A w_bar (and nothing), one for each wavefront; the sums likewise
  static_assert(kWaves == 16, "four groups of 16 lanes");
  const int v = lane & 15, set = lane >> 4, mine = 4 * min(set, 2) * kWaves + v;
  Moments b{lds[mine], lds[mine + kWaves], lds[mine + 2 * kWaves]};
  b = merge_level<0>(b);
  b = merge_level<1>(b);
  b = merge_level<2>(b);
  b = merge_level<3>(b);
  double sum = lds[(4 * set + 3) * kWaves + v];
  sum += butterfly<0>(sum);
  sum += butterfly<1>(sum);
  sum += butterfly<2>(sum);
  sum += butterfly<3>(sum);
  diag_formulas(b, sum, p, diag_out, status);
}

// ---- per-row coefficient of the gradient, rectification weight, loss ------------------------------------------------
// The inputs of N rows of a thread.
template <int N>
struct CoeffRows {
  float lt[N], roll[N], old[N], ref[N];
  unsigned char live[N];
  // FROM .. FROM + 3
  template <int FROM, typename F>
  __device__ __forceinline__ void load(const CoeffInputs& in, const CoeffRule& rule, F&& row) {
    int r[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      r[k] = row(FROM + k);
      lt[FROM + k] = in.logp_train[r[k]];
      roll[FROM + k] = in.logp_roll[r[k]];
      old[FROM + k] = ref[FROM + k] = 0.f;
      live[FROM + k] = 1;
    }
    if (rule.has_old) {
#pragma unroll
      for (int k = 0; k < 4; ++k) old[FROM + k] = in.logp_old[r[k]];
    }
    if (rule.kl) {
#pragma unroll
      for (int k = 0; k < 4; ++k) ref[FROM + k] = in.logp_ref[r[k]];
    }
    if (in.valid != nullptr) {
#pragma unroll
      for (int k = 0; k < 4; ++k) live[FROM + k] = in.valid[r[k]];
    }
  }
  __device__ __forceinline__ void next() {           // the rows take turns in one copy of the code
#pragma unroll
    for (int j = 0; j < N - 1; ++j) {
      lt[j] = lt[j + 1];
      roll[j] = roll[j + 1];
      old[j] = old[j + 1];
      ref[j] = ref[j + 1];
      live[j] = live[j + 1];
    }
  }
};

// The loss from every workgroup's partials, `words` of them in all, in the workgroup that finishes last.
__device__ __forceinline__ void loss_final(const Partials<1>& partials, int words, double* lds, double* loss_out) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  double acc = 0;
#pragma unroll 4
  for (int t = threadIdx.x; t < words; t += kThreads) acc += partials.get(t).v[0];
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

// Up to kSelfPlanResponses responses: every workgroup takes rows_each rows (see diag_rows_kernel).
__global__ __launch_bounds__(kThreads, 4) void coeff_rows_kernel(
    CoeffInputs in, int n_rows, int rows_each, double* partial, float* __restrict__ g_out, float* __restrict__ wtilde_out,
    float g_scale, double* __restrict__ loss_out, int* status, Tickets tickets) {
  __shared__ Responses resp;
  __shared__ float s_adv[kSelfPlanResponses];
  __shared__ double s_weight[kSelfPlanResponses], lds[kWaves];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int r0 = blockIdx.x * rows_each, r1 = n_rows - r0 < rows_each ? n_rows : r0 + rows_each;
  const CoeffRule rule(in.p, in.diag->alpha, in.lnC, in.logp_old != nullptr, in.logp_ref != nullptr);
  CoeffRows<kAtOnce> rows;
  WaveRows wave_rows(r0, r1, rows_each);
  const int turns = wave_rows.turns();
  auto load = [&](int k0) {                          // those of turns k0 .. k0 + 7 (rows past the end: the last)
    rows.load<0>(in, rule, [&](int k) { return wave_rows.row(k0 + k); });
    if (turns - k0 > 4) rows.load<4>(in, rule, [&](int k) { return wave_rows.row(k0 + k); });        // uniform
  };
  if (turns > 0) load(0);                            // uniform
  if (tid < in.n_resp) {
    s_adv[tid] = in.adv[tid];
    s_weight[tid] = response_weight(in.n_resp, in.count[tid]);
  }
  resp.init(in.cu_rows, in.n_resp, n_rows, status);
  __syncthreads();
  double acc = 0;
  for (int k0 = 0; k0 < turns; k0 += kAtOnce) {                          // uniform
    const int k1 = min(turns, k0 + kAtOnce);
#pragma unroll 1
    for (int k = k0; k < k1; ++k) {
      const bool one = wave_rows.common(resp, k);                        // uniform
      const int r = wave_rows.row(k), i = one ? wave_rows.i : resp.search(r, wave_rows.i, wave_rows.last);
      if (wave_rows.in(k)) {
        float g = 0.f, wt = 0.f;
        if (rows.live[0] != 0 && (one || resp.holds(i, r))) {
          const RowTerm t = row_term(rule, rows.lt[0], rows.roll[0], rows.old[0], rows.ref[0], (double)s_adv[i]);
          const double wgt = s_weight[i];
          acc -= wgt * t.obj;
          g = (float)(wgt * t.dobj * (double)g_scale);
          wt = (float)t.wtilde;
        }
        g_out[r] = g;
        if (wtilde_out != nullptr) wtilde_out[r] = wt;
      }
      rows.next();
    }
    if (k1 < turns) load(k1);
  }
  acc = wave_sum(acc);
  const Partials<1> partials{partial, 0};
  if (gridDim.x > 1) {                               // uniform
    if (lane == 0) partials.put(blockIdx.x * kWaves + wave, {acc});
    if (last_workgroup(tickets)) loss_final(partials, gridDim.x * kWaves, lds, loss_out);
    return;
  }
  if (lane == 0) lds[wave] = acc;
  __syncthreads();
  if (wave != 0) return;
  acc = lds[lane & (kWaves - 1)];
  acc += butterfly<0>(acc);
  acc += butterfly<1>(acc);
  acc += butterfly<2>(acc);
  acc += butterfly<3>(acc);
  if (tid == 0) *loss_out = acc;
}

// More responses: a tile of one response per wavefront.
__global__ __launch_bounds__(kThreads, 4) void row_coeff_kernel(
    CoeffInputs in, long long n_rows, const int* __restrict__ tile_off, TileRule rule, double* partial,
    float* __restrict__ g_out, float* __restrict__ wtilde_out, float g_scale, double* __restrict__ loss_out,
    Tickets tickets) {
  __shared__ double lds[kWaves];
  const CoeffRule coeff(in.p, in.diag->alpha, in.lnC, in.logp_old != nullptr, in.logp_ref != nullptr);
  const Tiling tiling{tile_off, in.cu_rows, in.n_resp, (int)n_rows};
  const int n_tiles = tiling.tiles();
  const Partials<1> partials{partial, 0};
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int per = (n_tiles + (int)gridDim.x - 1) / (int)gridDim.x;
  const int b0 = blockIdx.x * per, b1 = min(n_tiles, b0 + per);
  for (int b = b0 + wave; b < b1; b += kWaves) {               // uniform for the wavefront
    const Tile tile = tiling.tile(b);
    const double a = (double)in.adv[tile.resp], wgt = response_weight(in.n_resp, in.count[tile.resp]);
    CoeffRows<kLaneRows> rows;
    auto load = [&](int c0) {                        // (rows past the tile's end: its last)
      rows.load<0>(in, coeff, [&](int k) { return tile.row0 + min(c0 + 64 * k + lane, tile.len - 1); });
    };
    if (tile.len > 0) load(0);
    double acc = 0;
    for (int c0 = 0; c0 < tile.len; c0 += kChunkRows) {        // uniform for the wavefront
      const int n_k = min(kLaneRows, (tile.len - c0 + 63) >> 6);
#pragma unroll 1
      for (int k = 0; k < n_k; ++k) {
        float g = 0.f, wt = 0.f;
        const int r = c0 + 64 * k + lane;
        if (r < tile.len && rows.live[0] != 0) {
          const RowTerm t = row_term(coeff, rows.lt[0], rows.roll[0], rows.old[0], rows.ref[0], a);
          acc -= wgt * t.obj;
          g = (float)(wgt * t.dobj * (double)g_scale);
          wt = (float)t.wtilde;
        }
        if (r < tile.len) {
          g_out[tile.row0 + (unsigned)r] = g;
          if (wtilde_out != nullptr) wtilde_out[tile.row0 + (unsigned)r] = wt;
        }
        rows.next();
      }
      if (c0 + kChunkRows < tile.len) load(c0 + kChunkRows);
    }
    acc = wave_sum(acc);
    if (lane == 0) partials.put(b, {acc});
  }
  if (last_workgroup(tickets)) loss_final(partials, n_tiles, lds, loss_out);
}

// Workgroups that share the tiles of more than kSelfPlanResponses responses: four or more tiles each, on as many compute units
// as that gives.
int reduction_grid(const ais_ctx* ctx, int max_tiles) {
  const int per = std::max(4, (max_tiles + ctx->n_cus - 1) / ctx->n_cus);
  return (max_tiles + per - 1) / per;
}

// Workgroups that the rows are dealt out to.  Up to kAloneRows one, all alone: it takes no ticket and nothing goes through memory.
// Beyond, 256 rows each (a wavefront on every SIMD: with more they wait for each other's fp64 instructions) on up to
// kFewWorkgroups, since every ticket is a turn at one word; then 1,024 rows each.  Diagnostics and row coefficients, us, 256, 512
// and 1,024 rows each: 2,432 rows 8.1, 8.3, 8.6 and 4.9, 5.1, 5.3; 4,096 7.8, 8.0, 8.6 and 4.7, 4.8, 5.3; 8,192 8.2, 8.1, 8.6 and
// 4.8, 4.8, 5.3; 19,968 8.7, 8.4, 8.9 and 5.6, 5.2, 5.5; 41,643 9.0, 8.2, 8.1 and 6.7, 5.7, 5.6; 108,495 10.3, 10.0, 9.1 and 8.5, 7.8,
// 6.6.  Alone and with 256 each: 1,500 rows 6.9 and 7.2, 4.6 and 4.6; 2,048 7.4 and 7.3, 5.0 and 4.6.
constexpr int kAloneRows = 2048, kFewRows = 256, kFewWorkgroups = 32;
long long dealt_workgroups(long long n_rows, int n_cus) {
  if (n_rows <= kAloneRows) return 1;
  const long long few = std::min<long long>((n_rows + kFewRows - 1) / kFewRows, kFewWorkgroups);
  return std::min<long long>(std::max(few, (n_rows + kThreads - 1) / kThreads), std::min(n_cus, kMostWorkgroups));
}
int rows_each(const ais_ctx* ctx, long long n_rows) {
  const long long wgs = dealt_workgroups(n_rows, ctx->n_cus);
  if (wgs == 1) return (int)std::max<long long>(n_rows, 1);
  return (int)(((n_rows + wgs - 1) / wgs + 63) / 64 * 64);
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

// The tiling of batches of more than kSelfPlanResponses responses.
TileRule tile_rule(long long n_rows, int n_resp) {
  return TileRule{(int)((n_rows + kPlanTileRows - 1) / kPlanTileRows) + n_resp};
}

// Monotone in both arguments, so that a call at the largest batch sizes the workspace for all others: the partials have
// room for the tiles of a planned batch and for the workgroups' of any other (the sums over a workgroup's rows and a word of the
// counts, and one beside it per response; or its wavefronts' parts of the loss).
constexpr size_t kWorkgroupBytes = 128;
static_assert(sizeof(double) * kRowWords + sizeof(int) <= kWorkgroupBytes && sizeof(double) * kWaves <= kWorkgroupBytes, "");
WorkspaceLayout workspace_layout(long long n_rows, int n_resp) {
  auto up = [](size_t v) { return (v + 255) & ~size_t(255); };
  const size_t workgroups = (size_t)dealt_workgroups(n_rows, kMostWorkgroups);
  const size_t planned = (size_t)((n_rows + kPlanTileRows - 1) / kPlanTileRows) + (size_t)n_resp;
  WorkspaceLayout w;
  w.tile_off = 0;
  w.partial = up(w.tile_off + sizeof(int) * (size_t)(n_resp + 2));
  w.g = up(w.partial + std::max(kWorkgroupBytes * workgroups + sizeof(int) * (size_t)n_resp, sizeof(double) * kDiagWords * planned));
  w.total = up(w.g + sizeof(float) * (size_t)n_rows);
  return w;
}

// The documented limit of ais_diagnostics_static, 56 bytes for each of the tiles of 1,024 rows that the batch may have
// beside 4 for each response: at least what tiling and partials take beyond kSelfPlanResponses responses.
size_t static_scratch_bytes(long long n_rows, int n_resp) {
  auto up = [](size_t v) { return (v + 255) & ~size_t(255); };
  static_assert(sizeof(double) * kDiagWords <= 56, "partials of planned tiles fit what is documented");
  static_assert(2 * sizeof(int) * (kSelfPlanResponses + 2) + 256 + kWorkgroupBytes * kMostWorkgroups <= AIS_STATIC_SCRATCH_BYTES,
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
  const double lnC = std::log((double)p.C);
  if (n_resp <= kSelfPlanResponses) {
    const int each = rows_each(ctx, n_rows), grid = (int)std::max<long long>((n_rows + each - 1) / each, 1);
    int* counts = reinterpret_cast<int*>(partial + (size_t)kRowWords * grid);
    diag_rows_kernel<<<grid, kThreads, 0, ctx->stream>>>(
        logp_train, logp_roll, valid, (int)n_rows, each, cu_rows, n_resp, partial, counts, group_size, rewards, p, lnC, adv_out,
        count_out, diag_out, ctx->status_dev, take_tickets(ctx, in_static, grid));
    return hip_fail(ctx, hipGetLastError());
  }
  const TileRule rule = tile_rule(n_rows, n_resp);
  const int grid = reduction_grid(ctx, rule.max_tiles);
  diag_reduce_kernel<<<grid, kThreads, 0, ctx->stream>>>(
      logp_train, logp_roll, valid, n_rows, cu_rows, n_resp, tile_off, rule, partial, group_size, rewards, p, lnC, adv_out,
      count_out, diag_out, ctx->status_dev, take_tickets(ctx, in_static, grid));
  return hip_fail(ctx, hipGetLastError());
}

int launch_row_coeff(ais_ctx* ctx, const CoeffInputs& in, long long n_rows, int* tile_off, double* partial, float* g_out,
                     float* wtilde_out, double* loss_out, float g_scale) {
  if (in.n_resp <= kSelfPlanResponses) {
    const int each = rows_each(ctx, n_rows), grid = (int)std::max<long long>((n_rows + each - 1) / each, 1);
    coeff_rows_kernel<<<grid, kThreads, 0, ctx->stream>>>(in, (int)n_rows, each, partial, g_out, wtilde_out, g_scale, loss_out,
                                                          ctx->status_dev, take_tickets(ctx, false, grid));
    return hip_fail(ctx, hipGetLastError());
  }
  const TileRule rule = tile_rule(n_rows, in.n_resp);
  const int grid = reduction_grid(ctx, rule.max_tiles);
  row_coeff_kernel<<<grid, kThreads, 0, ctx->stream>>>(in, n_rows, tile_off, rule, partial, g_out, wtilde_out, g_scale,
                                                       loss_out, take_tickets(ctx, false, grid));
  return hip_fail(ctx, hipGetLastError());
}

}  // namespace ais
