// Per-row scalar work and the batch-wide reductions of the path.
//
// The batch is a set of variable-length segments (responses) of rows, some rows masked out.  Every response is cut
// into tiles of kTileRows rows (each workgroup works the tiling out for itself, for up to kSelfPlanResponses responses;
// beyond that a small plan kernel does it once); level 1 reduces one tile per workgroup
// (lane shuffles, then one exchange through LDS) to a partial; level 2, run by whichever workgroup of the
// same launch finishes last, folds the partials of each response in order, forms the group-relative
// advantages (Eq. 3) and the batch moments, and evaluates the three diagnostics and the mixing coefficient
// (Eq. 12-17).  Everything is accumulated in fp64 in a fixed order (no floating point atomics), so results
// are bit-reproducible from run to run; spreads are carried as pairwise-merged (count, mean, squared
// deviations) triples, never as differences of power sums.  These kernels move a few bytes per row (about a
// megabyte per batch) and are bound by the length of their dependent chains, not by bandwidth: 36 and 26 us
// for 1.2 million rows in 1,024 responses, 13 and 7 us for 512 rows in 8.
#include "ais_internal.h"

#include <cmath>
#include <type_traits>

namespace ais {
namespace {

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
__global__ __launch_bounds__(kTileThreads) void plan_kernel(const long long* __restrict__ cu_rows, int n_resp,
                                                            long long n_rows, int* __restrict__ tile_off,
                                                            int max_tiles, int* __restrict__ status) {
  __shared__ long long chunk_sum[kTileThreads];
  const int tid = threadIdx.x;
  const int per = (n_resp + kTileThreads - 1) / kTileThreads;
  const int i0 = min(n_resp, tid * per), i1 = min(n_resp, i0 + per);
  long long sum = 0;
  bool bad = false;
  for (int i = i0; i < i1; ++i) {
    long long lo, hi;
    response_rows(cu_rows, i, n_rows, lo, hi);
    bad |= (cu_rows[i] != lo) || (cu_rows[i + 1] != hi);
    sum += (hi - lo + kTileRows - 1) / kTileRows;
  }
  if (tid == 0 && n_resp > 0) bad |= (cu_rows[0] != 0) || (cu_rows[n_resp] != n_rows);
  chunk_sum[tid] = sum;
  __syncthreads();
  if (tid == 0) {
    long long run = 0;
    for (int t = 0; t < kTileThreads; ++t) {
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
    run += (hi - lo + kTileRows - 1) / kTileRows;
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

constexpr int kWaves = kTileThreads / 64;

// The tiling of the batch as a workgroup sees it: from the plan kernel's array in memory, or worked out by the
// workgroup itself into LDS.  The latter costs one read of cu_rows (8 KiB at most) and a scan where the former costs a
// launch and a chain of log2(n_resp) dependent reads in every workgroup: the two calls of 41,643 rows in 16
// responses take 34 instead of 39 us, of 1.2 million rows in 1,024 responses 62 instead of 64 us.
template <bool SELF>
struct Tiling;

template <>
struct Tiling<false> {
  const int* tile_off;
  const long long* cu_rows;
  long long n_rows;
  int n_resp;
  __device__ __forceinline__ void init(const int* off, const long long* cu, int resp, long long rows, int, int*) {
    tile_off = off;
    cu_rows = cu;
    n_resp = resp;
    n_rows = rows;
  }
  __device__ __forceinline__ int tiles() const { return tile_off[n_resp]; }
  __device__ __forceinline__ int first(int i) const { return tile_off[i]; }
  __device__ __forceinline__ int response_of(int b) const { return find_response(tile_off, n_resp, b); }
  __device__ __forceinline__ void rows(int i, long long& lo, long long& hi) const {
    response_rows(cu_rows, i, n_rows, lo, hi);
  }
};

template <>
struct Tiling<true> {
  int n_resp;
  long long n_rows;
  struct Shared {
    long long cu[kSelfPlanResponses + 1];
    int off[kSelfPlanResponses + 1];
    long long wave_tiles[kWaves];
  };
  __device__ static Shared& shared() {
    __shared__ Shared sh;
    return sh;
  }
  // Must be called by all threads of the workgroup.  Workgroup 0 reports a cu_rows that is no partition of the rows.
  __device__ __forceinline__ void init(const int*, const long long* __restrict__ cu, int resp, long long rows,
                                       int max_tiles, int* status) {
    Shared& sh = shared();
    n_resp = resp;
    n_rows = rows;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    for (int i = tid; i <= n_resp; i += kTileThreads) sh.cu[i] = cu[i];
    __syncthreads();
    constexpr int kPer = kSelfPlanResponses / kTileThreads;
    const int i0 = tid * kPer;
    long long mine[kPer], sum = 0;
    bool bad = tid == 0 && (sh.cu[0] != 0 || sh.cu[n_resp] != n_rows);
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
      mine[k] = sum;
      if (i0 + k < n_resp) {
        long long lo, hi;
        response_rows(sh.cu, i0 + k, n_rows, lo, hi);
        bad |= sh.cu[i0 + k] != lo || sh.cu[i0 + k + 1] != hi;
        sum += (hi - lo + kTileRows - 1) / kTileRows;
      }
    }
    long long incl = sum;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
      const long long o = __shfl_up(incl, off);
      incl += lane >= off ? o : 0;
    }
    if (lane == 63) sh.wave_tiles[wave] = incl;
    __syncthreads();
    long long before = incl - sum, total = 0;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
      if (w < wave) before += sh.wave_tiles[w];
      total += sh.wave_tiles[w];
    }
    bad |= total > max_tiles;                    // cannot happen when cu_rows is a partition of the rows
#pragma unroll
    for (int k = 0; k < kPer; ++k)
      if (i0 + k < n_resp) sh.off[i0 + k] = (int)clampll(before + mine[k], 0, max_tiles);
    if (tid == 0) sh.off[n_resp] = (int)clampll(total, 0, max_tiles);
    const bool any = __syncthreads_or(bad);
    if (any && blockIdx.x == 0 && tid == 0) atomicOr(status, AIS_STATUS_BAD_CU);
  }
  __device__ __forceinline__ int tiles() const { return shared().off[n_resp]; }
  __device__ __forceinline__ int first(int i) const { return shared().off[i]; }
  __device__ __forceinline__ int response_of(int b) const { return find_response(shared().off, n_resp, b); }
  __device__ __forceinline__ void rows(int i, long long& lo, long long& hi) const {
    response_rows(shared().cu, i, n_rows, lo, hi);
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

// Workgroup-wide sum: wavefront sums, then the kWaves partials through LDS in index order.  `lds` holds kWaves
// values; the result is valid in every thread.  Must be called by all threads of the workgroup.
template <typename V>
__device__ __forceinline__ V block_sum(V v, V* lds) {
  v = wave_sum(v);
  if ((threadIdx.x & 63) == 0) lds[threadIdx.x >> 6] = v;
  __syncthreads();
  V r = lds[0];
#pragma unroll
  for (int w = 1; w < kWaves; ++w) r += lds[w];
  __syncthreads();
  return r;
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

// (a thread pushes at most kTileRows / kTileThreads = 4 values: their reciprocals instead of a division)
__device__ __forceinline__ void push(Moments& m, double x) {
  static_assert(kTileRows / kTileThreads <= 4, "reciprocals below");
  m.n += 1.0;
  const double delta = x - m.mean;
  m.mean += delta * (m.n == 1.0 ? 1.0 : m.n == 2.0 ? 0.5 : m.n == 3.0 ? 1.0 / 3.0 : 0.25);
  m.m2 += delta * (x - m.mean);
}

template <int LEVEL>
__device__ __forceinline__ Moments merge_level(const Moments& m) {
  return merge(m, Moments{butterfly<LEVEL>(m.n), butterfly<LEVEL>(m.mean), butterfly<LEVEL>(m.m2)});
}

__device__ __forceinline__ Moments wave_merge(Moments m) {
  m = merge_level<0>(m);
  m = merge_level<1>(m);
  m = merge_level<2>(m);
  m = merge_level<3>(m);
  m = merge_level<4>(m);
  return merge_level<5>(m);
}

// One workgroup-wide reduction of everything a level of the diagnostics needs, with a single barrier pair: NM sets
// of moments, ND plain sums and NI integer sums.  `lds_d` holds (3 NM + ND) kWaves doubles, `lds_i` NI kWaves
// integers.  Results replace the arguments and are valid in every thread.  Must be called by all threads.
template <int NM, int ND, int NI>
__device__ __forceinline__ void block_reduce(Moments (&m)[NM], double (&d)[ND], long long (&c)[NI], double* lds_d,
                                             long long* lds_i) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
#pragma unroll
  for (int k = 0; k < NM; ++k) m[k] = wave_merge(m[k]);
#pragma unroll
  for (int k = 0; k < ND; ++k) d[k] = wave_sum(d[k]);
#pragma unroll
  for (int k = 0; k < NI; ++k) c[k] = wave_sum(c[k]);
  if (lane == 0) {
#pragma unroll
    for (int k = 0; k < NM; ++k) {
      lds_d[(3 * k + 0) * kWaves + w] = m[k].n;
      lds_d[(3 * k + 1) * kWaves + w] = m[k].mean;
      lds_d[(3 * k + 2) * kWaves + w] = m[k].m2;
    }
#pragma unroll
    for (int k = 0; k < ND; ++k) lds_d[(3 * NM + k) * kWaves + w] = d[k];
#pragma unroll
    for (int k = 0; k < NI; ++k) lds_i[k * kWaves + w] = c[k];
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < NM; ++k) {
    Moments r{lds_d[(3 * k + 0) * kWaves], lds_d[(3 * k + 1) * kWaves], lds_d[(3 * k + 2) * kWaves]};
#pragma unroll
    for (int v = 1; v < kWaves; ++v)
      r = merge(r, Moments{lds_d[(3 * k + 0) * kWaves + v], lds_d[(3 * k + 1) * kWaves + v],
                           lds_d[(3 * k + 2) * kWaves + v]});
    m[k] = r;
  }
#pragma unroll
  for (int k = 0; k < ND; ++k) {
    double r = lds_d[(3 * NM + k) * kWaves];
#pragma unroll
    for (int v = 1; v < kWaves; ++v) r += lds_d[(3 * NM + k) * kWaves + v];
    d[k] = r;
  }
#pragma unroll
  for (int k = 0; k < NI; ++k) {
    long long r = lds_i[k * kWaves];
#pragma unroll
    for (int v = 1; v < kWaves; ++v) r += lds_i[k * kWaves + v];
    c[k] = r;
  }
  __syncthreads();
}

// True in exactly one workgroup of the grid: the one that finishes last.  Every workgroup calls this once, after its own
// results have been written by thread 0 with put_device.  They have reached memory when thread 0 has waited for its
// stores, and only then is the ticket taken; the last workgroup reads them with get_device.  (A device-wide fence here
// instead, which writes a whole L2 back for the few bytes of a partial, makes the two calls of 1.2 million
// rows 79 instead of 62 us.)
// Level 2 of each reduction runs in that workgroup, which saves a kernel launch per reduction; the order in which level
// 2 folds the partials does not depend on which workgroup happens to be last, so results stay bit-reproducible.
struct Tickets {
  int* own;      // 0 when the launch begins and when it ends
  int* next;     // the launch's that comes after it
};

__device__ __forceinline__ bool last_workgroup(Tickets t) {
  __shared__ int s_last;
  if (threadIdx.x == 0) {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
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

// ---- level 2: responses -> advantages, batch moments, diagnostics, alpha --------------------------------------
// Runs in the last workgroup of diag_reduce_kernel.  A response's tiles are folded by a group of L lanes, L (a power of
// two up to 64) as large as the responses leave threads for: lane l folds tiles l, l + L, ... in order, then the lanes
// are merged in a fixed tree.  With one thread per response a batch of 4 responses of 1,000 tiles was a chain of 1,000
// dependent reads.
template <bool SELF>
__device__ void diag_final(const DiagPartial* partial, const Tiling<SELF>& tiling, int n_resp,
                           int group_size, const float* __restrict__ rewards, const ais_params& p,
                           float* __restrict__ adv_out, int* __restrict__ count_out, ais_diag* __restrict__ diag_out,
                           const int* status, double* lds_d, long long* lds_i) {
  Moments mw{0, 0, 0}, ma{0, 0, 0}, maw{0, 0, 0};     // of w_bar, of A and of A w_bar over the valid rows of the batch
  double sabs = 0, sd = 0, sdp = 0;
  long long cnt = 0, nclip = 0;
  int lanes = 1;
  while (lanes < 64 && 2 * lanes * n_resp <= kTileThreads) lanes <<= 1;
  const int l = threadIdx.x & (lanes - 1);
  const int per_pass = kTileThreads / lanes;
  for (int i0 = 0; i0 < n_resp; i0 += per_pass) {     // uniform: the lanes of a wavefront merge across groups below
    const int i = i0 + threadIdx.x / lanes;
    Moments r{0, 0, 0};
    long long r_cnt = 0;
    double a = 0.0;
    if (i < n_resp) {
      const int t1 = tiling.first(i + 1);
      auto read = [&](int t) {
        DiagPartial q;
        q.mean_w = get_device(&partial[t].mean_w);
        q.m2_w = get_device(&partial[t].m2_w);
        q.sabs = get_device(&partial[t].sabs);
        q.sd = get_device(&partial[t].sd);
        q.sdp = get_device(&partial[t].sdp);
        q.cnt = get_device(&partial[t].cnt);
        q.nclip = get_device(&partial[t].nclip);
        return q;
      };
      int t = tiling.first(i) + l;
      DiagPartial q;
      if (t < t1) q = read(t);                         // on its way while the advantage is formed
      // group-relative advantage (Eq. 3): reward minus the mean over the G responses of the prompt
      const int g0 = (i / group_size) * group_size;
      double mean = 0;
      for (int j = 0; j < group_size; ++j) mean += (double)rewards[g0 + j];
      mean /= group_size;
      a = (double)rewards[i] - mean;
      if (p.adv_mode == 1) {
        double var = 0;
        for (int j = 0; j < group_size; ++j) {
          const double e = (double)rewards[g0 + j] - mean;
          var += e * e;
        }
        const double den = sqrt(var / group_size) + (double)p.eps_std;
        a = den > 0.0 ? a / den : 0.0;     // eps_std = 0 and equal rewards: 0 / 0, read as 0
      }
      while (t < t1) {
        DiagPartial next = q;
        if (t + lanes < t1) next = read(t + lanes);    // in flight while this one is folded
        r = merge(r, Moments{(double)q.cnt, q.mean_w, q.m2_w});
        sabs += q.sabs;
        sd += q.sd;
        sdp += q.sdp;
        r_cnt += q.cnt;
        nclip += q.nclip;
        q = next;
        t += lanes;
      }
    }
    auto level = [&](auto k) {                         // uniform: every lane of the wavefront takes part
      constexpr int K = decltype(k)::value;
      if (lanes <= (1 << K)) return;
      r = merge_level<K>(r);
      r_cnt += butterfly<K>(r_cnt);
    };
    level(std::integral_constant<int, 0>{});
    level(std::integral_constant<int, 1>{});
    level(std::integral_constant<int, 2>{});
    level(std::integral_constant<int, 3>{});
    level(std::integral_constant<int, 4>{});
    level(std::integral_constant<int, 5>{});
    if (l != 0 || i >= n_resp) continue;               // lane 0 of the group goes on
    const float a32 = (float)a;
    adv_out[i] = a32;
    count_out[i] = (int)r_cnt;
    a = (double)a32;                     // the advantage every later step sees is the stored fp32 value
    // token-level moments of A and A w_bar: A is constant over the response's rows, so the response's rows
    // have mean A mean(w_bar) and squared deviations A^2 m2(w_bar)
    if (r_cnt == 0) continue;
    cnt += r_cnt;
    mw = merge(mw, r);
    ma = merge(ma, Moments{r.n, a, 0.0});
    maw = merge(maw, Moments{r.n, a * r.mean, a * a * r.m2});
  }
  {
    Moments m[3] = {mw, ma, maw};
    double d[3] = {sabs, sd, sdp};
    long long c[2] = {cnt, nclip};
    block_reduce(m, d, c, lds_d, lds_i);
    mw = m[0]; ma = m[1]; maw = m[2];
    sabs = d[0]; sd = d[1]; sdp = d[2];
    cnt = c[0]; nclip = c[1];
  }
  if (threadIdx.x != 0) return;

  ais_diag d;
  d.n_valid = cnt;
  d.status = get_device(status);
  d.reserved = 0;
  if (cnt == 0) {
    d.mean_w = d.var_w = d.cv2 = d.dbar = d.std_a = d.std_aw = d.dsigma = 0.0;
    d.ess_ratio = 1.0; d.alpha_ess = 1.0; d.alpha_mis = 0.0; d.alpha_var = 0.0; d.clip_frac = 0.0;
    d.alpha = 0.0; d.kl_roll_train = 0.0; d.mean_abs_dp = 0.0;
  } else {
    const double N = (double)cnt;
    d.mean_w = mw.mean;
    d.var_w = mw.m2 / N;
    // every truncated ratio underflowed to 0: CV^2 is 0 / 0; read as 0 (equal weights), like the empty batch
    const double cv = d.mean_w > 0.0 ? sqrt(d.var_w) / d.mean_w : 0.0;    // std / mean: mean^2 alone may underflow
    d.cv2 = cv * cv;
    d.ess_ratio = 1.0 / (1.0 + d.cv2);
    d.alpha_ess = 1.0 / sqrt(1.0 + d.cv2);                    // Eq. 12
    d.dbar = sabs / N;                                        // Eq. 13
    d.alpha_mis = fmin(1.0, d.dbar / (double)p.delta);        // Eq. 14
    d.std_a = sqrt(ma.m2 / N);
    d.std_aw = sqrt(maw.m2 / N);
    // Eq. 15; with eps_std = 0 and all advantages equal the ratio is 0 / 0: nothing to amplify, read as 0
    const double den = d.std_a + (double)p.eps_std;
    d.dsigma = den > 0.0 ? d.std_aw / den : 0.0;
    d.alpha_var = fmax(0.0, (d.dsigma - (double)p.gamma) / (double)p.gamma);   // Eq. 16
    const double rel = fmin(1.0, fmax(0.0, d.alpha_ess - (double)p.beta_var * d.alpha_var));
    d.alpha = rel * d.alpha_mis;                              // Eq. 17
    d.clip_frac = (double)nclip / N;
    d.kl_roll_train = -sd / N;       // tokens were drawn from pi_roll: mean of log pi_roll - log pi_train
    d.mean_abs_dp = sdp / N;
  }
  if (p.alpha_override >= 0.f) d.alpha = (double)p.alpha_override;
  *diag_out = d;
}

// Rows of a tile handled by each thread: their inputs are loaded together.
constexpr int kRowsPerThread = kTileRows / kTileThreads;

// ---- level 1: one tile of one response -> DiagPartial; level 2 in the last workgroup ------------------------
template <bool SELF>
__global__ __launch_bounds__(kTileThreads, 4) void diag_reduce_kernel(
    const float* __restrict__ logp_train, const float* __restrict__ logp_roll,
    const unsigned char* __restrict__ valid, long long n_rows, const long long* __restrict__ cu_rows, int n_resp,
    const int* __restrict__ tile_off, int max_tiles, DiagPartial* partial, int group_size,
    const float* __restrict__ rewards, ais_params p, double lnC, float* __restrict__ adv_out, int* __restrict__ count_out,
    ais_diag* __restrict__ diag_out, int* status, Tickets tickets) {
  __shared__ double lds_d[12 * kWaves];          // three sets of moments and three sums per wavefront
  __shared__ long long lds_i[2 * kWaves];
  Tiling<SELF> tiling;
  tiling.init(tile_off, cu_rows, n_resp, n_rows, max_tiles, status);
  const int n_tiles = tiling.tiles();
  for (int b = blockIdx.x; b < n_tiles; b += gridDim.x) {     // uniform for the workgroup
    const int i = tiling.response_of(b);
    long long lo, hi;
    tiling.rows(i, lo, hi);
    const long long r0 = lo + (long long)(b - tiling.first(i)) * kTileRows;
    const long long r1 = min(hi, r0 + kTileRows);
    float ltf[kRowsPerThread], lrf[kRowsPerThread];
    bool on[kRowsPerThread];
#pragma unroll
    for (int k = 0; k < kRowsPerThread; ++k) {
      const long long n = r0 + threadIdx.x + k * kTileThreads;
      on[k] = n < r1;
      ltf[k] = on[k] ? logp_train[n] : 0.f;
      lrf[k] = on[k] ? logp_roll[n] : 0.f;
      if (valid != nullptr) on[k] = on[k] && valid[n] != 0;
    }
    Moments mw{0, 0, 0};
    double sabs = 0, sd = 0, sdp = 0;
    long long cnt = 0, nclip = 0;
#pragma unroll
    for (int k = 0; k < kRowsPerThread; ++k) {
      if (!on[k]) continue;
      const double lt = (double)ltf[k], lr = (double)lrf[k];
      const double d = lt - lr;                                            // log rho (Alg. 1, sampler-trainer ratio)
      const double w = exp(fmin(d, lnC));                                  // w_bar = min(rho, C) (Eq. 10)
      push(mw, w);
      sabs += fabs(d);
      sd += d;
      sdp += fabs(exp(lt) - exp(lr));
      cnt += 1;
      nclip += (d > lnC) ? 1 : 0;
    }
    Moments m[1] = {mw};
    double d[3] = {sabs, sd, sdp};
    long long c[2] = {cnt, nclip};
    block_reduce(m, d, c, lds_d, lds_i);
    if (threadIdx.x == 0) {
      DiagPartial* t = partial + b;
      put_device(&t->mean_w, m[0].mean);
      put_device(&t->m2_w, m[0].m2);
      put_device(&t->sabs, d[0]);
      put_device(&t->sd, d[1]);
      put_device(&t->sdp, d[2]);
      put_device(&t->cnt, c[0]);
      put_device(&t->nclip, c[1]);
    }
  }
  // ---- level 2, in the workgroup that finishes last ----
  if (last_workgroup(tickets))
    diag_final<SELF>(partial, tiling, n_resp, group_size, rewards, p, adv_out, count_out, diag_out, status, lds_d,
                     lds_i);
}

// ---- per-row coefficient of the gradient, rectification weight, loss ------------------------------------------------
__device__ void loss_final(const double* partial, int n_tiles, double* __restrict__ loss_out, double* lds_d) {
  double acc = 0;
#pragma unroll 4
  for (int t = threadIdx.x; t < n_tiles; t += kTileThreads) acc += get_device(partial + t);
  acc = block_sum(acc, lds_d);
  if (threadIdx.x == 0) *loss_out = acc;
}

template <bool SELF>
__global__ __launch_bounds__(kTileThreads) void row_coeff_kernel(
    const float* __restrict__ logp_train, const float* __restrict__ logp_roll, const float* __restrict__ logp_old,
    const float* __restrict__ logp_ref, const unsigned char* __restrict__ valid, long long n_rows,
    const long long* __restrict__ cu_rows, int n_resp, const float* __restrict__ adv,
    const int* __restrict__ count, const ais_diag* __restrict__ diag, ais_params p, double lnC,
    const int* __restrict__ tile_off, int max_tiles, double* partial, float* __restrict__ g_out,
    float* __restrict__ wtilde_out, float g_scale, double* __restrict__ loss_out, int* status, Tickets tickets) {
  __shared__ double lds_d[kWaves];
  const double alpha = diag->alpha;
  Tiling<SELF> tiling;
  tiling.init(tile_off, cu_rows, n_resp, n_rows, max_tiles, status);
  const int n_tiles = tiling.tiles();
  const double lo_clip = 1.0 - (double)p.clip_eps, hi_clip = 1.0 + (double)p.clip_eps;
  const bool kl = (logp_ref != nullptr) && (p.beta_kl > 0.f);
  for (int b = blockIdx.x; b < n_tiles; b += gridDim.x) {     // uniform for the workgroup
    const int i = tiling.response_of(b);
    long long lo, hi;
    tiling.rows(i, lo, hi);
    const long long r0 = lo + (long long)(b - tiling.first(i)) * kTileRows;
    const long long r1 = min(hi, r0 + kTileRows);
    const double a = (double)adv[i];
    const int cnt = count[i];
    const double wgt = cnt > 0 ? 1.0 / ((double)n_resp * (double)cnt) : 0.0;   // 1/G and 1/|o_i| of Eq. 19 over all prompts
    float ltf[kRowsPerThread], rollf[kRowsPerThread], oldf[kRowsPerThread], reff[kRowsPerThread];
    bool on[kRowsPerThread];
#pragma unroll
    for (int k = 0; k < kRowsPerThread; ++k) {
      const long long n = r0 + threadIdx.x + k * kTileThreads;
      on[k] = n < r1;
      ltf[k] = on[k] ? logp_train[n] : 0.f;
      rollf[k] = on[k] ? logp_roll[n] : 0.f;
      oldf[k] = (on[k] && logp_old != nullptr) ? logp_old[n] : 0.f;
      reff[k] = (on[k] && kl) ? logp_ref[n] : 0.f;
      if (valid != nullptr) on[k] = on[k] && valid[n] != 0;
    }
    double acc = 0;
#pragma unroll
    for (int k = 0; k < kRowsPerThread; ++k) {
      const long long n = r0 + threadIdx.x + k * kTileThreads;
      if (n >= r1) continue;
      float g = 0.f, wt = 0.f;
      if (on[k]) {
        const double lt = (double)ltf[k];
        // the sampler-trainer ratio is taken at the checkpoint that generated the rollout (Alg. 1, "Sampler-Trainer
        // ratio"; Sec. 3.2: the two ratios are orthogonal), the old-new ratio between that checkpoint and theta
        const double l_old = logp_old != nullptr ? (double)oldf[k] : lt;
        const double wbar = exp(fmin(l_old - (double)rollf[k], lnC));
        const double wtilde = 1.0 + alpha * (wbar - 1.0);                       // Eq. 18 / Alg. 1 rectification weight
        const double rho_on = logp_old != nullptr ? exp(lt - l_old) : 1.0;
        const double clipped = fmin(fmax(rho_on, lo_clip), hi_clip);
        // the unclipped branch is the minimum (ties included) iff the ratio has not left the trust
        // region on the side the advantage pushes towards
        const bool active = (a >= 0.0) ? (rho_on <= hi_clip) : (rho_on >= lo_clip);
        const double s = active ? rho_on * a : clipped * a;
        double obj = wtilde * s;
        double dobj = active ? wtilde * a * rho_on : 0.0;
        if (kl) {
          const double q = (double)reff[k] - lt;
          const double eq = exp(q);
          obj -= (double)p.beta_kl * (eq - q - 1.0);
          dobj -= (double)p.beta_kl * (1.0 - eq);
        }
        acc -= wgt * obj;
        g = (float)(wgt * dobj * (double)g_scale);
        wt = (float)wtilde;
      }
      g_out[n] = g;
      if (wtilde_out != nullptr) wtilde_out[n] = wt;
    }
    acc = block_sum(acc, lds_d);
    if (threadIdx.x == 0) put_device(partial + b, acc);
  }
  if (last_workgroup(tickets)) loss_final(partial, n_tiles, loss_out, lds_d);
}

// Workgroups of a reduction: one per tile, but no more than the device holds at once (4 per compute unit by their
// registers); each then takes the same number of tiles, and works the tiling out once.  (One workgroup per tile up to
// 8 per compute unit: 88 us for 1.2 million rows, 4: 62 us.)
int reduction_grid(const ais_ctx* ctx, int max_tiles) {
  const int most = 4 * ctx->n_cus;
  const int rounds = (max_tiles + most - 1) / most;
  return rounds > 1 ? (max_tiles + rounds - 1) / rounds : max_tiles;
}

Tickets take_tickets(ais_ctx* ctx, bool in_static) {
  int* pair = ctx->status_dev + (in_static ? kStaticTicketWord : kTicketWord);
  const unsigned turn = (in_static ? ctx->static_turns : ctx->turns)++ & 1u;
  return Tickets{pair + turn, pair + (turn ^ 1u)};
}

}  // namespace

WorkspaceLayout workspace_layout(long long n_rows, int n_resp) {
  auto up = [](size_t v) { return (v + 255) & ~size_t(255); };
  WorkspaceLayout w;
  w.max_tiles = (int)((n_rows + kTileRows - 1) / kTileRows) + n_resp;
  w.tile_off = 0;
  w.partial = up(w.tile_off + sizeof(int) * (size_t)(n_resp + 2));
  w.g = up(w.partial + sizeof(DiagPartial) * (size_t)w.max_tiles);
  w.total = up(w.g + sizeof(float) * (size_t)n_rows);
  return w;
}

// Writes the tiling for batches of more responses than a workgroup works out for itself; nothing to do otherwise.
int launch_plan(ais_ctx* ctx, const long long* cu_rows, int n_resp, long long n_rows, int* tile_off,
                int max_tiles) {
  if (n_resp <= kSelfPlanResponses) return AIS_OK;
  plan_kernel<<<1, kTileThreads, 0, ctx->stream>>>(cu_rows, n_resp, n_rows, tile_off, max_tiles, ctx->status_dev);
  return hip_fail(ctx, hipGetLastError());
}

int launch_diagnostics(ais_ctx* ctx, const float* logp_train, const float* logp_roll, const unsigned char* valid,
                       long long n_rows, const long long* cu_rows, int n_resp, int group_size,
                       const float* rewards, const ais_params& p, int* tile_off, int max_tiles,
                       DiagPartial* partial, bool in_static, float* adv_out, int* count_out, ais_diag* diag_out) {
  auto kernel = n_resp <= kSelfPlanResponses ? diag_reduce_kernel<true> : diag_reduce_kernel<false>;
  kernel<<<reduction_grid(ctx, max_tiles), kTileThreads, 0, ctx->stream>>>(
      logp_train, logp_roll, valid, n_rows, cu_rows, n_resp, tile_off, max_tiles, partial, group_size, rewards, p,
      std::log((double)p.C), adv_out, count_out, diag_out, ctx->status_dev, take_tickets(ctx, in_static));
  return hip_fail(ctx, hipGetLastError());
}

int launch_row_coeff(ais_ctx* ctx, const float* logp_train, const float* logp_roll, const float* logp_old,
                     const float* logp_ref, const unsigned char* valid, long long n_rows,
                     const long long* cu_rows, int n_resp, const float* adv, const int* count,
                     const ais_diag* diag, const ais_params& p, int* tile_off, int max_tiles,
                     double* partial, float* g_out, float* wtilde_out, double* loss_out, float g_scale) {
  auto kernel = n_resp <= kSelfPlanResponses ? row_coeff_kernel<true> : row_coeff_kernel<false>;
  kernel<<<reduction_grid(ctx, max_tiles), kTileThreads, 0, ctx->stream>>>(
      logp_train, logp_roll, logp_old, logp_ref, valid, n_rows, cu_rows, n_resp, adv, count, diag, p,
      std::log((double)p.C), tile_off, max_tiles, partial, g_out, wtilde_out, g_scale, loss_out, ctx->status_dev,
      take_tickets(ctx, false));
  return hip_fail(ctx, hipGetLastError());
}

}  // namespace ais
