// The two vocabulary sweeps of the path, and a plain copy kernel used as a bandwidth yardstick.
//
//   token_logprob_kernel   one pass over a logits row with a running (max, sum) pair:
//                          lse = log sum_v exp(z_v / T), logp = z_y / T - lse, the latter evaluated as
//                          -log1p(sum_{v != y} exp((z_v - z_y) / T))
//                          (Alg. 1, "Compute full-precision log-probs")
//   dlogits_burst_kernel   second pass: dz_v = g (softmax_v - 1[v = y]) / T, written in the logits'
//                          dtype (gradient of Eq. 19 through the log-softmax; g is the row's coefficient)
//
// Both are bound by HBM bandwidth: nothing here is a contraction, so no matrix cores.  One workgroup
// owns one row (64 to 1,024 threads by number and width of the rows), so a row's partial
// results never leave its compute unit; consecutive lanes access consecutive 16-byte vectors (8 bf16 or
// 4 fp32 logits), i.e. each wavefront memory instruction covers 1 KiB of contiguous memory.  Logits are
// read and written with streaming (non-temporal) accesses: a batch is tens of GB and nothing survives in
// cache between the two sweeps (a temporal load costs the read-only sweep 11 % of its bandwidth).
#include "ais_internal.h"
#include "device_utils.h"

#include <type_traits>

namespace ais {
namespace {

using namespace dev;

// ---- sweep 1: token log-probability --------------------------------------------------------------
// grid.x = n_rows, block = THREADS.  ALIGNED: row base and pitch are 16-byte aligned, so a row is vectors from its
// first element on.  Otherwise the elements before the row's first 128-byte boundary are taken one by one together
// with those after the last vector.  (Until then such rows were read element by element, bound by the number of load
// instructions.  The three-call step over 12,345 x 50,257 bf16: 1,657 us element-wise, 636 us with vectors; over
// 4,096 x 32,003 fp32: 415 and 236 us.)  The vectors after the last whole round of UNROLL per thread are loaded together
// too, those past the end of the row masked, instead of one by one, each waiting for its own: 8,192 x 32,003 bf16 87.9 ->
// 84.8 us with 256 threads, no difference at 151,936.  (Three of them as four, one masked: 512 x 6,000 4.55 instead of 4.29
// us, 1,000 x 6,000 5.75 and 5.40.)
template <typename T, bool ALIGNED, int THREADS, int UNROLL>
__global__ __launch_bounds__(THREADS) void token_logprob_kernel(
    const T* __restrict__ logits, long long row_stride, int vocab, const int* __restrict__ token_ids,
    const unsigned char* __restrict__ valid, float inv_temperature, double exact, float* __restrict__ logp_out,
    float* __restrict__ lse_out, int* __restrict__ status) {
  static_assert(UNROLL == 4, "the last vectors of a row are loaded by one to four a thread");
  constexpr int N = Vec<T>::N;
  const long long row = blockIdx.x;
  const int tid = threadIdx.x;
  if (valid != nullptr && valid[row] == 0) {      // not evaluated: neither the row nor its token is read
    if (tid == 0) {
      logp_out[row] = 0.f;
      lse_out[row] = 0.f;
    }
    return;
  }
  const T* zr = logits + row * row_stride;
  const float scale = inv_temperature * kLog2e;   // 2^(z * scale) = exp(z / T)

  // The sampled token's own term is kept out of the running sum: with S_o = sum over the other tokens,
  // logp = -log1p(S_o / e^{z_y/T}) keeps its relative accuracy when the row is sharply peaked (p_y -> 1),
  // where z_y/T - lse would cancel.  Its logit is loaded first so that the latency hides behind the sweep.
  const int y = token_ids[row];
  const bool y_ok = (y >= 0) && (y < vocab);
  const float zy = y_ok ? Vec<T>::load1(zr + y) : 0.f;
  const int head = ALIGNED ? 0 : head_elements(zr, vocab);
  const int nvec = (vocab - head) / N;
  // vector index at which this thread meets the sampled token, or a value no index ever takes
  const int yb = y - head;                        // position of the sampled token from the first vector on
  const int yvec = (y_ok && yb >= 0 && yb < nvec * N && (yb / N) % THREADS == tid) ? yb / N : -(1 << 30);
  const int ysub = yb & (N - 1);

  MaxSum st{kNegHuge, 0.f};
  {
    const u32x4* zv = reinterpret_cast<const u32x4*>(zr + head);
    // COUNT vectors of every thread from vector `base` on, all in flight at once; TAIL: some lie past the end of the row
    auto batch = [&](int base, auto count, auto tail) {
      constexpr int COUNT = decltype(count)::value;
      constexpr bool TAIL = decltype(tail)::value;
      const int i = base + tid;
      u32x4 q[COUNT];
#pragma unroll
      for (int u = 0; u < COUNT; ++u)
        q[u] = load_stream(zv + (TAIL ? min(i + u * THREADS, nvec - 1) : i + u * THREADS));
      float x[COUNT * N];
#pragma unroll
      for (int u = 0; u < COUNT; ++u) {
        Vec<T>::unpack(q[u], x + u * N);
        if (TAIL && i + u * THREADS >= nvec) {
#pragma unroll
          for (int k = 0; k < N; ++k) x[u * N + k] = kMasked;
        }
      }
      if ((unsigned)(yvec - i) < (unsigned)(COUNT * THREADS)) {   // rare: once per row, one lane
        const int hit = ((yvec - i) / THREADS) * N + ysub;
#pragma unroll
        for (int k = 0; k < COUNT * N; ++k)
          if (k == hit) x[k] = kMasked;
      }
      accumulate<COUNT * N>(x, scale, st);
    };
    typedef std::integral_constant<int, 1> One;
    typedef std::integral_constant<int, 2> Two;
    typedef std::integral_constant<int, 3> Three;
    typedef std::integral_constant<int, UNROLL> All;
    int base = 0;
    for (; base + UNROLL * THREADS <= nvec; base += UNROLL * THREADS) batch(base, All{}, std::false_type{});
    const int left = nvec - base;                // uniform
    if (left > 3 * THREADS) batch(base, All{}, std::true_type{});
    else if (left > 2 * THREADS) batch(base, Three{}, std::true_type{});
    else if (left > THREADS) batch(base, Two{}, std::true_type{});
    else if (left > 0) batch(base, One{}, std::true_type{});
  }
  // the elements outside the vectors: at most 128 bytes before them, less than 16 after
  for (int r = tid; r < vocab - nvec * N; r += THREADS) {
    const int v = r < head ? r : r + nvec * N;
    float x = (y_ok && v == y) ? kMasked : Vec<T>::load1(zr + v);
    accumulate<1>(&x, scale, st);
  }

  st = wave_merge(st);
  __shared__ MaxSum lds[THREADS / 64];
  if ((tid & 63) == 0) lds[tid >> 6] = st;
  __syncthreads();
  if (tid >= 64) return;
  MaxSum t = lds[tid & (THREADS / 64 - 1)];         // the wavefronts' states, in lanes of the first
  if (THREADS > 64) t = merge_dpp<kDppQuadXor1>(t);
  if (THREADS > 128) t = merge_dpp<kDppQuadXor2>(t);
  if (THREADS > 256) t = merge_dpp<kDppRowHalfMirror>(t);
  if (THREADS > 512) t = merge_dpp<kDppRowMirror>(t);
  if (tid == 0) {
    if (y_ok) {
      // once per row, in fp64: r = S_o / e^{z_y/T};  logp = -log1p(r);  lse = z_y/T + log1p(r)
      const double l1p = log1p_scaled(t.s, ((double)t.m - (double)zy * (double)scale) * exact);
      logp_out[row] = (float)(-l1p);
      lse_out[row] = (float)((double)zy * (double)inv_temperature + l1p);
    } else {
      lse_out[row] = (t.m + log2_fast(t.s)) * kLn2;
      logp_out[row] = 0.f;
      atomicOr(status, AIS_STATUS_BAD_TOKEN);
    }
  }
}

// ---- sweep 2: gradient w.r.t. the logits -------------------------------------------------------------
// dz[v] = c * (2^(z_v * scale - lse * log2e) - 1[v = y]) with c = g / T.  Rows with g == 0 (not evaluated,
// zero advantage, or clipped away) are filled with zeros without being read.  In-place operation is safe:
// every element is read and written by the same thread, once.
//
// Element-wise form: the route when logits and gradient are not both 16-byte aligned and lie differently relative to a
// line, or are narrow.  grid.x = n_rows, block = kSweepThreads.
template <typename T>
__global__ __launch_bounds__(kSweepThreads) void dlogits_elementwise_kernel(
    const T* logits, long long row_stride, int vocab, const int* __restrict__ token_ids,
    const float* __restrict__ g, const unsigned char* __restrict__ valid, const float* __restrict__ lse,
    const float* __restrict__ logp, float inv_temperature, T* dlogits) {
  const long long row = blockIdx.x;
  const int tid = threadIdx.x;
  const T* zr = logits + row * row_stride;
  T* dr = dlogits + row * row_stride;
  // g == nullptr: unit coefficient on evaluated rows, i.e. the unscaled direction softmax - onehot
  const float gn = g != nullptr ? g[row] : ((valid == nullptr || valid[row] != 0) ? 1.f : 0.f);
  if (gn == 0.f) {
    for (int v = tid; v < vocab; v += kSweepThreads) Vec<T>::store1(dr + v, 0.f);
    return;
  }
  const float scale = inv_temperature * kLog2e;
  const float shift = -lse[row] * kLog2e;
  const float c = g != nullptr ? gn * inv_temperature : gn;
  int y = token_ids[row];
  if (y < 0 || y >= vocab) y = -1;               // flagged by the first sweep; no one-hot term
  // the sampled token's element is c (p_y - 1) = c expm1(logp): no cancellation when p_y is close to 1
  const float dzy = c * expm1f(logp[row]);
  for (int v = tid; v < vocab; v += kSweepThreads) {
    float p = c * exp2_fast(__builtin_fmaf(Vec<T>::load1(zr + v), scale, shift));
    if (v == y) p = dzy;
    Vec<T>::store1(dr + v, p);
  }
}

// Burst form: the route for every other row.  A workgroup of THREADS (1,024; narrow rows: 256) owns the row; every wavefront
// issues all of its loads (up to NV 16-byte vectors per lane, i.e. up to NV KiB per wavefront), transforms
// the vectors in place as they arrive, and only when its last load has landed issues all of its stores.
// Measured on MI355X, a read+write stream shaped this way (long load bursts followed by long store bursts,
// all wavefronts of a compute unit in step because they start together) sustains 5.8-6.0 TB/s where a loop
// that stores each vector as soon as it is computed, and every plain copy variant, saturate at 5.2-5.3 TB/s.
// grid.x = 8 * ceil(n_rows / 8), block = THREADS.  ALIGNED: both rows are 16-byte aligned; otherwise both lie the
// same way relative to 128-byte lines, and the elements before the row's first line boundary are handled one by one
// together with those after the last vector.  Rows wider than NV * 1024 vectors
// are processed in consecutive segments (there is no dependence between segments: lse is an input).
constexpr int kBurstThreads = 1024;

// Where a row's coefficient comes from: an array that the row-coefficient kernel has written (without one, g == nullptr, it
// is 1 on evaluated rows: the unscaled direction softmax - onehot) ...
struct GivenCoeff {
  static constexpr bool kOwn = false;
  const float* g;
  const unsigned char* valid;
  __device__ __forceinline__ float of_row(long long row) const {
    return g != nullptr ? g[row] : ((valid == nullptr || valid[row] != 0) ? 1.f : 0.f);
  }
  __device__ __forceinline__ float scale(float inv_temperature) const { return g != nullptr ? inv_temperature : 1.f; }
};
// ... or the workgroup itself, in small batches, whose coefficient kernel is a launch of 4 us and the gap before it.  One
// workgroup more, the grid's last, then forms the loss and the rectification weights of all rows.  The step over 512 rows
// of 1,024 fp32 logits: 24.0 us with the launch, 22.0 without.
struct OwnCoeff {
  static constexpr bool kOwn = true;
  CoeffInputs in;
  float* wtilde;
  double* loss;
  int* status;
  int n_rows;
  // Must be called by whole wavefronts.
  __device__ __forceinline__ float of_row(long long row) const {
    if (in.valid != nullptr && in.valid[row] == 0) return 0.f;           // uniform
    const int lane = threadIdx.x & 63;
    const float lt = in.logp_train[row], roll = in.logp_roll[row];
    const float old = in.logp_old != nullptr ? in.logp_old[row] : 0.f;
    const CoeffRule rule(in.p, in.diag->alpha, in.lnC, in.logp_old != nullptr, in.logp_ref != nullptr);
    const float ref = rule.kl ? in.logp_ref[row] : 0.f;
    bool here = false;
    if (lane < in.n_resp) here = in.cu_rows[lane] <= row && row < in.cu_rows[lane + 1];
    const unsigned long long mask = __ballot(here);
    if (mask == 0) return 0.f;                                           // no response's row: a faulty cu_rows, reported
    const int i = __builtin_ctzll(mask);
    const RowTerm t = row_term(rule, lt, roll, old, ref, (double)in.adv[i]);
    return (float)(response_weight(in.n_resp, in.count[i]) * t.dobj);
  }
  __device__ __forceinline__ float scale(float inv_temperature) const { return inv_temperature; }
  template <int THREADS>
  __device__ void loss_of_all() const {
    __shared__ long long cu[kOwnResponses + 1];
    __shared__ double sums[THREADS / 64];
    const int tid = threadIdx.x;
    if (tid <= in.n_resp) cu[tid] = in.cu_rows[tid];
    const CoeffRule rule(in.p, in.diag->alpha, in.lnC, in.logp_old != nullptr, in.logp_ref != nullptr);
    __syncthreads();
    if (tid < in.n_resp) {
      const long long lo = cu[tid], hi = cu[tid + 1];
      if (lo < 0 || hi < lo || hi > n_rows || (tid == 0 && lo != 0) || (tid == in.n_resp - 1 && hi != n_rows))
        atomicOr(status, AIS_STATUS_BAD_CU);
    }
    double acc = 0;
    for (int r = tid; r < n_rows; r += THREADS) {
      int i = 0, end = in.n_resp;                // the last response that begins at r or before it
      while (end - i > 1) {
        const int mid = (i + end) >> 1;
        if (cu[mid] <= r) i = mid; else end = mid;
      }
      if (r < cu[i] || r >= cu[i + 1]) continue;
      float wt = 0.f;
      if (in.valid == nullptr || in.valid[r] != 0) {
        const RowTerm t = row_term(rule, in.logp_train[r], in.logp_roll[r], in.logp_old != nullptr ? in.logp_old[r] : 0.f,
                                   rule.kl ? in.logp_ref[r] : 0.f, (double)in.adv[i]);
        acc -= response_weight(in.n_resp, in.count[i]) * t.obj;
        wt = (float)t.wtilde;
      }
      if (wtilde != nullptr) wtilde[r] = wt;
    }
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) acc += __shfl_xor(acc, off);
    if ((tid & 63) == 0) sums[tid >> 6] = acc;
    __syncthreads();
    if (tid != 0) return;
    for (int w = 1; w < THREADS / 64; ++w) acc += sums[w];
    *loss = acc;
  }
  static constexpr int kOwnResponses = 64;       // a lane for each
};

// NSEG > 0 promises that the row fits NSEG segments, which are then unrolled: the loop-free form is ~3 %
// faster than the same code inside a run-time loop.  NSEG = 0: run-time loop over as many segments as needed.
// KFULL promises that the row has at least KFULL * 1024 vectors: vectors 0 .. KFULL - 1 of every lane exist and
// are loaded and stored without a bounds branch (1.5 % faster at 19 vectors per lane).
template <typename T, bool ALIGNED, int THREADS, int NV, int NSEG, int KFULL, typename Coeff>
__global__ __launch_bounds__(THREADS) void dlogits_burst_kernel(
    const T* logits, long long row_stride, int vocab, const int* __restrict__ token_ids, Coeff coeff,
    const float* __restrict__ lse, const float* __restrict__ logp, float inv_temperature, T* dlogits, long long n_rows) {
  constexpr int N = Vec<T>::N;
  // Workgroups are dealt to the 8 XCDs round-robin by their index; every XCD walks a contiguous range of rows
  // (grid.x = 8 * ceil(n_rows / 8)).  Against rows dealt round-robin this is neutral on a batch of full rows
  // and 1-3 % faster where zero-filled rows mix with read+write rows.
  const long long rows_per_xcd = gridDim.x >> 3;
  if (Coeff::kOwn && blockIdx.x == (unsigned)rows_per_xcd * 8) {
    if constexpr (Coeff::kOwn) coeff.template loss_of_all<THREADS>();
    return;
  }
  const long long row = (long long)(blockIdx.x & 7) * rows_per_xcd + (blockIdx.x >> 3);
  if (row >= n_rows) return;
  const int tid = threadIdx.x;
  const T* zr = logits + row * row_stride;
  T* dr = dlogits + row * row_stride;
  const int head = ALIGNED ? 0 : head_elements(zr, vocab);
  const u32x4* zv = reinterpret_cast<const u32x4*>(zr + head);
  u32x4* dv = reinterpret_cast<u32x4*>(dr + head);
  const int nvec = (vocab - head) / N;
  const int rest = vocab - nvec * N;     // elements outside the vectors, one per thread for the first `rest` threads
  const int v_rest = tid < head ? tid : tid + nvec * N;
  const float gn = coeff.of_row(row);

  if (gn == 0.f) {
    const u32x4 zero = {0u, 0u, 0u, 0u};
    for (int i = tid; i < nvec; i += THREADS) store_stream(dv + i, zero);
    if (tid < rest) Vec<T>::store1(dr + v_rest, 0.f);
    return;
  }

  const float scale = inv_temperature * kLog2e;
  const float shift = -lse[row] * kLog2e;
  const float c = gn * coeff.scale(inv_temperature);
  int y = token_ids[row];
  if (y < 0 || y >= vocab) y = -1;               // flagged by the first sweep; no one-hot term
  // The sampled token's element is c (p_y - 1) = c expm1(logp): no cancellation when p_y is close to 1.  The
  // lane that holds it patches its packed output register before the store burst.
  const int yb = y - head;                       // its position from the first vector on
  const int yvec = (y >= 0 && yb >= 0 && yb < nvec * N && (yb / N) % THREADS == tid) ? yb / N : -1;
  const float dzy = c * expm1f(logp[row]);

  const int n_base = NSEG > 0 ? NSEG * NV * THREADS : nvec;
  constexpr int kUnrollSegments = NSEG > 0 ? NSEG : 1;
#pragma unroll kUnrollSegments
  for (int base = 0; base < n_base; base += NV * THREADS) {
    u32x4 q[NV];
#pragma unroll
    for (int k = 0; k < NV; ++k) {
      const int i = base + tid + k * THREADS;
      if (NSEG > 0 && base / THREADS + k < KFULL) q[k] = load_stream(zv + i);
      else q[k] = (i < nvec) ? load_stream(zv + i) : u32x4{0u, 0u, 0u, 0u};
    }
#pragma unroll
    for (int k = 0; k < NV; ++k) {                // in place, in order of arrival
      float x[N];
      Vec<T>::unpack(q[k], x);
#pragma unroll
      for (int j = 0; j < N; ++j) x[j] = c * exp2_fast(__builtin_fmaf(x[j], scale, shift));
      q[k] = Vec<T>::pack(x);
      __builtin_amdgcn_sched_barrier(0);
    }
    // every vector is made opaque here: no store can be issued before the last load has returned
#pragma unroll
    for (int k = 0; k < NV; ++k) asm volatile("" : "+v"(q[k]));
    if ((unsigned)(yvec - base - tid) < (unsigned)(NV * THREADS)) {   // one lane, once per row
      const int hit = (yvec - base - tid) / THREADS;
#pragma unroll
      for (int k = 0; k < NV; ++k)
        if (k == hit) q[k] = Vec<T>::put(q[k], yb & (N - 1), dzy);
    }
#pragma unroll
    for (int k = 0; k < NV; ++k) {
      const int i = base + tid + k * THREADS;
      if ((NSEG > 0 && base / THREADS + k < KFULL) || i < nvec) store_stream(dv + i, q[k]);
    }
  }
  if (tid < rest)
    Vec<T>::store1(dr + v_rest,
                   v_rest == y ? dzy : c * exp2_fast(__builtin_fmaf(Vec<T>::load1(zr + v_rest), scale, shift)));
}

template <typename T, bool ALIGNED>
void launch_dlogits_burst(ais_ctx* ctx, const T* z, long long n_rows, int vocab, long long row_stride,
                          const int* token_ids, const float* g, const unsigned char* valid, const float* lse,
                          const float* logp, float inv_t, T* dz) {
  const int need = (vocab / Vec<T>::N + kBurstThreads - 1) / kBurstThreads;
  dim3 grid((unsigned)(((n_rows + 7) / 8) * 8)), block(kBurstThreads);
  const GivenCoeff given{g, valid};
  if (!ALIGNED && need <= 1) {
    // A narrow row is no work for 1,024 threads, of which a compute unit holds two sets; of 256 it holds eight.  8,192
    // rows, us with 1,024 threads, element by element and with 256: bf16, 1,001 logits 46.0, 15.0, 17.0; 3,001 47.4, 28.2,
    // 21.2; 8,191 59.8, 67.7, 52.0; fp32, 1,001 34.9, 17.7, 15.7; 4,001 47.2, 43.9, 49.2.  1,000 rows: bf16, 3,001 10.5,
    // 7.5, 7.1; fp32, 4,001 10.8, 12.0, 8.9.
    dlogits_burst_kernel<T, false, 256, 4, 1, 0, GivenCoeff><<<grid, dim3(256), 0, ctx->stream>>>(
        z, row_stride, vocab, token_ids, given, lse, logp, inv_t, dz, n_rows);
    return;
  }
  // Aligned ones likewise, up to half that width.  41,643 rows, whole call, us with 1,024, 512, 256 and 64 threads: bf16, 1,000
  // logits 60.5, 34.9, 23.0, 24.1; 2,048 62.1, 36.9, 34.6, 35.7; 3,000 64.4, 51.0, 56.9, 60.2; 4,096 67.0, 61.1, 61.3, 61.8;
  // 6,000 91.0, 103, 108, 113; fp32, 256 59.6, 33.7, 21.5, 18.2; 2,048 66.9, 60.1, 61.4, 62.2; 3,000 89.9, 102, 105, 111.
  const int nvec = vocab / Vec<T>::N;
  if (ALIGNED && nvec <= 256) {
    dlogits_burst_kernel<T, true, 256, 1, 1, 0, GivenCoeff><<<grid, dim3(256), 0, ctx->stream>>>(
        z, row_stride, vocab, token_ids, given, lse, logp, inv_t, dz, n_rows);
    return;
  }
  if (ALIGNED && nvec <= 512) {
    dlogits_burst_kernel<T, true, 512, 1, 1, 0, GivenCoeff><<<grid, dim3(512), 0, ctx->stream>>>(
        z, row_stride, vocab, token_ids, given, lse, logp, inv_t, dz, n_rows);
    return;
  }
  // (vectors that surely exist, vectors per lane and burst, bursts): a row reaches a class only if it is wider than
  // the class before it, which is what the first figure states; an unaligned row may have lost up to 8 vectors to its
  // head, which the next lower figure covers
#define AIS_BURST_CASE(KFULL, NVAL, NSEG)                                                                      \
  dlogits_burst_kernel<T, ALIGNED, kBurstThreads, NVAL, NSEG, (ALIGNED || KFULL == 0 ? KFULL : KFULL - 1), GivenCoeff> \
      <<<grid, block, 0, ctx->stream>>>(z, row_stride, vocab, token_ids, given, lse, logp, inv_t, dz, n_rows)
  if (need <= 4) AIS_BURST_CASE(0, 4, 1);
  else if (need <= 8) AIS_BURST_CASE(4, 8, 1);
  else if (need <= 12) AIS_BURST_CASE(8, 12, 1);
  else if (need <= 13) AIS_BURST_CASE(12, 13, 1);
  else if (need <= 14) AIS_BURST_CASE(13, 14, 1);
  else if (need <= 15) AIS_BURST_CASE(14, 15, 1);
  else if (need <= 16) AIS_BURST_CASE(15, 16, 1);
  else if (need <= 17) AIS_BURST_CASE(16, 17, 1);
  else if (need <= 18) AIS_BURST_CASE(17, 18, 1);
  else if (need <= 19) AIS_BURST_CASE(18, 19, 1);
  else if (need <= 20) AIS_BURST_CASE(19, 20, 1);
  else if (need <= 32) AIS_BURST_CASE(20, 16, 2);   // wider rows: two or three bursts of 16 vectors per lane
  else if (need <= 48) AIS_BURST_CASE(32, 16, 3);
  else AIS_BURST_CASE(0, 16, 0);
#undef AIS_BURST_CASE
}

// ---- plain copy ------------------------------------------------------------------------------------------
__global__ __launch_bounds__(256) void copy_kernel(u32x4* __restrict__ dst, const u32x4* __restrict__ src,
                                                   long long nvec) {
  const long long stride = (long long)gridDim.x * blockDim.x;
  for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < nvec; i += stride)
    store_stream(dst + i, load_stream(src + i));
}

bool vec_ok(const void* base, long long row_stride, size_t esize) {
  return (reinterpret_cast<uintptr_t>(base) % 16 == 0) && ((row_stride * (long long)esize) % 16 == 0);
}
// Two arrays of one row pitch whose rows lie the same way relative to 128-byte lines.
bool same_lines(const void* a, const void* b) {
  return (reinterpret_cast<uintptr_t>(a) - reinterpret_cast<uintptr_t>(b)) % 128 == 0;
}

// Unaligned rows narrower than this go element by element: hardly more than a line's worth of vectors is left of them
// (8,192 rows of 511 bf16 logits 10.5 us, 16.2 with vectors; of 2,001 22.4 and 19.0; fp32, 511 12.4 and 13.7, 1,001 17.7
// and 15.7).
constexpr size_t kElementwiseBytes = 2048;

// 16-byte loads in flight per lane and loop iteration of the log-prob sweep
constexpr int kUnrollFwd = 4;

// Threads that share a row in the log-prob sweep.  256 leave a compute unit eight rows, which is what it takes to keep HBM
// busy.  Where there are hardly more rows than compute units they take more threads each; where there are many narrow ones
// they take fewer, so that more of them are on their way and fewer wavefronts meet at a row's end.  us, bf16 unless noted:
//   rows x logits         1,024   512     256         rows x logits          256     128     64
//   256 x 32,003            9.0    9.0    10.4        41,643 x 1,000          61.8    42.1    32.5
//   256 x 151,936          18.6   22.3    29.6        41,643 x 4,001          83.2    66.7    60.6
//   256 x 151,936 fp32     29.6   29.8    36.9        41,643 x 2,048 fp32     62.7    53.4    57.7
//   512 x 151,936          32.3   30.5    36.3        41,643 x 6,000         101.3    81.9    85.6
//   512 x 151,936 fp32     53.6   53.9    50.6        41,643 x 3,001 fp32     83.5    81.0    82.5
//   1,500 x 151,936        72.6   74.9    74.6        41,643 x 8,192         101.8   108.2   110.0
//   1,500 x 248,320 fp32  222.7  228.3   232.1        2,048 x 1,000 fp32       9.1     7.5     7.6
//   8,192 x 32,003         89.7   80.6    84.8        1,024 x 3,001            8.1     7.5     8.6
//   8,192 x 32,003 fp32   155.7  156.9   160.3        1,024 x 64               4.5     4.2     4.2
//   8,192 x 50,257        128.2  125.5   129.0        1,024 x 1,000            4.5     4.2     4.3
//   41,643 x 32,003       441.7  388.6   404.6
//   41,643 x 151,936      1,954  1,883   1,860
// and around the lines between 2,048 and 4,096 vectors (threads 1,024, 512, 256):
//   256 x 8,192 fp32        4.2    3.9     4.0        300 x 12,288 fp32        5.5     4.9     4.6
//   64 x 12,288 fp32        4.2    3.9     4.1        700 x 12,288 fp32        8.4     7.6     7.2
//   256 x 28,000, relative  0.76   0.79    0.96       300 x 20,000, relative   1.02    0.88    0.94
//   16,384 x 10,001 fp32           96.5   101         30,000 x 20,001                 187     181
//   16,384 x 24,001               117     121
//   1,024 x 50,264                21.7    20.6        700 x 16,600 fp32               9.5     9.0
//   850 x 49,600, relative        1.08    1.01        700 x 50,264, relative          0.96    0.99
int logprob_threads(const ais_ctx* ctx, long long n_rows, long long nvec, bool bf16) {
  const long long cus = ctx->n_cus;
  const bool few = n_rows < 8 * cus;
  if (nvec >= 2048 && n_rows <= cus) return nvec < 3500 ? 512 : 1024;
  if (nvec >= 8192 && n_rows <= 8 * cus) return n_rows > 2 * cus ? 1024 : bf16 ? 512 : 256;
  if (nvec >= (few == bf16 ? 2500 : few ? 3200 : 3000)) {
    const long long per_cu = (n_rows + cus - 1) / cus;       // 512 threads leave some of these compute units a round more
    return nvec >= 8192 || (bf16 ? per_cu == 4 || per_cu == 5 : per_cu == 3) ? 256 : 512;
  }
  // (256 threads that share a few vectors read some of them more than once)
  if (few) return nvec <= 64 ? 64 : nvec <= 128 ? 128 : 256;
  if (nvec >= 896) return 256;
  return nvec >= 512 ? 128 : 64;
}

}  // namespace

int launch_token_logprob(ais_ctx* ctx, const void* logits, ais_dtype dtype, long long n_rows, int vocab,
                         long long row_stride, const int* token_ids, const unsigned char* valid,
                         float inv_temperature, float* logp_out, float* lse_out) {
  if (n_rows == 0) return AIS_OK;
  ScopedTimer timer(ctx, AIS_K_LOGPROB);
  auto launch = [&](const auto* z) {
    typedef std::remove_cv_t<std::remove_pointer_t<decltype(z)>> T;
    const long long nvec = (long long)vocab / Vec<T>::N;
    auto run = [&](auto threads) {
      constexpr int kThreads = decltype(threads)::value;
      auto kernel = vec_ok(z, row_stride, sizeof(T)) ? token_logprob_kernel<T, true, kThreads, kUnrollFwd>
                                                     : token_logprob_kernel<T, false, kThreads, kUnrollFwd>;
      kernel<<<dim3((unsigned)n_rows), dim3(kThreads), 0, ctx->stream>>>(
          z, row_stride, vocab, token_ids, valid, inv_temperature, exact_exponents(inv_temperature), logp_out, lse_out,
          ctx->status_dev);
    };
    const int threads = logprob_threads(ctx, n_rows, nvec, std::is_same_v<T, bf16_t>);
    if (threads == 1024) run(std::integral_constant<int, 1024>{});
    else if (threads == 512) run(std::integral_constant<int, 512>{});
    else if (threads == 64) run(std::integral_constant<int, 64>{});
    else if (threads == 128) run(std::integral_constant<int, 128>{});
    else run(std::integral_constant<int, 256>{});
  };
  if (dtype == AIS_BF16) launch(static_cast<const bf16_t*>(logits));
  else launch(static_cast<const float*>(logits));
  return hip_fail(ctx, hipGetLastError());
}

int launch_dlogits(ais_ctx* ctx, const void* logits, ais_dtype dtype, long long n_rows, int vocab,
                   long long row_stride, const int* token_ids, const float* g, const unsigned char* valid,
                   const float* lse, const float* logp, float inv_temperature, void* dlogits) {
  if (n_rows == 0) return AIS_OK;
  dim3 grid((unsigned)n_rows), block(kSweepThreads);
  ScopedTimer timer(ctx, AIS_K_DLOGITS);
  auto launch = [&](const auto* z) {
    typedef std::remove_cv_t<std::remove_pointer_t<decltype(z)>> T;
    T* dz = static_cast<T*>(dlogits);
    if (vec_ok(z, row_stride, sizeof(T)) && vec_ok(dz, row_stride, sizeof(T)))
      launch_dlogits_burst<T, true>(ctx, z, n_rows, vocab, row_stride, token_ids, g, valid, lse, logp, inv_temperature,
                                    dz);
    else if (same_lines(z, dz) && vocab * sizeof(T) >= kElementwiseBytes)
      launch_dlogits_burst<T, false>(ctx, z, n_rows, vocab, row_stride, token_ids, g, valid, lse, logp, inv_temperature,
                                     dz);
    else
      dlogits_elementwise_kernel<T><<<grid, block, 0, ctx->stream>>>(z, row_stride, vocab, token_ids, g, valid, lse,
                                                                     logp, inv_temperature, dz);
  };
  if (dtype == AIS_BF16) launch(static_cast<const bf16_t*>(logits));
  else launch(static_cast<const float*>(logits));
  return hip_fail(ctx, hipGetLastError());
}

// Takes batches whose rows all have a workgroup on the chip at once, in up to 64 responses, with no more than two rows for
// each thread of the one that forms the loss.
bool try_loss_dlogits_small(ais_ctx* ctx, const CoeffInputs& in, const void* logits, ais_dtype dtype, long long n_rows,
                            int vocab, long long row_stride, const int* token_ids, const float* lse, float* wtilde_out,
                            double* loss_out, void* dlogits) {
  if (n_rows == 0 || n_rows > 1024 || in.n_resp > OwnCoeff::kOwnResponses) return false;
  auto launch = [&](const auto* z) {
    typedef std::remove_cv_t<std::remove_pointer_t<decltype(z)>> T;
    T* dz = static_cast<T*>(dlogits);
    const bool aligned = vec_ok(z, row_stride, sizeof(T)) && vec_ok(dz, row_stride, sizeof(T));
    if (!aligned && !(same_lines(z, dz) && vocab * sizeof(T) >= kElementwiseBytes)) return false;
    const int nvec = vocab / Vec<T>::N;
    auto run = [&](auto kernel, int threads) {
      if (n_rows > 2 * threads || n_rows > ctx->n_cus * (2048LL / threads)) return false;
      ScopedTimer timer(ctx, AIS_K_DLOGITS);
      kernel<<<dim3((unsigned)(((n_rows + 7) / 8) * 8 + 1)), dim3(threads), 0, ctx->stream>>>(
          z, row_stride, vocab, token_ids, OwnCoeff{in, wtilde_out, loss_out, ctx->status_dev, (int)n_rows}, lse,
          in.logp_train, in.p.inv_temperature, dz, n_rows);
      return true;
    };
    if (aligned) {
      if (nvec <= 256) return run(dlogits_burst_kernel<T, true, 256, 1, 1, 0, OwnCoeff>, 256);
      if (nvec <= 512) return run(dlogits_burst_kernel<T, true, 512, 1, 1, 0, OwnCoeff>, 512);
      if (nvec <= 4096) return run(dlogits_burst_kernel<T, true, 1024, 4, 1, 0, OwnCoeff>, 1024);
      if (nvec <= 8192) return run(dlogits_burst_kernel<T, true, 1024, 8, 1, 0, OwnCoeff>, 1024);
    } else {
      if (nvec <= 1024) return run(dlogits_burst_kernel<T, false, 256, 4, 1, 0, OwnCoeff>, 256);
      if (nvec <= 4096) return run(dlogits_burst_kernel<T, false, 1024, 4, 1, 0, OwnCoeff>, 1024);
      if (nvec <= 8192) return run(dlogits_burst_kernel<T, false, 1024, 8, 1, 0, OwnCoeff>, 1024);
    }
    return false;
  };
  return dtype == AIS_BF16 ? launch(static_cast<const bf16_t*>(logits)) : launch(static_cast<const float*>(logits));
}

int launch_copy(ais_ctx* ctx, void* dst, const void* src, long long bytes) {
  if (bytes == 0) return AIS_OK;
  const long long nvec = bytes / 16;
  long long blocks = (nvec + 255) / 256;
  if (blocks > 256 * 64) blocks = 256 * 64;   // 64 workgroups per compute unit, grid-stride beyond that
  ScopedTimer timer(ctx, AIS_K_COPY);
  copy_kernel<<<dim3((unsigned)blocks), dim3(256), 0, ctx->stream>>>(static_cast<u32x4*>(dst),
                                                                     static_cast<const u32x4*>(src), nvec);
  return hip_fail(ctx, hipGetLastError());
}

}  // namespace ais
