// FP8-E4M3 per-row quantisation of logits: the rollout-side perturbation (Sec. 2.1; Eq. 1 with the E4M3
// value grid, q_max = 448, in place of the integer grid; per-row scale s = max|z| / 448).
//
//   fp8_quantize_kernel          z -> (codes, s)        read 2 * e * V (two passes over the row), write V
//   fp8_dequantize_kernel        (codes, s) -> z_r      read V, write e * V
//   fp8_rollout_logprob_kernel   z, y -> log softmax(z_r)[y] without materialising codes or z_r
//
// gfx950's conversion instructions implement the OCP E4M3 format (round to nearest even); inputs are
// clamped to +-448 first, so the conversion never sees an overflow.  The arithmetic that decides a code is
// fp32: s = max|z| / 448 and q = z / s, both correctly rounded divisions (q through the per-row divider of
// fp8_utils.h).  Rows that fit the register file take the single-read kernels of fp8_table.hip and
// fp8_rows.hip, unless they are narrow.
#include "ais_internal.h"
#include "device_utils.h"
#include "fp8_utils.h"

#include <type_traits>

namespace ais {
namespace {

using namespace dev;

// Row abs-max (a NaN loses every comparison), shared by the workgroup through LDS.  The row's vectors start `head` elements
// into it, at its first 128-byte boundary.
template <typename T, int THREADS>
__device__ __forceinline__ float row_amax(const T* zr, int vocab, int head, float* lds) {
  constexpr int N = Vec<T>::N;
  const int tid = threadIdx.x;
  const int nvec = (vocab - head) / N;
  float amax = 0.f;
  {
    const u32x4* zv = reinterpret_cast<const u32x4*>(zr + head);
    for (int i = tid; i < nvec; i += THREADS) {
      float x[N];
      Vec<T>::unpack(zv[i], x);      // cached load: the row is read again right away
#pragma unroll
      for (int k = 0; k < N; ++k) amax = fmaxf(amax, fabsf(x[k]));
    }
  }
  for (int e = tid; e < vocab - nvec * N; e += THREADS)
    amax = fmaxf(amax, fabsf(Vec<T>::load1(zr + (e < head ? 0 : nvec * N) + e)));
  amax = wave_max(amax);
  if (THREADS == 64) return amax;
  if ((tid & 63) == 0) lds[tid >> 6] = amax;
  __syncthreads();
#pragma unroll
  for (int w = 0; w < THREADS / 64; ++w) amax = fmaxf(amax, lds[w]);
  return amax;
}

// The largest magnitude bits of a 16-byte aligned bf16 row, NaNs (above 0x7f80) included: as 16-bit integers, two to an
// instruction.
template <int THREADS>
__device__ __forceinline__ uint32_t row_top_bits(const bf16_t* zr, int vocab, uint32_t* lds) {
  typedef uint16_t u16x2 __attribute__((ext_vector_type(2)));
  const int tid = threadIdx.x;
  const int nvec = vocab / 8;
  u16x2 m = {0, 0};
  const u32x4* zv = reinterpret_cast<const u32x4*>(zr);
  for (int i = tid; i < nvec; i += THREADS) {
    const u32x4 q = zv[i];                 // cached load: the row is read again right away
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const uint32_t word = q[k] & 0x7fff7fffu;
      m = __builtin_elementwise_max(m, __builtin_bit_cast(u16x2, word));
    }
  }
  uint32_t top = max((uint32_t)m[0], (uint32_t)m[1]);
  if (tid < vocab - nvec * 8) top = max(top, (uint32_t)zr[nvec * 8 + tid] & 0x7fffu);
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) top = max(top, (uint32_t)__shfl_xor((int)top, off));
  if (THREADS == 64) return top;
  if ((tid & 63) == 0) lds[tid >> 6] = top;
  __syncthreads();
#pragma unroll
  for (int w = 0; w < THREADS / 64; ++w) top = max(top, lds[w]);
  __syncthreads();                         // `lds` may be used again
  return top;
}

// Where logits are larger than this, the difference between an exact and a rounded product of logit and log2(e) is no
// longer small (see accumulate_special).
constexpr float kLargeAmax = 16777216.f;

// As accumulate; where `rounded` is set (uniform), the products are rounded like the maximum's before it is subtracted: the
// maximum's own term is 1 whatever the magnitude, where the fma leaves the rounding of the maximum as its exponent (2^(1e3)
// at 1e11).  The rounding of the others is an error of 6e-8 of the product in their exponents, which is why ordinary rows
// keep the fma.
template <int n>
__device__ __forceinline__ void accumulate_special(const float* x, float scale, bool rounded, MaxSum& st) {
  float cm = x[0];
#pragma unroll
  for (int k = 1; k < n; ++k) cm = fmaxf(cm, x[k]);
  const float mn = fmaxf(st.m, cm * scale);
  auto term = [&](float v) {
#pragma clang fp contract(off)
    const float product = v * scale;
    return exp2_fast(rounded ? product - mn : __builtin_fmaf(v, scale, -mn));
  };
  float acc0 = st.s * exp2_fast(st.m - mn), acc1 = 0.f;
#pragma unroll
  for (int k = 0; k < n; k += 2) {
    acc0 += term(x[k]);
    if (k + 1 < n) acc1 += term(x[k + 1]);
  }
  st.m = mn;
  st.s = acc0 + acc1;
}

// A row's scale, how its elements are divided by it, and their code as an fp32 value (exact in E4M3).
// BITS: a 16-byte aligned bf16 row.  There, as in the table kernels that take the wider ones, a NaN has the code of the
// row's largest magnitude and its own sign; elsewhere a NaN's code is that of -448.  In a row with an infinity, whose scale
// is infinite, every infinity and every NaN is -448 and everything else a zero of its own sign, aligned or not.
template <typename T, int THREADS, bool BITS>
struct RowCoder {
  RowDivider d;
  float amax;
  bool special, large;                     // uniform for the workgroup; large: see accumulate_special
  __device__ __forceinline__ RowCoder(const T* zr, int vocab, int head, float* lds) {
    bool nan = false;
    if constexpr (BITS) {
      const uint32_t top = row_top_bits<THREADS>(zr, vocab, reinterpret_cast<uint32_t*>(lds));
      nan = top > 0x7f80u;
      amax = nan ? row_amax<T, THREADS>(zr, vocab, head, lds) : __uint_as_float(top << 16);
    } else {
      amax = row_amax<T, THREADS>(zr, vocab, head, lds);
    }
    d = make_divider(scale_of(amax));
    special = d.slow || nan;
    large = amax > kLargeAmax;
  }
  template <bool SPECIAL>
  __device__ __forceinline__ float quotient(float x) const {
    if (!SPECIAL) return divide<false>(x, d);
    if (!BITS) return divide<true>(x, d);
    const uint32_t mag = min(__float_as_uint(x) & 0x7fffffffu, __float_as_uint(amax));
    return __uint_as_float(mag) / d.s;
  }
  // two elements -> two codes in the low 16 bits
  template <bool SPECIAL>
  __device__ __forceinline__ uint32_t code2(float a, float b) const {
    uint32_t c = to_e4m3x2(quotient<SPECIAL>(a), quotient<SPECIAL>(b));
    if (SPECIAL && BITS) c |= (__float_as_uint(a) >> 24 & 0x80u) | (__float_as_uint(b) >> 16 & 0x8000u);
    return c;
  }
};

// VEC: the codes of a vector are aligned to their number; otherwise they are written one by one.
template <typename T, bool VEC, int THREADS, bool BITS>
__global__ __launch_bounds__(THREADS) void fp8_quantize_kernel(const T* __restrict__ logits, long long row_stride,
                                                               int vocab, unsigned char* __restrict__ codes,
                                                               long long codes_stride, float* __restrict__ scale_out) {
  constexpr int N = Vec<T>::N;
  __shared__ float lds[THREADS / 64];
  const long long row = blockIdx.x;
  const int tid = threadIdx.x;
  const T* zr = logits + row * row_stride;
  unsigned char* cr = codes + row * codes_stride;
  const int lead = BITS ? 0 : head_elements(zr, vocab);
  const RowCoder<T, THREADS, BITS> coder(zr, vocab, lead, lds);
  if (tid == 0) scale_out[row] = coder.d.s;
  const int head = VEC ? lead : 0;
  const int nvec = VEC ? (vocab - head) / N : 0;
  auto encode = [&](auto slow) {
    constexpr bool SLOW = decltype(slow)::value;
    if (VEC) {
      const u32x4* zv = reinterpret_cast<const u32x4*>(zr + head);
      unsigned char* cv = cr + head;
      for (int i = tid; i < nvec; i += THREADS) {
        float x[N];
        Vec<T>::unpack(load_stream(zv + i), x);
        uint32_t w[N / 4];
#pragma unroll
        for (int k = 0; k < N / 4; ++k)
          w[k] = coder.template code2<SLOW>(x[4 * k], x[4 * k + 1]) |
                 (coder.template code2<SLOW>(x[4 * k + 2], x[4 * k + 3]) << 16);
        if (N == 8) {
          uint2 o = {w[0], w[N / 4 - 1]};
          *reinterpret_cast<uint2*>(cv + (long long)i * N) = o;
        } else {
          *reinterpret_cast<uint32_t*>(cv + (long long)i * N) = w[0];
        }
      }
    }
    for (int e = tid; e < vocab - nvec * N; e += THREADS) {
      const int v = e < head ? e : e + nvec * N;
      cr[v] = (unsigned char)(coder.template code2<SLOW>(Vec<T>::load1(zr + v), 0.f) & 0xffu);
    }
  };
  if (coder.special) encode(std::true_type{}); else encode(std::false_type{});
}

template <typename T, bool VEC>
__global__ __launch_bounds__(kSweepThreads) void fp8_dequantize_kernel(const unsigned char* __restrict__ codes,
                                                                       long long codes_stride,
                                                                       const float* __restrict__ scale, int vocab,
                                                                       T* __restrict__ out, long long out_stride) {
  constexpr int THREADS = kSweepThreads;
  constexpr int N = Vec<T>::N;
  const long long row = blockIdx.x;
  const int tid = threadIdx.x;
  const unsigned char* cr = codes + row * codes_stride;
  T* orow = out + row * out_stride;
  const float s = scale[row];
  const int nvec = VEC ? vocab / N : 0;
  if (VEC) {
    u32x4* ov = reinterpret_cast<u32x4*>(orow);
    for (int i = tid; i < nvec; i += THREADS) {
      uint32_t w[2];
      if (N == 8) {
        const uint2 c = *reinterpret_cast<const uint2*>(cr + (long long)i * N);
        w[0] = c.x;
        w[1] = c.y;
      } else {
        w[0] = *reinterpret_cast<const uint32_t*>(cr + (long long)i * N);
        w[1] = 0;
      }
      float x[N];
#pragma unroll
      for (int k = 0; k < N / 4; ++k) {
        const f32x2v lo = from_e4m3x2(w[k] & 0xffffu), hi = from_e4m3x2(w[k] >> 16);
        x[4 * k] = lo[0] * s;
        x[4 * k + 1] = lo[1] * s;
        x[4 * k + 2] = hi[0] * s;
        x[4 * k + 3] = hi[1] * s;
      }
      store_stream(ov + i, Vec<T>::pack(x));
    }
  }
  for (int v = nvec * N + tid; v < vocab; v += THREADS) Vec<T>::store1(orow + v, from_e4m3x2(cr[v])[0] * s);
}

// log softmax(z_r)[y] with z_r = s * e4m3(z / s): abs-max pass, then a streaming log-sum-exp over the
// round-tripped values.
template <typename T, int THREADS, bool BITS>
__global__ __launch_bounds__(THREADS) void fp8_rollout_logprob_kernel(
    const T* __restrict__ logits, long long row_stride, int vocab, const int* __restrict__ token_ids,
    const unsigned char* __restrict__ valid, float* __restrict__ logp_out, int* __restrict__ status) {
  constexpr int N = Vec<T>::N;
  __shared__ float lds[THREADS / 64];
  __shared__ MaxSum lds_ms[THREADS / 64];
  const long long row = blockIdx.x;
  const int tid = threadIdx.x;
  if (valid != nullptr && valid[row] == 0) {
    if (tid == 0) logp_out[row] = 0.f;
    return;
  }
  const T* zr = logits + row * row_stride;
  const int head = BITS ? 0 : head_elements(zr, vocab);
  const RowCoder<T, THREADS, BITS> coder(zr, vocab, head, lds);
  const float s = coder.d.s;
  const int nvec = (vocab - head) / N;
  MaxSum st{kNegHuge, 0.f};
  // the round-tripped logit is s * decode(code): the row scale is folded into the exponent's multiplier (s > 0,
  // so the running maximum can be taken over the decoded values)
  const float scale = s * kLog2e;
  auto sweep = [&](auto slow) {
    constexpr bool SLOW = decltype(slow)::value;
    {
      const u32x4* zv = reinterpret_cast<const u32x4*>(zr + head);
      for (int i = tid; i < nvec; i += THREADS) {
        float x[N];
        Vec<T>::unpack(load_stream(zv + i), x);
#pragma unroll
        for (int k = 0; k < N; k += 2) {
          const f32x2v r = from_e4m3x2(coder.template code2<SLOW>(x[k], x[k + 1]));
          x[k] = r[0];
          x[k + 1] = r[1];
        }
        if (SLOW) accumulate_special<N>(x, scale, coder.large, st);
        else accumulate<N>(x, scale, st);
      }
    }
    for (int e = tid; e < vocab - nvec * N; e += THREADS) {
      float x = from_e4m3x2(coder.template code2<SLOW>(Vec<T>::load1(zr + (e < head ? 0 : nvec * N) + e), 0.f))[0];
      if (SLOW) accumulate_special<1>(&x, scale, coder.large, st);
      else accumulate<1>(&x, scale, st);
    }
  };
  if (coder.special || coder.large) sweep(std::true_type{}); else sweep(std::false_type{});
  st = wave_merge(st);
  if ((tid & 63) == 0) lds_ms[tid >> 6] = st;
  __syncthreads();
  if (tid == 0) {
    MaxSum t = lds_ms[0];
#pragma unroll
    for (int w = 1; w < THREADS / 64; ++w) t = merge(t, lds_ms[w]);
    const int y = token_ids[row];
    if (y >= 0 && y < vocab) {
      const float zy = from_e4m3x2(to_e4m3x2(Vec<T>::load1(zr + y) / s, 0.f))[0] * s;
      logp_out[row] = zy - (t.m + log2_fast(t.s)) * kLn2;
    } else {
      logp_out[row] = 0.f;
      atomicOr(status, AIS_STATUS_BAD_TOKEN);
    }
  }
}

bool aligned(const void* p, long long stride_bytes, int a) {
  return reinterpret_cast<uintptr_t>(p) % a == 0 && stride_bytes % a == 0;
}

// Rows that would take the table kernels if they were wider.
bool narrow_table_rows(const void* z, ais_dtype dtype, int vocab, long long row_stride) {
  return dtype == AIS_BF16 && aligned(z, row_stride * 2, 16) && vocab >= 8 && vocab <= kFp8NarrowRow;
}

// Runs `launch` with the number of threads that share a row (quantisation, log-prob) as a constant: one wavefront, which
// needs no barrier, where there are many rows of up to 4 KiB.  us, 64 and 256 threads: 41,643 rows of 1,000 bf16 logits
// quantised 25.6 and 42.4, log-prob 31.1 and 59.1; of 4,096 124.9 and 98.6, 100.7 and 120.7; 8,192 of 2,048 12.8 and 12.5, 14.5 and
// 16.6; of 4,096 26.8 and 19.0, 27.3 and 24.9; 41,643 of 1,024 fp32 39.4 and 47.9, 40.4 and 62.4; of 2,048 106.5 and 81.5,
// 84.2 and 90.7.
template <typename F>
void with_threads(const ais_ctx* ctx, long long n_rows, long long row_bytes, F launch) {
  if (row_bytes <= 4096 && n_rows >= 8 * ctx->n_cus) launch(std::integral_constant<int, 64>{});
  else launch(std::integral_constant<int, kSweepThreads>{});
}

}  // namespace

int launch_fp8_quantize(ais_ctx* ctx, const void* logits, ais_dtype dtype, long long n_rows, int vocab,
                        long long row_stride, unsigned char* codes, long long codes_stride, float* scale_out) {
  if (n_rows == 0) return AIS_OK;
  dim3 grid((unsigned)n_rows);
  ScopedTimer timer(ctx, AIS_K_FP8_QUANT);
  if (try_fp8_quantize_table(ctx, logits, dtype, n_rows, vocab, row_stride, codes, codes_stride, scale_out))
    return hip_fail(ctx, hipGetLastError());      // bf16 row held in registers, codes from a per-row table
  if (try_fp8_quantize_rows(ctx, logits, dtype, n_rows, vocab, row_stride, codes, codes_stride, scale_out))
    return hip_fail(ctx, hipGetLastError());      // row held in registers: one read of the logits
  const bool bits = narrow_table_rows(logits, dtype, vocab, row_stride);
  auto launch = [&](const auto* z) {
    typedef std::remove_cv_t<std::remove_pointer_t<decltype(z)>> T;
    constexpr int N = Vec<T>::N;
    // vectors start a multiple of N elements from any other place that is 16-byte aligned
    const bool vec = (reinterpret_cast<uintptr_t>(codes) - reinterpret_cast<uintptr_t>(z) / sizeof(T)) % N == 0 &&
                     (codes_stride - row_stride) % N == 0;
    with_threads(ctx, n_rows, (long long)vocab * sizeof(T), [&](auto threads) {
      constexpr int kThreads = decltype(threads)::value;
      auto kernel = vec ? fp8_quantize_kernel<T, true, kThreads, false> : fp8_quantize_kernel<T, false, kThreads, false>;
      if constexpr (sizeof(T) == 2) {
        if (vec && bits) kernel = fp8_quantize_kernel<T, true, kThreads, true>;
      }
      kernel<<<grid, dim3(kThreads), 0, ctx->stream>>>(z, row_stride, vocab, codes, codes_stride, scale_out);
    });
  };
  if (dtype == AIS_BF16) launch(static_cast<const bf16_t*>(logits));
  else launch(static_cast<const float*>(logits));
  return hip_fail(ctx, hipGetLastError());
}

int launch_fp8_dequantize(ais_ctx* ctx, const unsigned char* codes, long long codes_stride, const float* scale,
                          long long n_rows, int vocab, void* out, ais_dtype dtype, long long out_stride) {
  if (n_rows == 0) return AIS_OK;
  dim3 grid((unsigned)n_rows);
  ScopedTimer timer(ctx, AIS_K_FP8_DEQUANT);
  if (try_fp8_dequantize_burst(ctx, codes, codes_stride, scale, n_rows, vocab, out, dtype, out_stride))
    return hip_fail(ctx, hipGetLastError());
  auto launch = [&](auto* o) {
    typedef std::remove_pointer_t<decltype(o)> T;
    constexpr int N = Vec<T>::N;
    const bool vec = aligned(o, out_stride * (long long)sizeof(T), 16) && aligned(codes, codes_stride, N);
    auto kernel = vec ? fp8_dequantize_kernel<T, true> : fp8_dequantize_kernel<T, false>;
    kernel<<<grid, dim3(kSweepThreads), 0, ctx->stream>>>(codes, codes_stride, scale, vocab, o, out_stride);
  };
  if (dtype == AIS_BF16) launch(static_cast<bf16_t*>(out));
  else launch(static_cast<float*>(out));
  return hip_fail(ctx, hipGetLastError());
}

int launch_fp8_rollout_logprob(ais_ctx* ctx, const void* logits, ais_dtype dtype, long long n_rows, int vocab,
                               long long row_stride, const int* token_ids, const unsigned char* valid,
                               float* logp_out) {
  if (n_rows == 0) return AIS_OK;
  dim3 grid((unsigned)n_rows);
  ScopedTimer timer(ctx, AIS_K_FP8_LOGPROB);
  if (try_fp8_rollout_logprob_table(ctx, logits, dtype, n_rows, vocab, row_stride, token_ids, valid, logp_out))
    return hip_fail(ctx, hipGetLastError());      // bf16 row read once, terms of the sum from a per-row table
  const bool bits = narrow_table_rows(logits, dtype, vocab, row_stride);
  auto launch = [&](const auto* z) {
    typedef std::remove_cv_t<std::remove_pointer_t<decltype(z)>> T;
    with_threads(ctx, n_rows, (long long)vocab * sizeof(T), [&](auto threads) {
      constexpr int kThreads = decltype(threads)::value;
      auto kernel = fp8_rollout_logprob_kernel<T, kThreads, false>;
      if constexpr (sizeof(T) == 2) {
        if (bits) kernel = fp8_rollout_logprob_kernel<T, kThreads, true>;
      }
      kernel<<<grid, dim3(kThreads), 0, ctx->stream>>>(z, row_stride, vocab, token_ids, valid, logp_out,
                                                       ctx->status_dev);
    });
  };
  if (dtype == AIS_BF16) launch(static_cast<const bf16_t*>(logits));
  else launch(static_cast<const float*>(logits));
  return hip_fail(ctx, hipGetLastError());
}

}  // namespace ais
