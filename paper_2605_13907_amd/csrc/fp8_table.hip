// FP8-E4M3 per-row quantisation and rollout log-prob for bf16 logits by table lookup.
//
// A bf16 logit has 15 magnitude bits, and only the 20 binades below the row's abs-max can give a non-zero E4M3
// code (the quotient z / s of anything smaller lies below 2^-10, half the smallest E4M3 value).  So a row has at
// most 2,560 distinct magnitudes that matter, against 150,000 elements: once the row's scale s = max|z| / 448 is
// known (Eq. 1 with the E4M3 grid, Sec. 2.1), the workgroup evaluates
//     code(m) = e4m3(RN(m / s))            true fp32 division, then the hardware conversion (round to nearest even)
// once per magnitude m into a table in LDS, and every element then costs a table read instead of a correctly rounded
// division and a conversion.  The arithmetic that decides a code is exactly the plain definition's; it is only
// done once per distinct input.  For the rollout log-prob the table holds exp(z_r(m) - max_v z_r) for both signs
// directly, so the sweep over the row needs no division, no conversion and no exponential at all.
//
// One workgroup of 1,024 threads per row; the row is read from HBM once and waits in registers (up to 24 16-byte
// vectors per lane, 196,608 logits; 23 for the log-prob, which parks up to 8 more per lane in LDS: 253,952 logits)
// while the table is built.  Rows that are not 16-byte aligned are split at their first 128-byte boundary (see
// head_elements).  Wider or fp32 rows take the kernels of fp8_rows.hip / fp8.hip.
#include "ais_internal.h"
#include "device_utils.h"
#include "fp8_utils.h"

#include <type_traits>

namespace ais {
namespace {

using namespace dev;

constexpr int kRowThreads = 1024;
constexpr int kRowWaves = kRowThreads / 64;
constexpr int kTabEntries = 2560;             // 20 binades x 128 significands, ending at the row's abs-max
constexpr int kTabStride = 4096;              // floats between the two sign halves of the log-prob table
constexpr int kSlotBytes = kRowThreads * 16;  // one 16-byte vector per thread
typedef uint16_t u16x2 __attribute__((ext_vector_type(2)));
typedef __attribute__((address_space(3))) void* lds_ptr;
typedef const __attribute__((address_space(1))) void* glb_ptr;

// Copies vector min(tid + k * 1024, nvec - 1) of the row at zv into LDS slot `slot` (16 bytes per thread at index
// tid): lane i of a wavefront deposits its 16 bytes at the wavefront's base + 16 i.  nvec >= 1.
__device__ __forceinline__ void copy_to_slot(const u32x4* zv, int nvec, int k, u32x4* slot, int tid) {
  const int i = min(tid + k * kRowThreads, nvec - 1);
  __builtin_amdgcn_global_load_lds((glb_ptr)(zv + (unsigned)i), (lds_ptr)(slot + (tid & ~63)), 16, 0,
                                   2 /* non-temporal */);
}

__device__ __forceinline__ float bf16_bits_to_float(int bits) { return __uint_as_float((uint32_t)bits << 16); }

// E4M3 code of q (saturating, round to nearest even) and the value of a code.
__device__ __forceinline__ uint32_t code_of(float q) { return to_e4m3x2(q, 0.f) & 0xffu; }
__device__ __forceinline__ float value_of(uint32_t code) { return from_e4m3x2(code)[0]; }

// Where the parts of a row lie: `head` elements, then `nvec` vectors from `zv` on, then the rest.  The elements outside
// the vectors are handled one by one by the first `rest` threads.
template <bool ALIGNED>
struct RowParts {
  const bf16_t* zr;
  const u32x4* zv;
  int head, nvec, rest;
  __device__ __forceinline__ RowParts(const bf16_t* row, int vocab) : zr(row) {
    head = ALIGNED ? 0 : head_elements(row, vocab);
    nvec = (vocab - head) / 8;
    rest = vocab - nvec * 8;
    zv = reinterpret_cast<const u32x4*>(row + head);
  }
  // index of the element that thread `tid` < rest owns (from an opaque copy of the thread index: nothing of it is kept
  // in registers across the row loop)
  __device__ __forceinline__ int outside(int tid) const {
    asm volatile("" : "+v"(tid));
    return (ALIGNED || tid >= head ? nvec * 8 : 0) + tid;
  }
  // that element, or (the other threads) some element of the row: neither changes its extremes
  __device__ __forceinline__ float load_outside(int tid) const {
    asm volatile("" : "+v"(tid));
    return Vec<bf16_t>::load1(zr + (tid < rest ? outside(tid) : 0));
  }
  // Vector tid + 1024 k; past the end of the row (possible only if !full) its last vector, which changes neither
  // maximum nor minimum and is never summed.  nvec >= 1.
  __device__ __forceinline__ u32x4 load(int tid, int k, bool full) const {
    if (!full) return load_stream(zv + (unsigned)min(tid + k * kRowThreads, nvec - 1));
    // uniform base + one 32-bit offset for all vectors: an address costs a scalar addition and no vector instruction
    const u32x4* base = zv + k * kRowThreads;
    asm volatile("" : "+s"(base));
    return load_stream(base + (unsigned)tid);
  }
};

// Issues the loads of a row: q[k] is vector tid + 1024 k of the row, xt the thread's element outside the vectors.  KFULL:
// vectors 0 .. KFULL - 1 of every lane are certain to exist.
template <bool ALIGNED, int NV, int KFULL>
__device__ __forceinline__ void issue_row(const RowParts<ALIGNED>& row, u32x4 (&q)[NV], float& xt) {
  const int tid = threadIdx.x;
#pragma unroll
  for (int k = 0; k < NV; ++k) q[k] = row.load(tid, k, k < KFULL);
  xt = row.load_outside(tid);
}

typedef int16_t i16x2 __attribute__((ext_vector_type(2)));

template <int LEVEL>
__device__ __forceinline__ uint32_t lane_partner(uint32_t v) {        // butterfly partner, levels 0..5
  if (LEVEL >= 4) return __shfl_xor(v, 1 << LEVEL);
  constexpr int kCtrl = LEVEL == 0   ? kDppQuadXor1
                        : LEVEL == 1 ? kDppQuadXor2
                        : LEVEL == 2 ? kDppRowHalfMirror
                                     : kDppRowMirror;
  return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, kCtrl, 0xf, 0xf, true);
}

// The largest and smallest element by comparing numbers: the route for rows with a NaN (it loses every comparison).  Reads
// the row again, from memory.
template <bool ALIGNED>
__device__ __forceinline__ void row_minmax_streamed(const RowParts<ALIGNED>& row, float* lds, float& zmax,
                                                    float& zmin) {
  const int tid = threadIdx.x;
  float hi = row.load_outside(tid), lo = hi;
  for (int i = tid; i < row.nvec; i += kRowThreads) {
    float x[8];
    Vec<bf16_t>::unpack(load_stream(row.zv + i), x);
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      hi = fmaxf(hi, x[k]);
      lo = fminf(lo, x[k]);
    }
  }
  hi = wave_max(hi);
  lo = -wave_max(-lo);
  __syncthreads();                                          // `lds` is still being read by the caller's reduction
  if ((tid & 63) == 0) {
    lds[tid >> 6] = hi;
    lds[kRowWaves + (tid >> 6)] = lo;
  }
  __syncthreads();
  hi = lds[0];
  lo = lds[kRowWaves];
#pragma unroll
  for (int w = 1; w < kRowWaves; ++w) {
    hi = fmaxf(hi, lds[w]);
    lo = fminf(lo, lds[kRowWaves + w]);
  }
  zmax = hi == hi || !ALIGNED ? hi : 0.f;                   // nothing but NaNs (the largest is then one, see kLastEntry)
  zmin = lo == lo ? lo : 0.f;
}

// Largest and smallest element of the row held in q[], the NL LDS slots at lrow (slot j: 16 bytes per thread at index
// 1024 j + tid; every slot holds vectors of the row, possibly repeated ones) and xt, returned to every thread.
// `lds`: 2 * kRowWaves floats.
// The bits of bf16 numbers order them: as signed 16-bit integers the largest is the largest number if there is one
// without a sign, as unsigned integers it is the smallest number if there is one with a sign.  Two packed instructions
// per two logits instead of three.  In a row where every number has a sign the largest is the smallest unsigned integer,
// which a second look at the registers and slots finds (logits shifted below zero or log-probabilities are such rows: 2,632
// of 151,936 logits quantised in 259 us against 255 where signs are mixed, log-prob 160 and 153; 422 and 294 when they
// were read again from memory); a row with a NaN takes the route above.  (With no negative element the smallest is reported
// as 0, which is as good for a caller that asks for the largest magnitude.)
template <bool ALIGNED, int NV, int NL = 0>
__device__ __forceinline__ void row_minmax(u32x4 (&q)[NV], float xt, float* lds, float& zmax, float& zmin,
                                           const RowParts<ALIGNED>& row, const u32x4* lrow = nullptr) {
  const int tid = threadIdx.x;
  const uint32_t x2 = (__float_as_uint(xt) >> 16) * 0x00010001u;
  i16x2 s = __builtin_bit_cast(i16x2, x2);
  u16x2 u = __builtin_bit_cast(u16x2, x2);
  auto fold = [&](const u32x4& v) {
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      const uint32_t word = v[w];              // (a bit cast of the vector element itself would read the first one)
      s = __builtin_elementwise_max(s, __builtin_bit_cast(i16x2, word));
      u = __builtin_elementwise_max(u, __builtin_bit_cast(u16x2, word));
    }
  };
#pragma unroll
  for (int k = 0; k < NV; ++k) {
    fold(q[k]);
    __builtin_amdgcn_sched_barrier(0);
  }
  if (NL > 0) {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");       // the copies into the slots have landed
    int t1 = tid;
    asm volatile("" : "+v"(t1));
#pragma unroll
    for (int j = 0; j < NL; ++j) {
      fold(lrow[j * kRowThreads + t1]);
      __builtin_amdgcn_sched_barrier(0);
    }
  }
  auto level = [&](auto k) {
    constexpr int K = decltype(k)::value;
    s = __builtin_elementwise_max(s, __builtin_bit_cast(i16x2, lane_partner<K>(__builtin_bit_cast(uint32_t, s))));
    u = __builtin_elementwise_max(u, __builtin_bit_cast(u16x2, lane_partner<K>(__builtin_bit_cast(uint32_t, u))));
  };
  level(std::integral_constant<int, 0>{});
  level(std::integral_constant<int, 1>{});
  level(std::integral_constant<int, 2>{});
  level(std::integral_constant<int, 3>{});
  level(std::integral_constant<int, 4>{});
  level(std::integral_constant<int, 5>{});
  uint32_t* lds_u = reinterpret_cast<uint32_t*>(lds);
  if ((tid & 63) == 0) {
    lds_u[tid >> 6] = __builtin_bit_cast(uint32_t, s);
    lds_u[kRowWaves + (tid >> 6)] = __builtin_bit_cast(uint32_t, u);
  }
  __syncthreads();
#pragma unroll
  for (int w = 0; w < kRowWaves; ++w) {
    s = __builtin_elementwise_max(s, __builtin_bit_cast(i16x2, lds_u[w]));
    u = __builtin_elementwise_max(u, __builtin_bit_cast(u16x2, lds_u[kRowWaves + w]));
  }
  const int smax = max((int)s[0], (int)s[1]), umax = max((int)u[0], (int)u[1]);
  zmax = bf16_bits_to_float(smax);
  zmin = umax >= 0x8000 ? bf16_bits_to_float(umax) : 0.f;
  if (smax > 0x7f80 || umax > 0xff80) {                    // a NaN (uniform for the workgroup, as what follows)
    row_minmax_streamed<ALIGNED>(row, lds, zmax, zmin);
  } else if (smax < 0) {
    // where the registers are all in use: nothing but the element itself is kept for this (elsewhere it costs 2-5 %)
    if (NV > 20 && NL == 0) asm volatile("" : "+v"(xt));
    u16x2 m = __builtin_bit_cast(u16x2, (__float_as_uint(xt) >> 16) * 0x00010001u);
    auto fold_min = [&](const u32x4& v) {
#pragma unroll
      for (int w = 0; w < 4; ++w) {
        const uint32_t word = v[w];
        m = __builtin_elementwise_min(m, __builtin_bit_cast(u16x2, word));
      }
    };
#pragma unroll
    for (int k = 0; k < NV; ++k) {
      fold_min(q[k]);
      __builtin_amdgcn_sched_barrier(0);
    }
    if (NL > 0) {
      int t1 = tid;
      asm volatile("" : "+v"(t1));
#pragma unroll
      for (int j = 0; j < NL; ++j) {
        fold_min(lrow[j * kRowThreads + t1]);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    auto level_min = [&](auto k) {
      m = __builtin_elementwise_min(
          m, __builtin_bit_cast(u16x2, lane_partner<decltype(k)::value>(__builtin_bit_cast(uint32_t, m))));
    };
    level_min(std::integral_constant<int, 0>{});
    level_min(std::integral_constant<int, 1>{});
    level_min(std::integral_constant<int, 2>{});
    level_min(std::integral_constant<int, 3>{});
    level_min(std::integral_constant<int, 4>{});
    level_min(std::integral_constant<int, 5>{});
    __syncthreads();                                       // `lds` is still being read for the other extremes
    if ((tid & 63) == 0) lds_u[tid >> 6] = __builtin_bit_cast(uint32_t, m);
    __syncthreads();
#pragma unroll
    for (int w = 0; w < kRowWaves; ++w) m = __builtin_elementwise_min(m, __builtin_bit_cast(u16x2, lds_u[w]));
    zmax = bf16_bits_to_float(min((int)m[0], (int)m[1]));
  }
  // keep the row packed until the scale is known (the empty asm names the reduction result as an input)
#pragma unroll
  for (int k = 0; k < NV; ++k) asm volatile("" : "+v"(q[k]) : "v"(zmax));
}

// Workgroups of a kernel that a compute unit holds at once: with up to 8 vectors per lane (65,536 logits) a row leaves
// room for a second one, whose loads and sums overlap the first one's reductions and table.  Log-prob, 20,000 rows: of
// 32,000 logits 318 us with one, 287 with two; of 65,536 516 and 478.  Quantisation, where stores are the larger part of
// the traffic: of 32,000 676 and 659 (with the decoding), but of 65,536 1,342 and 1,373, so only up to 4 vectors.
constexpr int logprob_workgroups(int nv) { return nv <= 8 ? 2 : 1; }
constexpr int quantize_workgroups(int nv) { return nv <= 4 ? 2 : 1; }
// wavefronts per SIMD that the register budget has to allow for
constexpr int waves_of(int workgroups) { return workgroups * kRowThreads / 256; }

// Table index of a bf16 magnitude (15 bits): magnitudes below the table's first entry share it (their code is 0,
// as is the first entry's), and nothing finite lies above the last entry, the row's abs-max; a NaN's payload does,
// and is held at `last`: the last entry in aligned rows, and in the others an entry of its own behind it, which codes a
// NaN as the streaming kernels do, -448.
template <bool ALIGNED>
constexpr int kLastEntry = ALIGNED ? kTabEntries - 1 : kTabEntries;
__device__ __forceinline__ int table_index(uint32_t mag, int base, int last) { return min(max((int)mag - base, 0), last); }

// ---- quantise ----------------------------------------------------------------------------------------------
// Persistent grid (quantize_workgroups() per compute unit), rows dealt round-robin; the registers of a vector whose codes have
// been written are reloaded at once with the same vector of the workgroup's next row (see the log-prob kernel below
// for why).
template <bool ALIGNED, int NV, int KFULL>
__global__ __launch_bounds__(kRowThreads, waves_of(quantize_workgroups(NV))) void fp8_quantize_table_kernel(const bf16_t* __restrict__ logits,
                                                                         long long row_stride, int vocab,
                                                                         unsigned char* __restrict__ codes,
                                                                         long long codes_stride,
                                                                         float* __restrict__ scale_out,
                                                                         long long n_rows) {
  __shared__ float lds[2 * kRowWaves];
  constexpr int kLast = kLastEntry<ALIGNED>;
  __shared__ unsigned char table[kLast + 1];
  const int tid = threadIdx.x;
  long long row = blockIdx.x;
  if (row >= n_rows) return;
  RowParts<ALIGNED> at(logits + row * row_stride, vocab);
  u32x4 q[NV];
  float xt;
  issue_row<ALIGNED, NV, KFULL>(at, q, xt);
  for (; row < n_rows; row += gridDim.x) {
    unsigned char* cr = codes + row * codes_stride;
    // after its last row a workgroup fetches that row once more (into registers nobody reads again): the loop
    // body stays free of conditions, which keeps the reloaded registers the very ones that were just read
    const RowParts<ALIGNED> next(logits + (row + gridDim.x < n_rows ? row + gridDim.x : row) * row_stride, vocab);
    float zmax, zmin;
    row_minmax<ALIGNED, NV>(q, xt, lds, zmax, zmin, at);
    const float amax = fmaxf(fmaxf(zmax, -zmin), 0.f);       // (0: nothing but NaNs)
    const float s = scale_of(amax);
    if (tid == 0) scale_out[row] = s;
    // entry i belongs to the bf16 magnitude with bits base + i; the last entry is the abs-max itself
    const int base = (int)(__float_as_uint(amax) >> 16) - (kTabEntries - 1);
    const RowDivider by_s = make_divider(s);
    auto fill = [&](auto slow) {
      for (int i = tid; i < kTabEntries; i += kRowThreads)
        table[i] = (unsigned char)code_of(divide<decltype(slow)::value>(bf16_bits_to_float(max(base + i, 0)), by_s));
    };
    if (by_s.slow) fill(std::true_type{}); else fill(std::false_type{});
    if (!ALIGNED && tid == 0) table[kLast] = 0xfe;                  // the code of -448
    __syncthreads();
    auto code2 = [&](uint32_t w) -> uint32_t {           // two logits -> two codes in the low 16 bits
      const uint32_t c0 = table[table_index(w & 0x7fffu, base, kLast)];
      const uint32_t c1 = table[table_index((w >> 16) & 0x7fffu, base, kLast)];
      // the sign of the logit is the sign of the code, zero included
      return c0 | (c1 << 8) | ((w >> 8) & 0x80u) | ((w >> 16) & 0x8000u);
    };
    unsigned char* cv = cr + at.head;                    // a vector's codes: 8-byte aligned (the launcher checks)
#pragma unroll
    for (int k = 0; k < NV; ++k) {
      // the slot's index comes from a fresh opaque copy of the thread index: otherwise every slot's load and store
      // offsets are computed once, ahead of the row loop, and stay alive in four registers per slot
      int tk = tid;
      asm volatile("" : "+v"(tk));
      __builtin_assume(tk >= 0 && tk < kRowThreads);
      const int i = tk + k * kRowThreads;
      uint2 o;
      o.x = code2(q[k][0]) | (code2(q[k][1]) << 16);
      asm volatile("" : "+v"(o.x));                      // four table reads in flight at a time: fewer registers
      __builtin_amdgcn_sched_barrier(0);
      o.y = code2(q[k][2]) | (code2(q[k][3]) << 16);
      asm volatile("" : "+v"(o.y));                      // the codes are formed here, before the registers are reused
      __builtin_amdgcn_sched_barrier(0);
      if (k < KFULL || i < at.nvec) *reinterpret_cast<uint2*>(cv + (long long)i * 8) = o;
      // (uniform row base + 32-bit offset.  With scalar bases per vector as in the log-prob kernel the quantisation alone
      // is 4 % faster, 604 against 625 us, but followed by the decoding both take 1,143 us together instead of 1,136.)
      q[k] = load_stream(next.zv + (unsigned)(k < KFULL ? i : min(i, next.nvec - 1)));
      __builtin_amdgcn_sched_barrier(0);
    }
    if (tid < at.rest) cr[at.outside(tid)] = (unsigned char)(code2(__float_as_uint(xt) >> 16) & 0xffu);
    xt = next.load_outside(tid);
    at = next;
    __syncthreads();                                     // everyone has finished reading the table
  }
}

// ---- rollout log-prob ----------------------------------------------------------------------------------------
// logp[n] = z_r[y] - log sum_v exp(z_r[v]) with z_r = s * value(code(z / s)).  The table holds, for every
// magnitude and both signs, 2^(log2e (z_r - max_v z_r)): the row's largest term is exactly 1.
//
// A row (297 KiB at 151,936 logits) fills most of a compute unit's register file, so only one can be resident, and a
// workgroup that loaded, reduced and summed one row after the other would leave the memory system idle while it
// computes.  The grid is therefore persistent (logprob_workgroups() per compute unit, rows dealt round-robin), and the
// registers of the vector that the sum has just consumed are reloaded at once with the same vector of the
// workgroup's next row: by the time the sum is finished the next row is on its way or has landed.
// Bound by the vector ALU (and the LDS reads beside it), so instructions count: 10,411 rows of 151,936 took 597 us with
// three instructions per two logits for the extremes, a shift and an or where the multiply-add is, a 64-bit address per
// vector and a full division per table entry; 538 us (5.9 TB/s) now.  5,000 rows of 248,320: 488 and 438 us.
//
// Rows beyond 23 vectors per lane park vectors 23 .. 23 + NL - 1 of every lane in LDS slots (16 KiB each, filled by
// direct global -> LDS copies); a slot is refilled with the next row's vector by the thread that has just read its
// 16 bytes of it, so no thread ever waits for another.  With slots the two sign halves of the table are interleaved
// (8 bytes per magnitude, 20 KiB) instead of 16 KiB apart (32 KiB), which is what lets 8 slots fit beside it.
__device__ __forceinline__ uint32_t pk_mad(u16x2 t, int factor, uint32_t add) {      // t * factor + add in both halves
  uint32_t r;
  asm("v_pk_mad_u16 %0, %1, %2, %3 op_sel_hi:[1,0,1]" : "=v"(r) : "v"(t), "s"(factor), "v"(add));
  return r;
}

template <bool INTERLEAVED, int LAST>
struct LogprobTable {
  static_assert(LAST < kTabStride, "");
  static constexpr int kFloats = INTERLEAVED ? 2 * (LAST + 1) : 2 * kTabStride;
  // positions (in floats) of magnitude i's positive and negative entry
  static __device__ __forceinline__ int pos(int i) { return INTERLEAVED ? 2 * i : i; }
  static __device__ __forceinline__ int neg(int i) { return INTERLEAVED ? 2 * i + 1 : kTabStride + i; }
  // Byte offsets into the table of the two logits of a word, formed on both 16-bit halves at once: magnitude
  // minus base, saturating at 0 (smaller magnitudes share the first entry: their code is 0, as is its) and held
  // at the last entry (only a NaN's payload lies above the abs-max; see kLastEntry), times the entry pitch plus the sign's part in
  // one multiply-add.
  static __device__ __forceinline__ uint32_t offsets(uint32_t w, uint32_t base2) {
    u16x2 t = __builtin_bit_cast(u16x2, w & 0x7fff7fffu);
    t = __builtin_elementwise_sub_sat(t, __builtin_bit_cast(u16x2, base2));
    t = __builtin_elementwise_min(t, u16x2{LAST, LAST});
    if (INTERLEAVED) {
      static_assert(LAST * 8 + 4 < 0x10000, "an offset must fit a 16-bit half");
      return pk_mad(t, 8, (w >> 13) & 0x00040004u);                           // sign bit -> byte 4 of the entry
    }
    static_assert(kTabStride * 4 == 0x4000, "the sign bit of a half is moved to this bit of its offset");
    return pk_mad(t, 4, (w >> 1) & 0x40004000u);
  }
};

template <bool ALIGNED, int NV, int KFULL, int NL>
__global__ __launch_bounds__(kRowThreads, waves_of(logprob_workgroups(NV))) void fp8_rollout_logprob_table_kernel(
    const bf16_t* __restrict__ logits, long long row_stride, int vocab, const int* __restrict__ token_ids,
    const unsigned char* __restrict__ valid, float* __restrict__ logp_out, int* __restrict__ status,
    long long n_rows) {
  constexpr int kLast = kLastEntry<ALIGNED>;
  typedef LogprobTable<(NL > 0), kLast> Tab;
  __shared__ float lds_mm[2 * kRowWaves];
  __shared__ float lds_sum[kRowWaves];
  __shared__ float table[Tab::kFloats];                    // kTabEntries magnitudes x 2 signs in use
  extern __shared__ __align__(16) unsigned char lds_slots[];
  u32x4* lrow = reinterpret_cast<u32x4*>(lds_slots);       // NL slots
  static_assert(NL == 0 || KFULL >= NV - 1, "rows that need slots fill (all but the end of) every register vector");
  const int tid = threadIdx.x;
  // this workgroup's next evaluated row at or after `r`; rows that are not evaluated get their 0 on the way
  auto next_row = [&](long long r) -> long long {
    for (; r < n_rows; r += gridDim.x) {
      if (valid == nullptr || valid[r] != 0) break;        // uniform
      if (tid == 0) logp_out[r] = 0.f;
    }
    return r;
  };
  long long row = next_row(blockIdx.x);
  if (row >= n_rows) return;
  u32x4 q[NV];
  float xt;
  RowParts<ALIGNED> at(logits + row * row_stride, vocab);
  issue_row<ALIGNED, NV, KFULL>(at, q, xt);
  if (NL > 0) {
    int t0 = tid;
    asm volatile("" : "+v"(t0));
#pragma unroll
    for (int j = 0; j < NL; ++j) {
      copy_to_slot(at.zv, at.nvec, NV + j, lrow + j * kRowThreads, t0);
      __builtin_amdgcn_sched_barrier(0);
    }
  }
  while (row < n_rows) {
    const long long next = next_row(row + gridDim.x);
    // after its last row a workgroup fetches that row once more (into registers nobody reads again): the loop
    // body stays free of conditions, which keeps the reloaded registers the very ones that were just read
    const RowParts<ALIGNED> at_next(logits + (next < n_rows ? next : row) * row_stride, vocab);
    // the sampled token's logit: asked for before the prefetches below, which it would otherwise queue behind
    const int y = token_ids[row];
    const bool y_ok = y >= 0 && y < vocab;
    const float zy_raw = (tid == 0 && y_ok) ? Vec<bf16_t>::load1(at.zr + y) : 0.f;

    float zmax, zmin;
    row_minmax<ALIGNED, NV, NL>(q, xt, lds_mm, zmax, zmin, at, lrow);
    const float amax = fmaxf(fmaxf(zmax, -zmin), 0.f);     // (0: nothing but NaNs)
    const float s = scale_of(amax);
    const float scale = s * kLog2e;                        // z_r * log2e = value(code) * scale
    // quantisation is monotone: the largest round-tripped logit is that of the largest logit
    const float top = value_of(code_of(zmax / s)) * scale;
    // entry i belongs to the bf16 magnitude with bits base + i; the abs-max is the last entry or an earlier one
    const int base = max((int)(__float_as_uint(amax) >> 16) - (kTabEntries - 1), 0);
    const RowDivider by_s = make_divider(s);
    auto fill = [&](auto slow) {
      for (int i = tid; i < kTabEntries; i += kRowThreads) {
        const float v = value_of(code_of(divide<decltype(slow)::value>(bf16_bits_to_float(base + i), by_s)));
        table[Tab::pos(i)] = exp2_fast(__builtin_fmaf(v, scale, -top));
        table[Tab::neg(i)] = exp2_fast(__builtin_fmaf(-v, scale, -top));
      }
    };
    if (by_s.slow) fill(std::true_type{}); else fill(std::false_type{});
    if (!ALIGNED && tid == 0)
      table[Tab::pos(kLast)] = table[Tab::neg(kLast)] = exp2_fast(__builtin_fmaf(-kE4M3Max, scale, -top));
    __syncthreads();
    const uint32_t base2 = (uint32_t)base * 0x00010001u;
    auto entry = [&](uint32_t byte_offset) -> float {
      return *reinterpret_cast<const float*>(reinterpret_cast<const unsigned char*>(table) + byte_offset);
    };
    auto term = [&](uint32_t h) -> float { return entry(Tab::offsets(h, base2) & 0xffffu); };   // h: one bf16, low half
    // sum of the eight terms of one vector
    auto vector_sum = [&](const u32x4& v) -> float {
      float part = 0.f;
#pragma unroll
      for (int w = 0; w < 4; ++w) {
        const uint32_t o = Tab::offsets(v[w], base2);
        part = w == 0 ? entry(o & 0xffffu) : part + entry(o & 0xffffu);
        part += entry(o >> 16);
        if (w == 1) {
          asm volatile("" : "+v"(part));                   // the sum so far is formed here, not deferred
          __builtin_amdgcn_sched_barrier(0);               // four table reads in flight at a time: fewer registers
        }
      }
      asm volatile("" : "+v"(part));
      __builtin_amdgcn_sched_barrier(0);
      return part;
    };
    float acc0 = 0.f;
#pragma unroll
    for (int k = 0; k < NV; ++k) {
      const float part = vector_sum(q[k]);
      // slots past the end of the row hold copies of its last vector, which must not count again; the slot's index comes from a
      // fresh opaque copy of the thread index, so that no per-slot offset is kept alive across the row loop
      int tk = tid;
      asm volatile("" : "+v"(tk));
      __builtin_assume(tk >= 0 && tk < kRowThreads);
      const int i = tk + k * kRowThreads;
      const bool exists = k < KFULL || i < at.nvec;
      acc0 += exists ? part : 0.f;
      // this vector is done with: its registers take the same vector of the next row
      q[k] = at_next.load(tk, k, k < KFULL);
      __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int j = 0; j < NL; ++j) {
      int tk = tid;
      asm volatile("" : "+v"(tk));
      __builtin_assume(tk >= 0 && tk < kRowThreads);
      u32x4* slot = lrow + j * kRowThreads;
      const float part = vector_sum(slot[tk]);             // (the terms have been read out of LDS: `part` is formed)
      acc0 += (tk + (NV + j) * kRowThreads < at.nvec) ? part : 0.f;
      // the thread's 16 bytes of the slot are free: they take the next row's vector
      copy_to_slot(at_next.zv, at_next.nvec, NV + j, slot, tk);
      __builtin_amdgcn_sched_barrier(0);
    }
    if (tid < at.rest) acc0 += term(__float_as_uint(xt) >> 16);
    xt = at_next.load_outside(tid);
    const float acc = wave_sum(acc0);
    if ((tid & 63) == 0) lds_sum[tid >> 6] = acc;
    // also: everyone has finished reading the table.  With slots the barrier is written out: a workgroup fence would
    // wait for the copies of the next row that are on their way into the slots, which is what they are there to avoid
    // (nothing reads a slot before row_minmax has waited for them).
    if (NL > 0) asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    else __syncthreads();
    if (tid == 0) {
      float sum = lds_sum[0];
#pragma unroll
      for (int w = 1; w < kRowWaves; ++w) sum += lds_sum[w];
      if (y_ok) {
        const float zy = value_of(code_of(zy_raw / s)) * s;
        logp_out[row] = zy - (top + log2_fast(sum)) * kLn2;
      } else {
        logp_out[row] = 0.f;
        atomicOr(status, AIS_STATUS_BAD_TOKEN);
      }
    }
    row = next;
    at = at_next;
  }
  // copies of the row fetched once more may still be on their way into the slots
  if (NL > 0) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
}

bool row_aligned(const void* z, long long row_stride) {
  return reinterpret_cast<uintptr_t>(z) % 16 == 0 && (row_stride * 2) % 16 == 0;
}

// Vectors per lane of a bf16 row, or 0 when the row does not qualify for these kernels: too wide or narrow.
// lone: widest narrow row where each has a compute unit to itself.
int table_vectors_per_lane(const ais_ctx* ctx, const void* z, long long n_rows, int vocab, long long row_stride, int lone,
                           int most) {
  const int need = (vocab / 8 + kRowThreads - 1) / kRowThreads;
  const int narrow = n_rows <= ctx->n_cus && row_aligned(z, row_stride) ? lone : kFp8NarrowRow;
  return vocab > narrow && need <= most ? need : 0;
}

}  // namespace

// PREV: the widest row of the previous class; a row that reaches a class has more than PREV * 1024 vectors, of which an
// unaligned row may have lost up to 8 to its head
// Returns true when the table kernel was launched, false when the rows do not qualify (not bf16, wider than 24 vectors
// per lane, or the codes of a vector not 8-byte aligned).
bool try_fp8_quantize_table(ais_ctx* ctx, const void* logits, ais_dtype dtype, long long n_rows, int vocab,
                            long long row_stride, unsigned char* codes, long long codes_stride, float* scale_out) {
  if (dtype != AIS_BF16) return false;
  // a vector starts a multiple of 8 elements from any other place that is 16-byte aligned: its codes are 8-byte aligned
  // in every row if codes and logits have their first row and their pitch in common modulo 8 elements
  if ((reinterpret_cast<uintptr_t>(codes) - reinterpret_cast<uintptr_t>(logits) / 2) % 8 != 0 ||
      (codes_stride - row_stride) % 8 != 0)
    return false;
  const int need = table_vectors_per_lane(ctx, logits, n_rows, vocab, row_stride, kFp8NarrowLoneQuantize, 24);
  if (need == 0) return false;
  const bf16_t* z = static_cast<const bf16_t*>(logits);
  const long long resident = (long long)ctx->n_cus * quantize_workgroups(need <= 4 ? 4 : 24);
  dim3 grid((unsigned)(n_rows < resident ? n_rows : resident)), block(kRowThreads);     // persistent
  const bool aligned = row_aligned(logits, row_stride);
  // (classes of four for the middle widths; with one for every width 11,428 rows of 70,000 logits take 495 us instead of
  // 508, 7,971 of 100,352 470 and 480, 7,407 of 108,000 495 and 498, 6,325 of 126,464 493 both, 6,103 of 131,072 461 and 457)
#define AIS_CASE(PREV, NVAL)                                                                                    \
  if (need <= NVAL) {                                                                                           \
    auto kernel = aligned ? fp8_quantize_table_kernel<true, NVAL, PREV>                                         \
                          : fp8_quantize_table_kernel<false, NVAL, (PREV > 0 ? PREV - 1 : 0)>;                  \
    kernel<<<grid, block, 0, ctx->stream>>>(z, row_stride, vocab, codes, codes_stride, scale_out, n_rows);      \
    return true;                                                                                                \
  }
  AIS_CASE(0, 4)
  AIS_CASE(4, 8)
  AIS_CASE(8, 12)
  AIS_CASE(12, 16)
  AIS_CASE(16, 18)
  AIS_CASE(18, 19)
  AIS_CASE(19, 20)
  AIS_CASE(20, 24)
#undef AIS_CASE
  return false;
}

bool try_fp8_rollout_logprob_table(ais_ctx* ctx, const void* logits, ais_dtype dtype, long long n_rows, int vocab,
                                   long long row_stride, const int* token_ids, const unsigned char* valid,
                                   float* logp_out) {
  if (dtype != AIS_BF16) return false;
  // 23 vectors per lane in registers, 8 more in LDS slots beside the table
  const int need = table_vectors_per_lane(ctx, logits, n_rows, vocab, row_stride, kFp8NarrowLoneLogprob, 23 + 8);
  if (need == 0) return false;
  const bf16_t* z = static_cast<const bf16_t*>(logits);
  const long long resident = (long long)ctx->n_cus * logprob_workgroups(need <= 8 ? 8 : 24);
  dim3 grid((unsigned)(n_rows < resident ? n_rows : resident)), block(kRowThreads);     // persistent
  const bool aligned = row_aligned(logits, row_stride);
#define AIS_CASE(PREV, NVAL)                                                                                        \
  if (need <= NVAL) {                                                                                               \
    auto kernel = aligned ? fp8_rollout_logprob_table_kernel<true, NVAL, PREV, 0>                                   \
                          : fp8_rollout_logprob_table_kernel<false, NVAL, (PREV > 0 ? PREV - 1 : 0), 0>;            \
    kernel<<<grid, block, 0, ctx->stream>>>(z, row_stride, vocab, token_ids, valid, logp_out, ctx->status_dev,      \
                                            n_rows);                                                                \
    return true;                                                                                                    \
  }
  AIS_CASE(0, 4)
  AIS_CASE(4, 8)
  AIS_CASE(8, 12)
  // a class of its own for every width from here on: 8,192 rows of 100,352 logits 303 us, 335 in the class of 16
  AIS_CASE(12, 13)
  AIS_CASE(13, 14)
  AIS_CASE(14, 15)
  AIS_CASE(15, 16)
  AIS_CASE(16, 17)
  AIS_CASE(17, 18)
  AIS_CASE(18, 19)
  AIS_CASE(19, 20)
  AIS_CASE(20, 21)
  AIS_CASE(21, 22)
  AIS_CASE(22, 23)
#undef AIS_CASE
#define AIS_CASE(NEED, NLVAL)                                                                                       \
  if (need <= NEED) {                                                                                               \
    auto kernel = aligned ? fp8_rollout_logprob_table_kernel<true, 23, 23, NLVAL>                                   \
                          : fp8_rollout_logprob_table_kernel<false, 23, 22, NLVAL>;                                 \
    static std::once_flag once[2][kMaxDevices];            /* the attribute belongs to the function on one device */ \
    static bool ok[2][kMaxDevices];                                                                                 \
    if (!allow_dynamic_lds(ctx, reinterpret_cast<const void*>(kernel), NLVAL * kSlotBytes, once[aligned],           \
                           ok[aligned]))                                                                            \
      return false;                                        /* the caller falls back to the streaming kernel */     \
    kernel<<<grid, block, NLVAL * kSlotBytes, ctx->stream>>>(z, row_stride, vocab, token_ids, valid, logp_out,      \
                                                             ctx->status_dev, n_rows);                              \
    return true;                                                                                                    \
  }
  AIS_CASE(27, 4)
  AIS_CASE(31, 8)
#undef AIS_CASE
  return false;
}

}  // namespace ais
