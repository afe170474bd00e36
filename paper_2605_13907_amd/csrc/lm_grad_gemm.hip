// The two products that turn a chunk of dlogits into gradients of the hidden-state read-out (Alg. 1, "Policy Update"):
//
//   dweight[v, d] = sum_n ds[n, v] H[n, d]          both operands lie with the summed index along their rows
//   dhidden[n, d] (+)= sum_v ds[n, v] W[v, d]       ds lies with the summed index along its columns
//
// on the matrix cores, bf16 operands, fp32 accumulation and output, in one launch: the tiles of both fill the rounds of the
// chip together.  Written as C[b, a] = sum_k A[k, a] B(k, b): A is H or W (a = d), B is ds.  A 256-thread workgroup (4
// wavefronts, one to a SIMD, 128 a x 128 b each) computes 256 x 256 outputs, K in steps of 64; the schedule is that of the
// tile kernel in lm_head.hip: operand slices go straight from global memory into one of two LDS buffers, the fragments of a
// half step are read during the half step before, one barrier per step.
//
// dhidden has few tiles where there are few rows, each of them a sum over the whole chunk: its sum is then split, every part
// accumulates over the chunks in an array of its own, and the arrays are added at the end, in order.  So is dweight's where
// d_model or the vocabulary is small (its arrays are added chunk by chunk).
//
// An operand whose rows run along the summed index needs the transpose of what its rows are: its fragments come from LDS
// by ds_read_b64_tr_b16, which hands lane i of 16 the column i of a 4 x 16 block (checked on the device).  The 16 rows
// that such a read touches are 512 bytes apart; an XOR of the 32-byte column blocks with bits 0, 1 and 3 of the row
// spreads them over all banks.
//
// What bounds it: power nearly (the shader clock is 2.0 GHz, the matrix pipe busy 0.63 of the cycles), the outputs that leave at
// the end of a tile, and what a wavefront, alone on its SIMD, can issue beside its products.  4,052 rows x 8,192 entries x
// 4,096, both products: two launches of eight wavefronts of 128 x 64 outputs 458 us; one launch, copies with a select per lane
// for rows past the end and a 64-bit product per address 462; those once per item instead 424 (1.28 PFLOP/s).  The whole
// call against separate launches, in one part, of the library's product (rocBLAS) where tiles left the rounds too empty:
// 367 rows x 51,492 x 4,608 1,014 -> 792 us, 832 x 85,480 x 2,688 1,633 -> 1,288, 300 x 32,000 x 1,024 189 -> 115, 5,952 x
// 2,048 x 1,216 153 -> 108, 13,922 x 5,696 x 1,792 944 -> 762, 9,070 x 74,356 x 3,712 13.7 -> 12.7 ms, 20,000 x 32,000 x 512
// 2,607 -> 2,152 us, 41,643 x 16,384 x 4,096 14.0 -> 13.8 ms.
#include "ais_internal.h"
#include "device_utils.h"
#include "lm_tile.h"

#include <algorithm>

namespace ais {
namespace {

using namespace dev;
using namespace tile;

typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) void* lds_ptr;
typedef __attribute__((address_space(3))) bf16x4* lds_bf16x4;

constexpr int kThreads = 256;
constexpr int kTile = 256;                       // outputs along either index
constexpr int kStep = 64;                        // summed elements per step
constexpr int kSliceBytes = kTile * kStep * 2;   // 32 KiB
constexpr int kLdsBytes = 4 * kSliceBytes;       // two slices of A, then two of B
constexpr int kNI = 8, kNJ = 8;                  // 16 x 16 products per wavefront along a and b

__device__ __align__(16) const bf16_t kZeros[8] = {};

// Copies 16 bytes per lane from `src` + `ahead` elements (src per lane) to LDS at `base` + `at` + 16 * lane.  Written as
// instructions because the compiler, which does not see through the transposing reads, would wait for every copy in flight
// before each of them; the waits below are written out.  (It has no result but the address; a wait that the compiler places
// for loads of its own counts these copies too, which makes it wait longer, never shorter.)  The address is formed where m0,
// just written, may not be used yet.
// (m0 is said to be written although the compiler warns that it is a register of its own: it orders its own uses of m0
// by that.)
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
template <int AT>
__device__ __forceinline__ void copy_to_lds(const bf16_t* src, long long ahead, uint32_t base) {
  const bf16_t* from;
  asm volatile("s_add_i32 m0, %1, %4\n\tv_lshl_add_u64 %0, %3, 1, %2\n\tglobal_load_lds_dwordx4 %0, off"
               : "=&v"(from) : "s"(base), "v"(src), "s"(ahead), "n"(AT) : "m0", "scc", "memory");
}
#pragma clang diagnostic pop

// One product.
struct GemmArgs {
  const bf16_t* a;          // [k][ld_a]
  long long ld_a;
  const bf16_t* b;          // [k][ld_b], or [b][ld_b] (dhidden)
  long long ld_b;
  float* out;               // [b][m]; one such array for each part of the sum, part_stride elements apart
  long long part_stride;
  int m, n, k;              // outputs along a (a multiple of 32) and b; summed elements
  const int* k_dev;         // if not null: the number of summed elements is min(k, *k_dev)
  int accumulate, aligned;  // onto what is there; rows of out begin with 16 aligned bytes
  int a_tiles, b_tiles, parts, part_k, per_xcd;   // part_k: summed elements of a part, a multiple of 64
};

// Byte offset of the 16-byte chunk `pos` of row `row` in a slice with 512-byte rows, and the chunk that lies there.
__device__ __forceinline__ int row_swizzle(int row) { return (row & 3) | ((row >> 3) & 1) << 2; }

// Work item `item` of a product.  KC: B lies with the summed index along its rows' elements (dhidden).
template <bool KC>
__device__ __forceinline__ void gemm_item(const GemmArgs& g, int item, unsigned char* lds) {
  const int tiles = g.a_tiles * g.b_tiles;
  const int part = item / tiles, tile = item - part * tiles;
  const int group = tile / (4 * g.a_tiles), in = tile - group * 4 * g.a_tiles;
  const int rows_in = min(4, g.b_tiles - 4 * group);
  const int at = in / rows_in, bt = 4 * group + in - at * rows_in;
  const int a0 = at * kTile, b0 = bt * kTile;
  const int k_first = part * g.part_k;
  const int k_len = min((g.k_dev != nullptr ? min(g.k, *g.k_dev) : g.k) - k_first, g.part_k);
  const int n_steps = (max(k_len, 0) + kStep - 1) / kStep;

  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wa = wave & 1, wb = wave >> 1, quarter = lane >> 4, col = lane & 15;

  // ---- copies.  Rows along k: wavefront w moves rows 16 w + 2 q + (lane >> 5), q = 0..7, of a slice; the lane sits at
  // chunk lane & 31 of the row and fetches the chunk that belongs there.  (Columns of A past its end are columns of C
  // that nobody stores: any chunk of the row does.  ds holds whole tiles.)
  const int krow = 16 * wave + (lane >> 5);
  const bf16_t* ap[8];
  const bf16_t* bp[8];
#pragma unroll
  for (int q = 0; q < 8; ++q) {
    const int chunk = (lane & 31) ^ (row_swizzle(krow + 2 * q) << 1);
    ap[q] = g.a + (long long)(k_first + krow + 2 * q) * g.ld_a + min(a0 + chunk * 8, g.m - 8);
    if (KC) {                                      // rows along b: 128-byte rows, eight to an instruction
      const int crow = 8 * wave + (lane >> 3);
      bp[q] = g.b + (long long)min(b0 + crow + 32 * q, g.n - 1) * g.ld_b + k_first + ((lane & 7) ^ ((crow >> 1) & 7)) * 8;
    } else {
      bp[q] = g.b + (long long)(k_first + krow + 2 * q) * g.ld_b + b0 + chunk * 8;
    }
  }
  int c_step = 0;                                  // step being copied; stays at the last one
  long long a_ahead = 0, b_ahead = 0;              // elements from ap, bp to it
  const long long a_step = kStep * g.ld_a, b_step = KC ? kStep : kStep * g.ld_b;
  // Once the cursor is at the last step: rows past the end of the sum are zeros (of both operands, so that an infinity in one
  // does not meet the zeros of the other).
  auto end_rows = [&] {
    const int left = k_len - c_step * kStep;
    if (c_step + 1 != n_steps || left >= kStep) return;                        // uniform
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      if (krow + 2 * q >= left) {
        ap[q] = kZeros - a_ahead;
        if (!KC) bp[q] = kZeros - b_ahead;
      }
    }
  };
  const uint32_t lds0 = (uint32_t)(uintptr_t)(lds_ptr)lds;
  const uint32_t a_base = lds0 + wave * (16 * 512), b_base = lds0 + 2 * kSliceBytes + wave * (KC ? 8 * 128 : 16 * 512);
  auto copy_part = [&](int buf, auto part_number) __attribute__((always_inline)) {   // 0..15: the eight parts of A and B in turn
    constexpr int p = decltype(part_number)::value, q = p >> 1;
    if constexpr ((p & 1) == 0) copy_to_lds<2 * q * 512>(ap[q], a_ahead, a_base + buf);
    else copy_to_lds<KC ? 32 * q * 128 : 2 * q * 512>(bp[q], b_ahead, b_base + buf);
    if constexpr (p == 15) {
      if (c_step + 1 < n_steps) {
        ++c_step;
        a_ahead += a_step;
        b_ahead += b_step;
        end_rows();
      }
    }
  };

  // ---- fragments.  Transposed: the lane addresses row 8 quarter + 4 h + (col >> 2) of a 32-row half slice and 4 of the
  // 16 columns; the read gives it rows 8 quarter + 4 h .. + 3 of its own column.  16-column blocks: bits 5..8 of the offset.
  const int tr_row = 8 * quarter + (col >> 2);
  const int tr_off = tr_row * 512 + (row_swizzle(tr_row) << 5) + (col & 3) * 8;
  const int a_off = tr_off ^ (wa << 8);
  const int bt_off = 2 * kSliceBytes + (tr_off ^ (wb << 8));
  const int bk_row = 2 * kSliceBytes + wb * 128 * 128 + col * 128;
  const int bk_off[2] = {bk_row + ((quarter ^ ((col >> 1) & 7)) << 4), bk_row + (((4 + quarter) ^ ((col >> 1) & 7)) << 4)};
  bf16x8 a[2][kNI], b[2][kNJ];
  auto read_tr = [&](int offset) {
    const bf16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4)(lds + offset));
    const bf16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4)(lds + offset + 4 * 512));
    return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
  };
  // the fragments of half step kk in the order in which its products need them: A's first, B's, the others of A
  auto read_part = [&](int buf, int kk, int p) {
    if (p == 0 || p > kNJ) {
      const int i = p == 0 ? 0 : p - kNJ;
      a[kk][i] = read_tr(buf + (a_off ^ (i << 5)) + kk * 32 * 512);
    } else {
      const int j = p - 1;
      if (KC) b[kk][j] = *reinterpret_cast<const bf16x8*>(lds + buf + bk_off[kk] + j * 2048);
      else b[kk][j] = read_tr(buf + (bt_off ^ (j << 5)) + kk * 32 * 512);
    }
  };

  f32x4 acc[kNI][kNJ];
  {
    const Clear clear;
    unrolled<kNI * kNJ>([&](auto k) __attribute__((always_inline)) { clear.first(acc[k.value / kNJ][k.value % kNJ]); });
  }
  if (n_steps > 0) {                               // uniform
    int now = 0, next = kSliceBytes;
    end_rows();
    unrolled<16>([&](auto p) __attribute__((always_inline)) { copy_part(now, p); });
    unrolled<16>([&](auto p) __attribute__((always_inline)) { copy_part(next, p); });
    // copies complete in order: all but the last sixteen are step 0's
    asm volatile("s_waitcnt vmcnt(16)\n\ts_barrier" ::: "memory");
#pragma unroll
    for (int p = 0; p < kNI + kNJ; ++p) read_part(now, 0, p);
#define AIS_PIN __builtin_amdgcn_sched_barrier(0)
    // (see the tile kernel in lm_head.hip for why the reads, the barrier and the copies are where they are)
    // A fragment of two transposing reads and their address is what fits beside one product, and so is a copy: reads after
    // every third product, copies after every third from the barrier on, never both after the same one.
    constexpr int kHalf = kNI * kNJ, kBarrierAt = 54, kCopiesFrom = 56;
    for (int s = 0; s < n_steps; ++s) {
      AIS_PIN;
      unrolled<2 * kHalf>([&](auto product) __attribute__((always_inline)) {
        constexpr int m = decltype(product)::value, kk = m / kHalf, at = m % kHalf, i = at / kNJ, j = at % kNJ;
        multiply(acc[i][j], a[kk][i], b[kk][j]);
        AIS_PIN;
        if constexpr (at % 3 == 0 && at / 3 < kNI + kNJ) read_part(kk == 0 ? now : next, kk ^ 1, at / 3);
        if constexpr (m == kBarrierAt) {
          asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
          AIS_PIN;
        }
        if constexpr (m >= kCopiesFrom && (m - kCopiesFrom) % 3 == 0 && (m - kCopiesFrom) / 3 < 16)
          copy_part(now, std::integral_constant<int, (m - kCopiesFrom) / 3>{});
        AIS_PIN;
      });
      const int n = now;
      now = next;
      next = n;
    }
#undef AIS_PIN
    // copies re-fetched after the last step are still on their way into LDS
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  }
  settle();

  // ---- outputs: element v of product (i, j) is C[b = 16 j + col][a = 16 i + 4 quarter + v]
  float* out = g.out + part * g.part_stride + a0 + wa * 128 + 4 * quarter;
  const int a_left = g.m - (a0 + wa * 128 + 4 * quarter);       // outputs of the lane's row from here on
  unrolled<kNJ>([&](auto column) __attribute__((always_inline)) {
    constexpr int j = decltype(column)::value;
    f32x4 c[kNI];
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < kNI; ++i) {
      asm volatile("" : "+a"(acc[i][j]));
      c[i] = acc[i][j];
    }
    const int bi = b0 + wb * 128 + 16 * j + col;
    if (bi < g.n) {
      float* row = out + (long long)bi * g.m;
      if (g.aligned) {
        f32x4 old[kNI];
        if (g.accumulate) {
#pragma unroll
          for (int i = 0; i < kNI; ++i) old[i] = 16 * i < a_left ? *reinterpret_cast<const f32x4*>(row + 16 * i) : c[i];
#pragma unroll
          for (int i = 0; i < kNI; ++i) c[i] += old[i];
        }
#pragma unroll
        for (int i = 0; i < kNI; ++i)
          if (16 * i < a_left) *reinterpret_cast<f32x4*>(row + 16 * i) = c[i];
      } else {
#pragma unroll
        for (int i = 0; i < kNI; ++i)
#pragma unroll
          for (int v = 0; v < 4; ++v)
            if (16 * i < a_left) row[16 * i + v] = g.accumulate ? row[16 * i + v] + c[i][v] : c[i][v];
      }
    }
  });
}

// Every XCD takes a contiguous range of the work items of either product, four b tiles under each a tile: the 32 resident
// workgroups of an XCD then share 8 slices of A and 4 of B through its L2.  The product with the longer items goes first.
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(1, 1))) void lm_grad_products_kernel(
    GemmArgs dweight, GemmArgs dhidden, int dhidden_first) {
  extern __shared__ __align__(16) unsigned char lds[];
  const int xcd = blockIdx.x & 7;
  int local = blockIdx.x >> 3;
  const int first = dhidden_first ? dhidden.per_xcd : dweight.per_xcd;
  const bool hidden = (local < first) == (dhidden_first != 0);                 // uniform for the workgroup, as all of this
  if (local >= first) local -= first;
  const int per_xcd = hidden ? dhidden.per_xcd : dweight.per_xcd;
  const int item = xcd * per_xcd + local;
  const int items = hidden ? dhidden.a_tiles * dhidden.b_tiles * dhidden.parts
                           : dweight.a_tiles * dweight.b_tiles * dweight.parts;
  if (local >= per_xcd || item >= items) return;
  if (hidden) gemm_item<true>(dhidden, item, lds);
  else gemm_item<false>(dweight, item, lds);
}

// out[n, :] = sum over the parts of part[p][row, :], in order, row = n or pos[n] (zeros where that is negative).  One
// workgroup per row.
__global__ __launch_bounds__(256) void lm_add_parts_kernel(const float* __restrict__ part, long long part_stride,
                                                              int parts, const int* __restrict__ pos, int d_model,
                                                              float* __restrict__ out, int aligned) {
  const int n = blockIdx.x;
  const int row = pos != nullptr ? pos[n] : n;
  const float* src = part + (long long)(row < 0 ? 0 : row) * d_model;
  float* dst = out + (long long)n * d_model;
  for (int c = threadIdx.x * 4; c < d_model; c += 1024) {
    f32x4 sum = {0.f, 0.f, 0.f, 0.f};
    if (row >= 0) {
      sum = *reinterpret_cast<const f32x4*>(src + c);
#pragma unroll 4
      for (int p = 1; p < parts; ++p) sum += *reinterpret_cast<const f32x4*>(src + p * part_stride + c);
    }
    if (aligned) {
      *reinterpret_cast<f32x4*>(dst + c) = sum;
    } else {
#pragma unroll
      for (int v = 0; v < 4; ++v) dst[c + v] = sum[v];
    }
  }
}

// Time of a launch whose `n0` items of length l0 come before `n1` of length l1 <= l0, in units of a step: whoever is done
// first takes the next item.
long long launch_time(int n_cus, long long n0, long long l0, long long n1, long long l1) {
  const long long full = n0 / n_cus, rest = n0 % n_cus;          // `rest` compute units have one more
  long long t = full * l0 + (rest != 0 ? l0 : 0);
  if (n1 == 0) return t;
  auto room = [&](long long until) {
    const long long early = std::max<long long>(until - full * l0, 0), late = std::max<long long>(until - (full + 1) * l0, 0);
    return (n_cus - rest) * (early / l1) + rest * (late / l1);
  };
  long long lo = t, hi = t + (n1 / n_cus + 2) * l1;              // smallest time that has room for the n1
  while (lo < hi) {
    const long long mid = (lo + hi) / 2;
    if (room(mid) >= n1) hi = mid;
    else lo = mid + 1;
  }
  return lo;
}

// Length of an item in steps: its sum, and what its start and its outputs take besides.
constexpr int kItemSteps = 8;

}  // namespace

// Parts of either sum: those that make the launch of both products shortest, and fewer arrays to add up unless it is so by
// 2 %.  dweight's is a sum over all rows: few tiles, each of them long, where d_model or the vocabulary is small.  Sums of at most
// kWholeSteps (1,024 rows) stay whole: what parts save there is less than the launch that adds them.  us a call in parts and whole:
// 590 rows x 1,133 x 1,024 in chunks of 512 162 and 150, 449 x 9,048 x 512 in 4,096 155 and 142, 900 (half) x 13,433 x 1,408 in 256
// 3,339 and 2,875, 4,533 (a tenth) x 58,572 x 512 in 2,048 1,561 and 1,275, 554 x 1,951 x 1,216 61.3 and 58.3, 741 x 2,510 x 576
// 55.8 and 57.0; but 1,252 x 12,151 x 768 in 2,048 368 and 408, 1,768 x 2,944 x 1,344 in 1,024 214 and 239.
constexpr int kWholeSteps = 16;
LmParts lm_grad_parts(int n_cus, long long n_rows, long long d, long long n_v) {
  return lm_grad_parts(n_cus, n_rows, d, n_v, kLmPartsBytes);
}
LmParts lm_grad_parts(int n_cus, long long n_rows, long long d, long long n_v, long long bytes_each) {
  const long long a_tiles = (d + kTile - 1) / kTile;
  const long long h_tiles = a_tiles * ((n_rows + kTile - 1) / kTile), w_tiles = a_tiles * ((n_v + kTile - 1) / kTile);
  const long long h_steps = (n_v + kStep - 1) / kStep, w_steps = (n_rows + kStep - 1) / kStep;
  const bool split_w = 2 * w_tiles < n_cus && n_v <= kLmGradChunk && w_steps > kWholeSteps;
  LmParts best{1, 1};
  long long best_time = -1;
  for (int w = 1; w <= (split_w ? kLmMaxWeightParts : 1) && w <= w_steps; ++w) {
    if (w > 1 && w * n_v * d * 4 > bytes_each) break;
    const long long w_len = (w_steps + w - 1) / w + kItemSteps + (w > 1 ? 4 : 0);
    for (int h = 1; h <= kLmMaxParts && h <= h_steps; ++h) {
      if (h > 1 && h * n_rows * d * 4 > bytes_each) break;
      const long long h_len = (h_steps + h - 1) / h + kItemSteps + (h > 1 ? 2 : 0);
      const long long time = h_len >= w_len ? launch_time(n_cus, h_tiles * h, h_len, w_tiles * w, w_len)
                                            : launch_time(n_cus, w_tiles * w, w_len, h_tiles * h, h_len);
      if (best_time < 0 || 50 * time < 49 * best_time) {
        best = LmParts{w, h};
        best_time = time;
      }
    }
  }
  return best;
}

// Most bytes that the parts of dweight take, in chunks of n_v entries, whatever the rows.
static size_t dweight_parts_bytes(long long n_v, long long d, int n_cus, long long bytes_each) {
  if (n_v > kLmGradChunk || 2 * ((d + kTile - 1) / kTile) * ((n_v + kTile - 1) / kTile) >= n_cus) return 0;
  return (size_t)std::min<long long>(bytes_each, kLmMaxWeightParts * n_v * d * 4);
}

// Whether the 256 x 256 tiles of an [n, m] product keep `percent` of the compute units busy over all rounds.
static bool rounds_full(int n_cus, long long m, long long n, int percent) {
  const long long tiles = ((m + kTile - 1) / kTile) * ((n + kTile - 1) / kTile);
  const long long rounds = (tiles + n_cus - 1) / n_cus;
  return tiles > 0 && tiles <= (1 << 28) && 100 * tiles >= percent * rounds * n_cus;
}

// Chunks of 8,192 vocabulary entries (32 tiles; lm_grad_even_chunk keeps them beyond 65,536 rows, and where there is no room for
// wider ones), narrowed to the widest of 22 to 31 tiles that fills dweight's rounds where 32 do not: d_model 2,304 (28 tiles),
// 2,560 (25), 2,816 (23), 4,352 (30), 4,608 (28), 4,864 (26), 6,400 (30).  With both products in one launch the two are within
// a per cent of each other (70,000 rows x 30,000 x 2,560 26.8 ms and 27.0 with 8,192, x 40,000 x 2,304 32.3 and 32.0).  Never
// wider: the chunk fits the workspace of 8,192 entries.
long long lm_grad_chunk_for(long long chunk, long long vocab, long long d_model, int n_cus) {
  if (chunk != kLmGradChunk || vocab < 3 * chunk || rounds_full(n_cus, d_model, chunk, 80)) return chunk;
  for (long long width = chunk - kTile; width >= 22 * kTile; width -= kTile)
    if (rounds_full(n_cus, d_model, width, 95)) return width;
  return chunk;
}

// Room for a call over n_rows rows of which m_rows are gone through (fewer: by a list).  roomy: wide chunks and parts; 0: the
// narrow chunks, and sums in one part, for where there is no room for those.  Every array's place follows from the chunk and
// the parts that the launches take; what is asked for beyond the last one's end is for calls over fewer rows, whose chunks may
// be wider and whose sums may have more parts (dhidden's only with so few rows that two of them fit: their dlogits and parts
// often lie where the dlogits of many rows do).
LmGradRoom lm_grad_room(long long n_rows, long long m_rows, long long d, long long vocab, long long asked, int n_cus,
                        int roomy) {
  auto up = [](size_t b) { return (b + 255) & ~size_t(255); };
  const bool list = m_rows < n_rows;
  const long long bytes_each = asked == 0 ? kLmPartsBytes : kLmAskedPartsBytes;
  LmGradRoom r{};
  r.chunk = lm_grad_chunk(m_rows, vocab, asked, n_cus);
  if (asked == 0) {
    const long long even = roomy ? lm_grad_even_chunk(r.chunk, m_rows, vocab) : r.chunk;
    r.chunk = even != r.chunk ? even : lm_grad_chunk_for(r.chunk, vocab, d, n_cus);
  }
  const long long n_v = std::min(r.chunk, vocab);                // entries of the widest chunk
  r.parts = roomy ? lm_grad_parts(n_cus, m_rows, d, n_v, bytes_each) : LmParts{1, 1};
  auto dh_bytes = [&](long long rows, int parts) { return list || parts > 1 ? up((size_t)rows * (size_t)d * 4 * parts) : 0; };
  const size_t dh = dh_bytes(m_rows, r.parts.h), dw = r.parts.w > 1 ? up((size_t)n_v * (size_t)d * 4 * r.parts.w) : 0;
  r.plan = up(2 * (size_t)m_rows * (size_t)r.chunk);
  r.mask = r.plan + 256;
  r.index = r.mask + (list ? up((size_t)n_rows) : 0);
  r.pos = r.index + (list ? up((size_t)n_rows * 4) : 0);
  r.hidden = r.pos + (list ? up((size_t)n_rows * 4) : 0);
  r.dhidden = r.hidden + (list ? up((size_t)m_rows * (size_t)d * 2) : 0);
  r.dweight = r.dhidden + dh;
  r.end = r.dweight + dw;
  // dlogits and dhidden's parts, no fewer bytes than over any smaller number of rows
  auto ds_most = [&](long long rows) {
    const size_t own = lm_grad_dlogits_bytes(rows, vocab, asked, n_cus);
    return up(roomy && asked == 0 ? std::max(own, lm_grad_wide_bytes(rows, vocab)) : own);
  };
  size_t most = ds_most(m_rows) + dh_bytes(m_rows, 1), dw_most = 0;
  if (roomy) {
    const long long few = std::min(m_rows, bytes_each / (8 * d));                 // most rows whose dhidden has parts
    most = std::max(most, ds_most(few) + up((size_t)std::min<long long>(bytes_each, kLmMaxParts * few * d * 4)));
    dw_most = up(dweight_parts_bytes(std::min(asked != 0 ? asked : kLmGradChunk, vocab), d, n_cus, bytes_each));
  }
  r.all = std::max(r.end, r.end - r.plan - dh - dw + most + dw_most);
  return r;
}

// dweight[n_v, d] = ds^T h over the first k rows (min(k, *k_dev) if k_dev is given), and dhidden[n_rows, d] (+)= ds w over the
// n_v entries of the chunk (ds is zero from there to the next multiple of 256 columns); where there are several parts of a
// sum, the part p of it, that many elements of the stride further.  ds rows of pitch ds_stride; pitches of ds, h, w and
// their bases are 16-byte aligned, d a multiple of 32, the outputs' rows contiguous.
int launch_lm_grad_products(ais_ctx* ctx, const void* ds, long long ds_stride, const void* h, long long ld_h, const void* w,
                            long long ld_w, int n_rows, const int* n_rows_dev, int n_v, int d, float* dweight,
                            float* dhidden, LmParts parts, long long w_stride, long long h_stride, bool accumulate) {
  static std::once_flag once[kMaxDevices];
  static bool ok[kMaxDevices];
  if (!allow_dynamic_lds(ctx, reinterpret_cast<const void*>(lm_grad_products_kernel), kLdsBytes, once, ok))
    return hip_fail(ctx, hipErrorInvalidValue);
  const bf16_t* p = static_cast<const bf16_t*>(ds);
  const int a_tiles = (d + kTile - 1) / kTile;
  GemmArgs gw{static_cast<const bf16_t*>(h), ld_h, p, ds_stride, dweight, w_stride, d, n_v, n_rows, n_rows_dev, 0, 0,
              a_tiles, (n_v + kTile - 1) / kTile, parts.w, 0, 0};
  GemmArgs gh{static_cast<const bf16_t*>(w), ld_w, p, ds_stride, dhidden, h_stride, d, n_rows, n_v, nullptr,
              accumulate ? 1 : 0, 0, a_tiles, (n_rows + kTile - 1) / kTile, parts.h, 0, 0};
  for (GemmArgs* g : {&gw, &gh}) {
    g->aligned = reinterpret_cast<uintptr_t>(g->out) % 16 == 0;
    g->part_k = ((g->k + g->parts - 1) / g->parts + kStep - 1) / kStep * kStep;
    g->per_xcd = (int)(((long long)g->a_tiles * g->b_tiles * g->parts + 7) / 8);
  }
  const long long grid = 8LL * (gw.per_xcd + (long long)gh.per_xcd);
  if (grid > 0x7fffffff) return AIS_ERR_SIZE;
  lm_grad_products_kernel<<<(unsigned)grid, kThreads, kLdsBytes, ctx->stream>>>(gw, gh, gh.part_k >= gw.part_k ? 1 : 0);
  return hip_fail(ctx, hipGetLastError());
}

// The sums of the parts, their rows in the order of the list where there is one.
int launch_lm_add_parts(ais_ctx* ctx, const float* part, long long part_stride, int parts, const int* row_pos,
                           long long n_rows, int d, float* out) {
  lm_add_parts_kernel<<<(unsigned)n_rows, 256, 0, ctx->stream>>>(part, part_stride, parts, row_pos, d, out,
                                                                    reinterpret_cast<uintptr_t>(out) % 16 == 0 ? 1 : 0);
  return hip_fail(ctx, hipGetLastError());
}

}  // namespace ais
