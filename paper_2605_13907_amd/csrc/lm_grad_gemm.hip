// The two products that turn a chunk of dlogits into gradients of the hidden-state read-out (Alg. 1, "Policy Update"):
//
//   dweight[v, d] = sum_n ds[n, v] H[n, d]          both operands lie with the summed index along their rows
//   dhidden[n, d] (+)= sum_v ds[n, v] W[v, d]       ds lies with the summed index along its columns
//
// on the matrix cores, bf16 operands, fp32 accumulation and output.  Written as C[b, a] = sum_k A[k, a] B(k, b): A is H
// or W (a = d), B is ds.  A 512-thread workgroup (8 wavefronts, 128 a x 64 b each) computes 256 x 256 outputs, K in
// steps of 64; the schedule is that of the tile kernel in lm_head.hip: operand slices go straight from global memory into
// one of two LDS buffers, fragments pass through a ring of registers, one barrier per step.
//
// An operand whose rows run along the summed index needs the transpose of what its rows are: its fragments come from LDS
// by ds_read_b64_tr_b16, which hands lane i of 16 the column i of a 4 x 16 block (checked on the device).  The 16 rows
// that such a read touches are 512 bytes apart; an XOR of the 32-byte column blocks with bits 0, 1 and 3 of the row
// spreads them over all banks.
//
// Power-limited like that kernel.  Against the library's products for the same layouts, which these replace where their
// tiles fill the chip: 4,052 rows x 8,192 entries x 4,096, dweight 271-304 -> 225 us (1.21 PFLOP/s), dhidden 223-230 ->
// 214 us (1.27).
#include "ais_internal.h"
#include "device_utils.h"

namespace ais {
namespace {

using namespace dev;

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) void* lds_ptr;
typedef __attribute__((address_space(3))) bf16x4* lds_bf16x4;

constexpr int kThreads = 512;
constexpr int kTile = 256;                       // outputs along either index
constexpr int kStep = 64;                        // summed elements per step
constexpr int kSliceBytes = kTile * kStep * 2;   // 32 KiB
constexpr int kBufferBytes = 2 * kSliceBytes;    // A slice, then B slice
constexpr int kLdsBytes = 2 * kBufferBytes;
constexpr int kNI = 8, kNJ = 4;                  // 16 x 16 products per wavefront along a and b

__device__ __align__(16) const bf16_t kZeros[8] = {};

// Copies 16 bytes per lane from `src` (per lane) to LDS at `base` + 16 * lane.  Written as an instruction because the
// compiler, which does not see through the transposing reads, would wait for every copy in flight before each of them;
// the waits below are written out.  (It has no result register; a wait that the compiler places for loads of its own
// counts these copies too, which makes it wait longer, never shorter.)
// (m0 is said to be written although the compiler warns that it is a register of its own: it orders its own uses of m0
// by that.)
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
__device__ __forceinline__ void copy_to_lds(const bf16_t* src, const unsigned char* base) {
  const uint32_t at = (uint32_t)(uintptr_t)(lds_ptr)base;               // uniform
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" : : "s"(at), "v"(src) : "m0", "memory");
}
#pragma clang diagnostic pop

struct GemmArgs {
  const bf16_t* a;          // [k][ld_a]
  long long ld_a;
  const bf16_t* b;          // [k][ld_b], or [b][ld_b] (KC)
  long long ld_b;
  float* out;               // [b][ld_out]
  long long ld_out;
  int m, n, k;              // outputs along a (a multiple of 4) and b; summed elements
  const int* k_dev;         // if not null: the number of summed elements is min(k, *k_dev)
  int accumulate;
  int a_tiles, b_tiles, per_xcd;
};

// Byte offset of the 16-byte chunk `pos` of row `row` in a slice with 512-byte rows, and the chunk that lies there.
__device__ __forceinline__ int row_swizzle(int row) { return (row & 3) | ((row >> 3) & 1) << 2; }

template <bool KC>
__global__ __launch_bounds__(kThreads) void lm_grad_gemm_kernel(GemmArgs g) {
  extern __shared__ __align__(16) unsigned char lds[];
  // every XCD takes a contiguous range of tiles, four b tiles under each a tile: the 32 resident workgroups of an XCD
  // then share 8 slices of A and 4 of B through its L2
  const int item = (blockIdx.x & 7) * g.per_xcd + (blockIdx.x >> 3);
  if ((int)(blockIdx.x >> 3) >= g.per_xcd || item >= g.a_tiles * g.b_tiles) return;     // uniform for the workgroup
  const int group = item / (4 * g.a_tiles), in = item - group * 4 * g.a_tiles;
  const int rows_in = min(4, g.b_tiles - 4 * group);
  const int at = in / rows_in, bt = 4 * group + in - at * rows_in;
  const int a0 = at * kTile, b0 = bt * kTile;
  const int k_len = g.k_dev != nullptr ? min(g.k, *g.k_dev) : g.k;
  const int n_steps = (k_len + kStep - 1) / kStep;

  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wa = wave & 1, wb = wave >> 1, quarter = lane >> 4, col = lane & 15;

  // ---- copies.  Rows along k: wavefront w moves rows 8 w + 2 q + (lane >> 5), q = 0..3, of a slice; the lane sits at
  // chunk lane & 31 of the row and fetches the chunk that belongs there.
  const int krow = 8 * wave + (lane >> 5);
  const int chunk0 = (lane & 31) ^ (row_swizzle(krow) << 1);             // q even; q odd: bit 1 of the row flips
  const bf16_t* ap = g.a + (long long)krow * g.ld_a + a0;
  const bool a_in0 = a0 + chunk0 * 8 < g.m, a_in1 = a0 + (chunk0 ^ 4) * 8 < g.m;
  const bf16_t* bp[4];
  bool b_in0 = true, b_in1 = true;
  if (KC) {                                        // rows along b: 128-byte rows, eight to an instruction
    const int crow = 8 * wave + (lane >> 3);
#pragma unroll
    for (int q = 0; q < 4; ++q)
      bp[q] = g.b + (long long)min(b0 + crow + 64 * q, g.n - 1) * g.ld_b + ((lane & 7) ^ ((crow >> 1) & 7)) * 8;
  } else {
    bp[0] = g.b + (long long)krow * g.ld_b + b0;
    b_in0 = b0 + chunk0 * 8 < g.n;
    b_in1 = b0 + (chunk0 ^ 4) * 8 < g.n;
  }
  uint32_t zeros_lo = (uint32_t)reinterpret_cast<uintptr_t>(kZeros);
  uint32_t zeros_hi = (uint32_t)(reinterpret_cast<uintptr_t>(kZeros) >> 32);
  asm volatile("" : "+v"(zeros_lo), "+v"(zeros_hi));
  auto either = [&](bool in, const bf16_t* src) {   // src or the zeros: two selects, no branch
    const uint64_t p = reinterpret_cast<uint64_t>(src);
    const uint32_t lo = in ? (uint32_t)p : zeros_lo, hi = in ? (uint32_t)(p >> 32) : zeros_hi;
    return reinterpret_cast<const bf16_t*>((uint64_t)hi << 32 | lo);
  };
  int c_step = 0;                                  // step being copied; stays at the last one
  auto copy_part = [&](int buf, int p) {           // p = 0..7: the four parts of A and B in turn
    const int q = p >> 1, k0 = c_step * kStep;
    unsigned char* base = lds + buf * kBufferBytes;
    const int chunk = (q & 1) ? chunk0 ^ 4 : chunk0;
    const bool k_in = k0 + krow + 2 * q < k_len;
    if ((p & 1) == 0) {
      const bf16_t* src = ap + (long long)(k0 + 2 * q) * g.ld_a + chunk * 8;
      copy_to_lds(either(k_in & ((q & 1) ? a_in1 : a_in0), src), base + (8 * wave + 2 * q) * 512);
    } else if (KC) {
      copy_to_lds(bp[q] + k0, base + kSliceBytes + (8 * wave + 64 * q) * 128);
    } else {
      const bf16_t* src = bp[0] + (long long)(k0 + 2 * q) * g.ld_b + chunk * 8;
      copy_to_lds(either(k_in & ((q & 1) ? b_in1 : b_in0), src), base + kSliceBytes + (8 * wave + 2 * q) * 512);
    }
    if (p == 7 && c_step + 1 < n_steps) ++c_step;
  };

  // ---- fragments.  Transposed: the lane addresses row 8 quarter + 4 h + (col >> 2) of a 32-row half slice and 4 of the
  // 16 columns; the read gives it rows 8 quarter + 4 h .. + 3 of its own column.
  const int tr_row = 8 * quarter + (col >> 2);
  const int tr_off = tr_row * 512 + (row_swizzle(tr_row) << 5) + (col & 3) * 8;
  const int a_off = tr_off ^ (wa << 8);            // 16-column blocks 8 wa + i: bits 5..8 of the offset
  const int bt_off = kSliceBytes + (tr_off ^ (wb << 7));      // 16-column blocks 4 wb + j
  const int bk_off[2] = {kSliceBytes + wb * 64 * 128 + col * 128 + ((quarter ^ ((col >> 1) & 7)) << 4),
                         kSliceBytes + wb * 64 * 128 + col * 128 + (((4 + quarter) ^ ((col >> 1) & 7)) << 4)};
  bf16x4 a[4][2], b[2][kNJ][2];
  auto read_tr = [&](int offset) { return __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4)(lds + offset)); };
  auto read_a = [&](int buf, int gr) {             // fragment of group gr (0..15): block gr & 7, half gr >> 3
    const int at_block = buf * kBufferBytes + (a_off ^ ((gr & 7) << 5)) + (gr >> 3) * 32 * 512;
    a[gr & 3][0] = read_tr(at_block);
    a[gr & 3][1] = read_tr(at_block + 4 * 512);
  };
  auto read_b = [&](int buf, int kk, int j) {
    if (KC) {
      const bf16x8 v = *reinterpret_cast<const bf16x8*>(lds + buf * kBufferBytes + bk_off[kk] + j * 2048);
      b[kk][j][0] = __builtin_shufflevector(v, v, 0, 1, 2, 3);
      b[kk][j][1] = __builtin_shufflevector(v, v, 4, 5, 6, 7);
    } else {
      const int at_block = buf * kBufferBytes + (bt_off ^ (j << 5)) + kk * 32 * 512;
      b[kk][j][0] = read_tr(at_block);
      b[kk][j][1] = read_tr(at_block + 4 * 512);
    }
  };
  auto whole = [](const bf16x4 (&v)[2]) -> bf16x8 { return __builtin_shufflevector(v[0], v[1], 0, 1, 2, 3, 4, 5, 6, 7); };

  f32x4 acc[kNI][kNJ];
#pragma unroll
  for (int i = 0; i < kNI; ++i)
#pragma unroll
    for (int j = 0; j < kNJ; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

  if (n_steps > 0) {                               // uniform
#pragma unroll
    for (int p = 0; p < 8; ++p) copy_part(0, p);
#pragma unroll
    for (int p = 0; p < 3; ++p) copy_part(1, p);
    // copies complete in order: all but the last three are step 0's
    asm volatile("s_waitcnt vmcnt(3)\n\ts_barrier" ::: "memory");
#pragma unroll
    for (int j = 0; j < kNJ; ++j) read_b(0, 0, j);
#pragma unroll
    for (int gr = 0; gr < 3; ++gr) read_a(0, gr);
  }
#define AIS_PIN __builtin_amdgcn_sched_barrier(0)
  for (int s = 0; s < n_steps; ++s) {
    const int buf = s & 1;
#pragma unroll
    for (int gr = 0; gr < 16; ++gr) {
      const int kk = gr >> 3, i = gr & 7;
#pragma unroll
      for (int j = 0; j < kNJ; ++j)
        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(whole(a[gr & 3]), whole(b[kk][j]), acc[i][j], 0, 0, 0);
      AIS_PIN;
      // (see the tile kernel in lm_head.hip for why the reads and copies are where they are)
      if (gr <= 10) read_a(buf, gr + 3);
      if (gr == 11) {
        read_a(buf, 14);
        read_a(buf, 15);
      }
      if (gr >= 2 && gr < 6) read_b(buf, 1, gr - 2);
      if (gr < 5) copy_part(buf ^ 1, gr + 3);
      AIS_PIN;
      if (gr == 12) {
        asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
        AIS_PIN;
        read_a(buf ^ 1, 0);
        read_b(buf ^ 1, 0, 0);
        read_b(buf ^ 1, 0, 1);
      }
      if (gr == 13) {
        read_b(buf ^ 1, 0, 2);
        read_b(buf ^ 1, 0, 3);
        read_a(buf ^ 1, 1);
      }
      if (gr == 14) read_a(buf ^ 1, 2);
      if (gr >= 13) copy_part(buf, gr - 13);
      AIS_PIN;
    }
  }
#undef AIS_PIN
  // copies re-fetched after the last step are still on their way into LDS
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");

  // ---- outputs: element v of product (i, j) is C[b = 16 j + col][a = 16 i + 4 quarter + v]
#pragma unroll
  for (int j = 0; j < kNJ; ++j) {
    const int bi = b0 + wb * 64 + 16 * j + col;
    if (bi >= g.n) continue;
    float* row = g.out + (long long)bi * g.ld_out;
#pragma unroll
    for (int i = 0; i < kNI; ++i) {
      const int ai = a0 + wa * 128 + 16 * i + 4 * quarter;
      if (ai >= g.m) continue;
      f32x4* p = reinterpret_cast<f32x4*>(row + ai);
      *p = g.accumulate ? *p + acc[i][j] : acc[i][j];
    }
  }
}

template <bool KC>
int launch_gemm(ais_ctx* ctx, GemmArgs g) {
  static std::once_flag once[kMaxDevices];
  static bool ok[kMaxDevices];
  if (!allow_dynamic_lds(ctx, reinterpret_cast<const void*>(lm_grad_gemm_kernel<KC>), kLdsBytes, once, ok))
    return hip_fail(ctx, hipErrorInvalidValue);
  g.a_tiles = (g.m + kTile - 1) / kTile;
  g.b_tiles = (g.n + kTile - 1) / kTile;
  g.per_xcd = (g.a_tiles * g.b_tiles + 7) / 8;
  lm_grad_gemm_kernel<KC><<<8 * g.per_xcd, kThreads, kLdsBytes, ctx->stream>>>(g);
  return hip_fail(ctx, hipGetLastError());
}

}  // namespace

// Whether the 256 x 256 tiles of an [n, m] product keep enough of the compute units busy over all rounds to beat the
// library's product, which has smaller tiles and can split the sum.  With full rounds dweight takes 0.78-0.82 of the
// library's time and dhidden 0.93-0.96, so that is about how full the rounds have to be: dhidden of 14,000 rows x 1,024
// (86 % full) takes 216 against 194 us, of 6,000 rows x 2,048 (75 %) 175 against 165, of 2,600 rows x 5,120 (86 %) the
// same; dweight of 8,192 entries x 5,120 (83 %) 210 against 262, of 8,192 x 1,024 (50 %) 314 against 233.  Between those
// the line of dweight matters little: the whole call over 4,096 rows x 4,096 takes 276 us with its own product at 69 % full
// and 283 with the library's, at 75 % 287 and 291, at 81 % 301 and 326 (dhidden with it), over 8,192 rows at 62 % 507 and
// 503.
static bool rounds_full(int n_cus, long long m, long long n, int percent) {
  const long long tiles = ((m + kTile - 1) / kTile) * ((n + kTile - 1) / kTile);
  const long long rounds = (tiles + n_cus - 1) / n_cus;
  return tiles > 0 && tiles <= (1 << 28) && 100 * tiles >= percent * rounds * n_cus;
}
bool lm_dweight_fits(const ais_ctx* ctx, long long d, long long n_v) { return rounds_full(ctx->n_cus, d, n_v, 80); }
bool lm_dhidden_fits(const ais_ctx* ctx, long long d, long long n_rows) { return rounds_full(ctx->n_cus, d, n_rows, 95); }

// The library's chunk of 8,192 vocabulary entries (32 tiles), narrowed to the widest of 22 to 31 tiles that fills dweight's
// rounds where 32 leave them too empty for the own product: d_model 2,304 (28 tiles), 2,560 (25), 2,816 (23), 4,352 (30),
// 4,608 (28), 4,864 (26), 6,400 (30).  Whole call against chunks of 8,192, in this order, over 3,300 to 12,000 rows and
// vocabularies of 24,600 to 151,936: 0.79-0.91, 0.82-0.99, 0.79-0.96, 0.83-0.91, 0.96-1.00, 0.92-0.94, 0.91-0.98 (6,144 rows x
// 50,257 x 2,304: 4,525 -> 3,590 us).  Fewer tiles (21, d_model 3,072: 0.96-1.07) shorten the recomputation's work items too
// far; vocabularies of two or three chunks are left with too small a last one (0.85-1.02).  Never wider: the chunk fits the
// workspace of 8,192 entries.
long long lm_grad_chunk_for(long long chunk, long long vocab, long long d_model, int n_cus) {
  if (chunk != kLmGradChunk || vocab < 3 * chunk || rounds_full(n_cus, d_model, chunk, 80)) return chunk;
  for (long long width = chunk - kTile; width >= 22 * kTile; width -= kTile)
    if (rounds_full(n_cus, d_model, width, 95)) return width;
  return chunk;
}

// dweight[n_v, d] = ds^T h over the first k rows (min(k, *k_dev) if k_dev is given); ds rows of pitch ds_stride.
// Row pitches and bases are 16-byte aligned, d a multiple of 32, ds defined up to a multiple of 256 columns.
int launch_lm_dweight(ais_ctx* ctx, const void* ds, long long ds_stride, const void* h, long long ld_h, int k,
                      const int* k_dev, int n_v, int d, float* dweight) {
  GemmArgs g{static_cast<const bf16_t*>(h), ld_h, static_cast<const bf16_t*>(ds), ds_stride, dweight, d, d, n_v, k, k_dev,
             0, 0, 0, 0};
  return launch_gemm<false>(ctx, g);
}

// dhidden[n_rows, d] (+)= ds w over n_v vocabulary entries (ds is zero from there to the next multiple of 64 columns).
int launch_lm_dhidden(ais_ctx* ctx, const void* ds, long long ds_stride, const void* w, long long ld_w, int n_v,
                      int n_rows, int d, bool accumulate, float* dhidden) {
  GemmArgs g{static_cast<const bf16_t*>(w), ld_w, static_cast<const bf16_t*>(ds), ds_stride, dhidden, d, d, n_rows, n_v,
             nullptr, accumulate ? 1 : 0, 0, 0, 0};
  return launch_gemm<true>(ctx, g);
}

}  // namespace ais
