// Token log-probabilities straight from the final hidden states and the output-embedding matrix:
// the [rows x vocab] logits are produced tile by tile on the matrix cores and folded into a running
// (max, sum) per token while they are still in the accumulators, so they never reach memory.
//
//   z[t, v] = sum_d H[t, d] W[v, d],   logp_t = z[t, y_t] / T - log sum_v exp(z[t, v] / T)
//
// This is a dense contraction (2 * rows * vocab * d_model flops against (rows + vocab) * d_model inputs),
// a matrix-core kernel, unlike the sweeps over materialised logits, which are bound by HBM.
//
// Layout of the work.  The product is taken transposed, C^T[v, t] = W H^T, with v_mfma_f32_16x16x32_bf16:
// a lane of the wavefront then owns one *token* column of every 16x16 tile and 4 vocabulary entries of
// it, so the running softmax state of a token lives in four lanes' registers and the reduction over the
// vocabulary needs no cross-lane traffic until the very end.  A 256-thread workgroup (4 wavefronts, one to a SIMD,
// 2 along the vocabulary x 2 along the tokens, 128 x 128 outputs each) computes 256 vocabulary entries x
// 256 tokens per tile.  It owns one block of up to 256 tokens (all blocks alike) and a contiguous chunk of vocabulary tiles; per
// token and chunk it emits a partial (max, sum), and a small second kernel merges the partials and
// subtracts.  Workgroups are numbered so that those resident on one XCD (which share an L2) work on a few
// token blocks x all vocabulary chunks at the same time, and therefore share both operands.
//
// Operand slices of 64 elements of d_model (a row of a slice is a whole 128-byte line) are copied from global memory
// straight into LDS, and copies, LDS reads and MFMAs are interleaved.  The slices lie in LDS with an XOR swizzle of
// their 16-byte chunks, which makes the fragment reads free of bank conflicts.
//
// What bounds it.  With 256 x 256 tiles every 32 K flops need 256 bytes from L2 and, with 128 x 128 outputs per
// wavefront, 512 bytes of fragments from LDS; under a sustained run with real (toggling) data the part is power-limited
// (the shader clock settles near 1.9 GHz instead of 2.4), so time follows energy.  That is why the products are 16 x 16
// x 32 and not 32 x 32 x 16, which move twice the accumulators per flop: MFMAs alone on random operands in registers
// run at 2,090 against 1,845 TFLOP/s; and why a wavefront has 128 x 128 outputs, all of its SIMD's accumulation registers:
// with eight wavefronts of 128 x 64 (768 bytes of fragments) 41,643 rows x 151,936 x 4,096 took 37.8 ms, with these 37.0 (1.40
// PFLOP/s; matrix pipe busy 0.68 of the cycles); 4,096 x 126,464 x 4,096 3,037 -> 2,896 us (0.77), 64 x 151,936 x 4,096 241 ->
// 214.  What it costs: alone on its SIMD, a wavefront has nothing beside its start and its soft-max, so contractions below 512
// are up to 20 % slower (9,506 rows x 24,897 x 64 80 -> 95 us).
#include "ais_internal.h"
#include "device_utils.h"
#include "lm_tile.h"

#include <algorithm>

namespace ais {
namespace {

using namespace dev;
using namespace tile;

constexpr int kLmThreads = 256;
constexpr int kLmTileV = 256;      // vocabulary entries per tile
constexpr int kLmTileT = 256;      // tokens per tile
constexpr int kLmTileK = 64;       // d_model elements per step
constexpr int kLmWaveV = 128;      // per wavefront: 8 MFMA tiles along the vocabulary
constexpr int kLmWaveT = 128;      //                8 along the tokens
constexpr int kLmNI = kLmWaveV / 16;
constexpr int kLmNJ = kLmWaveT / 16;
constexpr int kLmOperandBytes = kLmTileV * kLmTileK * 2;            // 32 KiB: one operand slice
// Operand slices in LDS: two of W (DEEP: three), then two of H.
constexpr int lm_lds_bytes(bool deep) { return (deep ? 5 : 4) * kLmOperandBytes; }

// A row of an operand slice is 128 bytes, eight 16-byte chunks; chunk c lies at position c ^ swizzle(row), so that the 16 rows
// that a fragment read touches at the same logical chunk lie in 16 different 16-byte bank groups (two rows fill the banks
// once).  The 16 rows of a fragment are consecutive ones of H; of W they are four fours, eight rows apart (see lm_entry).
__device__ __forceinline__ int lds_swizzle_h(int row) { return (row >> 1) & 7; }
__device__ __forceinline__ int lds_swizzle_w(int row) { return (row >> 1 & 1) | (row >> 2 & 6); }
// Token blocks that walk the vocabulary chunks together (see LmItem::init).  1 = token block major: the workgroups
// resident on an XCD share a few hidden-state blocks and sit on all chunks of the vocabulary.  Measured at 41,643
// rows x 151,936 x 4,096: 43.9 ms; groups of 2 / 4 / 8 / 16 / 32 token blocks on the same chunk (more sharing of the
// output-embedding tiles, less of the hidden-state block, which a work item re-reads for every vocabulary tile):
// 44.3 / 47.4 / 47.5 / 50.1 / 52.9 ms.  Where there are fewer than 8 token blocks every one of them fits the L2 beside
// the tiles, and sharing the tiles is what counts: 390 rows 618 us alone, 601 us in twos; 1,500 rows 1,734 us alone,
// 1,670 us in fours; from 2,000 rows on no difference beyond the noise.
__host__ __device__ inline int lm_token_block_group(int n_tblocks) { return n_tblocks < 8 ? (n_tblocks < 4 ? n_tblocks : 4) : 1; }

__device__ __forceinline__ bf16x8 as_bf16x8(u32x4 q) { return __builtin_bit_cast(bf16x8, q); }


// ---- pieces of the tile kernel ---------------------------------------------------------------------

// Decomposition of the evaluated rows into work items, decided on the device where a mask makes their number known only
// there (lm_head_setup_kernel), by lm_head_plan otherwise: n_tblocks blocks of block_rows (a multiple of 16, at most 256) evaluated rows x n_chunks chunks of tiles_per_chunk
// vocabulary tiles, per_xcd work items for each of the 8 XCDs.
struct LmDevPlan {
  int n_eval, n_tblocks, n_chunks, tiles_per_chunk, per_xcd, n_items, tb_group, block_rows;
};

// The decomposition as a kernel gets it: in memory, or (at == nullptr) with its arguments, which saves the launch that would
// put it there: us of 266 rows x 1,216 x 832 25.0 -> 21, of 390 x 151,936 x 4,096 452 -> 447.
struct LmPlanArg {
  const LmDevPlan* at;
  LmDevPlan given;
  __device__ __forceinline__ LmDevPlan get() const { return at != nullptr ? *at : given; }
};

// Cost of splitting n_vtiles vocabulary tiles into `chunks` equal chunks, or -1 where that gives more than max_items work
// items.  Workgroups are bound to XCDs by their index, so what counts is the rounds of the busiest XCD (n_cus / 8 units
// each) times the length of a work item, to which its start adds about three tiles; and what those rounds have to fetch:
// the workgroups resident on an XCD sit on b chunks of n_cus / (8 b) token blocks, so every tile of the embedding serves
// that many of them and every token block b.  41,643 rows x 151,936 x 4,096, ms, 3 chunks (2 rounds) 38.2, 6 (4 rounds)
// 38.6, 14 (9 rounds, which counting rounds alone prefers by 1 %) 40.6, 8 (6 rounds) 44.9; 32,768 rows 2 chunks (one
// round) 33.1, 3 37.4, 6 (3 rounds) 29.8, 8 (4 rounds) 30.1; chosen by this and by the rounds alone: 41,643 rows 38.0 and
// 38.4-40.6, 32,768 28.7 and 31.4, 20,000 18.4 and 18.9, 10,240 9.3 and 9.9, 6,144 5.7 and 5.9.
__host__ __device__ inline long long lm_chunks_cost(int chunks, int n_tblocks, int n_vtiles, int n_cus,
                                                    long long max_items, int* n_chunks, int* tiles_per_chunk) {
  const int cus_per_xcd = n_cus >= 8 ? n_cus / 8 : 1;
  const int tpc = (n_vtiles + chunks - 1) / chunks;
  const int real = (n_vtiles + tpc - 1) / tpc;
  *n_chunks = real;
  *tiles_per_chunk = tpc;
  const long long items = (long long)n_tblocks * real;
  if (items > max_items && chunks > 1) return -1;
  const long long per_xcd = (items + 7) / 8;
  const long long rounds = (per_xcd + cus_per_xcd - 1) / cus_per_xcd;
  const int b = real < cus_per_xcd ? real : cus_per_xcd;
  return rounds * (tpc + 3) * (256 + 77 * b / cus_per_xcd + 77 / b);
}

// Most chunks the vocabulary is split into: 64, or as many as give two work items per compute unit where there are only
// a few token blocks.  (With 64 for everyone a batch of 390 rows x 151,936 x 4,096 was 120 work items on 256 compute
// units and took 1,030 us; with more chunks 618 us, 256 rows 1,060 -> 391 us.)
__host__ __device__ inline int lm_chunk_limit(int n_tblocks, int n_vtiles, int n_cus) {
  const int fill = n_tblocks > 0 ? (2 * n_cus + n_tblocks - 1) / n_tblocks : 64;
  const int limit = fill > 64 ? fill : 64;
  return n_vtiles < limit ? n_vtiles : limit;
}

// What `chunks` chunks make of `total` evaluated rows.
__host__ __device__ inline LmDevPlan lm_decomposition(int total, int chunks, int n_vtiles, int n_cus, long long max_items) {
  LmDevPlan d;
  d.n_eval = total;
  d.n_tblocks = (total + kLmTileT - 1) / kLmTileT;
  lm_chunks_cost(chunks, d.n_tblocks, n_vtiles, n_cus, max_items, &d.n_chunks, &d.tiles_per_chunk);
  d.n_items = d.n_tblocks * d.n_chunks;
  d.per_xcd = (d.n_items + 7) / 8;
  d.tb_group = d.n_tblocks > 0 ? lm_token_block_group(d.n_tblocks) : 1;
  // as many rows in every block: a block's time goes with its columns of 16 (see LmItem)
  d.block_rows = d.n_tblocks > 0 ? ((total + d.n_tblocks - 1) / d.n_tblocks + 15) / 16 * 16 : kLmTileT;
  return d;
}

// The rows to evaluate.  With a mask, `index` lists the evaluated rows in order (built by
// lm_head_setup_kernel); without one, every row is evaluated.
struct LmRows {
  const int* index;
  // source row of evaluated position p (positions past the end repeat the last one; their results are discarded)
  __device__ __forceinline__ int row(int p, int n_eval) const {
    p = min(p, n_eval - 1);
    return index != nullptr ? index[p] : p;
  }
};

// Which part of the problem this workgroup owns, and where the thread sits in its tile.
struct LmItem {
  int tb, ch, vt0, vt1, t0, t_end, n_eval, n_chunks;
  int lane, wave, wv, wt, quarter, col;
  int col0, n_cols;      // first of the wavefront's columns of 16 tokens inside the block, and their number, 0 to 8
  __device__ __forceinline__ bool init(const LmDevPlan& plan, int n_vtiles) {
    // Workgroups are dealt to the 8 XCDs round-robin; every XCD takes a contiguous, equally long range of work
    // items (token block major): its resident workgroups then share a few token blocks' hidden-state slices and
    // each other's vocabulary tiles through the L2.
    const int xcd = blockIdx.x & 7, local = blockIdx.x >> 3;
    const int item = xcd * plan.per_xcd + local;
    if (local >= plan.per_xcd || item >= plan.n_items) return false;   // uniform for the workgroup
    n_eval = plan.n_eval;
    n_chunks = plan.n_chunks;
    const int tiles_per_chunk = plan.tiles_per_chunk;
    // items are ordered group by group of tb_group token blocks, chunk by chunk inside a group, token block by
    // token block inside a chunk: the workgroups resident on an XCD then sit on tb_group token blocks x a few chunks
    const int group = plan.tb_group, per_group = group * n_chunks;
    const int g = item / per_group, j = item - g * per_group;
    const int gsize = min(group, plan.n_tblocks - g * group);     // the last group may be smaller
    ch = j / gsize;
    tb = g * group + (j - ch * gsize);
    vt0 = ch * tiles_per_chunk;
    vt1 = min(n_vtiles, vt0 + tiles_per_chunk);
    t0 = tb * plan.block_rows;
    t_end = min(t0 + plan.block_rows, n_eval);
    lane = threadIdx.x & 63;
    wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    wv = wave & 1;                                               // position of the wavefront in the tile
    wt = wave >> 1;
    // the block's columns are dealt evenly to the two wavefronts along the tokens
    const int cols = __builtin_amdgcn_readfirstlane((min(plan.block_rows, n_eval - t0) + 15) >> 4);
    n_cols = (cols + 1 - wt) >> 1;
    col0 = wt * ((cols + 1) >> 1);
    quarter = lane >> 4;
    col = lane & 15;
    return true;
  }
};

typedef f32x4 LmAcc[kLmNI][kLmNJ];

// First of the four vocabulary entries, inside the wavefront's 128, that MFMA tile i leaves in a lane of this quarter: two
// tiles are 32 entries, eight consecutive ones to a lane.
__device__ __forceinline__ int lm_entry(int i, int quarter) { return 32 * (i >> 1) + 8 * quarter + 4 * (i & 1); }

// Copies the accumulators of MFMA tiles I .. I + N - 1 of column J out, to z[0 ..] if I = 0 and N = 2, to their places in a
// column otherwise, before whatever follows.
template <int J, int I, int N>
__device__ __forceinline__ void lm_take(LmAcc& acc, float* z) {
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int i = I; i < I + N; ++i) asm volatile("" : "+a"(acc[i][J]));      // where the products left them until here
#pragma unroll
  for (int k = 0; k < 4 * N; ++k) {
    float v = acc[I + (k >> 2)][J][k & 3];
    asm volatile("" : "+v"(v));
    z[N == 2 ? k : 4 * I + k] = v;
  }
  __builtin_amdgcn_sched_barrier(0);
}

// Per-lane soft-max state of the lane's token columns, up to eight, in the base-2 domain (logit * scale).
struct LmSoftmax {
  float run_m[kLmNJ], run_s[kLmNJ];
  int tok0, y[kLmNJ];
  // tok0 + 16 j: evaluated position of the lane's token column j; y[j]: its sampled token, -1 if there is none to find
  __device__ __forceinline__ void init(const LmItem& it, const LmRows& rows, int vocab,
                                       const int* __restrict__ token_ids) {
    tok0 = it.t0 + 16 * it.col0 + it.col;
#pragma unroll
    for (int j = 0; j < kLmNJ; ++j) {
      run_m[j] = kNegHuge;
      run_s[j] = 0.f;
      y[j] = -1;
      if (j < it.n_cols && tok0 + 16 * j < it.n_eval) {
        const int id = token_ids[rows.row(tok0 + 16 * j, it.n_eval)];
        y[j] = (id >= 0 && id < vocab) ? id : -1;
      }
    }
  }
  // Folds column j of the finished tile `vt` into the running state.  Accumulator element v of MFMA tile i holds vocabulary
  // entry  vbase + lm_entry(i, quarter) + v.  Leaves the column at zero.
  template <int J>
  __device__ __forceinline__ void fold(LmAcc& acc, const LmItem& it, int vt, int vocab, float scale,
                                       float* __restrict__ zy_out, const Clear& clear) {
    const int vbase = vt * kLmTileV + it.wv * kLmWaveV;
    float z[4 * kLmNI];
    lm_take<J, 0, kLmNI>(acc, z);
    if (vt * kLmTileV + kLmTileV > vocab) {                      // uniform: only the last tile of the vocabulary
      // entries past the end of the vocabulary become -inf: they never win the max (which starts from a
      // finite value) and add exp2(-inf) = 0 to the sum
      int left = vocab - vbase - 8 * it.quarter;
      asm volatile("" : "+v"(left));             // keeps the comparisons below in this branch
#pragma unroll
      for (int k = 0; k < 4 * kLmNI; ++k) z[k] = lm_entry(k >> 2, 0) + (k & 3) < left ? z[k] : -__builtin_inff();
    }
    float tmax = kNegHuge;
#pragma unroll
    for (int k = 0; k < 4 * kLmNI; ++k) tmax = fmaxf(tmax, z[k]);
    const float m_new = fmaxf(run_m[J], tmax * scale);           // finite: run_m is, and -inf never wins
    float sum = 0.f;
    unrolled<4>([&](auto part) __attribute__((always_inline)) {
#pragma unroll
      for (int k = 8 * part.value; k < 8 * part.value + 8; ++k) sum += exp2_fast(fmaf(z[k], scale, -m_new));
      asm volatile("" : "+v"(sum));                              // summed here, not with all other columns at the end
      clear(acc[2 * part.value][J]);
      clear(acc[2 * part.value + 1][J]);
    });
    run_s[J] = fmaf(run_s[J], exp2_fast(run_m[J] - m_new), sum);
    run_m[J] = m_new;
    // the sampled token's own logit: held by exactly one lane of one wavefront of one workgroup
    const int rel = y[J] - vbase;
    if ((unsigned)rel < (unsigned)kLmWaveV && ((rel >> 3) & 3) == it.quarter) {
      int idx = (rel >> 5) * 8 + (rel & 7), tok = tok0 + 16 * J;
      asm volatile("" : "+v"(idx), "+v"(tok));                   // keeps what is formed from them in this branch
      float zy = 0.f;
#pragma unroll
      for (int k = 0; k < 4 * kLmNI; ++k) zy = k == idx ? z[k] : zy;
      zy_out[tok] = zy;
    }
  }
  // Merges the four lane quarters, then the two wavefronts along the vocabulary (through `xch`, 2 KiB of LDS that
  // no one uses any more), and writes the chunk's partial (max, sum) of every token of the block.
  __device__ __forceinline__ void finish(const LmItem& it, float* xch, float* __restrict__ part_m,
                                         float* __restrict__ part_s) {
#pragma unroll
    for (int j = 0; j < kLmNJ; ++j)
#pragma unroll
      for (int off = 16; off <= 32; off <<= 1) {
        const float om = __shfl_xor(run_m[j], off), os = __shfl_xor(run_s[j], off);
        const float m = fmaxf(run_m[j], om);
        run_s[j] = run_s[j] * exp2_fast(run_m[j] - m) + os * exp2_fast(om - m);
        run_m[j] = m;
      }
    __syncthreads();                                            // everyone is done with the staging buffers
    float* xm = xch;                                            // [2 token groups][128 tokens] max, then sum
    float* xs = xch + 256;
    if (it.wv == 1 && it.quarter == 0) {
#pragma unroll
      for (int j = 0; j < kLmNJ; ++j) {
        xm[it.wt * 128 + j * 16 + it.col] = run_m[j];
        xs[it.wt * 128 + j * 16 + it.col] = run_s[j];
      }
    }
    __syncthreads();
    if (it.wv == 0 && it.quarter == 0) {
#pragma unroll
      for (int j = 0; j < kLmNJ; ++j) {
        const float om = xm[it.wt * 128 + j * 16 + it.col], os = xs[it.wt * 128 + j * 16 + it.col];
        const float m = fmaxf(run_m[j], om);
        const float s = run_s[j] * exp2_fast(run_m[j] - m) + os * exp2_fast(om - m);
        const int tok = tok0 + 16 * j;
        if (j < it.n_cols && tok < it.n_eval) {
          part_m[(long long)it.ch * it.n_eval + tok] = m;
          part_s[(long long)it.ch * it.n_eval + tok] = s;
        }
      }
    }
  }
};

// What the gradient variant of the tile kernel needs besides the operands: per-row lse, log-prob and
// coefficient (inputs), and the block of dlogits it writes: rows x a chunk of the vocabulary, bf16, row-major.
struct LmGradArgs {
  const float* lse;        // [n_rows]  log sum_v exp(z / T), as written by the log-prob call
  const float* logp;       // [n_rows]  log-prob of the sampled token
  const float* coeff;      // [n_rows]  d loss / d (row's log-prob) times 1 / T; 0 on rows without gradient
  bf16_t* ds;              // [n_rows, ds_stride]  coeff (softmax - onehot) over this chunk of the vocabulary
  long long ds_stride;     // elements, a multiple of 256 (stores are of eight)
  int y_off;               // first vocabulary entry of the chunk: token ids are global, tile indices local
  int compact;             // != 0: row p of ds belongs to the p-th listed row (LmRows::index), not to source row p
};

// Per-lane state of the gradient variant: for each of the lane's token columns the row it writes to, the
// sampled token's position inside the chunk, -lse in the base-2 domain, the coefficient and the sampled token's
// own element coeff (p_y - 1) = coeff expm1(logp), which would cancel if it were formed from p_y.
struct LmGrad {
  int row[kLmNJ], y[kLmNJ];
  float shift[kLmNJ], c[kLmNJ], dy[kLmNJ];
  __device__ __forceinline__ void init(const LmItem& it, const LmRows& rows, int vocab,
                                       const int* __restrict__ token_ids, const LmGradArgs& ga) {
#pragma unroll
    for (int j = 0; j < kLmNJ; ++j) {
      const int tok = it.t0 + 16 * (it.col0 + j) + it.col;
      row[j] = -1;
      y[j] = -1;
      shift[j] = 0.f;
      c[j] = 0.f;
      dy[j] = 0.f;
      if (j < it.n_cols && tok < it.n_eval) {
        const int r = rows.row(tok, it.n_eval);
        row[j] = ga.compact ? tok : r;
        c[j] = ga.coeff[r];
        if (c[j] != 0.f) {                  // rows without gradient: lse may be 0 there, and nothing is exponentiated
          const int id = token_ids[r] - ga.y_off;
          y[j] = (id >= 0 && id < vocab) ? id : -1;
          shift[j] = -ga.lse[r] * kLog2e;
          dy[j] = c[j] * expm1f(ga.logp[r]);
        }
      }
    }
  }
  // Writes column j of the finished tile `vt`, zeros past the end of the chunk (a row of ds holds whole tiles, and the
  // products that read it take whole steps).  Two MFMA tiles hold eight consecutive entries of the column's row: 16 bytes.
  // Leaves the column at zero.
  template <int J>
  __device__ __forceinline__ void emit(LmAcc& acc, const LmItem& it, int vt, int vocab, float scale, const LmGradArgs& ga,
                                       const Clear& clear) {
    const int vbase = vt * kLmTileV + it.wv * kLmWaveV;
    bf16_t* out = ga.ds + (long long)row[J] * ga.ds_stride;
    unrolled<kLmNI / 2>([&](auto pair) __attribute__((always_inline)) {
      constexpr int i = 2 * pair.value;
      const int v0 = vbase + lm_entry(i, it.quarter);
      float z[8], x[8];
      lm_take<J, i, 2>(acc, z);
      clear(acc[i][J]);
      clear(acc[i + 1][J]);
#pragma unroll
      for (int e = 0; e < 8; ++e) x[e] = c[J] != 0.f ? c[J] * exp2_fast(fmaf(z[e], scale, shift[J])) : 0.f;
      if (vt * kLmTileV + kLmTileV > vocab) {                    // uniform: only the last tile of the chunk
        int left = vocab - v0;
        asm volatile("" : "+v"(left));           // keeps the comparisons below in this branch
#pragma unroll
        for (int e = 0; e < 8; ++e) x[e] = e < left ? x[e] : 0.f;
      }
      int at = y[J] - v0;
      if ((unsigned)at < 8u) {                                   // one lane of one wavefront in the whole row
        asm volatile("" : "+v"(at));
#pragma unroll
        for (int e = 0; e < 8; ++e) x[e] = e == at ? dy[J] : x[e];
      }
      u32x4 q = Vec<bf16_t>::pack(x);
      if (row[J] >= 0) *reinterpret_cast<u32x4*>(out + v0) = q;
    });
  }
};

typedef __attribute__((address_space(3))) void* lds_ptr;
typedef const __attribute__((address_space(1))) void* glb_ptr;

// ---- the tile kernel: any d_model that is a multiple of 8 -------------------------------------------------------
// Steps of 64 elements of d_model; the two operand slices of a step (2 x 32 KiB) go from global memory straight into
// one of two LDS buffers (DEEP: of three for W; global_load_lds_dwordx4: lane i of a wavefront deposits its 16 bytes at base + 16 i, so the
// swizzle is applied by choosing which chunk each lane fetches).  A row of a slice is a whole 128-byte line, so a copy
// instruction of a wavefront asks L2 for 8 full lines.
// A step is two half steps of 32 elements: with eight columns of tokens 64 MFMAs each, every one of the half's eight
// fragments of W with every one of its token fragments.  All fragments of a half step are in registers before it begins: they
// are read during the half before, one after every second or third MFMA.  The instruction order is pinned: a wavefront has its
// SIMD to itself, so what it issues between two MFMAs has to fit beside one (16 cycles).  Reads and copies in groups after
// every eighth MFMA left the matrix pipe busy 0.59 of the cycles, spread out 0.76.
// One barrier per step, after three quarters of its first half: every wavefront has then received all it reads of the step's
// slices and its own copies of the next step, so the barrier publishes the next step and frees the slices; the copies of the
// step after next go into them at once, spread over a half step's worth of MFMAs, and are awaited a step later.  Reads over
// 4 to 6 eighths of a half step, the barrier at 5 to 7, copies over 6 to 9: no difference beyond the noise, but for copies
// over 6 eighths (1-2 % slower).  Folding a tile beside the next one's first products: nothing at d_model 4,096 or 960.
// DEEP: W has a third slice in LDS (160 KiB in all) and is copied two steps ahead instead of one, H first in every set of
// copies so that the wait can leave W's last eight in flight.  See lm_deep for where that pays.
// A wavefront multiplies as many columns of 16 tokens as its block gives it, 0 to 8, in a loop of its own for each number.
// RAGGED: d_model is not a multiple of 64; lanes whose chunk of a tile's last step lies past the end of d_model fetch
// zeros (both operands, so that an infinity in one does not meet the zeros of the other).
// GRAD = false: every finished tile is folded into the running soft-max state (log-prob call).  GRAD = true: every
// finished tile is written out as coeff (softmax - onehot) in bf16, lse being an input (gradient call).
__device__ __align__(16) const bf16_t kLmZeros[8] = {};

template <bool GRAD, bool RAGGED, bool DEEP>
__global__ __launch_bounds__(kLmThreads) __attribute__((amdgpu_waves_per_eu(1, 1))) void lm_head_tile_kernel(
    const bf16_t* __restrict__ hidden, long long ld_h, const bf16_t* __restrict__ weight, long long ld_w,
    LmRows rows, LmPlanArg plan, int d_model, int vocab, const int* __restrict__ token_ids,
    float scale, int n_vtiles, float* __restrict__ part_m, float* __restrict__ part_s,
    float* __restrict__ zy_out, LmGradArgs ga) {
  extern __shared__ __align__(16) unsigned char lds[];
  LmItem it;
  if (!it.init(plan.get(), n_vtiles)) return;
  const int lane = it.lane, wave = it.wave;

  // ---- copies: wavefront w moves rows 8 w .. 8 w + 7 (+ 32 j, j = 0..7) of each slice; a lane sits at chunk
  // position lane & 7 of row lane >> 3 and therefore fetches logical chunk (lane & 7) ^ swizzle(row), which is
  // the same for the eight rows 32 apart
  const int crow = 8 * wave + (lane >> 3);
  const int hchunk = (lane & 7) ^ lds_swizzle_h(crow), wchunk = (lane & 7) ^ lds_swizzle_w(crow);
  const bf16_t* hp[8];
  const bf16_t* wp[8];
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    // (rows past the block's are one row again and again: a line of L2 instead of eight for what nobody multiplies)
    const int trow = rows.row(min(it.t0 + crow + 32 * j, it.t_end - 1), it.n_eval);
    hp[j] = hidden + (long long)trow * ld_h + hchunk * 8;
  }
  auto point_w = [&](int vt) {
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const int vrow = min(vt * kLmTileV + crow + 32 * j, vocab - 1);
      wp[j] = weight + (long long)vrow * ld_w + wchunk * 8;
    }
  };
  const int n_ksteps = (d_model + kLmTileK - 1) / kLmTileK;
  const int n_steps = (it.vt1 - it.vt0) * n_ksteps;
  // One of the eight copy instructions (rows, then those 32, 64, ... rows further) that bring a step's slice of W into the
  // slice at byte `at`, or of H; the eighth advances the cursor.  Once the cursor of W has reached the last step it stays
  // there: the copies issued after that re-fetch the last step into a slice nobody reads any more, which keeps the loop free
  // of branches.  (H has the same rows for every tile: its cursor goes round.)
  int w_step = 0, w_kt = 0, w_vt = it.vt0, h_kt = 0;
  point_w(w_vt);
  auto copy = [&](const bf16_t* row, int k0, int chunk, int at, int q) {
    const bf16_t* src = row + k0;
    if (RAGGED) src = k0 + chunk * 8 < d_model ? src : kLmZeros;
    __builtin_amdgcn_global_load_lds((glb_ptr)src, (lds_ptr)(lds + at + (8 * wave + 32 * q) * 128), 16, 0, 0);
  };
  auto copy_w = [&](int at, int q) {
    copy(wp[q], w_kt * kLmTileK, wchunk, at, q);
    if (q == 7 && w_step + 1 < n_steps) {
      ++w_step;
      if (++w_kt == n_ksteps) {
        w_kt = 0;
        ++w_vt;
        point_w(w_vt);
      }
    }
  };
  auto copy_h = [&](int at, int q, int n) {                      // n: of that many
    copy(hp[q], h_kt * kLmTileK, hchunk, at, q);
    if (q == n - 1) h_kt = h_kt + 1 == n_ksteps ? 0 : h_kt + 1;
  };

  // ---- fragments of a half step (32 elements): lane reads chunk 4 kk + quarter of a 128-byte row
  const int arow = 8 * (it.col >> 2) + (it.col & 3);           // tile i: rows 32 (i >> 1) + 4 (i & 1) + arow, see lm_entry
  const int a_off[2] = {arow * 128 + ((it.quarter ^ lds_swizzle_w(arow)) << 4) + it.wv * kLmWaveV * 128,
                        arow * 128 + (((4 + it.quarter) ^ lds_swizzle_w(arow)) << 4) + it.wv * kLmWaveV * 128};
  const int b_off[2] = {it.col * 128 + ((it.quarter ^ lds_swizzle_h(it.col)) << 4) + it.col0 * 16 * 128,
                        it.col * 128 + (((4 + it.quarter) ^ lds_swizzle_h(it.col)) << 4) + it.col0 * 16 * 128};
  bf16x8 a[2][kLmNI], b[2][kLmNJ];
  auto read_a = [&](int at, int kk, int i) {
    a[kk][i] = as_bf16x8(*reinterpret_cast<const u32x4*>(lds + at + a_off[kk] + (i >> 1) * 4096 + (i & 1) * 512));
  };
  auto read_b = [&](int at, int kk, int j) {
    b[kk][j] = as_bf16x8(*reinterpret_cast<const u32x4*>(lds + at + b_off[kk] + j * 2048));
  };

  LmSoftmax sm;
  LmGrad gr;
  if (GRAD) gr.init(it, rows, vocab, token_ids, ga);
  else sm.init(it, rows, vocab, token_ids);

#define AIS_PIN __builtin_amdgcn_sched_barrier(0)
  // All tiles of the work item, by a wavefront with NJ columns of tokens.  Every wavefront issues the same copies and comes
  // to the same barriers, whatever its NJ.
  auto walk = [&](auto columns) {
    constexpr int NJ = decltype(columns)::value;
    LmAcc acc;
    // Copies that bring the block's rows of H, 32 to each: the block has at most one column more than twice the wavefront's.  With
    // few rows a step's copies are what it waits for (64 KiB at 64 bytes a cycle).  Log-prob, us, all eight and these: 198 rows (a
    // tenth evaluated) x 4,239 x 1,920 30.6 and 25.6, 124 (a tenth) x 8,033 x 960 22.8 and 20.1, 331 (a tenth) x 10,317 x 1,856 33.1
    // and 28.5; gradient of 201 (a tenth) x 3,070 x 3,392 in chunks of 2,048 118 and 100.  With more columns eight as ever: 390 x
    // 151,936 x 4,096 (six and seven) 454 and 456.
    constexpr int kHCopies = NJ <= 4 ? NJ + 1 : 8, kCopies = 8 + kHCopies;
    // The copies of a set, in order: those of H first where W runs a step further ahead, in turns otherwise.
    auto copy_part = [&](int w_at, int h_at, int p) {
      if (DEEP ? p < kHCopies : p < 2 * kHCopies && (p & 1) != 0) copy_h(h_at, DEEP ? p : p >> 1, kHCopies);
      else copy_w(w_at, DEEP || p >= 2 * kHCopies ? p - kHCopies : p >> 1);
    };
    // slices of the step at hand, of the next one and (DEEP: of W) of the one after that
    constexpr int kH = (DEEP ? 3 : 2) * kLmOperandBytes;
    int w0 = 0, w1 = kLmOperandBytes, w2 = DEEP ? 2 * kLmOperandBytes : 0, h0 = kH, h1 = kH + kLmOperandBytes;
    // ---- prologue: step 0 published, those after it in flight
#pragma unroll
    for (int p = 0; p < kCopies; ++p) copy_part(w0, h0, p);
    if (DEEP) {
#pragma unroll
      for (int q = 0; q < 8; ++q) copy_w(w1, q);
    }
#pragma unroll
    for (int p = 0; p < kCopies; ++p) copy_part(DEEP ? w2 : w1, h1, p);
    // copies complete in order: all but the last set (DEEP: and eight) are step 0's
    asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"(DEEP ? kCopies + 8 : kCopies) : "memory");
    // the reads of a half step in the order in which its products need them
    auto read_part = [&](int w_at, int h_at, int kk, int p) {
      if (p == 0) read_a(w_at, kk, 0);
      else if (p <= NJ) read_b(h_at, kk, p - 1);
      else if (p < NJ + kLmNI) read_a(w_at, kk, p - NJ);
    };
    if (NJ > 0) {
#pragma unroll
      for (int p = 0; p < NJ + kLmNI; ++p) read_part(w0, h0, 0, p);
    }
    // slices change places after a step
    auto turn = [&] {
      const int w = w0, h = h0;
      w0 = w1;
      w1 = DEEP ? w2 : w;
      w2 = w;
      h0 = h1;
      h1 = h;
    };
    // every copy in flight is of step s + 1 (DEEP: or one of the last eight, W of step s + 2)
    auto meet = [&] {
      if (DEEP) asm volatile("s_waitcnt vmcnt(8) lgkmcnt(0)\n\ts_barrier" ::: "memory");
      else asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
      AIS_PIN;
    };
    if constexpr (NJ == 0) {                             // copies and barriers only
      for (int s = 0; s < n_steps; ++s) {
        meet();
#pragma unroll
        for (int p = 0; p < kCopies; ++p) copy_part(w0, h0, p);
        turn();
      }
    } else {
      // Products of a half step, its reads, and where in the step (counted in products) reads end, the barrier comes and
      // copies end.  The p-th of n things that are spread over a span of products comes after product p * span / n.
      constexpr int kHalf = kLmNI * NJ, kReads = kLmNI + NJ;
      constexpr int kReadSpan = kHalf * 5 / 8, kBarrierAt = kHalf * 6 / 8, kCopySpan = kHalf;
      auto half_step = [&](auto which) __attribute__((always_inline)) {
        constexpr int kk = decltype(which)::value;
        AIS_PIN;
        unrolled<kHalf>([&](auto product) __attribute__((always_inline)) {
          constexpr int in = decltype(product)::value, m = kk * kHalf + in, i = in / NJ, j = in % NJ;
          multiply(acc[i][j], a[kk][i], b[kk][j]);
          AIS_PIN;
          constexpr int r0 = (in * kReads + kReadSpan - 1) / kReadSpan, r1 = ((in + 1) * kReads + kReadSpan - 1) / kReadSpan;
#pragma unroll
          for (int p = r0; p < r1; ++p) {
            if (kk == 0) read_part(w0, h0, 1, p);
            else read_part(w1, h1, 0, p);
          }
          if constexpr (m == kBarrierAt) meet();
          if constexpr (m >= kBarrierAt) {               // into the slices that the barrier has freed
            constexpr int after = m - kBarrierAt;
            constexpr int c0 = (after * kCopies + kCopySpan - 1) / kCopySpan;
            constexpr int c1 = ((after + 1) * kCopies + kCopySpan - 1) / kCopySpan;
#pragma unroll
            for (int p = c0; p < (c1 < kCopies ? c1 : kCopies); ++p) copy_part(w0, h0, p);
          }
          AIS_PIN;
        });
      };
      {
        const Clear clear;
        unrolled<kHalf>([&](auto k) __attribute__((always_inline)) { clear.first(acc[k.value / NJ][k.value % NJ]); });
      }
      for (int vt = it.vt0; vt < it.vt1; ++vt) {
        for (int kt = 0; kt < n_ksteps; ++kt) {
          half_step(std::integral_constant<int, 0>{});
          half_step(std::integral_constant<int, 1>{});
          turn();
        }
        settle();
        const Clear clear;
        unrolled<NJ>([&](auto column) __attribute__((always_inline)) {
          constexpr int j = decltype(column)::value;
          if constexpr (GRAD) gr.template emit<j>(acc, it, vt, vocab, scale, ga, clear);
          else sm.template fold<j>(acc, it, vt, vocab, scale, zy_out, clear);
        });
      }
    }
  };
  if (it.n_cols == 8) walk(std::integral_constant<int, 8>{});
  else if (it.n_cols == 7) walk(std::integral_constant<int, 7>{});
  else if (it.n_cols == 6) walk(std::integral_constant<int, 6>{});
  else if (it.n_cols == 5) walk(std::integral_constant<int, 5>{});
  else if (it.n_cols == 4) walk(std::integral_constant<int, 4>{});
  else if (it.n_cols == 3) walk(std::integral_constant<int, 3>{});
  else if (it.n_cols == 2) walk(std::integral_constant<int, 2>{});
  else if (it.n_cols == 1) walk(std::integral_constant<int, 1>{});
  else walk(std::integral_constant<int, 0>{});
#undef AIS_PIN
  // copies of the last steps may still be in flight, and they land in LDS that finish() is about to reuse
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  if (!GRAD) sm.finish(it, reinterpret_cast<float*>(lds), part_m, part_s);
}

// What lm_head_setup_kernel decides a decomposition for: a vocabulary width (0: none), the grid that was sized for it,
// and the most partials per evaluated row times evaluated rows that its workspace holds.
struct LmSetupGoal {
  int n_vtiles, max_items;
  long long max_partials;
};

// One workgroup, before the main kernel.  With a mask it lists the rows to evaluate (index[p] = p-th row with
// valid != 0, pos[n] = position of row n in that list or -1); in both cases it then decides the decomposition for the
// number of evaluated rows, once per goal (plan[0] and plan[1]).
// n_cap >= 0: the list holds at most n_cap rows; further rows are dropped (pos = -1) and reported in *status.
// It is latency-bound, one workgroup in front of a large kernel: every wavefront owns a contiguous run of rows and ranks
// them 64 at a time by ballot, and the candidate decompositions are tried by one thread each.  (Before, a serial scan
// over 1,024 counters and a serial search took 15-20 us without and 28-33 us with a mask of 8,192 rows.)
__global__ __launch_bounds__(1024) void lm_head_setup_kernel(const unsigned char* __restrict__ valid, int n_rows,
                                                             LmSetupGoal goal0, LmSetupGoal goal1, int n_cus,
                                                             int* __restrict__ index, int* __restrict__ pos,
                                                             LmDevPlan* __restrict__ plan, int n_cap,
                                                             int* __restrict__ status) {
  __shared__ int wave_count[16];
  __shared__ unsigned long long best[2];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  if (tid < 2) best[tid] = ~0ull;
  int total = n_rows;
  if (valid != nullptr) {
    const long long run = (((long long)n_rows + 15) / 16 + 63) & ~63ll;
    const int r0 = (int)min((long long)n_rows, wave * run), r1 = (int)min((long long)n_rows, r0 + run);
    int cnt = 0;
#pragma unroll 4
    for (int n = r0 + lane; n < r1; n += 64) cnt += valid[n] != 0;
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) cnt += __shfl_xor(cnt, off);
    if (lane == 0) wave_count[wave] = cnt;
    __syncthreads();
    total = 0;
    int p = 0;
#pragma unroll
    for (int w = 0; w < 16; ++w) {
      if (w == wave) p = total;
      total += wave_count[w];
    }
    const int cap = n_cap >= 0 ? n_cap : n_rows;
    for (int n0 = r0 + lane; n0 - lane < r1; n0 += 256) {
      bool on[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) on[u] = n0 + 64 * u < r1 && valid[n0 + 64 * u] != 0;
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int n = n0 + 64 * u;
        const unsigned long long mask = __ballot(on[u]);
        const int mine = p + (int)__popcll(mask & ((1ull << lane) - 1));
        if (on[u] && mine < cap) index[mine] = n;
        if (n < r1) pos[n] = on[u] && mine < cap ? mine : -1;
        p += (int)__popcll(mask);
      }
    }
    if (total > cap) {
      total = cap;
      if (tid == 0 && status != nullptr) atomicOr(status, AIS_STATUS_LIVE_OVERFLOW);
    }
  } else {
    __syncthreads();
  }
  const int n_tblocks = (total + kLmTileT - 1) / kLmTileT;
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    const LmSetupGoal goal = k == 0 ? goal0 : goal1;
    if (goal.n_vtiles == 0) continue;
    int limit = lm_chunk_limit(n_tblocks, goal.n_vtiles, n_cus), real, tpc;
    if (total > 0) limit = (int)min((long long)limit, goal.max_partials / total);
    // at least one chunk, whatever the limits; the fewest chunks win among equals
    for (int c = tid + 1; c <= max(limit, 1); c += 1024) {
      const long long cost = lm_chunks_cost(c, n_tblocks, goal.n_vtiles, n_cus, goal.max_items, &real, &tpc);
      if (cost >= 0) atomicMin(&best[k], ((unsigned long long)cost << 16) | (unsigned)c);
    }
  }
  __syncthreads();
  if (tid < 2) {
    const LmSetupGoal goal = tid == 0 ? goal0 : goal1;
    if (goal.n_vtiles == 0) return;
    plan[tid] = lm_decomposition(total, (int)(best[tid] & 0xffffu), goal.n_vtiles, n_cus, goal.max_items);
  }
}

// lse and log-prob from the per-chunk partials, which are stored by evaluated position.  16 rows per workgroup, the
// chunks of a row over 16 threads, whose sums are added in order; beyond 16 chunks eight partials of a thread are asked for
// together.  (One thread per row and all its chunks in turn took 33 us for 390 rows of 60 chunks, 16 us for 41,643 rows of
// 14; one partial of a thread at a time and eight: 300 rows x 65,536 of which 30 evaluated, 256 chunks, 11.0 and 6.2 us,
// 129 of 257 x 100,000 10.3 and 6.2; up to 16 chunks, 41,643 rows, 5.0 and 5.3.)
constexpr int kMergeRows = 16;
constexpr int kMergeWays = 16;
constexpr int kMergeAtOnce = 8;
__global__ __launch_bounds__(kMergeRows * kMergeWays) void lm_head_merge_kernel(
    const float* __restrict__ part_m, const float* __restrict__ part_s, const float* __restrict__ zy, int n_rows,
    LmPlanArg plan, int vocab, const int* __restrict__ token_ids, const int* __restrict__ pos,
    float inv_temperature, float* __restrict__ logp_out, float* __restrict__ lse_out, int* __restrict__ status) {
  __shared__ float way_m[kMergeWays][kMergeRows];
  __shared__ double way_s[kMergeWays][kMergeRows];
  const int r = threadIdx.x % kMergeRows, way = threadIdx.x / kMergeRows;
  const long long n = (long long)blockIdx.x * kMergeRows + r;
  const LmDevPlan decomposition = plan.get();
  const int n_chunks = decomposition.n_chunks;
  const long long stride = decomposition.n_eval;
  const int p = n >= n_rows ? -1 : (pos != nullptr ? pos[n] : (int)n);
  const bool some = p >= 0 && way < n_chunks;
  const int last = some ? way + (n_chunks - 1 - way) / kMergeWays * kMergeWays : 0;       // (past it: the last again)
  float m = kNegHuge;
  if (some) {
    m = part_m[way * stride + p];
    for (int k0 = way + kMergeWays; k0 < n_chunks; k0 += kMergeAtOnce * kMergeWays) {
#pragma unroll
      for (int u = 0; u < kMergeAtOnce; ++u) m = fmaxf(m, part_m[min(k0 + u * kMergeWays, last) * stride + p]);
    }
  }
  way_m[way][r] = m;
  __syncthreads();
#pragma unroll
  for (int w = 0; w < kMergeWays; ++w) m = fmaxf(m, way_m[w][r]);
  double s = 0.0;
  if (some) {
    s = (double)part_s[way * stride + p] * (double)exp2_fast(part_m[way * stride + p] - m);
    for (int k0 = way + kMergeWays; k0 < n_chunks; k0 += kMergeAtOnce * kMergeWays) {
      float ps[kMergeAtOnce], pm[kMergeAtOnce];
#pragma unroll
      for (int u = 0; u < kMergeAtOnce; ++u) {
        const long long at = min(k0 + u * kMergeWays, last) * stride + p;
        ps[u] = part_s[at];
        pm[u] = part_m[at];
      }
#pragma unroll
      for (int u = 0; u < kMergeAtOnce; ++u)
        if (k0 + u * kMergeWays < n_chunks) s += (double)ps[u] * (double)exp2_fast(pm[u] - m);
    }
  }
  way_s[way][r] = s;
  __syncthreads();
  if (way != 0 || n >= n_rows) return;
  if (p < 0) {
    logp_out[n] = 0.f;
    lse_out[n] = 0.f;
    return;
  }
#pragma unroll
  for (int w = 1; w < kMergeWays; ++w) s += way_s[w][r];
  const double lse = ((double)m + log2(s)) * 0.6931471805599453;
  lse_out[n] = (float)lse;
  const int id = token_ids[n];
  if (id >= 0 && id < vocab) {
    logp_out[n] = (float)((double)zy[p] * (double)inv_temperature - lse);
  } else {
    logp_out[n] = 0.f;
    atomicOr(status, AIS_STATUS_BAD_TOKEN);
  }
}

// ---- rows that take part in the gradient call, gathered ------------------------------------------------------
__global__ __launch_bounds__(256) void lm_live_mask_kernel(const float* __restrict__ coeff, int n_rows,
                                                           unsigned char* __restrict__ mask) {
  const int n = blockIdx.x * 256 + threadIdx.x;
  if (n < n_rows) mask[n] = coeff[n] != 0.f;
}

// out[p, :] = hidden[index[p], :] for the listed rows, zeros for p in [n_eval, n_cap).  One workgroup per row.
__global__ __launch_bounds__(256) void lm_gather_rows_kernel(const bf16_t* __restrict__ hidden, long long ld_h,
                                                             const int* __restrict__ index,
                                                             const LmDevPlan* __restrict__ plan, int d_model,
                                                             bf16_t* __restrict__ out) {
  const int p = blockIdx.x;
  const bool live = p < plan->n_eval;
  const u32x4* src = reinterpret_cast<const u32x4*>(hidden + (live ? (long long)index[p] * ld_h : 0));
  u32x4* dst = reinterpret_cast<u32x4*>(out + (long long)p * d_model);
  const u32x4 zero = {0u, 0u, 0u, 0u};
  for (int c = threadIdx.x; c < d_model / 8; c += 256) dst[c] = live ? src[c] : zero;
}

}  // namespace

// Worst case of the decomposition (every row evaluated): sizes the grid and the workspace.
LmHeadPlan lm_head_plan(long long n_rows, int vocab, int n_cus) {
  LmHeadPlan p;
  const int n_tblocks = (int)((n_rows + kLmTileT - 1) / kLmTileT);
  p.n_vtiles = (vocab + kLmTileV - 1) / kLmTileV;
  p.max_chunks = lm_chunk_limit(n_tblocks, p.n_vtiles, n_cus);
  long long best = -1, items = 1;
  p.chunks = 1;
  for (int c = 1; c <= p.max_chunks; ++c) {
    int real, tpc;
    const long long cost = lm_chunks_cost(c, n_tblocks, p.n_vtiles, n_cus, 1LL << 40, &real, &tpc);
    if (best < 0 || cost < best) {
      best = cost;
      items = (long long)n_tblocks * real;
      p.chunks = c;
    }
  }
  p.max_items = (int)((items + 7) / 8 * 8);
  // with a mask fewer rows may be evaluated, in more chunks: two work items per compute unit are what they can use
  p.max_items_masked = p.max_items > 2 * n_cus ? p.max_items : (2 * n_cus + 7) / 8 * 8;
  return p;
}

// Workspace of the log-prob call: the partials (max, sum) of max_chunks chunks per row, three words per row, the plan.
// More rows than before never ask for less (a context's users size it with one call at their largest batch), although
// few rows take more chunks each: what is asked for is the most that any number of rows up to n_rows takes.  From
// 64 * 256 / (2 n_cus) token blocks on every batch has the same number of chunks, so the rows below are few to look at.
size_t lm_head_logprob_bytes(long long n_rows, int vocab, int n_cus) {
  const int n_vtiles = (vocab + kLmTileV - 1) / kLmTileV;
  size_t most = 0;
  for (long long blocks = 1;; ++blocks) {
    const bool steady = lm_chunk_limit((int)blocks, n_vtiles, n_cus) == lm_chunk_limit(1 << 30, n_vtiles, n_cus);
    const long long rows = steady || blocks * kLmTileT > n_rows ? n_rows : blocks * kLmTileT;
    const size_t words = 2 * (size_t)lm_chunk_limit((int)blocks, n_vtiles, n_cus) + 3;
    most = std::max(most, sizeof(float) * (size_t)rows * words);
    if (rows == n_rows) return most + 256;
  }
}

// Vocabulary entries per chunk of the gradient call; asked == 0: the library's choice.  8,192 entries are 32 tiles, which
// with 16 token blocks (4,096 rows) are two work items per compute unit.  Up to 12 token blocks take chunks of as many
// tiles as make two for every compute unit in one round of the recomputation.  Time against chunks of 8,192, over d_model
// 1,024 to 8,192 and vocabularies of 50,257 and 128,256: 1 block 0.45-0.51, 2 0.56-0.72, 3 0.66-0.87, 4 0.72-0.94, 5
// 0.74-1.04, 6 0.83-1.09, 7 0.90-1.15, 8 0.84-0.98, 9 0.78-1.03, 10 0.87-1.02, 11 0.82-1.10, 12 0.87-1.07; 13 0.90-1.15, 14
// 0.91-1.18, 15 0.98-1.15.  (Rounded up to a tile more, which takes a second round or items of three tiles, 6 blocks
// 0.86-1.16, 7 0.97-1.23, 9 0.81-1.12, 14 1.00-1.22.)
constexpr long long kLmGradFewBlocks = 12;
long long lm_grad_chunk(long long m_rows, long long vocab, long long asked, int n_cus) {
  const long long whole = (vocab + kLmTileV - 1) / kLmTileV * kLmTileV;
  const long long blocks = std::max<long long>(1, (m_rows + kLmTileT - 1) / kLmTileT);
  long long chunk = asked != 0 ? asked : kLmGradChunk;
  if (asked == 0 && blocks <= kLmGradFewBlocks) chunk = std::max(chunk, kLmTileV * (2 * (n_cus / blocks)));
  return std::min(chunk, whole);
}

// Bytes of a chunk's dlogits.  Where the library chooses the chunk, no fewer than it takes over any smaller number of rows
// (whose chunks are wider): a call never needs more than one over more rows before it.
size_t lm_grad_dlogits_bytes(long long m_rows, long long vocab, long long asked, int n_cus) {
  const size_t own = 2 * (size_t)m_rows * (size_t)lm_grad_chunk(m_rows, vocab, asked, n_cus);
  if (asked != 0) return own;
  const long long whole = (vocab + kLmTileV - 1) / kLmTileV * kLmTileV;
  const long long tiles = std::max<long long>(2 * n_cus, kLmGradFewBlocks * (kLmGradChunk / kLmTileV));
  return std::max(own, 2 * (size_t)std::min(kLmTileT * kLmTileV * tiles, kLmGradFewBlocks * kLmTileT * whole));
}

// The width that the call takes where the choice is the library's: chunks alike, as few as kLmWideBytes of dlogits allow, of
// a multiple of 16 or 8 tiles (so that the token blocks' items of whole tiles fill the rounds), or `chunk`, the narrower choice
// above, where it is no narrower.  Wide chunks are longer sums and fewer of them: dhidden is read and written once per chunk.
// Whole call, 8,192 entries and this: 3,300 rows x 100,000 x 2,560 4,935 and 4,264 us, 4,000 x 128,256 x 2,304 6,402 and
// 5,716, 5,128 x 40,360 x 1,152 1,485 and 1,339, 6,000 x 151,936 x 1,024 5,373 and 4,950, 33,000 x 50,257 x 2,560 22.8 and 21.4
// ms, 16,576 x 20,800 x 1,920 3,666 and 3,440 us; at d_model 4,096 within a per cent; 20,000 x 32,000 x 1,024 3,559 and 3,662.
constexpr long long kLmWideBytes = 1LL << 30, kLmWideChunk = 65536;
long long lm_grad_even_chunk(long long chunk, long long m_rows, long long vocab) {
  const long long tiles = (vocab + kLmTileV - 1) / kLmTileV;
  const long long wide = std::min(kLmWideChunk, kLmWideBytes / (2 * std::max<long long>(m_rows, 1)));
  if (wide <= chunk) return chunk;
  const long long most = wide / kLmTileV, n = (tiles + most - 1) / most, even = (tiles + n - 1) / n;
  for (long long of : {16, 8}) {
    const long long up = (even + of - 1) / of * of;
    if (up <= most && up < tiles) return up * kLmTileV;
  }
  return even * kLmTileV;
}
size_t lm_grad_wide_bytes(long long m_rows, long long vocab) {
  const long long whole = (vocab + kLmTileV - 1) / kLmTileV * kLmTileV;
  return (size_t)std::min(kLmWideBytes, 2 * m_rows * std::min(whole, kLmWideChunk));
}

template <bool GRAD, bool DEEP>
int launch_lm_tile(ais_ctx* ctx, int grid, const void* hidden, long long ld_h, const void* weight, long long ld_w,
                     LmRows rows, const LmPlanArg& decomposition, int d_model, int vocab, const int* token_ids, float scale,
                     int n_vtiles, float* part_m, float* part_s, float* zy, const LmGradArgs& ga) {
  static std::once_flag once[2][kMaxDevices];                          // per function and device
  static bool ok[2][kMaxDevices];
  const int ragged = d_model % kLmTileK != 0 ? 1 : 0;
  auto kernel = ragged ? lm_head_tile_kernel<GRAD, true, true> : lm_head_tile_kernel<GRAD, false, DEEP>;
  const int lds = lm_lds_bytes(DEEP || ragged);                        // (ragged: see lm_deep)
  if (!allow_dynamic_lds(ctx, reinterpret_cast<const void*>(kernel), lds, once[ragged], ok[ragged]))
    return hip_fail(ctx, hipErrorInvalidValue);
  ScopedTimer timer(ctx, GRAD ? AIS_K_LM_HEAD_GRAD : AIS_K_LM_HEAD);
  kernel<<<grid, kLmThreads, lds, ctx->stream>>>(static_cast<const bf16_t*>(hidden), ld_h,
                                                         static_cast<const bf16_t*>(weight), ld_w, rows, decomposition, d_model,
                                                         vocab, token_ids, scale, n_vtiles, part_m, part_s, zy, ga);
  return hip_fail(ctx, hipGetLastError());
}

// Whether the log-prob call's W runs two steps ahead: where few token blocks share what the embedding brings and it is more than
// the Infinity Cache's 256 MB, so that its way from HBM is what a step waits for, or the contraction is long.  Log-prob, us without
// and with: 64 rows x 151,936 x 4,096 270 and 214, x 1,024 73 and 56, 390 x 4,096 500 and 450, x 1,024 138 and 122, 1,000 x 4,096
// 983 and 918, 2,000 1,920 and 1,839, 4,096 x 126,464 x 4,096 3,022 and 2,896; but 5,000 x 128,256 x 4,096 3,797 and 3,849, 6,500
// 4,935 and 5,042, 30,000 x 151,936 27.1 and 29.1 ms (between, 8,192 to 20,000 rows of 4,096, it would gain 1 to 3 %, at 25,000
// lose 2).  Embeddings that the cache holds, long contractions: 256 rows (half evaluated) x 16,384 x 2,560 57.2 and 50.4, 600 (a
// tenth) x 16,384 x 4,096 62.8 and 52.2, 128 x 8,000 x 3,072 48.8 and 42.0, 64 x 4,099 x 3,072 42.6 and 31.9; but 1,800 x 46,336 x
// 960 143 and 153, 390 x 50,257 x 1,024 51.5 and 52.6, 1,000 95.2 and 96.7, 390 x 151,936 x 576 74.9 and 76.7, 2,000 x 50,257 x
// 2,048 327 and 325.  In between (d_model 1,024 to 2,047) it pays for one token block and, where a mask may leave as few rows, for a
// few, with tiles enough for every workgroup to go through several: 106 rows x 10,748 x 1,728 31.2 and 28.3, 114 x 20,750 x 1,472
// 29.5 and 26.4, 199 (half) x 10,542 x 1,600 35.2 and 30.5, 331 (a tenth) x 10,317 x 1,856 33.9 and 26.9, 899 (a tenth) x 17,984 x
// 1,024 31.8 and 30.1, 1,640 (a tenth) x 27,476 x 1,344 41.0 and 40.5; but 491 x 14,490 x 1,024 32.4 and 32.8, 1,825 x 7,444 x
// 1,792 50.4 and 51.9, 3,853 (half) x 26,531 x 1,152 117 and 119, and 309 (a tenth) x 1,816 x 1,792 23.6 and 23.2.
// The gradient's chunks are short items, most of them in their first tiles: 4,052 rows x 126,464 x 4,096 10.23 and 9.97 ms, 3,000
// x 50,257 x 1,024 1.148 and 1.117, 8,192 x 126,464 x 576 4.81 and 4.66, 600 x 50,257 x 1,024 464 and 438 us, but 2,500 x 32,000 x
// 512 501 and 504: always two steps ahead.
// At any size where the embedding's rows do not begin with a 128-byte line, as with a ragged d_model: a slice's rows then lie
// across two lines each, and one step is too short for them (with eight wavefronts to a workgroup 300 rows x 151,936 x 2,056
// 356 without and 268 with, 8,192 rows 4,974 and 3,957).
// masked: n_rows is a guess, half of the rows given.
bool lm_deep(long long n_rows, bool masked, int d_model, long long vocab, const void* weight, long long ld_w) {
  if (d_model % kLmTileK != 0 || reinterpret_cast<uintptr_t>(weight) % 128 != 0 || ld_w % 64 != 0) return true;
  if (d_model >= 2048 || vocab * d_model >= 128LL << 20) return n_rows <= 4608;
  return d_model >= 1024 && vocab >= 8192 && n_rows <= (masked ? 1024 : kLmTileT);
}

int launch_lm_head_logprob(ais_ctx* ctx, const void* hidden, long long ld_h, const void* weight, long long ld_w,
                           long long n_rows, int d_model, int vocab, const int* token_ids,
                           const unsigned char* valid, float inv_temperature, const LmHeadPlan& plan,
                           float* part_m, float* part_s, float* zy, int* row_index, int* row_pos, void* dev_plan,
                           float* logp_out, float* lse_out) {
  // The grid covers the work items of the worst case; with fewer evaluated rows the device-side plan may use
  // more, shorter chunks, but never more items than that, and the workgroups left over leave at once.
  const int max_items = valid != nullptr ? plan.max_items_masked : plan.max_items;
  LmDevPlan* dplan = static_cast<LmDevPlan*>(dev_plan);
  LmPlanArg decomposition{nullptr, lm_decomposition((int)n_rows, plan.chunks, plan.n_vtiles, ctx->n_cus, max_items)};
  if (valid != nullptr) {
    lm_head_setup_kernel<<<1, 1024, 0, ctx->stream>>>(
        valid, (int)n_rows, LmSetupGoal{plan.n_vtiles, max_items, (long long)plan.max_chunks * n_rows}, LmSetupGoal{},
        ctx->n_cus, row_index, row_pos, dplan, -1, nullptr);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return hip_fail(ctx, e);
    decomposition.at = dplan;
  }
  LmRows rows{valid != nullptr ? row_index : nullptr};
  // (how many rows a mask leaves is known on the device only: half of them is the guess)
  const bool masked = valid != nullptr;
  auto launch = lm_deep(masked ? n_rows / 2 : n_rows, masked, d_model, vocab, weight, ld_w) ? launch_lm_tile<false, true>
                                                                                            : launch_lm_tile<false, false>;
  const int rc = launch(ctx, max_items, hidden, ld_h, weight, ld_w, rows, decomposition, d_model, vocab, token_ids,
                                       inv_temperature * kLog2e, plan.n_vtiles, part_m, part_s, zy, LmGradArgs{});
  if (rc != AIS_OK) return rc;
  lm_head_merge_kernel<<<(unsigned)((n_rows + kMergeRows - 1) / kMergeRows), kMergeRows * kMergeWays, 0, ctx->stream>>>(
      part_m, part_s, zy, (int)n_rows, decomposition, vocab, token_ids, valid != nullptr ? row_pos : nullptr,
      inv_temperature, logp_out, lse_out, ctx->status_dev);
  return hip_fail(ctx, hipGetLastError());
}

// The list of rows with a gradient (with live_mask: at most n_cap of them) and the decompositions of the gradient
// call's chunks: plan 0 for chunks of `width` vocabulary entries, plan 1 for a last chunk of width_last (0: none).
int launch_lm_head_grad_setup(ais_ctx* ctx, const unsigned char* live_mask, long long n_rows, int n_cap, int width,
                              int width_last, int* row_index, int* row_pos, void* dev_plan) {
  if (live_mask == nullptr) return AIS_OK;         // every row: the decompositions go with the launches
  auto goal = [&](int w) {
    if (w == 0) return LmSetupGoal{};
    const LmHeadPlan plan = lm_head_plan(n_cap, w, ctx->n_cus);
    return LmSetupGoal{plan.n_vtiles, plan.max_items_masked, 1LL << 62};
  };
  lm_head_setup_kernel<<<1, 1024, 0, ctx->stream>>>(live_mask, (int)n_rows, goal(width), goal(width_last), ctx->n_cus,
                                                    row_index, row_pos, static_cast<LmDevPlan*>(dev_plan), n_cap,
                                                    ctx->status_dev);
  return hip_fail(ctx, hipGetLastError());
}

// dlogits of one chunk of the vocabulary, from hidden states and the chunk's rows of the output embedding, into
// ds[n_rows, ds_stride] (bf16).  `weight` points at the chunk's first row, `vocab` is the chunk's width, `y_off` its
// first vocabulary entry, `which` the plan for its width.  Every row is processed (rows whose coefficient is 0 come out
// as zeros).
// With a list (row_index != nullptr: the rows with a gradient, at most n_cap of them) row p of ds belongs to the p-th
// listed row; rows past the end of the list are left as they are.
int launch_lm_head_dlogits_chunk(ais_ctx* ctx, const void* hidden, long long ld_h, const void* weight,
                                 long long ld_w, long long n_rows, int d_model, int vocab, int y_off,
                                 const int* token_ids, const float* lse, const float* logp, const float* coeff,
                                 float inv_temperature, const void* dev_plan, int which, void* ds, long long ds_stride,
                                 const int* row_index, int n_cap) {
  const LmHeadPlan plan = lm_head_plan(row_index != nullptr ? n_cap : n_rows, vocab, ctx->n_cus);
  const int max_items = row_index != nullptr ? plan.max_items_masked : plan.max_items;
  const LmDevPlan* dplan = static_cast<const LmDevPlan*>(dev_plan) + which;
  const LmPlanArg decomposition{row_index != nullptr ? dplan : nullptr,
                                lm_decomposition((int)n_rows, plan.chunks, plan.n_vtiles, ctx->n_cus, max_items)};
  LmRows rows{row_index};
  LmGradArgs ga{lse, logp, coeff, static_cast<bf16_t*>(ds), ds_stride, y_off, row_index != nullptr ? 1 : 0};
  return launch_lm_tile<true, true>(ctx, max_items, hidden, ld_h, weight, ld_w, rows, decomposition, d_model, vocab,
                                        token_ids, inv_temperature * kLog2e, plan.n_vtiles, nullptr, nullptr, nullptr,
                                        ga);
}

int launch_lm_live_mask(ais_ctx* ctx, const float* coeff, long long n_rows, unsigned char* mask) {
  lm_live_mask_kernel<<<(unsigned)((n_rows + 255) / 256), 256, 0, ctx->stream>>>(coeff, (int)n_rows, mask);
  return hip_fail(ctx, hipGetLastError());
}

// The hidden states of the listed rows, in order (zeros past the end of the list, up to row n_cap - 1).
int launch_lm_gather_rows(ais_ctx* ctx, const void* hidden, long long ld_h, int d_model, const int* row_index,
                          const void* dev_plan, int n_cap, void* gathered) {
  lm_gather_rows_kernel<<<(unsigned)n_cap, 256, 0, ctx->stream>>>(
      static_cast<const bf16_t*>(hidden), ld_h, row_index, static_cast<const LmDevPlan*>(dev_plan), d_model,
      static_cast<bf16_t*>(gathered));
  return hip_fail(ctx, hipGetLastError());
}

}  // namespace ais
