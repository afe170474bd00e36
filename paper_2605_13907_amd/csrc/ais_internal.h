// Internal declarations shared by the translation units of the library (not installed).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <mutex>
#include <vector>

#include "ais.h"
#include "row_coeff.h"

namespace ais {

constexpr int kSweepThreads = 256;     // one workgroup (4 wavefronts) streams one logits row
constexpr int kPlanThreads = 256;      // workgroup of the plan kernel
constexpr int kPlanTileRows = 1024;    // rows of a tile that it lays out
// Most responses that the scalar kernels know each of (a thread of a workgroup reads one's rows), so that the rows are dealt out
// evenly; beyond, tiles are laid out by the plan kernel.  Diagnostics and row coefficients, us a call, dealt out and planned (the
// plan kernel's launch is part of the first): 41,643 rows in 16 responses 8.1 and 18.1, 5.6 and 10.3; 200,000 in 64 10.3 and 19.7, 8.0
// and 10.8; 200,000 in 512 10.5 and 20.2, 8.2 and 11.0; 1,200,000 in 1,024 15.2 and 28.2, 13.7 and 14.8; 4,000,000 in 1,024 25.3 and
// 49.3, 24.3 and 26.3.
constexpr int kSelfPlanResponses = 1024;
// Words of the status allocation that count the finished workgroups of a reduction: a pair for the calls that work in the
// context's workspace, a pair for the static call, which may run beside them.
constexpr int kTicketWord = 32, kStaticTicketWord = 48;
// Widest bf16 row (two vectors for each of 1,024 threads) that the streaming FP8 kernels take from the table kernels.  There the
// extremes and the table take the same time for every row, and a compute unit works on two rows at most; the streaming
// kernels have eight or more of them on their way.  us, streaming and table, 8,192 rows: quantisation, 1,000 logits 8.5 and
// 91.7, 4,096 19.0 and 93.2, 8,192 39.2 and 97.3, 16,384 97.6 and 99.3, 20,001 127 and 119; log-prob, 1,000 9.1 and 94.6,
// 8,192 44.8 and 97.7, 16,384 82.2 and 104.3, 24,001 120 and 122, 28,001 139 and 122.  41,643 rows of 1,000: 25.6 and 452.4;
// 31.1 and 467.5.  300 rows of 16,001 13.4 and 14.0, of 20,001 14.8 and 14.3.
constexpr int kFp8NarrowRow = 16391;
// ... and where every row has a compute unit to itself and is 16-byte aligned: 256 threads then read the row twice with
// nothing beside them, which takes longer from about six vectors for each thread on.  us, streaming and table, 1 and 256
// rows: quantisation, 12,288 logits 4.6 and 5.0, 5.2 and 5.8; 14,000 5.0 and 5.0, 5.8 and 5.8; 15,000 5.4 and 5.0, 6.2 and
// 5.9; log-prob, 12,288 5.3 and 5.5, 5.9 and 6.2; 13,312 5.7 and 5.6, 6.2 and 6.2; 16,384 6.3 and 5.5, 6.8 and 6.2.  300 rows
// of 16,384: 6.5 and 8.3, 7.9 and 8.7.
constexpr int kFp8NarrowLoneQuantize = 14336, kFp8NarrowLoneLogprob = 12800;
constexpr int kMaxDevices = 64;        // device indices a context may be created on
constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;
// What turns a difference of two logits' exponents as the fp32 `inv_temperature * kLog2e` gives it into the one with that
// factor as fp64 has it: the fp32 constant alone is 1.3e-8 off, which ten units of difference make 1.3e-7 of a small log-prob
// (rms relative error of log-probs over 4,096 rows of 32,003 fp32 logits 9.9e-8 without and 5.0e-8 with).  Formed on the
// host: a kernel that does it holds registers for it and is 0.05 to 0.1 us longer (2 % of 64 rows of 500 logits).
inline double exact_exponents(float inv_temperature) {
  return (double)inv_temperature * 1.4426950408889634074 / (double)(inv_temperature * kLog2e);
}

// Per-tile partial results of the diagnostics reduction (level 1 -> level 2), word k of tile b at [k * max_tiles + b], so
// that lanes which read consecutive tiles read consecutive words.  The spread of w_bar travels as (count, mean, sum of
// squared deviations from the mean), merged pairwise: a variance never comes out of the difference of two large sums.
enum DiagWord {
  kMeanW,    // mean of w_bar over the tile's valid rows
  kM2W,      // sum of (w_bar - mean)^2
  kSumAbs,   // sum of |log pi_train - log pi_roll|
  kSumD,     // sum of (log pi_train - log pi_roll)
  kSumDp,    // sum of |pi_train - pi_roll|
  kCounts,   // valid rows + 2^32 * rows with rho > C (a bit pattern, not a double)
  kDiagWords
};

// How a batch of more than kSelfPlanResponses responses is cut into tiles of kPlanTileRows: at most max_tiles of them.
struct TileRule {
  int max_tiles;
};
TileRule tile_rule(long long n_rows, int n_resp);

// Byte offsets of the regions of the context workspace for a call with (n_rows, n_resp).
struct WorkspaceLayout {
  size_t tile_off;   // int [n_resp + 2]   first tile of each response, and the total (n_resp > kSelfPlanResponses)
  size_t partial;    // of tiles: double [kDiagWords][max_tiles] (the loss: [max_tiles]); where rows are dealt out evenly: double
                     // [14][workgroups], then int [n_resp + workgroups] (the loss: double [16 workgroups])
  size_t g;          // float [n_rows]     per-row gradient coefficient
  size_t total;
};
WorkspaceLayout workspace_layout(long long n_rows, int n_resp);
size_t static_scratch_bytes(long long n_rows, int n_resp);   // what ais_diagnostics_static accepts a batch by

// Decomposition of the hidden-state read-out when every row is evaluated: token blocks x chunks of vocabulary
// tiles.  The decomposition actually used is decided on the device from the number of evaluated rows.
struct LmHeadPlan {
  int n_vtiles;          // tiles of 256 vocabulary entries
  int max_chunks;        // most chunks the device-side decision can use (sizes the workspace)
  int max_items;         // work items, rounded up to a multiple of 8 (sizes the grid)
  int max_items_masked;  // the same where fewer rows than that may be evaluated
  int chunks;            // chunks where every row is evaluated
};
LmHeadPlan lm_head_plan(long long n_rows, int vocab, int n_cus);
// Workspace of the read-out's two calls (the gradient call's: of a chunk's dlogits) and the gradient call's chunk width.
size_t lm_head_logprob_bytes(long long n_rows, int vocab, int n_cus);
constexpr long long kLmGradChunk = 8192;
long long lm_grad_chunk(long long m_rows, long long vocab, long long asked, int n_cus);
long long lm_grad_even_chunk(long long chunk, long long m_rows, long long vocab);
size_t lm_grad_wide_bytes(long long m_rows, long long vocab);
long long lm_grad_chunk_for(long long chunk, long long vocab, long long d_model, int n_cus);
// Parts that the sums of the gradient's two products over a chunk are split into, at most so many and so many bytes of each:
// fewer where the caller chose the chunk, which is how it bounds the workspace: 96 MiB and a quarter is less than the 150 MiB
// beside the workspace that a handle of the library's products held, which ran at these sizes before.  us a call with those,
// with up to 128 and with up to 48 MiB of each sum, chunks of 8,192: 300 rows x 50,257 x 4,096 1,228, 1,000, 1,021; 2,000 x
// 50,257 x 1,024 994, 708, 744; 20,000 x 32,000 x 512 2,489, 2,047, 2,237; chunks of 4,096: 5,000 x 32,000 x 512 976, 750, 777.
struct LmParts {
  int w, h;                  // of dweight and of dhidden
};
constexpr int kLmMaxParts = 32, kLmMaxWeightParts = 8;
constexpr long long kLmPartsBytes = 128LL << 20, kLmAskedPartsBytes = 48LL << 20;
LmParts lm_grad_parts(int n_cus, long long n_rows, long long d, long long n_v);
LmParts lm_grad_parts(int n_cus, long long n_rows, long long d, long long n_v, long long bytes_each);
size_t lm_grad_dlogits_bytes(long long m_rows, long long vocab, long long asked, int n_cus);
// The gradient call's chunk, the parts of its sums and where its arrays lie in the workspace, which begins with the chunk's
// dlogits (byte offsets).
struct LmGradRoom {
  long long chunk;
  LmParts parts;
  size_t plan;                 // decompositions of the recompute kernel
  size_t mask, index, pos;     // with a row list: rows with a gradient, their list, its inverse,
  size_t hidden, dhidden;      // the listed rows' hidden states and their gradient; the parts of dhidden
  size_t dweight;              // the parts of dweight
  size_t end;                  // end of the last of them
  size_t all;                  // what is asked for: no less, and no less than any call over fewer rows asks for
};
LmGradRoom lm_grad_room(long long n_rows, long long m_rows, long long d, long long vocab, long long asked, int n_cus,
                        int roomy);

}  // namespace ais

struct ais_ctx {
  int device = 0;
  hipStream_t stream = nullptr;
  void* ws = nullptr;
  size_t ws_bytes = 0;
  int* status_dev = nullptr;     // 256 bytes: the status word and the tickets, which are 0 between launches
  unsigned turns = 0, static_turns = 0;   // reductions launched with either pair of tickets
  int n_cus = 256;               // compute units of the device
  int last_hip_error = 0;
  bool profiling = false;
  struct Timed { hipEvent_t start, stop; int which; };
  std::vector<Timed> timed;      // events of measured launches
  std::vector<hipEvent_t> pool;  // recycled events
  // The row tiling that the last ais_diagnostics call left in the workspace (batches of more than kSelfPlanResponses
  // responses).  The calls that follow it in a step reuse the tiling instead of launching the plan kernel again when they
  // name the same cu_rows array, sizes and stream; anything else that writes the workspace clears it.
  struct Plan {
    const long long* cu_rows = nullptr;
    long long n_rows = -1;
    int n_resp = -1;
    hipStream_t stream = nullptr;
    bool valid = false;
  } plan;
  bool ws_recorded = false;         // a call that was recorded into a graph uses ws: replaced only for a call that it cannot hold
  void* static_scratch = nullptr;   // address, on this context's device, of the library's static scratch array
};

namespace ais {

int ensure_workspace(ais_ctx* ctx, size_t bytes);
int hip_fail(ais_ctx* ctx, hipError_t e);

// Raises the dynamic-LDS limit of kernel `fn` to `bytes` on the context's device, once per (kernel, device): `once`
// and `ok` are the caller's function-local tables of kMaxDevices entries.  False if the runtime refuses.
inline bool allow_dynamic_lds(ais_ctx* ctx, const void* fn, int bytes, std::once_flag* once, bool* ok) {
  std::call_once(once[ctx->device], [&] {
    ok[ctx->device] = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, bytes) == hipSuccess;
    if (!ok[ctx->device]) (void)hipGetLastError();
  });
  return ok[ctx->device];
}

// Brackets one launch with events when profiling is on.
struct ScopedTimer {
  ais_ctx* ctx;
  int idx = -1;
  ScopedTimer(ais_ctx* c, int which);
  ~ScopedTimer();
};

// Launchers (each checks nothing: arguments were validated by the entry point).
int launch_token_logprob(ais_ctx* ctx, const void* logits, ais_dtype dtype, long long n_rows, int vocab,
                         long long row_stride, const int* token_ids, const unsigned char* valid,
                         float inv_temperature, float* logp_out, float* lse_out);
int launch_dlogits(ais_ctx* ctx, const void* logits, ais_dtype dtype, long long n_rows, int vocab,
                   long long row_stride, const int* token_ids, const float* g, const unsigned char* valid,
                   const float* lse, const float* logp, float inv_temperature, void* dlogits);
int launch_fused_logprob_softmax(ais_ctx* ctx, const void* logits, ais_dtype dtype, long long n_rows, int vocab,
                                 long long row_stride, const int* token_ids, const unsigned char* valid,
                                 float inv_temperature, float* logp_out, float* lse_out, void* sgrad,
                                 bool* used_registers);
int launch_plan(ais_ctx* ctx, const long long* cu_rows, int n_resp, long long n_rows, int* tile_off);
int launch_diagnostics(ais_ctx* ctx, const float* logp_train, const float* logp_roll, const unsigned char* valid,
                       long long n_rows, const long long* cu_rows, int n_resp, int group_size,
                       const float* rewards, const ais_params& p, int* tile_off, double* partial,
                       bool in_static, float* adv_out, int* count_out, ais_diag* diag_out);
int launch_row_coeff(ais_ctx* ctx, const CoeffInputs& in, long long n_rows, int* tile_off, double* partial, float* g_out,
                     float* wtilde_out, double* loss_out, float g_scale);
// Coefficients, loss and gradient in one launch, for batches small enough; false where this one is not.
bool try_loss_dlogits_small(ais_ctx* ctx, const CoeffInputs& in, const void* logits, ais_dtype dtype, long long n_rows,
                            int vocab, long long row_stride, const int* token_ids, const float* lse, float* wtilde_out,
                            double* loss_out, void* dlogits);
int launch_copy(ais_ctx* ctx, void* dst, const void* src, long long bytes);
int launch_fp8_quantize(ais_ctx* ctx, const void* logits, ais_dtype dtype, long long n_rows, int vocab,
                        long long row_stride, unsigned char* codes, long long codes_stride, float* scale_out);
bool try_fp8_quantize_rows(ais_ctx* ctx, const void* logits, ais_dtype dtype, long long n_rows, int vocab,
                           long long row_stride, unsigned char* codes, long long codes_stride, float* scale_out);
int launch_fp8_dequantize(ais_ctx* ctx, const unsigned char* codes, long long codes_stride, const float* scale,
                          long long n_rows, int vocab, void* out, ais_dtype dtype, long long out_stride);
bool try_fp8_dequantize_burst(ais_ctx* ctx, const unsigned char* codes, long long codes_stride, const float* scale,
                              long long n_rows, int vocab, void* out, ais_dtype dtype, long long out_stride);
bool try_fp8_quantize_table(ais_ctx* ctx, const void* logits, ais_dtype dtype, long long n_rows, int vocab,
                            long long row_stride, unsigned char* codes, long long codes_stride, float* scale_out);
bool try_fp8_rollout_logprob_table(ais_ctx* ctx, const void* logits, ais_dtype dtype, long long n_rows, int vocab,
                                   long long row_stride, const int* token_ids, const unsigned char* valid,
                                   float* logp_out);
int launch_fp8_rollout_logprob(ais_ctx* ctx, const void* logits, ais_dtype dtype, long long n_rows, int vocab,
                               long long row_stride, const int* token_ids, const unsigned char* valid,
                               float* logp_out);

int launch_lm_head_grad_setup(ais_ctx* ctx, const unsigned char* live_mask, long long n_rows, int n_cap, int width,
                              int width_last, int* row_index, int* row_pos, void* dev_plan);
int launch_lm_head_dlogits_chunk(ais_ctx* ctx, const void* hidden, long long ld_h, const void* weight,
                                 long long ld_w, long long n_rows, int d_model, int vocab, int y_off,
                                 const int* token_ids, const float* lse, const float* logp, const float* coeff,
                                 float inv_temperature, const void* dev_plan, int which, void* ds, long long ds_stride,
                                 const int* row_index, int n_cap);
int launch_lm_grad_products(ais_ctx* ctx, const void* ds, long long ds_stride, const void* h, long long ld_h, const void* w,
                            long long ld_w, int n_rows, const int* n_rows_dev, int n_v, int d, float* dweight,
                            float* dhidden, LmParts parts, long long w_stride, long long h_stride, bool accumulate);
int launch_lm_add_parts(ais_ctx* ctx, const float* part, long long part_stride, int parts, const int* row_pos,
                           long long n_rows, int d, float* out);
int launch_lm_live_mask(ais_ctx* ctx, const float* coeff, long long n_rows, unsigned char* mask);
int launch_lm_gather_rows(ais_ctx* ctx, const void* hidden, long long ld_h, int d_model, const int* row_index,
                          const void* dev_plan, int n_cap, void* gathered);
int launch_lm_head_logprob(ais_ctx* ctx, const void* hidden, long long ld_h, const void* weight, long long ld_w,
                           long long n_rows, int d_model, int vocab, const int* token_ids,
                           const unsigned char* valid, float inv_temperature, const LmHeadPlan& plan,
                           float* part_m, float* part_s, float* zy, int* row_index, int* row_pos, void* dev_plan,
                           float* logp_out, float* lse_out);

}  // namespace ais
