// Launch wrappers of the GPU library's kernels (host-callable).
#pragma once

#include <algorithm>
#include <stddef.h>
#include <stdint.h>

#include "common.h"

namespace ebrl {

// ------------------------------------------------------------------ GEMM --
enum EpiKind {
    EPI_F32 = 0,     // C f32 [M, ldc] = acc
    EPI_ACT = 1,     // C act dtype = acc (bf16 or f32)
    EPI_RESID = 2,   // C f32 += acc (residual stream)
    EPI_REMAP = 3,   // C f32 row row_base[m/group] + m%group = acc (+ add row m%group)
    EPI_SWIGLU = 4,  // packed gate/up -> C act [M, N/2] = silu(gate) * up
    EPI_QKV = 5      // rotary-paired Q/K/V rows -> rotated Q (act) + paged K/V cache (see RopeKVArgs)
};
struct RopeKVArgs;

struct GemmArgs {
    bool bf16 = true;
    const void* A = nullptr; int lda = 0;   // [M, K] activations
    const void* B = nullptr; int ldb = 0;   // [N, K] weights
    int M = 0, N = 0, K = 0;
    EpiKind epi = EPI_F32;
    void* C = nullptr; int ldc = 0;
    const int* row_base = nullptr; int group = 1;
    const void* add = nullptr; int add_ld = 0;
    const RopeKVArgs* rope = nullptr;           // EPI_QKV parameters
    float* ws = nullptr; size_t ws_floats = 0;  // split-K workspace
    // gemm_counter_words() zeroed words; bf16 GEMMs with K splits leave them
    // zero again.  Calls that share a workspace must not overlap in time.
    unsigned* counters = nullptr;
    // Decode GEMMs (M = batch, at most 256) may split K; the split count then
    // depends on (N, K) only, so an element's summation order -- and its bits
    // -- do not depend on the batch size.  Without splitting, every kernel
    // variant sums K in the same 64-wide steps, so results do not depend on M
    // either.
    bool split_ok = false;
    // GEMMs with a paired epilogue (EPI_QKV, EPI_SWIGLU) that gemm_row_norm_ok
    // allows (bf16 decode with one K split; all fp32): A holds un-normalised
    // rows and every output row is scaled by 1/sqrt(mean_k A[m][k]^2 +
    // norm_eps), i.e. the unit-gain RMSNorm of the input folded into the
    // projection.
    bool row_norm = false; float norm_eps = 1e-6f;
    // EPI_RESID: also store the updated rows in bf16 here (nullable).
    void* xb = nullptr; int ldxb = 0;
    // Compute units the launch stream may use (its CU mask): the decode
    // kernel's column-slice width and the large-M kernel's macro tile are
    // priced in rounds over this many CUs.  Neither choice changes an
    // element's summation order.
    int cus = 256;
};
// Decode GEMMs (split_ok) plan their K splits for at most this many rows;
// callers that need batch-size-independent bits keep calls within it.
constexpr int DECODE_MAX_ROWS = 256;
// Returns the number of K splits used (1 = single pass).
int gemm(const GemmArgs& a, hipStream_t s);
// What gemm() launches for a product: {kernel, tile rows, tile columns, K splits,
// workgroups, LDS stages of the decode kernel, tiles that the large-M kernel
// deals evenly, parts that it cuts each other tile into}; what a kernel has not
// is 0.
enum { GEMM_K_TILES = 0, GEMM_K_LARGE, GEMM_K_RING, GEMM_K_DECODE, GEMM_K_FP32 };
void gemm_plan_info(bool bf16, int M, int N, int K, size_t ws_floats, bool split_ok, int cus, int32_t* out);
bool gemm_row_norm_ok(bool bf16, int M, int N, int K, size_t ws_floats);
size_t gemm_counter_words();
// Workspace floats the plan for (M, N, K) writes (0 without a K split).
size_t gemm_ws_floats_used(bool bf16, int M, int N, int K, size_t ws_floats, bool split_ok);

// ------------------------------------------------------------- attention --
// Paged KV: layer base pointer; physical block b holds
// [2 (K, V)][kv_heads][16 tokens][head_dim] elements.
struct PagedKV {
    void* base = nullptr;            // this layer's first block
    const int* block_table = nullptr;  // [max_envs][bt_stride]
    int bt_stride = 0;
    int kv_heads = 0, head_dim = 0;
};

// Flash attention over query tiles of ATTN_Q_TILE rows.  Tile t covers rows
// [tile_q0[t], +ATTN_Q_TILE) of sequence tile_seq[t].
constexpr int ATTN_Q_TILE = 64;
struct AttnPrefillArgs {
    bool bf16 = true;
    const void* Q = nullptr; int ldq = 0;  // [rows, q_heads*hd]
    void* O = nullptr; int ldo = 0;        // [rows, q_heads*hd]
    int q_heads = 0;
    PagedKV kv;
    const int* seq_env = nullptr;   // [n] block-table row of each sequence
    const int* q_off = nullptr;     // [n] first Q/O row
    const int* q_len = nullptr;     // [n]
    const int* q_pos0 = nullptr;    // [n] absolute position of the first query
    const int* kv_len = nullptr;    // [n]
    const int* tile_seq = nullptr;  // [n_tiles]
    const int* tile_q0 = nullptr;   // [n_tiles]
    int n_tiles = 0;
    bool causal = true;
    int max_kv_len = 0;             // fp32 path: scores buffer size
};
void attn_prefill(const AttnPrefillArgs& a, hipStream_t s);
// bf16 attention kernels stage a sequence's block table in LDS: at most this
// many 16-token blocks (4096 tokens) per sequence.
constexpr int ATTN_BT_MAX = 256;

// One query per sequence against kv_len[i] keys, split over the sequence in
// chunks (fp32: ATTN_DEC_CHUNK keys; bf16: at most 512 keys at head dim 128,
// 1024 at 64) merged in chunk order.
constexpr int ATTN_DEC_CHUNK = 64;
struct AttnDecodeArgs {
    bool bf16 = true;
    const void* Q = nullptr; int ldq = 0;  // [n, q_heads*hd]
    void* O = nullptr; int ldo = 0;
    int q_heads = 0;
    PagedKV kv;
    const int* seq_env = nullptr;
    const int* kv_len = nullptr;
    int n = 0;
    int max_splits = 0;            // ceil(longest kv_len / ATTN_DEC_CHUNK) the buffers are sized for
    float* part = nullptr;         // [n][q_heads][max_splits][hd + 2]
    // bf16: [n][q_heads] zeroed words (left zero after the call)
    unsigned* counters = nullptr;
};
void attn_decode(const AttnDecodeArgs& a, hipStream_t s);

// ----------------------------------------------------------------- misc --
// Y[row] = rmsnorm(X[src_row]) ; src_row = rows ? rows[i] : i
void rmsnorm_rows(bool bf16_out, const float* X, int ldx, const int* rows, void* Y, int ldy,
                  int n_rows, int d, float eps, hipStream_t s);

// Rotary embedding + paged KV write of the fused QKV projection, applied in
// the GEMM epilogue (EPI_QKV): rotated queries go to Q (act dtype), rotated
// keys and the values to the paged cache.  row_dst[m] = {position of row m in
// its sequence, physical block of that position}: one load per row, where the
// chain row -> sequence -> env -> block table took three dependent ones at the
// end of every QKV launch.  use_rope = false skips rotation.  The QKV weight
// rows are packed per head so that rows e and e + hd/2 sit in the two 16-row
// halves of one 32-row group.
struct RopeKVArgs {
    int q_heads = 0;
    void* Q = nullptr; int ldq = 0;
    PagedKV kv;
    const int2* row_dst = nullptr;
    const float* cos_tab = nullptr;  // [max_pos][hd/2]
    const float* sin_tab = nullptr;
    bool use_rope = true;
};

// X[dst_rows[i]] = E[ids[src[i]]] as float; ids outside [0, n_rows_e) give zero rows.
void embed_rows(bool bf16, const void* E, int n_rows_e, int d, const int* ids, const int* src, const int* dst_rows,
                float* X, int ldx, int n, hipStream_t s);

// images f32 [n, cams, H, W, 3] -> patches [n*cams*(H/P)*(W/P), kpad] (zero-padded columns)
void im2col(bool bf16, const float* img, int n, int cams, int H, int W, int P, void* out,
            int kpad, hipStream_t s);

// Action head: logits = W_act . rmsnorm(x_row), argmax (ties -> lowest), top-2 margin,
// bin -> action.  Writes column `col` of [n, ntok] outputs and, with `emb`, the
// chosen tokens' embedding rows as the next step's input rows 0 .. n - 1.
struct LogitsArgs {
    bool bf16 = true;
    const float* X = nullptr; int ldx = 0;
    const int* rows = nullptr;      // gather rows of X (nullable: identity)
    const void* W = nullptr;        // [n_bins, d]
    int d = 0, n_bins = 256, n = 0;
    float eps = 1e-6f;
    int* tokens = nullptr; float* actions = nullptr; float* margins = nullptr;
    int ntok = 7, col = 0;
    const void* emb = nullptr;      // [n_bins, d]
    float* nx = nullptr; int ldnx = 0;   // next input rows
    void* nxb = nullptr; int ldnxb = 0;  // the same in bf16 (nullable)
    // logits scratch [n][n_bins] and n zeroed counters (left zero after the call)
    float* lg = nullptr; unsigned* counters = nullptr;
};
void action_logits(const LogitsArgs& a, hipStream_t s);

// Streaming read of `bytes` (multiple of 16) with non-temporal loads (HBM read reference).
void stream_read(const void* buf, size_t bytes, unsigned* out, hipStream_t s);

// Last prefix row of each sequence: h_pre[env] = X[row]; h_norm[env] = rmsnorm(X[row]).
void gather_last(const float* X, int ldx, const int* seq_env, const int* last_row, int n, int d,
                 float eps, float* h_pre, float* h_norm, hipStream_t s);

// out[r][n] = sum_k in[r][k] * W[n][k]  (W act dtype), optional silu on the input.
void small_linear(bool bf16, const float* in, int R, int K, const void* W, int N, float* out,
                  bool silu_input, hipStream_t s);

// The expert's ends of a denoising step, for one or two modalities (rows = 0:
// none): with `last`, the output head on H and the Euler update x_out = x - v /
// n_steps; then, with `first`, the input projection of x (updated or not) plus
// the time vector, written to H.  A modality's token r lives in row
// (r / per_in) * per_out + off + r % per_in of H.  d % 64 == 0, adim <= 64.
struct FlowMod {
    const float* x = nullptr; float* x_out = nullptr;   // [rows, adim]; may be the same buffer
    float* v_out = nullptr;                             // velocities (nullable)
    const void* w_in = nullptr;                         // [d, adim]
    const void* w_out = nullptr;                        // [adim, d]
    int adim = 0, rows = 0, per_in = 1, off = 0;
};
struct FlowStepArgs {
    bool bf16 = true, last = false, first = false;
    FlowMod mod[2];
    float* H = nullptr; int ldh = 0;
    int d = 0, per_out = 0;
    const float* tvec = nullptr;
    float eps = 1e-6f, n_steps = 1.f;
};
void flow_step(const FlowStepArgs& a, hipStream_t s);

// Element copy (device) with f32 -> f32.
void copy_f32(const float* src, float* dst, size_t n, hipStream_t s);
// The first `count` elements of a decode call's tokens (and, where the
// destination is not NULL, actions and margins) to the caller's buffers.
void copy_decode_out(const int* tok, const float* act, const float* mar, int count, int* out_tok, float* out_act,
                     float* out_mar, hipStream_t s);
// Standard normals for `rows` rows of per_row floats: Philox4x32-10 with
// counter (pair, calls[i], env[i], stream) under the seed, Box-Muller.
void normal_noise(float* out, int rows, int per_row, const int* env, const int* calls, uint64_t seed,
                  uint32_t stream, hipStream_t s);

}  // namespace ebrl
