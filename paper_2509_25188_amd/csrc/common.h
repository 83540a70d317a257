// Internal declarations shared by the HIP translation units of libl2pd.
#pragma once
#include <hip/hip_runtime.h>
#include <hip/hip_bf16.h>
#include <stdint.h>

#include <atomic>

#include "../../include/l2pd.h"

namespace l2pd {

typedef __hip_bfloat16 bf16;

// Division of a number by one that only the launch knows: two multiplications instead of some 40 instructions (with one or
// two wavefronts on a SIMD, 0.1 us each).  m = ceil(2^31 / d), so the product is the quotient or one more: exact for
// 0 <= x < 2^30.
struct Div {
  unsigned m, d;
  Div(int d_ = 1) : m((unsigned)(((1ull << 31) + d_ - 1) / d_)), d(d_) {}
  __device__ __forceinline__ int operator()(int x) const {
    const unsigned q = __umulhi((unsigned)x << 1, m);
    return (int)(q - (q * d > (unsigned)x ? 1 : 0));
  }
};

// Device control block (int32 words).  Written by k_prepare at the start of every step.  The words
// from CTL_SEQ_GB on hold the active block of every sequence: the batch's common one in lock step,
// the sequence's own with per-sequence block pointers.
// After them (from CTL_SEQ_GB + max_batch on; k_prepare is told where) one word per sequence: 1 once it is done.
enum { CTL_GB = 0, CTL_ALL_DONE = 1, CTL_ACTIVE = 2, CTL_TMAX = 3, CTL_WORDS = 8, CTL_SEQ_GB = 8 };

// Every kernel of a step is gated: once decoding has stopped (or, with the prefix cache, once the
// block the host enqueued it for is finished) it returns at once, so steps that the host enqueued
// ahead of the device's progress cost a launch and nothing else.
// A kernel asks for the two words first, sends off its first loads, and only then looks at them: the round trip to the
// control block (0.2 us, in each of the 60 to 230 kernels of a step) is not waited for.
struct Gate {
  const int* ctl;     // the control block, for kernels that read more of it; nullptr: there is none
  int expect_gb;      // >= 0: skip unless the active block is this one
  const int2* words;  // never null: (active block, all done) of the control block, or zeros
  bool cold;          // no gate, but as much the same for every launch of a bf16 model: its weights do not fit the memory-side cache,
                      // none of them is there when a pass wants it
};
static_assert(CTL_GB == 0 && CTL_ALL_DONE == 1, "the gate's two words");
__device__ __forceinline__ int2 gate_words(const Gate& g) { return *g.words; }
__device__ __forceinline__ bool gate_closed(const Gate& g, int2 w) {
  return (w.y != 0) | ((g.expect_gb >= 0) & (w.x != g.expect_gb));
}
__device__ __forceinline__ bool gate_skip(const Gate& g) { return gate_closed(g, gate_words(g)); }

// Maps a compact row index r (b * rows_per_seq + j) to a row of a [B, seq_stride] array:
//   b * seq_stride + off_base + gb_b * off_per_gb + j,  gb_b = sequence b's active block from the control block.
struct RowMap {
  int rows_per_seq, seq_stride, off_base, off_per_gb;
};
__device__ __forceinline__ int map_row(const RowMap& m, int r, const int* ctl) {
  int gb = (m.off_per_gb && ctl) ? ctl[CTL_SEQ_GB + r / m.rows_per_seq] : 0;
  return (r / m.rows_per_seq) * m.seq_stride + m.off_base + gb * m.off_per_gb + (r % m.rows_per_seq);
}

// whether map_row moves any of the first `rows` rows
inline bool row_map_moves(const RowMap& m, int rows) {
  return m.off_base || m.off_per_gb || (rows > m.rows_per_seq && m.seq_stride != m.rows_per_seq);
}

// exp(-x) for x >= 0: the product with log2(e) in two parts, the small one applied to the result to first order
// (about 1 ulp, a third of the instructions of expf).  Beyond 200 the result is 0 (and the two parts would be
// infinities of opposite sign); NaN stays NaN.
__device__ __forceinline__ float exp_neg(float x) {
  x = x > 200.f ? 200.f : x;
  const float l2e = 1.44269504089f, l2e_lo = 1.92596303e-8f;   // log2(e) = l2e + l2e_lo
  const float hi = -x * l2e, lo = -fmaf(x, l2e, hi) - x * l2e_lo;
  const float e = __builtin_amdgcn_exp2f(hi);
  return fmaf(e, lo * 0.69314718056f, e);
}

// Raises a kernel's dynamic-LDS limit once per device: the attribute belongs to the device's copy of
// the kernel, and launchers may be called from several host threads (setting it twice is harmless).
struct DynLdsAttr {
  std::atomic<unsigned long long> done{0};
  void ensure(const void* kernel, int bytes) {
    int dev = 0;
    (void)hipGetDevice(&dev);
    const unsigned long long bit = 1ull << (dev & 63);
    if (done.load(std::memory_order_acquire) & bit) return;
    (void)hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
    done.fetch_or(bit, std::memory_order_release);
  }
};

// ---- small kernels (kernels_misc.hip) ----
void launch_fill_u32(uint32_t* p, size_t n, uint32_t v, hipStream_t s);
// (cos, sin) of pos * base^(-2i / head_dim), [max_pos, head_dim / 2]
void launch_rope_table(float2* table, int max_pos, int head_dim, float base, hipStream_t s);
void launch_init_decode(int32_t* X, const int32_t* prompt, int B, int P, int G, int mask_id, int32_t* state,
                        int* ctl, hipStream_t s);
void launch_prepare(const int32_t* state, int B, int n_blocks, int ragged, int* ctl, hipStream_t s,
                    int done_at = 0);   // done_at > 0: also ctl[done_at + b] = sequence b's done flag
void launch_embed(float* h, const bf16* emb, const int32_t* tokens, RowMap tokmap, int rows, int d,
                  Gate g, hipStream_t s);
// h (+= the sum part[0] + ... + part[n_parts-1], formed first, in that order, when given) -> y = rmsnorm(h) * gain, rows taken
// through `src`.  part z is at parts + z * part_stride, laid out like h.  The sum is written back to h
// when `write_back` is set; the final norm before the LM head leaves h alone (h is dead after it, and
// two head rows may map to one row of h, so a write-back would race).
// h_out: the parts are laid out like y and the sum goes to h_out, laid out like y too, instead of back to h.
void launch_rmsnorm(float* h, const float* parts, int n_parts, size_t part_stride, RowMap src, const bf16* gain,
                    bf16* y, int rows, int d, float eps, bool write_back, Gate g, hipStream_t s,
                    float* h_out = nullptr);
constexpr int kFilterMaxLayers = 4;
struct UpdateArgs {
  int32_t* X;            // [B, T]
  int32_t* state;        // [B, 3]
  int B, P, T, s, n_blocks, mask_id, eos_id, eotp;
  const float* part_max; // [B*s, n_part]
  const float* part_sum;
  const int32_t* part_idx;
  int n_part;
  // the filter as it goes to LDS, filled in by launch_update: layer k's weights (nw) at `at`, its biases (nb) behind them;
  // layers that there are not stand for one number of the first.  total 0: it does not fit, or there is none
  struct Staged { const float *w[kFilterMaxLayers], *b[kFilterMaxLayers]; int nw[kFilterMaxLayers], nb[kFilterMaxLayers], at[kFilterMaxLayers], total; } staged;
  // filter: n_layers layers of widths s -> hidden -> ... -> hidden -> s (layer k: fw[k] [out, in], fb[k] [out])
  const float* fw[kFilterMaxLayers];
  const float* fb[kFilterMaxLayers];
  int n_layers, hidden;
  float tau;
  float* conf_out;       // optional taps [B, s]
  int32_t* pred_out;
  float* filt_out;
  uint8_t* unmask_out;
  int* ctl;
  const int* teff;       // step-granular EoTP: per-sequence length in force (else null)
  // EGP rollout (Alg. 1): unmask where the prediction equals the reference answer; one training row per step
  const int32_t* reference;   // [B, gen_len] or null
  float* egp_conf;            // [B, gen_len, s]: row = step index of the sequence
  float* egp_label;
  int gen_len;
  int next_ctl, ragged;       // B == 1: also leave the control block as launch_prepare would for the state afterwards
};
void launch_update(UpdateArgs a, Gate g, hipStream_t s);
void launch_finalize(const int32_t* X, const int32_t* state, const int* teff, const int32_t* perm, int B, int P,
                     int G, int s_len, int mask_id, int32_t* tokens_out, int32_t* steps_out, int32_t* dlen_out,
                     hipStream_t s);
// live sequences to the leading rows (stable), src copies -> dst copies; perm_src nullptr = identity
void launch_compact(const int32_t* X_src, int32_t* X_dst, const int32_t* state_src, int32_t* state_dst,
                    const int32_t* perm_src, int32_t* perm_dst, int B, int T, hipStream_t s);
// `epochs` full-batch AdamW steps on the binary cross-entropy of Eq. 6 for a filter of n_layers layers
// (widths s -> hidden -> ... -> hidden -> s), in place.
struct TrainArgs {
  float* w[kFilterMaxLayers];   // device, updated in place; layer k: [out, in]
  float* b[kFilterMaxLayers];
  int n_layers, s, hidden;
  const float* conf;          // [n, s]
  const float* label;         // [n, s]
  long long n;
  int epochs;
  float lr, beta1, beta2, eps, weight_decay;
  float* opt_state;           // [2 * n_params], never read before it is written; holds the moments at the end
  float* loss_out;            // [epochs] or null
};
int filter_param_count(int s, int hidden, int n_layers);
int filter_train_supported(int s, int hidden, int n_layers);
// `ws` (16-byte aligned, filter_train_split_bytes of it; null: one workgroup does it all): rows over workgroups
void launch_filter_train(const TrainArgs& a, float* ws, hipStream_t s);
constexpr size_t kTrainSplitFloats = 2560000;   // filter_train_split_bytes never asks for more: 10.2 MB
size_t filter_train_split_bytes(int s, int hidden, int n_layers, long long n);   // 0: one workgroup is the better choice
void launch_seq_len(const int32_t* X, int B, int P, int G, int eos_id, int* teff, int* ctl, hipStream_t s);
// keys[b] = base + ctl[CTL_SEQ_GB + b] * per_gb: keys a sequence's block rows may see under the prefix cache
void launch_block_keys(const int* ctl, int B, int base, int per_gb, int* keys, hipStream_t s);

struct BiasArgs {
  int token_id, gen_pos_from, block_len;
  float value;           // 0: off
};
struct LmHeadEpilogue {
  float* logits;         // optional [M, V]
  float* part_max;       // optional [M, n_part]: per part of the columns max, sum exp(x - max), argmax (lowest id on ties),
  float* part_sum;       // mask_id excluded
  int32_t* part_idx;
  int n_part;
  int mask_id;
  BiasArgs bias;         // applied when value != 0 (needs ctl for the active block)
};

// ---- fp32 path (kernels_f32.hip) ----
// One product of a layer with what comes before and behind it:
//   F32_QKV     rows of A, RMS-normalised with `gain`, times W[0..2]: rotated q into C [rows, H * Dh], rotated k and v into the
//               [B, Tmax, H * Dh] stores at pos0 + t (seq_gb / pos_per_gb: per-sequence offsets as in QkvEpilogue).
//               N = 3 * H * Dh / 2 pairs
//   F32_SWIGLU  normalised rows times W[0], W[1]: silu(.) * . into C [rows, N]
//   F32_LMHEAD  normalised rows times W[0]: logits and partials, f32_lmhead_n_part of them a row
//   F32_PLAIN   C [rows, N] (+)= A W[0]^T
enum { F32_PLAIN = 0, F32_QKV = 1, F32_SWIGLU = 2, F32_LMHEAD = 3 };
struct F32Product {
  const float* A;          // row r of the product is row map_row(rows, r) of A [., K], or of the table A at that token
  RowMap rows;
  const int32_t* tokens;   // null: rows of A as they are
  float* h_out;            // optional (with tokens): the rows as they are, [M, K]
  const float* gain;
  float eps;
  const float* W[3];
  int M, N, K;
  float* C;
  int accumulate;
  float *kstore, *vstore;
  const float2* rope;
  int Tq, pos0, Tmax, H, Dh;
  const int* seq_gb;
  int pos_per_gb;
  LmHeadEpilogue lm;
  Gate gate;
  // filled in by launch_product_f32: rows are not simply 0, 1, ...; divisions by H * Dh / 2, Dh / 2 and Tq
  int mapped;
  Div per_mat, half, per_seq;
};
void launch_product_f32(F32Product a, int kind, hipStream_t s);
int f32_lmhead_n_part(int V);
void launch_attn_f32(const float* q, const float* kstore, const float* vstore, float* out, int B, int Tq, int Tk,
                     int Tmax, int H, int Dh, const int* tk_dev, Gate g, hipStream_t s);

// ---- bf16 path ----
struct QkvEpilogue {
  bf16* q;               // [rows, d]
  bf16* kstore;          // [B, Tpad, d]
  bf16* vtstore;         // [B, H, Dh, Tpad]
  const float2* rope;    // [max_pos, Dh/2] (cos, sin)
  int Tq, pos0, Tpad, H, Dh, d;
  // per-sequence block pointers with a K/V cache: row t of sequence b sits at position
  // pos0 + seq_gb[b] * pos_per_gb + t (seq_gb = the control block's per-sequence active blocks); null: pos0 + t
  const int* seq_gb;
  int pos_per_gb;
};
__device__ __forceinline__ int seq_pos_offset(const int* seq_gb, int per_gb, int b) {
  return seq_gb ? seq_gb[b] * per_gb : 0;
}
void launch_gemm_qkv_bf16(const bf16* A, const bf16* wq, const bf16* wk, const bf16* wv, int M, int K,
                          const QkvEpilogue& e, Gate g, hipStream_t s);
// partial[z][M,N] = A[:, z-th K slice] * W[:, slice]^T, z < wide_splits(M, N, K, pass_rows).  The rows may be some of a
// pass over pass_rows >= M: they sum in the order of that pass, however few they are.
// add (wide_splits == 1): parts is the residual stream [M, N]; the sum is added to it in place instead of written.
void launch_gemm_partial_bf16(const bf16* A, const bf16* W, float* parts, size_t part_stride, int M, int N, int K,
                              int pass_rows, bool add, Gate g, hipStream_t s);
int k_ranges(int pass_rows, int N, int K);   // K ranges that a [pass_rows, N] projection sums in (more than 64 rows)
// Few-row GEMMs (block-only steps of the cached decode modes, at most kSkinnyRows rows) stream their
// weights once; K is split until a launch has a few hundred workgroups, each K range staying a
// multiple of the 64-wide stage.
constexpr int kSkinnyRows = 64;
constexpr int kSkinnyRowsAttn = 64;   // B * Tq up to which attention may chunk the keys across workgroups
int skinny_splits(int N, int K);
int wide_splits(int M, int N, int K, int pass_rows);   // partial buffers the wide path's [d, d] / [d, F] projections write, at most 8
size_t partial_floats(long long rows, int d, int F);   // split-K partials of any pass of up to `rows` rows
void launch_gemm_skinny_bf16(const bf16* A, const bf16* w0, const bf16* w1, int n_sub, float* parts,
                             size_t part_stride, int M, int N, int K, int splits, Gate g, hipStream_t s);
// sums of the skinny GEMM's partials -> SiLU(gate) * up
void launch_skinny_swiglu_finish(const float* parts, int n_parts, size_t part_stride, int rows, int F, bf16* act,
                                 Gate g, hipStream_t s);
// act[M, F] = silu(A Wg^T) * (A Wu^T).  Few rows: launch_gemm_swiglu_bf16 (GATE_UP_TILES), launch_gemm_few_rows_swiglu_bf16
// (GATE_UP_WIDE), or K ranges and a finishing kernel (GATE_UP_RANGES).
enum GateUpPath { GATE_UP_TILES, GATE_UP_WIDE, GATE_UP_RANGES };
GateUpPath few_rows_gate_up(int F, int K, bool ranges);
void launch_gemm_swiglu_bf16(const bf16* A, const bf16* wg, const bf16* wu, bf16* act, int M, int F, int K, Gate g,
                             hipStream_t s);
void launch_gemm_few_rows_swiglu_bf16(const bf16* A, const bf16* wg, const bf16* wu, bf16* act, int M, int F, int K, Gate g,
                                      hipStream_t s);
int lmhead_n_part(int V);
void launch_gemm_lmhead_bf16(const bf16* A, const bf16* W, int M, int V, int K, const LmHeadEpilogue& e, Gate g,
                             hipStream_t s);
// `sel`: only n query rows of every sequence are wanted, from base + seq_gb[b] * per_gb on (seq_gb null: base); out is
// then [B * n, d].  n == 0: all of them.
struct QueryRows {
  int n, base, per_gb;
  const int* seq_gb;
};
void launch_attn_bf16(const bf16* q, const bf16* kstore, const bf16* vtstore, bf16* out, int B, int Tq, int Tk,
                      int Tpad, int H, int Dh, float* chunk_ws, size_t chunk_ws_bytes, const int* tk_dev, QueryRows sel,
                      Gate g, hipStream_t s);
// bytes of chunk workspace that lets launch_attn_bf16 spread few queries' keys over workgroups
inline size_t attn_chunk_ws_bytes(int H, int Dh) { return (size_t)kSkinnyRowsAttn * H * 16 * (Dh + 2) * 4; }

}  // namespace l2pd
