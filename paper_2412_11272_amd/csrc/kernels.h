// Internal launcher interface between the host runtime (encoder.hip) and the gfx950 kernels.
// Nothing here is part of the public ABI (include/wf_encoder.h is).
#pragma once
#include <hip/hip_runtime.h>
#include <stdarg.h>
#include <stdint.h>

namespace wf {

typedef uint16_t bf16_raw;   // storage type of a bfloat16 value in host-visible structs

// How the GEMM reads its activation operand.
enum AMode : int {
  A_PLAIN = 0,   // row r of the operand is A + r * lda
  A_CONV3 = 1,   // row r is a contiguous window of 3*C elements starting at row_src[r] * C of a
                 // [rows, C] matrix: the three taps of a width-3 convolution.  row_flags[r] bit 0
                 // zeroes tap 0 (first frame of a stream), bit 1 zeroes tap 2 (last frame).
  A_LN = 2,      // small-batch kernel only: A is an fp32 matrix x (row stride lda) and the operand is LayerNorm(x) with
                 // ln_g / ln_b / ln_eps, normalised on the way in
};

// What the GEMM does with acc = A . W^T.
enum Epilogue : int {
  EPI_BIAS = 0,            // out = acc + bias                          (QKV projection)
  EPI_BIAS_GELU = 1,       // out = GELU(acc + bias)                    (fc1, first convolution)
  EPI_BIAS_RESID = 2,      // out(fp32) += acc + bias, in place         (out-projection, fc2)
  EPI_BIAS_GELU_POS = 3,   // out(fp32) = GELU(acc + bias) + pos[row_pos[r]]   (second convolution)
  EPI_BIAS_F32 = 4,        // out(fp32) = acc + bias                    (logits)
  EPI_PARTIAL = 5,         // out(fp32)[s][M][N] = acc of the s-th of k_splits parts of the reduction; the LayerNorm that
                           // follows adds the parts and the bias to the residual stream
};

struct GemmArgs {
  const void *A;            // activations: bf16 (MFMA path) or fp32 (debug path)
  const void *W;            // weights [N, K] row-major, same element type as A; K zero-padded
  const float *bias;        // [N]
  void *out;                // [M, ldo]; bf16 for EPI_BIAS / EPI_BIAS_GELU on the MFMA path, else fp32
  int32_t M, N, K;          // K is the padded reduction length (multiple of 64 on the MFMA path)
  int32_t lda, ldo;
  // work-unit split of the direct-load GEMM (set by its launcher): full tiles, then half-width units
  int32_t n_full, n_half, full_per_xcd, half_per_xcd;
  int32_t group_n;          // tiles walk column groups of this many tile columns (>= tiles per row: plain row-major)
  uint32_t div_group, div_row, div_last, div_split;      // order_mul of the tile order's divisors (set by the launchers): tiles of a group,
                            // columns of a group, of the last group, parts of a cut reduction
  // Panel layout (direct-load GEMM only): instead of row-major, a matrix is stored as [rows/256][cols/64][256][64],
  // i.e. every (256-row panel, 64-column chunk) is one contiguous 32 KB block -- exactly one K step of a
  // tile's operand.  a_panels: A is read in that layout; w_panels: W is (rows = output features, padded to a
  // multiple of 256); out_panels: a bf16 result is written in it.
  int32_t a_panels, w_panels, out_panels;
  // A_CONV3 only
  const int32_t *row_src;   // [M], ascending; -1 is a window that starts before the matrix, with its first tap masked
  const int32_t *row_flags;
  int32_t C;                // channels per tap; 3*C <= K, elements at k >= 3*C read as zero
  // EPI_BIAS_GELU_POS only
  const float *pos;         // [n_pos, N]
  const int32_t *row_pos;   // [M]
  // A_LN only
  const float *ln_g, *ln_b; // [K]
  float ln_eps;
  // bf16 results only (EPI_BIAS on the MFMA path): columns [n_split, N) of the result go to out2 (row stride ldo2) instead
  // of out, starting at its column 0 -- one product feeding two buffers (queries | keys and values).  n_split % 8 == 0.
  void *out2;
  int32_t n_split, ldo2;
  // EPI_BIAS_F32 only: columns [n_valid, N) of the result are not stored (the weight rows that pad a vocabulary to whole
  // tiles), ldo = n_valid may be odd; 0: all columns, ldo a multiple of 4
  int32_t n_valid;
  // One product over several weight matrices side by side (bf16 results, no panels): columns [g n_group, (g + 1) n_group) of the result go
  // to out + g group_stride (elements), row stride ldo.  n_group is a multiple of every tile's width; 0: one matrix.
  int32_t n_group;
  int64_t group_stride;
  int32_t k_splits;         // EPI_PARTIAL only
  int32_t shares_chip;      // another lane's kernels run beside this one
  int32_t prefer_large;     // never the small-batch kernel (a product that streams a huge weight matrix, a wide model)
  int32_t prefer_small;     // run on the small-batch kernels even if M is above their usual limit (the first convolution
                            // of a small batch has twice as many rows as the batch has tokens) or the model is wide
};

// Memory a later kernel will read (weights), fetched towards the caches by workgroups that a kernel with few of its own adds to its grid.
struct Prefetch {
  const void *p;
  uint32_t bytes;           // a multiple of 16; 0: none
  int32_t blocks;
};

struct AttnArgs {
  // Head h owns columns [64h, 64h+64) counted from each of the three base pointers.  Queries of stream i
  // are rows [cu_q[i], cu_q[i+1]) of q (row stride ldq elements), its keys/values rows
  // [cu_kv[i], cu_kv[i+1]) of k and v (row stride ldkv).  Encoder self-attention: one [M, 3d] matrix
  // q | k | v and cu_q == cu_kv.  causal != 0 (needs cu_q == cu_kv): query r sees keys 0..r of its stream.
  const void *q, *k, *v;
  void *out;                // [Mq, d_model]
  int32_t ldq, ldkv;
  const int32_t *cu_q, *cu_kv;   // [B+1] each
  const int32_t *work;      // [n_work][2]: (stream, first query row inside the stream), longest first
  int32_t n_work, n_heads, d_model, B, M;   // M = total query rows
  int32_t Mkv;              // total key rows, 0: M
  int32_t n_work_batch;     // work items of the whole batch where this launch is one lane of it, 0: n_work
  int32_t causal;
  float scale;              // 1/sqrt(64)
  Prefetch pf;
};

struct PrepArgs {
  const void *mel;          // caller's frames [*, n_mels]
  const void *hush;         // [H, n_mels] same dtype as the packed output
  void *packed;             // [total_frames, n_mels]
  const int32_t *cu_frames, *cu_seqlens, *frame_offset, *n_frames;
  int32_t *frame_src, *frame_flags;            // [total_frames]  conv1 row map
  int32_t *tok_src, *tok_flags, *tok_pos;      // [M]             conv2 row map + position index
  int32_t B, n_mels, total_frames, M, mel_is_bf16;
};

// bf16 MFMA path -------------------------------------------------------------------------------
hipError_t launch_gemm_bf16(const GemmArgs &a, AMode amode, Epilogue epi, hipStream_t s);
// small batches (kSmallRows rows) of narrow models: reduction split over the waves, or LayerNorm fused into the operand.  An encoder whose
// whole batch is that small runs all of its products there, so the other streams of such a batch do not change the order of a row's
// sums in any product.  Elsewhere (wf_op_linear, wide models, larger batches) the number of rows has a say in the kernel and with it in
// the last bits: products that fill the chip with tiles, or that few enough rows make faster here, go by their tile counts.
constexpr int32_t kSmallRows = 1024;
bool gemm_small_applies(int32_t M, int32_t N, int32_t K);
bool gemm_slice_applies(int32_t M, int32_t N, int32_t K, bool may_cut);     // products of a few hundred rows of a wide model
bool gemm_slice_reaches(int64_t rows, int64_t values);      // of a convolution: windows that lie in this many rows of so many values
int gemm_small_choice(int32_t M, int32_t N, int32_t K, Epilogue epi, int32_t *bm, int32_t *bn);      // waves that share K, and the tile (diagnostic)
bool gemm_small_few_rows(int32_t M, int32_t N, int32_t K, Epilogue epi);      // plain products of a few rows, any width
hipError_t launch_gemm_small(const GemmArgs &a, AMode amode, Epilogue epi, hipStream_t s);
// products with at most one tile per compute unit, and convolutions whose taps are no whole K steps
bool gemm_pipe_applies(int32_t M, int32_t N, int32_t K);
bool gemm_pipe_tile(int32_t M, int32_t N, int32_t K, int32_t *bm, int32_t *bn);      // the same, with the tile it takes
bool gemm_pipe_logits_applies(int32_t M, int32_t N);      // EPI_BIAS_F32
hipError_t launch_gemm_pipe(const GemmArgs &a, AMode amode, Epilogue epi, hipStream_t s);
// Parts the reduction of a residual product should be cut into (1: none); k_splits * M * N <= kPartialFloats
constexpr int64_t kPartialFloats = 256L * 128 * 128;
int gemm_split_choice(int32_t M, int32_t N, int32_t K);
double gemm_cut_estimate(int32_t M, int32_t N, int32_t K);     // us of that product, cut or not (infinite: not on the pipelined kernel)
// Forms of the non-causal attention (attention_bf16.hip); the choice is a function of the whole batch's sizes
enum AttnForm : int { ATTN_PLAIN = 0, ATTN_KEYS2 = 1, ATTN_KEYS4 = 2, ATTN_KEYS4_TWO_BUFFERS = 3 };
AttnForm attention_form(int32_t n_heads, int32_t B, int64_t M, int64_t Mkv, int64_t n_work);
hipError_t launch_attention_bf16(const AttnArgs &a, hipStream_t s);
// Parts of the residual product in front of a LayerNorm (EPI_PARTIAL): x += part[0] + .. + part[n - 1] + bias first
struct Partials {
  const float *part;        // [n][M][d]
  const float *bias;        // [d]
  int32_t n, M;             // n = 0: none
};
// out[i] = LayerNorm(x[rows[i]]), rows == NULL: x[i].  x is written only with partials and without rows.
hipError_t launch_layernorm(float *x, const int32_t *rows, const float *g, const float *b, void *out, int out_bf16,
                            int32_t M, int32_t d, float eps, hipStream_t s, Partials pt = {}, Prefetch pf = {});
// The first kernel of a call may bring the call's index arrays along in its arguments (at most kInlineInts of them: a launch takes
// 4 KB) and leave them at `dst` for the kernels after it, which spares the call a copy ahead of its first kernel.
constexpr int32_t kInlineInts = 960;
constexpr size_t kLaunchBytes = 4096;          // all arguments of a launch together
struct InlineInts {
  int32_t *dst;             // device, n ints
  const int32_t *src;       // host
  int32_t n;                // 0: the arrays are on the device already
};
// Threads of the packing kernel: one per eight features of a frame, one per token.
inline int64_t prep_threads(int64_t total_frames, int64_t n_mels, int64_t tokens) { return total_frames * (n_mels / 8) + tokens; }
// Do a batch's n_ints index values travel in the packing kernel's arguments?  That form counts its threads in 32 bits.
inline bool prep_takes_ints(int64_t n_ints, int64_t threads) { return n_ints <= kInlineInts && threads < ((int64_t)1 << 31); }
// (a.cu_frames, cu_seqlens, frame_offset and n_frames are the first 4 (B + 1) of the ints, in that order)
hipError_t launch_prep(const PrepArgs &a, int packed_bf16, hipStream_t s, InlineInts in = {});
// x[r, :] = table[tok[r], :] + pos[pos_idx[r], :]  (fp32 out; table bf16 or fp32, pos fp32); tok and pos_idx are the first 2 rows
// of the ints, in that order
hipError_t launch_embed(const void *table, int table_bf16, const float *pos, const int32_t *tok, const int32_t *pos_idx,
                        float *x, int32_t rows, int32_t d, hipStream_t s, InlineInts in = {});
int attention_q_tile();     // query rows per attention work item
int gemm_dl_tile_map(int32_t M, int32_t N, int32_t bm, int32_t bn, int32_t *units, int32_t cap);   // diagnostic, host only
void gemm_tile_choice(int32_t M, int32_t N, int32_t *bm, int32_t *bn);                                                  // diagnostic, host only
int gemm_kernel_choice(int32_t M, int32_t N, int32_t K, Epilogue epi, int32_t *bm, int32_t *bn);                        // diagnostic, host only

// fp32 debug path ------------------------------------------------------------------------------
hipError_t launch_gemm_f32(const GemmArgs &a, AMode amode, Epilogue epi, hipStream_t s);
hipError_t launch_attention_f32(const AttnArgs &a, hipStream_t s);

// thread-local error text behind wf_last_error(), shared by all translation units
int set_error(int code, const char *fmt, va_list ap);
char *error_buffer();

// one-time per-process kernel attribute setup (dynamic LDS limits)
hipError_t init_kernels();

}  // namespace wf
