// Shared declarations of the early-exit decode library: types, memory layouts, launch interfaces.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "ee_decode.h"

namespace ee {

typedef __bf16 bf16_t;
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

// ---------------------------------------------------------------------------------------------------
// Error reporting (host)
// ---------------------------------------------------------------------------------------------------
void set_error(const char* fmt, ...);
#define EE_FAIL(code, ...)      \
  do {                          \
    ee::set_error(__VA_ARGS__); \
    return (code);              \
  } while (0)
#define EE_HIP(expr)                                                                        \
  do {                                                                                      \
    hipError_t e_ = (expr);                                                                 \
    if (e_ != hipSuccess) EE_FAIL(EE_ERR_HIP, "%s failed: %s", #expr, hipGetErrorString(e_)); \
  } while (0)

// ---------------------------------------------------------------------------------------------------
// Layouts of the bf16 path.
//
// XT ("operand tiles"): a [rows m][cols k] bf16 activation matrix stored in the order in which the
//   32x32x16 MFMA wants its second operand: [m/32][k/16][lane][8] with lane = (m%32) + 32*((k%16)/8) and
//   element k%8, so a wavefront fetches one 32x16 operand tile as 1 KiB of consecutive bytes.
// The fp32 residual stream is plain row-major [Mpad][d].  The output and down projections do not add into it:
//   each contraction slice writes its partial result to a slice of its own ([slices][Mpad][d], plain stores), and
//   the normalisation kernel that follows sums the slices in slice order, adds them to the residual row and
//   normalises it.  (Up to eight rows, gemm_small.hip, they do: a workgroup has whole contractions and adds each to its element
//   of the residual rows, and activations are plain rows.)  No float atomics anywhere, so the bf16 path is reproducible bit for bit.
// ---------------------------------------------------------------------------------------------------
__host__ __device__ inline size_t xt_index(int m, int k, int K) {
  return ((size_t)(m >> 5) * (size_t)(K >> 4) + (size_t)(k >> 4)) * 512 + (size_t)((((k >> 3) & 1) << 5) + (m & 31)) * 8 +
         (size_t)(k & 7);
}
__host__ __device__ inline int round_up(int x, int to) { return (x + to - 1) / to * to; }

// Packed weight row order: packed tile `nt`, row r (0..31) holds plain output row
//   f_lo(nt, r%16) + (r/16) * pair_stride,   f_lo = (nt / tpb) * 2*pair_stride + 16*(nt % tpb) + r%16,  tpb = pair_stride/16.
// pair_stride 16 is the identity order.
__host__ __device__ inline int packed_row_lo(int nt, int r16, int pair_stride) {
  const int tpb = pair_stride >> 4;
  return (nt / tpb) * 2 * pair_stride + ((nt % tpb) << 4) + r16;
}

// ---------------------------------------------------------------------------------------------------
// Per-iteration device state
// ---------------------------------------------------------------------------------------------------
struct IterState {
  int32_t* status;            // [B] sticky exit status
  int32_t* exit_layer;        // [B]
  int32_t* n_exited;          // [1]
  int32_t* done;              // [1] 1 once every sequence of the batch is accepted
  int32_t* batch_exit_layer;  // [1] output_layer of Algorithm 1
};

// Compaction of the rows that are still active (per-sequence exit at more than 128 rows): position p < *n_active of a
// compacted operand holds batch row perm[p]; cpos is the inverse map.
// The map is rebuilt after every exit check and is constant inside a layer.
struct RowMap {
  int32_t* perm;      // [Mpad]; nullptr = no compaction (every row, in place)
  int32_t* cpos;      // [Mpad] batch row -> position, -1 for a sequence that has left
  int32_t* n_active;  // [1]
};

// Epilogue parameter blocks ---------------------------------------------------------------------------
struct QkvEpi {                 // rotary embedding + paged cache write (+ q output)
  float* q;                     // [M][d] fp32 or nullptr (KV filling)
  void* k_pool;                 // layer base of the pools ([num_blocks][H][16][dh])
  void* v_pool;
  const int32_t* context_lens;  // [M]
  const int32_t* block_tables;  // [M][max_blocks]
  const int32_t* row_table;     // nullptr, or [M]: row m uses row row_table[m] of block_tables
  const int32_t* fill_from;     // nullptr, or [M]: only rows with fill_from[m] + fill_lead < layer are written (KV filling, which has no q)
  int fill_from_stride;         // 1 = per row, 0 = one value for the whole batch
  int fill_lead;                // layers behind fill_from that have been cached as well
  int layer;
  int max_blocks, n_heads, head_dim, d_model;
  float rope_theta;
  const float2* rope;           // [M][dh/2] (cos, sin) of the rotary angles at context_lens[m] (rope_theta > 0)
  int num_blocks;               // blocks per layer of the pools: a slot whose block id or position is out of range is not written
  int table_rows;               // rows of block_tables (the batch size): a row_table entry outside 0..table_rows-1 is read as 0
};
// Whether KV filling has nothing to do for row m (no row of other projections).
__device__ inline bool kv_filled(const QkvEpi& e, int m) {
  return e.fill_from && !(e.fill_from[(size_t)m * e.fill_from_stride] + e.fill_lead < e.layer);
}
struct AccEpi {                 // residual update
  float* h;                     // fp32 path and gemm_small.hip: the residual stream [M][n_out], added to in place (one contributor per element).
                                // else: partial results [slices][Mpad][n_out]; slice s receives the sum over the
                                // s-th part of the contraction (operand row m -> row m: compacted operands stay compacted)
  int Mpad;                     // row count of a slice, or 0 (added in place)
  int n_out;
  const int32_t* skip;          // added in place: nullptr, or [M]: rows with skip[m] != 0 keep their hidden state
  const float* h_in;            // fp32 path: nullptr (added in place), or what is added to, with h the result
};
struct GateUpEpi {              // act = silu(gate) * up
  void* act;                    // XT bf16 [Mpad][f] (bf16 path), plain bf16 [M][f] (gemm_small.hip) or plain float [M][f]
  int d_ffn;
};
struct LmEpi {                  // per-tile softmax statistics of the scaled logits
  float4* partials;             // [M][n_parts]: {max logit (unscaled), sum exp(scale*(z - max)), 2nd max, arg max as int bits}
  float* logits;                // fp32 path: [M][vocab] logits of the row times the gains, short of
  float* row_scale;             // [M] the row's 1 / sqrt(mean square + eps); bf16 path: nullptr, both
  int n_parts;
  int vocab;
  float scale;                  // logit_scale * layer
  const int32_t* perm;          // nullptr, or [M]: operand row m is batch row perm[m] (compacted operand)
};

// ---------------------------------------------------------------------------------------------------
// Launchers (each enqueues on `st`).  A launch carries a predicate on a device word: its kernels return at once
// unless (*flag != 0) == run_when.  The layer loop runs while the all-exited flag is 0, KV filling once it is 1.
// ---------------------------------------------------------------------------------------------------
struct Pred {
  const int32_t* flag;  // nullptr = always run
  int run_when;         // run when (*flag != 0) == run_when
};

// misc.hip
void launch_copy_f32(const float* src, float* dst, size_t n, hipStream_t st);
void launch_rope_table(const int32_t* context_lens, float2* table, int B, int head_dim, float theta, hipStream_t st);
struct GainTable {
  const void* g[EE_MAX_LAYERS];
};
// Optional second job of a normalisation launch (confidence measures that need no LM head, Section 2.1):
// dots[m] = sum_k h[m][k] * other, where other is the previous hidden state (per_row: [Mpad][d], the similarity
// measure) or one weight row shared by all rows ([d], the dedicated classifier); snapshot, if set, receives h
// (it may be the buffer `other` points to: every element is read before it is written, by the same thread).
struct RowDot {
  const float* other;
  float* snapshot;
  float* dots;      // [Mpad]
  int per_row;
};
// Rebuilds the row map from the status words (active rows keep their order).
void launch_compact(const int32_t* status, int B, const RowMap& rm, Pred pred, hipStream_t st);
// Residual update + RMSNorm of the bf16 path, one workgroup per batch row:
//   h[m] += y[0][p] + y[1][p] + .. (slice order; p = m, or cpos[m] with a row map; not for rows that have left),
//   rowsq_out[m] = sum_k h[m][k]^2, and for each gain j: x[j] row = bf16(h * rsqrt(rowsq/d + eps) * gain[j]) in
//   operand-tile order (at row m, or at position cpos[m] of a compacted operand, which is zero from *n_active on).
struct NormArgs {
  const float* h_in;      // [rows][d]
  float* h_out;           // nullptr (nothing to add) or the same buffer
  const float* y;         // [S][Mpad][d]
  int S;
  const int32_t* skip;    // nullptr, or [B] status words: rows with skip[m] != 0 have left and keep their hidden state
  RowMap rm;              // perm == nullptr: no compaction
  const bf16_t* gain[2];
  bf16_t* x[2];           // nullptr = unused
  int compacted[2];
  float* rowsq_out;       // nullptr or [Mpad]
  RowDot rd;
  float eps;
  int B, Mpad, d;
};
void launch_finish_norm(const NormArgs& a, Pred pred, hipStream_t st);
// Start of an iteration: state reset, embedding (residual rows [B][d]), rotary table, and on the bf16 path the first
// layer's operand x (RMSNorm with `gain`), the rows' sums of squares and the identity row map.
struct BeginArgs {
  IterState s;
  float* conf_out;        // nullptr or [n_layers][B]
  const int32_t* context_lens;
  const int32_t* tokens;
  float2* rope;
  const bf16_t* embed;    // bf16 path
  const float* embed_f32; // fp32 path
  const bf16_t* gain;
  float* h;
  float* snapshot;        // nullptr, or a copy of h (h_0 of the similarity measure)
  bf16_t* x;
  float* rowsq_out;
  RowMap rm;              // perm == nullptr: none
  float theta, eps;
  int B, Mpad, d, vocab, n_layers, head_dim;
};
void launch_iter_begin(const BeginArgs& a, hipStream_t st);
void launch_iter_begin_f32(const BeginArgs& a, hipStream_t st);
// KV filling: x slab of layer l = bf16(RMSNorm(h; gains.g[l-1])) for every layer some row needs (fill_from + fill_lead < l).
// rope.table != nullptr: the same launch also tabulates the rotary angles.
struct RopeJob {
  const int32_t* context_lens;
  float2* table;
  int head_dim;
  float theta;
};
void launch_fill_prep(const float* h, const GainTable& gains, int n_layers, bf16_t* x_slabs, float eps,
                      const int32_t* fill_from, int fill_from_stride, int fill_lead, int B, int Mpad, int d, Pred pred, const RopeJob& rope,
                      hipStream_t st);
struct CombineArgs {
  const float4* partials;
  int n_parts;
  int B;
  int layer;           // 1-based; 0 = final token selection (no status update)
  float scale;         // logit_scale * layer
  float threshold;
  int conf_mode;
  const int32_t* forced_exit_layer;
  IterState s;
  int32_t* argmax_out;  // [B] or nullptr
  float* conf_out;      // [B] or nullptr
  const int32_t* left;  // nullptr, or [B]: rows with left[m] != 0 are not touched (per-sequence exit: token and state stay)
};
void launch_combine(const CombineArgs& a, Pred pred, hipStream_t st);
// The same where the predicate holds, and always dst[m][..] = src[m][..] over d floats for every row (dst may be nullptr).
void launch_combine_copy(const CombineArgs& a, Pred pred, const float* src, float* dst, int d, hipStream_t st);
// Exit decision from a measure that is one dot product per row (conf_mode 2: cosine of consecutive hidden
// states = dots / sqrt(sq_a * sq_b); conf_mode 3: logistic function of dots * rsqrt(sq_b / d + eps) + bias[0],
// the classifier's unit applied to the hidden state at unit root mean square).
struct DecideArgs {
  const float* dots;   // [B] (bf16 path)
  const float* sq_a;   // [B] squared norms (conf_mode 2; bf16 path)
  const float* sq_b;
  const float* bias;   // device, this layer's bias (conf_mode 3)
  int d;               // width of the hidden state
  float eps;
  int B;
  int layer;
  float threshold;
  int conf_mode;
  const int32_t* forced_exit_layer;
  IterState s;
  float* conf_out;
};
void launch_decide(const DecideArgs& a, Pred pred, hipStream_t st);
// fp32 path: the decision of every row from its own logits [B][vocab] and their scale [B] (LmEpi; conf_mode 0, 1; layer 0: token
// selection), one launch; dst as in launch_combine_copy.
void launch_head_decide_f32(const float* logits, const float* row_scale, int vocab, const CombineArgs& a, Pred pred, const float* src, float* dst, int d,
                            hipStream_t st);
// fp32 path: the sums of a one-dot-product measure and the decision from them; other is the previous hidden state [B][d]
// (per_row; it becomes h) or one row [d].
void launch_measure_decide_f32(const float* h, float* other, int per_row, const DecideArgs& a, Pred pred, hipStream_t st);
// The exit decision of layer i may ride along with the QKV projection launch of layer i+1 instead of taking a
// launch of its own (see launch_gemm_qkv_bf16): n_wg leading workgroups of that launch (a multiple of 8) take it.
// kind 1: softmax-response measures, workgroup m < a.B runs combine_row for batch row m.
// kind 2: one-dot-product measures, workgroup 0 runs decide_from_dot for every row.  n_wg == 0: none.
struct CombineJob {
  CombineArgs a;
  DecideArgs d;
  int kind;
  int n_wg;
};

// pack.hip
void launch_pack_weight(const bf16_t* w, int n_out, int n_in, int pair_stride, bf16_t* packed, hipStream_t st);

// gemm_mfma.hip (bf16 path).  w: packed; x: XT [Mpad][K].  tiles [tile_begin, tile_begin + n_tiles).
struct GemmShape {
  const void* w;
  const void* x;
  int K;            // contraction length
  int M;            // valid rows
  int tile_begin;   // first packed 32-row tile
  int n_tiles;      // tiles to compute
  int pair_stride;  // row order of the packed matrix
  int unused_;      // (kept so that aggregate initialisers stay positional)
  // QKV projection with one batch tile: the last split_tiles tiles (tiles without a rotation: V) are each computed
  // by two workgroups, 16 of the 32 output rows each, dispatched first; see gemm_mfma.hip.  0 = off.
  int split_tiles;
  // Block kernel only: nullptr, or the device-side number of valid operand rows (<= M).  Row blocks beyond it
  // return at once, rows beyond it are not written.
  const int32_t* n_rows_dev;
  int grid_y;   // set by the launcher (tiled kernel): batch chunks x contraction slices per group of output tiles
  int keep;     // set by the launcher (tiled kernel): weights stay cached
  int even_wgs; // set by the launcher (tiled kernel): > 0 = the tiles are dealt out evenly over this many workgroups
};
// Whether a projection of more than 128 rows onto n_tiles packed tiles takes a compacted operand (n_rows_dev and the epilogues' perm):
// whole groups of four tiles.
bool gemm_bf16_takes_compacted(int n_tiles);
// One-time host-side set-up of the projection kernels (function attributes) that the first launch would otherwise do.
void gemm_bf16_prepare();
// with_combine != nullptr (only where gemm_qkv_carries_combine(M) holds): the launch also takes the exit decision
// of the previous layer.  The projection then runs SPECULATIVELY when that decision ends the iteration (its
// predicate word may or may not show the new value yet): what it caches for its layer is what KV filling
// (Section 3.2) caches there, and KV filling starts one layer further on.
void launch_gemm_qkv_bf16(const GemmShape& g, const QkvEpi& e, Pred pred, hipStream_t st,
                          const CombineArgs* with_combine = nullptr, const DecideArgs* with_decide = nullptr);
bool gemm_qkv_carries_combine(int M);
// Contraction slices the accumulate launch of this shape writes (the launch below uses exactly this many).
int gemm_acc_slices(int M, int n_tiles, int K);
// Rows of partial results (all slices) to set aside for accumulate launches of up to M rows onto n_tiles tiles over a contraction of K.
size_t gemm_acc_rows(int M, int n_tiles, int K);
void launch_gemm_acc_bf16(const GemmShape& g, const AccEpi& e, Pred pred, hipStream_t st);
void launch_gemm_gateup_bf16(const GemmShape& g, const GateUpEpi& e, Pred pred, hipStream_t st);
void launch_gemm_lm_bf16(const GemmShape& g, const LmEpi& e, Pred pred, hipStream_t st);
// KV filling over layers first..n in one launch: per-layer weights / x slabs / pools.
struct FillLayers {
  const void* w_qkv[EE_MAX_LAYERS];
};
void launch_gemm_kvfill_bf16(const FillLayers& fl, int n_layers, const bf16_t* x_slabs, size_t x_slab_elems,
                             size_t pool_layer_elems, const GemmShape& g, const QkvEpi& e, Pred pred, hipStream_t st);

// gemm_small.hip (bf16 path, up to eight rows).  w: packed.  QKV, gate/up and the LM head take the residual rows [M][K] and multiply
// RMSNorm(x; gain); the output projection takes float rows, the down projection bf16 rows [M][K], and both add to the residual rows in place
// (AccEpi as on the fp32 path).  gate/up leaves plain rows [M][d_ffn].
struct SmallShape {
  const void* w;
  const void* x;
  const bf16_t* gain;
  float eps;
  int K, M;
  int pair_stride;
  int whole, halves;   // output tiles that are finished whole, and 16-row halves of the tiles behind them
  int wgs;             // set by the launcher
};
// Whether they take an iteration of B rows (head_tiles: of the LM heads of its exit checks, 0 without), and an exit check on its own.
bool gemm_small_takes(int B, int d, int head_tiles);
bool gemm_small_takes_check(int B, int d, int head_tiles);
void launch_small_qkv(const SmallShape& g, const QkvEpi& e, Pred pred, hipStream_t st, const CombineArgs* with_combine);
// The first layer's, which begins the iteration as well (x unused; the embedding table starts on 16 bytes).
void launch_small_begin_qkv(const BeginArgs& begin, const SmallShape& g, const QkvEpi& e, hipStream_t st);
void launch_small_oproj(const SmallShape& g, const AccEpi& e, Pred pred, hipStream_t st);
void launch_small_gateup(const SmallShape& g, const GateUpEpi& e, Pred pred, hipStream_t st);
void launch_small_down(const SmallShape& g, const AccEpi& e, Pred pred, hipStream_t st);
void launch_small_lm(const SmallShape& g, const LmEpi& e, Pred pred, hipStream_t st);

// gemm_simple.hip (fp32 path).  w: plain [n_out][K]; x: plain [M][K]; QKV, gate/up and the LM head take the residual rows
// as x and multiply RMSNorm(x; gain), the accumulate projections take x as it is (gain unused).
struct SimpleShape {
  const float* w;
  const float* x;
  const float* gain;
  float eps;
  int K, M;
  int row_begin;    // first output row
  int n_rows;       // output rows to compute (even)
  int pair_stride;  // rows (f, f + pair_stride) are computed together
  // gate/up (of up to 256 channels) behind attention that has multiplied by the columns of the output projection, head by head: the operand is
  // x + parts[0] + parts[1] + .. ([n_parts][M][K]; rows with left[m] != 0: x alone), and is left in x_out [M][K].  parts == nullptr: x.
  const float* parts;
  int n_parts;
  float* x_out;
  const int32_t* left;
};
// An exit decision on materialised logits that rides along with a projection launch (one workgroup per row, in front).
struct SimpleDecision {
  CombineArgs a;
  const float* logits;
  const float* row_scale;
  int vocab;
  int n_wg;   // set by the launch
};
void launch_simple_qkv(const SimpleShape& g, const QkvEpi& e, Pred pred, hipStream_t st, const SimpleDecision* with = nullptr);
// The first layer's, which begins the iteration (launch_iter_begin_f32) as well: g.x is the embedding table.
// Up to 256 channels.
void launch_simple_begin_qkv(const BeginArgs& begin, const SimpleShape& g, const QkvEpi& e, hipStream_t st);
// The LM head in the launch of the next layer's QKV projection, or of KV filling (each by its own predicate: with a measure that has no head both
// run).  Up to 256 rows and 256 channels.
void launch_simple_head_qkv(const SimpleShape& gh, const LmEpi& eh, const SimpleShape& g, const QkvEpi& e, Pred pred, hipStream_t st);
void launch_simple_acc(const SimpleShape& g, const AccEpi& e, Pred pred, hipStream_t st);
void launch_simple_gateup(const SimpleShape& g, const GateUpEpi& e, Pred pred, hipStream_t st);
void launch_simple_lm(const SimpleShape& g, const LmEpi& e, Pred pred, hipStream_t st);
// KV filling over layers 1..n_layers in one launch (e.fill_from set; e.k_pool / e.v_pool: pools of layer 1).
struct SimpleFill {
  FillLayers layers;
  GainTable gains;
  size_t pool_layer_bytes;
};
void launch_simple_kvfill(const SimpleFill& fill, int n_layers, const SimpleShape& g, const QkvEpi& e, Pred pred, hipStream_t st);
void launch_simple_head_kvfill(const SimpleShape& gh, const LmEpi& eh, Pred ph, const SimpleFill& fill, int n_layers, const SimpleShape& g, const QkvEpi& e,
                               Pred pred, hipStream_t st);

// attention.hip
// Block ids and positions come from device memory the caller filled in; the kernels never let them reach outside
// the pools or the block table (the result for such a sequence is unspecified, the access is not).
__host__ __device__ inline int safe_block(int blk, int num_blocks) { return (unsigned)blk < (unsigned)num_blocks ? blk : 0; }
__host__ __device__ inline int safe_row(int row, int n_rows) { return (unsigned)row < (unsigned)n_rows ? row : 0; }

// Block-table entries per sequence that the attention kernels stage in LDS (contexts up to 262144 tokens).  The
// entry points check ee_batch.max_blocks against it before anything is enqueued.
constexpr int kAttnMaxBlocks = 16384;

struct AttnArgs {
  const float* q;               // [B][H*dh] fp32, rotary applied
  const void* k_pool;           // layer base
  const void* v_pool;
  const int32_t* context_lens;  // attends positions 0..context_lens[b] inclusive
  const int32_t* block_tables;
  int max_blocks, B, n_heads, head_dim;
  void* out;                    // fp32 plain [B][H*dh], or XT bf16 [Mpad][H*dh]
  int out_xt;                   // 1: XT bf16
  const int32_t* skip;          // nullptr, or [B]: sequences with skip[b] != 0 are not attended (they have left)
  const int32_t* row_table;     // nullptr, or [B]: row b uses row row_table[b] of block_tables
  const int32_t* out_pos;       // nullptr, or [B]: the result of sequence b goes to row out_pos[b] of out (compacted operand)
  int num_blocks;               // blocks per layer of the pools: a block id outside 0..num_blocks-1 is read as block 0
  // Few (sequence, head) pairs and long contexts: split_parts > 1 workgroups share one pair, each over a contiguous
  // range of the sequence's blocks; their partial results (running maximum, sum and unnormalised output:
  // head_dim + 2 floats each) meet in split_ws [B][H][split_parts][head_dim + 2] and a second launch merges them in
  // part order.  1 (or split_ws == nullptr) = one workgroup per pair.  Not with row_table.
  float* split_ws;
  int split_parts;
};
int launch_attention(const AttnArgs& a, int dtype, Pred pred, hipStream_t st);
// fp32 path: attention of one workgroup per (sequence, head) that multiplies its result by the head's columns of the output projection w_o
// [d][d] (parts [H][B][d], see SimpleShape), and takes the exit decision `with` of the layer before, if there is one, in leading workgroups.
void launch_attention_f32(const AttnArgs& a, const float* w_o, float* parts, Pred pred, hipStream_t st, const SimpleDecision* with);
// Host-side set-up for the current device (function attributes) that the first launch over prompt rows would otherwise do.
void attention_prepare();
// How many workgroups should share one (sequence, head) pair for this batch, and the floats of split_ws that takes.
int attn_split_parts(int B, int n_heads, int max_blocks);
inline size_t attn_split_floats(int B, int n_heads, int head_dim, int parts) {
  return parts > 1 ? (size_t)B * n_heads * parts * (head_dim + 2) : 0;
}
constexpr int kAttnMaxSplit = 8;
constexpr int kAttnSplitMaxPairs = 64;   // (sequence, head) pairs up to which the split form is used

}  // namespace ee
