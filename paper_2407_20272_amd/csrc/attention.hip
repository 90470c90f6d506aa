// Single-query attention over the paged KV cache (the attention inside one layer of the decode step).
//
// Bandwidth-bound: every cached K and V value of the sequence is read once (about one flop per byte), so the
// kernel is organised around the reads.  One workgroup owns one (sequence, head); its four wavefronts take the
// sequence's 16-token blocks round-robin.  A block of one head is 16 tokens x head_dim values of consecutive
// memory (4 KiB for bf16 x 128), which a wavefront fetches with 16-byte loads per lane, every load instruction
// covering 1 KiB of consecutive bytes; the next block's K and V are in flight while the current one is reduced.
// Lanes that share a token add their partial dot products with a butterfly; every group of lanes keeps its own
// running softmax (max, sum, weighted V) over the tokens it sees, and the groups, then the wavefronts, are merged
// once at the end.  No score is ever written to memory.
#include <atomic>
#include <type_traits>

#include "ee_common.h"
#include "ee_epilogue.h"
#include "ee_decide.h"

namespace ee {
namespace {

constexpr int NW = 4;
constexpr float NEG_BIG = -1.0e30f;

template <class T>
struct Elems;
template <>
struct Elems<float> {
  static constexpr int N = 4;
  __device__ static void unpack(const uint4& v, float (&f)[4]) {
    f[0] = __uint_as_float(v.x);
    f[1] = __uint_as_float(v.y);
    f[2] = __uint_as_float(v.z);
    f[3] = __uint_as_float(v.w);
  }
};
template <>
struct Elems<bf16_t> {
  static constexpr int N = 8;
  __device__ static void unpack(const uint4& v, float (&f)[8]) {
    f[0] = __uint_as_float(v.x << 16);
    f[1] = __uint_as_float(v.x & 0xffff0000u);
    f[2] = __uint_as_float(v.y << 16);
    f[3] = __uint_as_float(v.y & 0xffff0000u);
    f[4] = __uint_as_float(v.z << 16);
    f[5] = __uint_as_float(v.z & 0xffff0000u);
    f[6] = __uint_as_float(v.w << 16);
    f[7] = __uint_as_float(v.w & 0xffff0000u);
  }
};

// Sum over the LPT lanes that share a token; every lane of the group ends up with the total.
// Within a 16-lane row the butterfly runs on the DPP cross-lane network (quad permutes, half-row and row
// mirrors); only a 32-lane group needs one LDS-crossbar shuffle on top.
template <int LPT>
__device__ inline float group_sum(float v) {
  v += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0xB1, 0xF, 0xF, true));   // quad_perm [1,0,3,2]
  v += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x4E, 0xF, 0xF, true));   // quad_perm [2,3,0,1]
  v += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x141, 0xF, 0xF, true));  // row_half_mirror
  if constexpr (LPT >= 16)
    v += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x140, 0xF, 0xF, true));  // row_mirror
  if constexpr (LPT >= 32) v += __shfl_xor(v, 16);
  return v;
}

// 16 bytes of the cache, read once per iteration and never again: a streaming (non-temporal) load, which leaves
// the caches to the data that is reused.
template <class T>
__device__ inline uint4 load_stream(const T* p) {
  typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
  const u32x4 v = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(p));
  return make_uint4(v.x, v.y, v.z, v.w);
}

// Sixteen bytes of zeros (never written; not const, so that it lives in the same address space as the cache).
// A lane whose token lies after the sequence's last position reads its V values from here instead of from the
// cache: what an earlier owner of the block, or nobody, left in those slots is weighted with zero, and 0 * NaN
// would still be NaN.  The choice is made on the ADDRESS; the load itself stays unconditional.
__device__ uint4 k_zero16;

constexpr int TABLE_LDS_MAX = kAttnMaxBlocks;   // block-table entries staged in LDS

// What attention of the float path may do besides (launch_attention_f32).
struct NoOproj {};
struct Oproj {
  const float* w;
  float* parts;
  SimpleDecision job;   // n_wg: rows of leading workgroups (0: no decision)
};

template <class T, int DH, bool OUT_XT, bool SPLIT, class Op, class Skip>
__device__ __forceinline__ void attn_decode(const AttnArgs& a, const Op& op, int b, Skip skip) {
  constexpr bool OPROJ = std::is_same<Op, Oproj>::value;
  constexpr int EPL = Elems<T>::N;         // values per 16-byte lane load
  constexpr int LPT = DH / EPL;            // lanes per token
  constexpr int TPL = 64 / LPT;            // tokens per wavefront load
  constexpr int LPB = 16 / TPL;            // loads per 16-token block
  static_assert(LPT >= 8 && LPT <= 32, "unsupported head_dim for this element type");

  const int head = blockIdx.x;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int sub = lane % LPT;              // which EPL-wide slice of the head this lane holds
  const int grp = lane / LPT;              // which token of a load this lane sees
  const int32_t* table = a.block_tables + (size_t)(a.row_table ? safe_row(a.row_table[b], a.B) : b) * a.max_blocks;

  extern __shared__ int32_t tbl[];
  if constexpr (OPROJ)   // (what the launch was given is fetched ahead of the predicate, not in a second trip behind it)
    asm volatile("" ::"s"(a.q), "s"(a.k_pool), "s"(a.v_pool), "s"(a.context_lens), "s"(a.block_tables), "s"(a.max_blocks), "s"(a.num_blocks), "s"(op.w));
  if (skip()) return;
  // Everything the first K/V load needs is requested before any of it is waited for: the context length, the
  // start of the block-table row (its width is known without the length) and q: one memory round trip, not
  // three in a row.
  const int t0 = (int)threadIdx.x < a.max_blocks ? safe_block(table[threadIdx.x], a.num_blocks) : 0;
  const int len = a.context_lens[b];
  int left = 0;
  if constexpr (OPROJ) {
    if (a.skip) left = op.job.n_wg ? left_before(op.job.a.s, b, op.job.a.layer) : ctl_load(a.skip + b);
  } else {
    left = a.skip ? ctl_load(a.skip + b) : 0;
  }
  const int out_row = a.out_pos ? a.out_pos[b] : b;
  float q[EPL];
  {
    const float* qp = a.q + ((size_t)b * a.n_heads + head) * DH + sub * EPL;
#pragma unroll
    for (int i = 0; i < EPL; ++i) q[i] = qp[i];
  }
  if (left != 0) return;   // the sequence has left at an earlier layer: nothing to attend, nothing read
  // positions 0..p inclusive, never beyond the block table's width
  const int n_ctx = min(len + 1, a.max_blocks * 16);
  const int n_blocks = (n_ctx + 15) >> 4;

  // The sequence's block table goes to LDS once (max_blocks entries of dynamic LDS).  The block loop must not
  // read it from memory: the wait for such a read would also wait for every K/V load issued before it.
  if ((int)threadIdx.x < a.max_blocks) tbl[threadIdx.x] = t0;
  for (int i = threadIdx.x + blockDim.x; i < n_blocks; i += blockDim.x) tbl[i] = safe_block(table[i], a.num_blocks);

  // q slice, pre-scaled so that exp2 can be used: softmax(x) = 2^(x*log2 e)
  {
    const float sc = 1.4426950408889634f / sqrtf((float)DH);
#pragma unroll
    for (int i = 0; i < EPL; ++i) q[i] *= sc;
  }
  __syncthreads();

  float m_run = NEG_BIG, l_run = 0.0f, o[EPL];
#pragma unroll
  for (int i = 0; i < EPL; ++i) o[i] = 0.0f;

  const size_t head_off = (size_t)head * 16 * DH;             // elements, inside a block
  const size_t block_elems = (size_t)a.n_heads * 16 * DH;
  const T* kbase = reinterpret_cast<const T*>(a.k_pool) + head_off + (size_t)grp * DH + sub * EPL;
  const T* vbase = reinterpret_cast<const T*>(a.v_pool) + head_off + (size_t)grp * DH + sub * EPL;

  struct Blk {
    uint4 k[LPB], v[LPB];
  };
  const T* zero_src = reinterpret_cast<const T*>(&k_zero16);
  auto fetch = [&](Blk& x, int lb) {
    const int phys = tbl[lb];
    const size_t off = (size_t)phys * block_elems;
#pragma unroll
    for (int i = 0; i < LPB; ++i) {
      x.k[i] = load_stream(kbase + off + (size_t)i * TPL * DH);
      x.v[i] = load_stream(lb * 16 + i * TPL + grp < n_ctx ? vbase + off + (size_t)i * TPL * DH : zero_src);
    }
  };
  auto consume = [&](const Blk& x, int lb) {
    float s[LPB];
    float m_new = m_run;
#pragma unroll
    for (int i = 0; i < LPB; ++i) {
      float kf[EPL];
      Elems<T>::unpack(x.k[i], kf);
      float d = 0.0f;
#pragma unroll
      for (int e = 0; e < EPL; ++e) d = fmaf(q[e], kf[e], d);
      d = group_sum<LPT>(d);
      const int tok = lb * 16 + i * TPL + grp;
      s[i] = tok < n_ctx ? d : NEG_BIG;
      m_new = fmaxf(m_new, s[i]);
    }
    const float alpha = __builtin_amdgcn_exp2f(m_run - m_new);
    l_run *= alpha;
#pragma unroll
    for (int e = 0; e < EPL; ++e) o[e] *= alpha;
#pragma unroll
    for (int i = 0; i < LPB; ++i) {
      const int tok = lb * 16 + i * TPL + grp;
      const float p = tok < n_ctx ? __builtin_amdgcn_exp2f(s[i] - m_new) : 0.0f;
      l_run += p;
      float vf[EPL];
      Elems<T>::unpack(x.v[i], vf);
#pragma unroll
      for (int e = 0; e < EPL; ++e) o[e] = fmaf(p, vf[e], o[e]);
    }
    m_run = m_new;
  };

  // Two blocks of this wavefront in flight at any time.  The steady loop has no conditional load: a load under
  // a condition makes the compiler wait for every outstanding load where the paths join, which would drain
  // the stream once per block; the scheduling fences keep each block's loads together ahead of the arithmetic.
  // SPLIT: this workgroup is part blockIdx.z of gridDim.z and walks a contiguous range of the sequence's blocks
  // (possibly empty: a short sequence in a wide table); otherwise all of them.
  int lb_begin = 0, lb_end = n_blocks;
  if constexpr (SPLIT) {
    const int per = (n_blocks + (int)gridDim.z - 1) / (int)gridDim.z;
    lb_begin = min(n_blocks, (int)blockIdx.z * per);
    lb_end = min(n_blocks, lb_begin + per);
  }
  Blk A, B;
  int lb = lb_begin + wave;
  if (lb < lb_end) fetch(A, lb);
  if (lb + NW < lb_end) fetch(B, lb + NW);
  // The head's columns of this workgroup's rows of the output projection, LPT lanes a row, are on their way while the keys are
  // looked at.
  constexpr int RPI = NW * TPL, AHEAD = OPROJ ? 64 / RPI : 1;   // (256 channels at most: 64 rows a workgroup)
  float4 wo[AHEAD];
  [[maybe_unused]] const float* wrow = nullptr;
  [[maybe_unused]] int d_out = 0, rows = 0;
  if constexpr (OPROJ) {
    d_out = a.n_heads * DH;
    rows = d_out / (int)gridDim.z;   // (whole iterations of RPI rows: d_out is a multiple of 64)
    if (op.w) {
      wrow = op.w + (size_t)(blockIdx.z * rows + wave * TPL + grp) * d_out + head * DH + sub * EPL;
#pragma unroll
      for (int i = 0; i < AHEAD; ++i) wo[i] = *reinterpret_cast<const float4*>(wrow + (size_t)min(i * RPI, rows - RPI) * d_out);
    }
  }
  for (; lb + 3 * NW < lb_end; lb += 2 * NW) {
    consume(A, lb);
    __builtin_amdgcn_sched_barrier(0);
    fetch(A, lb + 2 * NW);
    __builtin_amdgcn_sched_barrier(0);
    consume(B, lb + NW);
    __builtin_amdgcn_sched_barrier(0);
    fetch(B, lb + 3 * NW);
    __builtin_amdgcn_sched_barrier(0);
  }
  // at most three blocks left: lb (in A), lb + NW (in B), lb + 2 NW (not fetched yet)
  if (lb < lb_end) {
    consume(A, lb);
    const bool third = lb + 2 * NW < lb_end;
    if (third) fetch(A, lb + 2 * NW);
    if (lb + NW < lb_end) consume(B, lb + NW);
    if (third) consume(A, lb + 2 * NW);
  }

  // merge the TPL lane groups of the wavefront
#pragma unroll
  for (int x = LPT; x < 64; x <<= 1) {
    const float m_o = __shfl_xor(m_run, x);
    const float l_o = __shfl_xor(l_run, x);
    const float m_new = fmaxf(m_run, m_o);
    const float wa = __builtin_amdgcn_exp2f(m_run - m_new), wb = __builtin_amdgcn_exp2f(m_o - m_new);
    l_run = l_run * wa + l_o * wb;
#pragma unroll
    for (int e = 0; e < EPL; ++e) {
      const float o_o = __shfl_xor(o[e], x);
      o[e] = o[e] * wa + o_o * wb;
    }
    m_run = m_new;
  }

  // merge the wavefronts
  __shared__ __align__(16) float sm[NW], sl[NW], so[NW][DH];
  if (grp == 0) {
#pragma unroll
    for (int e = 0; e < EPL; ++e) so[wave][sub * EPL + e] = o[e];
    if (sub == 0) {
      sm[wave] = m_run;
      sl[wave] = l_run;
    }
  }
  __syncthreads();
  if (threadIdx.x < DH) {
    float M = sm[0];
#pragma unroll
    for (int w = 1; w < NW; ++w) M = fmaxf(M, sm[w]);
    float L = 0.0f, acc = 0.0f;
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      const float wgt = __builtin_amdgcn_exp2f(sm[w] - M);
      L += sl[w] * wgt;
      acc += so[w][threadIdx.x] * wgt;
    }
    if constexpr (SPLIT) {
      // this part's running maximum, sum and unnormalised output; the merge launch takes it from here
      float* ws = a.split_ws + (((size_t)b * a.n_heads + head) * gridDim.z + blockIdx.z) * (DH + 2);
      if (threadIdx.x == 0) {
        ws[0] = M;
        ws[1] = L;
      }
      ws[2 + threadIdx.x] = acc;
    } else {
      const float r = acc / L;
      const int col = head * DH + threadIdx.x;
      if (OPROJ && wrow) {
        so[0][threadIdx.x] = r;   // (this thread was the last to read it)
      } else if constexpr (OUT_XT) {
        reinterpret_cast<bf16_t*>(a.out)[xt_index(out_row, col, a.n_heads * DH)] = (bf16_t)r;
      } else {
        reinterpret_cast<float*>(a.out)[(size_t)out_row * a.n_heads * DH + col] = r;
      }
    }
  }
  if constexpr (OPROJ) {
    if (!wrow) return;
    __syncthreads();
    const float4 x = *reinterpret_cast<const float4*>(&so[0][sub * EPL]);
    float* part = op.parts + ((size_t)head * a.B + b) * d_out + blockIdx.z * rows + wave * TPL + grp;
    auto row = [&](const float4& w, int i) {
      const float v = group_sum<LPT>(fmaf(w.w, x.w, fmaf(w.z, x.z, fmaf(w.y, x.y, w.x * x.x))));
      if (sub == 0) part[i * RPI] = v;
    };
#pragma unroll
    for (int i = 0; i < AHEAD; ++i)
      if (i * RPI < rows) row(wo[i], i);
  }
}

template <class T, int DH, bool OUT_XT, bool SPLIT>
__global__ __launch_bounds__(256) void attn_decode_kernel(AttnArgs a, Pred pred) {
  attn_decode<T, DH, OUT_XT, SPLIT>(a, NoOproj{}, blockIdx.y, [&] { return pred_skip(pred); });
}

// fp32 path: attention and output projection in one launch, with the exit decision of the layer before in leading workgroups.  All of
// them apply the decision's own rule (layer_ran, and left_before for a sequence), not the live words: the attention of the layer after the
// batch exit layer, or of a sequence that leaves by this decision, runs, and nobody reads its result.
template <int DH>
__global__ __launch_bounds__(256) void attn_f32_kernel(AttnArgs a, Pred pred, Oproj op) {
  if ((int)blockIdx.y < op.job.n_wg) {
    if (blockIdx.z || !layer_ran(op.job.a.s, op.job.a.layer)) return;
    __shared__ float4 red[4];
    const int m = blockIdx.y * gridDim.x + blockIdx.x;
    if (m < op.job.a.B) decide_row_f32(op.job.logits, op.job.row_scale, op.job.vocab, op.job.a, m, red);
    return;
  }
  attn_decode<float, DH, false, false>(a, op, (int)blockIdx.y - op.job.n_wg,
                                       [&] { return op.job.n_wg ? !layer_ran(op.job.a.s, op.job.a.layer) : pred_skip(pred); });
}

// Second launch of the split form: one workgroup of DH threads per (sequence, head) adds the parts in part order.
template <int DH, bool OUT_XT>
__global__ __launch_bounds__(DH) void attn_merge_kernel(AttnArgs a, Pred pred) {
  if (pred_skip(pred)) return;
  const int head = blockIdx.x, b = blockIdx.y;
  const int left = a.skip ? __hip_atomic_load(a.skip + b, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0;
  if (left != 0) return;
  const int out_row = a.out_pos ? a.out_pos[b] : b;
  const float* ws = a.split_ws + ((size_t)b * a.n_heads + head) * a.split_parts * (DH + 2);
  // (everything is asked for at once: the maxima first and the rest behind them were two trips to memory; 7B shape, one sequence
  // at 1000 positions, two layers 254 -> 250 us, 16384 positions 45.3 -> 44.2 us a call)
  float m[kAttnMaxSplit], l[kAttnMaxSplit], o[kAttnMaxSplit];
#pragma unroll
  for (int s = 0; s < kAttnMaxSplit; ++s) {
    m[s] = NEG_BIG;
    l[s] = o[s] = 0.0f;
    if (s < a.split_parts) {
      const float* p = ws + (size_t)s * (DH + 2);
      m[s] = p[0];
      l[s] = p[1];
      o[s] = p[2 + threadIdx.x];
    }
  }
  float M = NEG_BIG;
#pragma unroll
  for (int s = 0; s < kAttnMaxSplit; ++s) M = fmaxf(M, m[s]);
  float L = 0.0f, acc = 0.0f;
#pragma unroll
  for (int s = 0; s < kAttnMaxSplit; ++s) {
    if (s >= a.split_parts) break;
    const float wgt = __builtin_amdgcn_exp2f(m[s] - M);   // an empty part has the maximum -1e30: weight 0
    L += l[s] * wgt;
    acc += o[s] * wgt;
  }
  const float r = acc / L;
  const int col = head * DH + threadIdx.x;
  if constexpr (OUT_XT) {
    reinterpret_cast<bf16_t*>(a.out)[xt_index(out_row, col, a.n_heads * DH)] = (bf16_t)r;
  } else {
    reinterpret_cast<float*>(a.out)[(size_t)out_row * a.n_heads * DH + col] = r;
  }
}

// ---------------------------------------------------------------------------------------------------------
// Several batch rows of ONE sequence per workgroup (a chunk of a prompt pushed through the decode step: rows
// that share a block table).  A workgroup owns R consecutive batch rows of one head; rows of the same sequence
// form a run, and the run's K/V blocks are streamed once and multiplied against every row of the run, each row
// masking the positions after its own.  A workgroup whose rows span several sequences walks its runs one after
// the other.  Per row the arithmetic is that of the single-row kernel above; only the K/V traffic is shared.
// ---------------------------------------------------------------------------------------------------------
template <class T, int DH, int R, bool OUT_XT>
__global__ __launch_bounds__(256) void attn_rows_kernel(AttnArgs a, Pred pred) {
  constexpr int EPL = Elems<T>::N;
  constexpr int LPT = DH / EPL;
  constexpr int TPL = 64 / LPT;
  constexpr int LPB = 16 / TPL;
  extern __shared__ int32_t tbl[];
  if (pred_skip(pred)) return;

  const int head = blockIdx.x, row0 = blockIdx.y * R;
  const int nrows = min(R, a.B - row0);
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int sub = lane % LPT, grp = lane / LPT;

  int seq[R], npos[R];
  float q[R][EPL], m_run[R], l_run[R], o[R][EPL];
  const float sc = 1.4426950408889634f / sqrtf((float)DH);
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const bool valid = r < nrows;
    seq[r] = valid ? safe_row(a.row_table[row0 + r], a.B) : -1;
    npos[r] = valid ? min(a.context_lens[row0 + r] + 1, a.max_blocks * 16) : 0;
    const float* qp = a.q + ((size_t)(valid ? row0 + r : row0) * a.n_heads + head) * DH + sub * EPL;
#pragma unroll
    for (int i = 0; i < EPL; ++i) {
      q[r][i] = qp[i] * sc;
      o[r][i] = 0.0f;
    }
    m_run[r] = NEG_BIG;
    l_run[r] = 0.0f;
  }

  const size_t head_off = (size_t)head * 16 * DH;
  const size_t block_elems = (size_t)a.n_heads * 16 * DH;
  const T* kbase = reinterpret_cast<const T*>(a.k_pool) + head_off + (size_t)grp * DH + sub * EPL;
  const T* vbase = reinterpret_cast<const T*>(a.v_pool) + head_off + (size_t)grp * DH + sub * EPL;
  struct Blk {
    uint4 k[LPB], v[LPB];
  };

  int r_begin = 0;
  while (r_begin < nrows) {
    // the run: rows r_begin .. r_end-1 of one sequence (uniform over the workgroup)
    int r_end = r_begin + 1, run_ctx = 0, run_seq = -1;
#pragma unroll
    for (int r = 0; r < R; ++r)
      if (r == r_begin) run_seq = seq[r];
#pragma unroll
    for (int r = 1; r < R; ++r)
      if (r == r_end && r < nrows && seq[r] == run_seq) ++r_end;
#pragma unroll
    for (int r = 0; r < R; ++r)
      if (r >= r_begin && r < r_end) run_ctx = max(run_ctx, npos[r]);
    const int n_blocks = (run_ctx + 15) >> 4;
    const int32_t* table = a.block_tables + (size_t)run_seq * a.max_blocks;
    __syncthreads();   // the previous run's table is no longer read
    for (int i = threadIdx.x; i < n_blocks; i += blockDim.x) tbl[i] = safe_block(table[i], a.num_blocks);
    __syncthreads();

    const T* zero_src = reinterpret_cast<const T*>(&k_zero16);
    auto fetch = [&](Blk& x, int lb) {
      const size_t off = (size_t)tbl[lb] * block_elems;
#pragma unroll
      for (int i = 0; i < LPB; ++i) {
        x.k[i] = load_stream(kbase + off + (size_t)i * TPL * DH);
        x.v[i] = load_stream(lb * 16 + i * TPL + grp < run_ctx ? vbase + off + (size_t)i * TPL * DH : zero_src);
      }
    };
    auto consume = [&](const Blk& x, int lb) {
      float kf[LPB][EPL], vf[LPB][EPL];
#pragma unroll
      for (int i = 0; i < LPB; ++i) {
        Elems<T>::unpack(x.k[i], kf[i]);
        Elems<T>::unpack(x.v[i], vf[i]);
      }
#pragma unroll
      for (int r = 0; r < R; ++r) {
        if (r < r_begin || r >= r_end) continue;   // uniform: rows of other runs keep their state
        float s[LPB];
        float m_new = m_run[r];
#pragma unroll
        for (int i = 0; i < LPB; ++i) {
          float d = 0.0f;
#pragma unroll
          for (int e = 0; e < EPL; ++e) d = fmaf(q[r][e], kf[i][e], d);
          d = group_sum<LPT>(d);
          const int tok = lb * 16 + i * TPL + grp;
          s[i] = tok < npos[r] ? d : NEG_BIG;
          m_new = fmaxf(m_new, s[i]);
        }
        const float alpha = __builtin_amdgcn_exp2f(m_run[r] - m_new);
        l_run[r] *= alpha;
#pragma unroll
        for (int e = 0; e < EPL; ++e) o[r][e] *= alpha;
#pragma unroll
        for (int i = 0; i < LPB; ++i) {
          const int tok = lb * 16 + i * TPL + grp;
          const float p = tok < npos[r] ? __builtin_amdgcn_exp2f(s[i] - m_new) : 0.0f;
          l_run[r] += p;
#pragma unroll
          for (int e = 0; e < EPL; ++e) o[r][e] = fmaf(p, vf[i][e], o[r][e]);
        }
        m_run[r] = m_new;
      }
    };

    // one block in flight behind the one being multiplied (the multiplies of R rows hide the load)
    Blk A, B;
    int lb = wave;
    if (lb < n_blocks) fetch(A, lb);
    for (; lb + NW < n_blocks; lb += 2 * NW) {
      fetch(B, lb + NW);
      consume(A, lb);
      if (lb + 2 * NW < n_blocks) fetch(A, lb + 2 * NW);
      consume(B, lb + NW);
    }
    if (lb < n_blocks) consume(A, lb);
    r_begin = r_end;
  }

  // merge the lane groups of each wavefront, then the wavefronts, row by row
  __shared__ float sm[NW][R], sl[NW][R], so[NW][R][DH];
#pragma unroll
  for (int r = 0; r < R; ++r) {
#pragma unroll
    for (int x = LPT; x < 64; x <<= 1) {
      const float m_o = __shfl_xor(m_run[r], x);
      const float l_o = __shfl_xor(l_run[r], x);
      const float m_new = fmaxf(m_run[r], m_o);
      const float wa = __builtin_amdgcn_exp2f(m_run[r] - m_new), wb = __builtin_amdgcn_exp2f(m_o - m_new);
      l_run[r] = l_run[r] * wa + l_o * wb;
#pragma unroll
      for (int e = 0; e < EPL; ++e) {
        const float o_o = __shfl_xor(o[r][e], x);
        o[r][e] = o[r][e] * wa + o_o * wb;
      }
      m_run[r] = m_new;
    }
    if (grp == 0) {
#pragma unroll
      for (int e = 0; e < EPL; ++e) so[wave][r][sub * EPL + e] = o[r][e];
      if (sub == 0) {
        sm[wave][r] = m_run[r];
        sl[wave][r] = l_run[r];
      }
    }
  }
  __syncthreads();
  for (int t = threadIdx.x; t < nrows * DH; t += blockDim.x) {
    const int r = t / DH, c = t - r * DH;
    float M = sm[0][r];
#pragma unroll
    for (int w = 1; w < NW; ++w) M = fmaxf(M, sm[w][r]);
    float L = 0.0f, acc = 0.0f;
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      const float wgt = __builtin_amdgcn_exp2f(sm[w][r] - M);
      L += sl[w][r] * wgt;
      acc += so[w][r][c] * wgt;
    }
    const float res = acc / L;
    const int col = head * DH + c;
    if constexpr (OUT_XT) {
      reinterpret_cast<bf16_t*>(a.out)[xt_index(row0 + r, col, a.n_heads * DH)] = (bf16_t)res;
    } else {
      reinterpret_cast<float*>(a.out)[(size_t)(row0 + r) * a.n_heads * DH + col] = res;
    }
  }
}

// ---------------------------------------------------------------------------------------------------------
// Rows of a prompt chunk on the matrix cores (bf16 cache).  A workgroup of eight wavefronts owns up to R <= 64
// consecutive batch rows of one head, in one or two groups of 32; rows of one sequence form a run, and the 32-token steps
// of all its runs' contexts, one after the other, are dealt out to the slices (each wavefront a slice, or each pair with
// two groups).  A wavefront multiplies its steps against its group's rows with v_mfma_f32_32x32x16_bf16; rows of other
// runs, and positions after a row's own, are masked:
//   scores^T [token][row] = K [token][dh] . q^T [dh][row]
//   out^T    [dh][row]   += V^T [dh][token] . p^T [token][row]
// With the transposed products a lane holds 16 of the 32 scores of ONE row (row = lane % 32; lane ^ 32 holds the others),
// so the online softmax needs one shuffle per step, and the probabilities go from the score registers into the next
// product without leaving the lane (its contraction slots are numbered in the order the first product delivers tokens).
// q and the probabilities stay float in effect: each is split into a bf16 head and a bf16 remainder and multiplied twice.
//
// What bounds it is the compute unit's intake of K and V (about 55 bytes a nanosecond, whatever cache they come from), so
// the two groups share every tile: each of a slice's two wavefronts brings one of the step's two blocks, from memory to
// LDS directly in whole kilobytes, into the slice's other buffer while this step is multiplied; the pair meets once per step.
// The lanes of a load choose WHICH 16 bytes of a token they fetch, which permutes a token's channels in LDS so that
// neither the fragment reads of K nor the transposing reads of V (ds_read_b64_tr_b16: four tokens x 16 channels per 16
// lanes) meet in one bank.
// 512 rows of four sequences at 0 to 3128 positions, 32 heads x 128: 129 us with 16 rows per workgroup, each streaming
// the whole context, and V transposed through 2-byte LDS stores; 56 us now.  A step takes a slice 2.1 us (one prompt of 512
// rows: 20.6 us at 4 steps a slice, 88.3 at 35): a wavefront's multiplies are 1024 cycles of that and two wavefronts share a
// SIMD's matrix core, 40 % together; the rest is softmax, LDS and the meeting.  16 rows of 12 sequences at up to 1000 positions: 141 us
// (runs one after the other, each through all four wavefronts) -> 28 us; 200 rows of four at up to 100: 16 -> 12 us.
// ---------------------------------------------------------------------------------------------------------
typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef unsigned int u32x4_t __attribute__((ext_vector_type(4)));
typedef short s16x4_t __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) void* lds_void_ptr;
typedef __attribute__((address_space(3))) unsigned char* lds_uchar_ptr;
typedef __attribute__((address_space(1))) const void* global_void_ptr;

constexpr int PW = 8;            // wavefronts per workgroup
constexpr int PROMPT_ROWS = 64;  // most batch rows a workgroup owns

// Two floats rounded to bf16 (nearest even), the first in the low half.
__device__ inline unsigned pack_bf16(float a, float b) {
  typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
  return __builtin_bit_cast(unsigned, bf16x2_t{(__bf16)a, (__bf16)b});
}

// Transposing LDS reads at four (or two) lane addresses, two rows of tokens each (the second 8 tokens on), and the wait for
// them.  (In asm: in front of the builtin the compiler waits for every direct-to-LDS load in flight, the next K tile's too.)
template <int OFF, int STEP>
__device__ inline void read_tr(const unsigned (&at)[4], s16x4_t (&p)[4][2]) {
  asm volatile(
      "ds_read_b64_tr_b16 %0, %8 offset:%12\n\tds_read_b64_tr_b16 %1, %8 offset:%13\n\t"
      "ds_read_b64_tr_b16 %2, %9 offset:%12\n\tds_read_b64_tr_b16 %3, %9 offset:%13\n\t"
      "ds_read_b64_tr_b16 %4, %10 offset:%12\n\tds_read_b64_tr_b16 %5, %10 offset:%13\n\t"
      "ds_read_b64_tr_b16 %6, %11 offset:%12\n\tds_read_b64_tr_b16 %7, %11 offset:%13\n\t"
      "s_waitcnt lgkmcnt(0)"
      : "=&v"(p[0][0]), "=&v"(p[0][1]), "=&v"(p[1][0]), "=&v"(p[1][1]), "=&v"(p[2][0]), "=&v"(p[2][1]), "=&v"(p[3][0]), "=&v"(p[3][1])
      : "v"(at[0]), "v"(at[1]), "v"(at[2]), "v"(at[3]), "n"(OFF), "n"(OFF + STEP)
      : "memory");
}
template <int OFF, int STEP>
__device__ inline void read_tr(const unsigned (&at)[2], s16x4_t (&p)[2][2]) {
  asm volatile(
      "ds_read_b64_tr_b16 %0, %4 offset:%6\n\tds_read_b64_tr_b16 %1, %4 offset:%7\n\t"
      "ds_read_b64_tr_b16 %2, %5 offset:%6\n\tds_read_b64_tr_b16 %3, %5 offset:%7\n\t"
      "s_waitcnt lgkmcnt(0)"
      : "=&v"(p[0][0]), "=&v"(p[0][1]), "=&v"(p[1][0]), "=&v"(p[1][1])
      : "v"(at[0]), "v"(at[1]), "n"(OFF), "n"(OFF + STEP)
      : "memory");
}

// The same rows one at a time, a wavefront each, every row over its own positions alone: for workgroups that met an Inf or NaN
// (see the end of the walk below).  64 scores at a time, a token per lane; then a channel or two per lane.
template <int DH, bool OUT_XT>
__device__ inline void prompt_rows_alone(const AttnArgs& a, int row0, int nrows, int head, int wave, int lane) {
  constexpr int CPL = DH / 64;   // channels per lane
  const float sc = 1.4426950408889634f / sqrtf((float)DH);
  const size_t block_elems = (size_t)a.n_heads * 16 * DH;
  const bf16_t* kpool = reinterpret_cast<const bf16_t*>(a.k_pool) + (size_t)head * 16 * DH;
  const bf16_t* vpool = reinterpret_cast<const bf16_t*>(a.v_pool) + (size_t)head * 16 * DH;
  for (int row = row0 + wave; row < row0 + nrows; row += PW) {
    const int32_t* table = a.block_tables + (size_t)safe_row(a.row_table[row], a.B) * a.max_blocks;
    const int npos = max(0, min(a.context_lens[row], a.max_blocks * 16 - 1) + 1);
    const float* q = a.q + ((size_t)row * a.n_heads + head) * DH;
    float m = NEG_BIG, l = 0.0f, acc[CPL];
#pragma unroll
    for (int i = 0; i < CPL; ++i) acc[i] = 0.0f;
    for (int t0 = 0; t0 < npos; t0 += 64) {
      const int n = min(64, npos - t0), t = t0 + min(lane, n - 1);
      const size_t at = (size_t)safe_block(table[t >> 4], a.num_blocks) * block_elems + (size_t)(t & 15) * DH;
      float z = 0.0f;
#pragma unroll 8
      for (int c = 0; c < DH; ++c) z = fmaf(q[c], (float)kpool[at + c], z);
      z = lane < n ? z * sc : NEG_BIG;
      float mx = fmaxf(m, z);
#pragma unroll
      for (int x = 1; x < 64; x <<= 1) mx = fmaxf(mx, __shfl_xor(mx, x));
      const float alpha = __builtin_amdgcn_exp2f(m - mx), p = lane < n ? __builtin_amdgcn_exp2f(z - mx) : 0.0f;
      float sum = p;
#pragma unroll
      for (int x = 1; x < 64; x <<= 1) sum += __shfl_xor(sum, x);
      m = mx;
      l = l * alpha + sum;
#pragma unroll
      for (int i = 0; i < CPL; ++i) acc[i] *= alpha;
      for (int j = 0; j < n; ++j) {
        const float pj = __shfl(p, j);
        const bf16_t* v = vpool + (size_t)__shfl((unsigned long long)at, j) + lane * CPL;
#pragma unroll
        for (int i = 0; i < CPL; ++i) acc[i] = fmaf(pj, (float)v[i], acc[i]);
      }
    }
#pragma unroll
    for (int i = 0; i < CPL; ++i) {
      const int col = head * DH + lane * CPL + i;
      const float r = acc[i] * (1.0f / l);
      if constexpr (OUT_XT) reinterpret_cast<bf16_t*>(a.out)[xt_index(row, col, a.n_heads * DH)] = (bf16_t)r;
      else reinterpret_cast<float*>(a.out)[(size_t)row * a.n_heads * DH + col] = r;
    }
  }
}

template <int DH>
constexpr int prompt_lds_bytes() { return PW * 2 * 32 * DH * 2; }

template <int DH, bool OUT_XT>
__global__ __launch_bounds__(PW * 64) void attn_prompt_kernel(AttnArgs a, int R, Pred pred) {
  constexpr int CS = DH / 16;            // contraction steps of q . K
  constexpr int CT = DH / 32;            // 32-channel tiles of the output
  constexpr int CPT = DH / 8;            // 16-byte pieces of a token
  constexpr int TPI = 64 / CPT;          // tokens per load instruction
  constexpr int JB = 16 / TPI;           // load instructions per 16-token block
  constexpr int TILE = 32 * DH * 2;      // bytes of a 32-token tile
  // two groups: [slice][buffer][K, V]; one group: [wavefront][K, V]; at the end [wavefront][32 rows][DH] floats
  extern __shared__ __align__(16) unsigned char psm[];
  __shared__ int s_first[PROMPT_ROWS + 1];                        // first step of every run, and their total
  __shared__ int s_seq[PROMPT_ROWS], s_ctx[PROMPT_ROWS], s_rows[PROMPT_ROWS];   // of every run: sequence, positions, begin | end << 8
  __shared__ float sm[PW][32], sl[PW][32];
  __shared__ int s_meet[PW], s_alone;
  if (pred_skip(pred)) return;

  const int head = blockIdx.x, row0 = blockIdx.y * R;
  const int nrows = min(R, a.B - row0);
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int l32 = lane & 31, h = lane >> 5;
  // More than 32 rows: wavefront (slice, group) of four slices, each wavefront bringing block `group` of every step for
  // both.  Otherwise eight slices of one group, each wavefront on its own.
  const bool two = nrows > 32;
  const int nsl = two ? PW / 2 : PW, slice = two ? wave >> 1 : wave, grp = two ? wave & 1 : 0;
  const int my = grp * 32 + l32;                                  // this lane's row (of the workgroup's)
  const bool row_ok = my < nrows;

  const int seq_l = lane < nrows ? safe_row(a.row_table[row0 + lane], a.B) : -1;
  // (a negative context attends nothing: the counts of steps below must not go backwards)
  const int npos_l = lane < nrows ? max(0, min(a.context_lens[row0 + lane], a.max_blocks * 16 - 1) + 1) : 0;
  // q of this lane's row, channels c*16 + h*8 .. +8 of every contraction step, scaled, as bf16 head + remainder
  u32x4_t qh[CS], ql[CS];
  {
    const float sc = row_ok ? 1.4426950408889634f / sqrtf((float)DH) : 0.0f;
    const float* qp = a.q + ((size_t)(row0 + (row_ok ? my : 0)) * a.n_heads + head) * DH + h * 8;
#pragma unroll
    for (int c = 0; c < CS; ++c) {
      const float4 lo = *reinterpret_cast<const float4*>(qp + c * 16);
      const float4 hi = *reinterpret_cast<const float4*>(qp + c * 16 + 4);
      const float v[8] = {lo.x * sc, lo.y * sc, lo.z * sc, lo.w * sc, hi.x * sc, hi.y * sc, hi.z * sc, hi.w * sc};
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const unsigned hd = pack_bf16(v[2 * e], v[2 * e + 1]);
        qh[c][e] = hd;
        ql[c][e] = pack_bf16(v[2 * e] - __uint_as_float(hd << 16), v[2 * e + 1] - __uint_as_float(hd & 0xffff0000u));
      }
    }
  }

  // The runs: every lane that starts one finds its end, its longest row and the steps before it (the same in every wavefront).
  const int n_runs = [&] {
    const int before = __shfl_up(seq_l, 1);   // (outside the condition: a shuffle reads nothing from a lane that is masked off)
    const bool starts = lane < nrows && (lane == 0 || before != seq_l);
    const unsigned long long bal = __ballot(starts);
    const unsigned long long after = lane < 63 ? bal >> (lane + 1) : 0;
    const int end = after ? lane + 1 + __builtin_ctzll(after) : nrows;
    int ctx = npos_l;
#pragma unroll
    for (int x = 1; x < 64; x <<= 1) {
      const int o = __shfl_down(ctx, x);
      if (lane + x < end) ctx = max(ctx, o);
    }
    const int steps = starts ? (ctx + 31) >> 5 : 0;
    int upto = steps;
#pragma unroll
    for (int x = 1; x < 64; x <<= 1) {
      const int o = __shfl_up(upto, x);
      if (lane >= x) upto += o;
    }
    if (wave == 0) {
      if (starts) {
        const int j = __popcll(bal & ((1ull << lane) - 1ull));
        s_first[j] = upto - steps;
        s_seq[j] = seq_l;
        s_ctx[j] = ctx;
        s_rows[j] = lane | end << 8;
      }
      if (lane == 63) s_first[__popcll(bal)] = upto;
      if (lane < PW) s_meet[lane] = 0;
      if (lane == 0) s_alone = 0;
    }
    return __popcll(bal);
  }();
  __syncthreads();
  const int n_steps = __builtin_amdgcn_readfirstlane(s_first[n_runs]);
  // Steps of this wavefront, over all runs one after the other; both wavefronts of a pair take part in every step of
  // their slice.  One past the end repeats the last.
  const int nk = slice < n_steps ? (n_steps - slice + nsl - 1) / nsl : 0;

  const size_t block_elems = (size_t)a.n_heads * 16 * DH;
  const bf16_t* kpool = reinterpret_cast<const bf16_t*>(a.k_pool) + (size_t)head * 16 * DH;
  const bf16_t* vpool = reinterpret_cast<const bf16_t*>(a.v_pool) + (size_t)head * 16 * DH;
  // piece c of token t lies at piece c ^ perm(t) of its row: K t % CPT, V 2 * (t % (CPT / 2))
  int koff[JB], voff[JB];
#pragma unroll
  for (int j = 0; j < JB; ++j) {
    const int t = j * TPI + lane / CPT, c = lane % CPT;
    koff[j] = t * DH + (c ^ (t & (CPT - 1))) * 8;
    voff[j] = t * DH + (c ^ (2 * (t & (CPT / 2 - 1)))) * 8;
  }
  // lane offsets of the transposing reads: token h*4 + (lane%16)/4 (+ 8, 16, 24), channels d*32 + (lane/16%2)*16 + lane%4*4
  unsigned voff_tr[CT];
#pragma unroll
  for (int d = 0; d < CT; ++d) {
    const int t = h * 4 + ((lane & 15) >> 2);
    const int piece = (d * 4 + ((lane >> 4) & 1) * 2 + ((lane & 3) >> 1)) ^ (2 * (t & (CPT / 2 - 1)));
    voff_tr[d] = t * (DH * 2) + piece * 16 + (lane & 1) * 8;
  }

  // The blocks of 32 steps at a time sit in one pair of registers (bytes from the pool's start), two lanes per step.  An
  // odd block count reads the last block twice (its second copy is masked).
  int off_lo = 0, off_hi = 0, ids_from = 0;
  auto step_of = [&](int k) { return min(slice + k * nsl, n_steps - 1); };
  auto load_ids = [&](int k0) {
    const int g = step_of(k0 + (lane >> 1));
    int j = 0;
    while (j + 1 < n_runs && s_first[j + 1] <= g) ++j;
    const int lb = min(2 * (g - s_first[j]) + (lane & 1), ((s_ctx[j] + 15) >> 4) - 1);
    const int blk = safe_block(a.block_tables[(size_t)s_seq[j] * a.max_blocks + lb], a.num_blocks);
    const size_t off = (size_t)blk * (block_elems * sizeof(bf16_t));
    off_lo = (int)(unsigned)off;
    off_hi = (int)(unsigned)(off >> 32);
    ids_from = k0;
  };
  auto block_at = [&](const bf16_t* pool, int k, int hb) {
    const int i = 2 * (k - ids_from) + hb;
    const unsigned lo = __builtin_amdgcn_readlane(off_lo, i), hi = __builtin_amdgcn_readlane(off_hi, i);
    return reinterpret_cast<const bf16_t*>(reinterpret_cast<const char*>(pool) + ((size_t)hi << 32 | lo));
  };
  // The run of the step that is loaded / multiplied (both only move forward).
  struct Run {
    int j, first, next, ctx, rows;
  };
  auto run_at = [&](int j) {
    Run r;
    r.j = j;
    r.first = __builtin_amdgcn_readfirstlane(s_first[j]);
    r.next = __builtin_amdgcn_readfirstlane(s_first[j + 1]);
    r.ctx = __builtin_amdgcn_readfirstlane(s_ctx[j]);
    r.rows = __builtin_amdgcn_readfirstlane(s_rows[j]);
    return r;
  };
  Run ld = run_at(0);
  // block hb (0 / 1) of step k: K tile to kt, V tile to kt + TILE
  auto issue_k = [&](int k, int hb, unsigned char* kt) {
    const bf16_t* kb = block_at(kpool, k, hb);
#pragma unroll
    for (int j = 0; j < JB; ++j)
      __builtin_amdgcn_global_load_lds((global_void_ptr)(kb + koff[j]), (lds_void_ptr)(kt + hb * (TILE / 2) + j * 1024), 16, 0, 0);
  };
  auto issue_v = [&](int k, int hb, unsigned char* kt) {
    const bf16_t* vb = block_at(vpool, k, hb);
    const int g = step_of(k);
    while (g >= ld.next) ld = run_at(ld.j + 1);
    const int t0 = (g - ld.first) * 32 + hb * 16;
    unsigned char* vt = kt + TILE + hb * (TILE / 2);
    if (t0 + 16 <= ld.ctx) {
#pragma unroll
      for (int j = 0; j < JB; ++j)
        __builtin_amdgcn_global_load_lds((global_void_ptr)(vb + voff[j]), (lds_void_ptr)(vt + j * 1024), 16, 0, 0);
    } else {   // positions from the run's end on (also the second copy of a repeated last block) come from the zeros
      for (int j = 0; j < JB; ++j) {
        const int t = j * TPI + lane / CPT, c = lane % CPT;
        const bf16_t* src = vb + t * DH + (c ^ (2 * (t & (CPT / 2 - 1)))) * 8;
        if (t0 + t >= ld.ctx) src = reinterpret_cast<const bf16_t*>(&k_zero16);
        __builtin_amdgcn_global_load_lds((global_void_ptr)src, (lds_void_ptr)(vt + j * 1024), 16, 0, 0);
      }
    }
  };
  unsigned char* ring = psm + (size_t)(two ? slice * 4 : wave * 2) * TILE;
  if (nk > 0) {
    load_ids(0);
    if (two) {
      issue_k(0, grp, ring);
      issue_v(0, grp, ring);
    } else {
      issue_k(0, 0, ring);
      issue_k(0, 1, ring);
      issue_v(0, 0, ring);
      issue_v(0, 1, ring);
    }
  }

  float m_run = NEG_BIG, l_run = 0.0f;
  f32x16 o[CT];
#pragma unroll
  for (int d = 0; d < CT; ++d)
#pragma unroll
    for (int i = 0; i < 16; ++i) o[d][i] = 0.0f;

  auto walk = [&](auto two_c) {
    constexpr bool TWO = decltype(two_c)::value;
    Run mu = run_at(0);
    mu.next = -1;                 // taken up at the first step
    mu.j = -1;
    int npos = 0;                 // positions this lane's row attends of the run (0: the row is another run's)
    int longest = 0, full = 0;    // longest / shortest row of the group (shortest: 0 if not all of its rows are the run's)
    int meet = 0;
    for (int k = 0; k < nk; ++k) {
      const int g = slice + k * nsl;
      if (g >= mu.next) {
        do mu = run_at(mu.j + 1);
        while (g >= mu.next);
        const int rb = mu.rows & 255, re = mu.rows >> 8;
        npos = __shfl(npos_l, my);
        if (my < rb || my >= re) npos = 0;
        longest = npos;
        full = row_ok ? npos : 0x7fffffff;
#pragma unroll
        for (int x = 1; x < 32; x <<= 1) {
          longest = max(longest, __shfl_xor(longest, x));
          full = min(full, __shfl_xor(full, x));
        }
        longest = __builtin_amdgcn_readfirstlane(longest);
        full = __builtin_amdgcn_readfirstlane(full);
      }
      if (k + 1 - ids_from == 32) load_ids(k + 1);
      const unsigned char* kt = ring;
      if constexpr (TWO) {
        // This wavefront's half of step k is in LDS and it has read step k-1: say so, and wait for the other's word.
        // (Only the pair meets, and both make every step, so the wait ends; the slices run free of each other.)
        asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
        ++meet;
        __hip_atomic_store(&s_meet[wave], meet, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        while (__hip_atomic_load(&s_meet[wave ^ 1], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) < meet) {
        }
        asm volatile("" ::: "memory");
        unsigned char* other = ring + ((k + 1) & 1) * 2 * TILE;
        issue_k(k + 1, grp, other);                  // (the one past the end is never used)
        issue_v(k + 1, grp, other);
        kt = ring + (k & 1) * 2 * TILE;
      } else {
        asm volatile("s_waitcnt vmcnt(%0)" ::"n"(2 * JB) : "memory");   // K of step k is in LDS, V may still be on its way
      }
      const int tok0 = (g - mu.first) * 32;
      if (TWO && tok0 >= longest) continue;          // nothing for this group
      f32x16 st;
#pragma unroll
      for (int i = 0; i < 16; ++i) st[i] = 0.0f;
      {
        bf16x8_t kk[CS];
#pragma unroll
        for (int c = 0; c < CS; ++c)
          kk[c] = *reinterpret_cast<const bf16x8_t*>(kt + l32 * (DH * 2) + ((2 * c + h) ^ (l32 & (CPT - 1))) * 16);
#pragma unroll
        for (int c = 0; c < CS; ++c) {
          st = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kk[c], __builtin_bit_cast(bf16x8_t, qh[c]), st, 0, 0, 0);
          st = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kk[c], __builtin_bit_cast(bf16x8_t, ql[c]), st, 0, 0, 0);
        }
      }
      if constexpr (!TWO) {
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // the K tile has been read: its space takes the next one
        issue_k(k + 1, 0, ring);
        issue_k(k + 1, 1, ring);
      }
      // accumulator i of a lane is token (i/4)*8 + h*4 + i%4 of the step
      const bool masked = tok0 + 32 > full;
      if (masked) {
#pragma unroll
        for (int i = 0; i < 16; ++i) st[i] = tok0 + (i >> 2) * 8 + h * 4 + (i & 3) < npos ? st[i] : NEG_BIG;
      }
      float mx = m_run;
#pragma unroll
      for (int i = 0; i < 16; ++i) mx = fmaxf(mx, st[i]);
      mx = fmaxf(mx, __shfl_xor(mx, 32));
      // The sums are taken relative to m_run, which follows the maximum only when some row's has grown by a factor of sqrt(2)
      // or more: the output is rescaled less often (a new maximum by any margin turns up in some row of 32 at most steps).
      // 512 rows of the case above, and relative error against float64 there: following every maximum 59.8 us, 2.83e-6; this
      // margin 59.1, 2.83e-6; 2^2 57.0, 2.84e-6; 2^8 55.8, 2.86e-6 and single rows up to a fifth worse, in this order at every
      // shape measured.  The margin is about the largest that costs no precision.
      if (__any(mx > m_run + 0.5f)) {
        const float alpha = __builtin_amdgcn_exp2f(m_run - mx);
        m_run = mx;
        l_run *= alpha;
#pragma unroll
        for (int d = 0; d < CT; ++d)
#pragma unroll
          for (int i = 0; i < 16; ++i) o[d][i] *= alpha;
      }
#pragma unroll
      for (int i = 0; i < 16; ++i) st[i] = __builtin_amdgcn_exp2f(st[i] - m_run);
      if (masked) {
#pragma unroll
        for (int i = 0; i < 16; ++i) st[i] = tok0 + (i >> 2) * 8 + h * 4 + (i & 3) < npos ? st[i] : 0.0f;
      }
      u32x4_t ph[2], pl[2];
#pragma unroll
      for (int i = 0; i < 16; i += 2) {
        l_run += st[i];
        l_run += st[i + 1];
        const unsigned hd = pack_bf16(st[i], st[i + 1]);
        ph[i >> 3][(i & 7) >> 1] = hd;
        pl[i >> 3][(i & 7) >> 1] = pack_bf16(st[i] - __uint_as_float(hd << 16), st[i + 1] - __uint_as_float(hd & 0xffff0000u));
      }
      if constexpr (!TWO) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(2 * JB) : "memory");   // V of step k is in LDS
      // contraction slot 8h + e of 16 tokens is token (e/4)*8 + 4h + e%4: the order ph / pl hold them in
      unsigned va[CT];
#pragma unroll
      for (int d = 0; d < CT; ++d) va[d] = (unsigned)(size_t)(lds_uchar_ptr)(kt + TILE) + voff_tr[d];
      auto output_product = [&](auto uc) {
        constexpr int u = decltype(uc)::value;
        typedef short s16x8_t __attribute__((ext_vector_type(8)));
        s16x4_t part[CT][2];
        read_tr<u * 16 * DH * 2, 8 * DH * 2>(va, part);
#pragma unroll
        for (int d = 0; d < CT; ++d) {
          const s16x8_t v8 = __builtin_shufflevector(part[d][0], part[d][1], 0, 1, 2, 3, 4, 5, 6, 7);
          o[d] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, v8), __builtin_bit_cast(bf16x8_t, ph[u]), o[d], 0, 0, 0);
          o[d] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, v8), __builtin_bit_cast(bf16x8_t, pl[u]), o[d], 0, 0, 0);
        }
      };
      output_product(std::integral_constant<int, 0>{});
      output_product(std::integral_constant<int, 1>{});
      if constexpr (!TWO) {   // (the V tile has been read: read_tr waits)
        issue_v(k + 1, 0, ring);
        issue_v(k + 1, 1, ring);
      }
    }
  };
  if (two)
    walk(std::true_type{});
  else
    walk(std::false_type{});
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // the loads past the end still target LDS
  // A row takes part in the steps of the group's other runs, and in what is after its own position, with probabilities of 0.
  // That leaves its sums alone unless a V of the step is not finite: 0 times Inf is NaN, and what one sequence cached must
  // not reach another.  So where a row's sums are not finite, the rows are done again, each by itself.  (The look at the sums
  // costs 0 to 0.5 us a launch; leaving such rows out of each step needs registers the walk does not have.)
  float zero = 0.0f;
#pragma unroll
  for (int d = 0; d < CT; ++d)
#pragma unroll
    for (int i = 0; i < 16; ++i) zero = fmaf(o[d][i], 0.0f, zero);   // NaN if one of them is not finite
  if (row_ok && zero != 0.0f) s_alone = 1;
  __syncthreads();                                   // every tile has been read: the space now holds the partial outputs
  if (__builtin_amdgcn_readfirstlane(s_alone)) {
    prompt_rows_alone<DH, OUT_XT>(a, row0, nrows, head, wave, lane);
    return;
  }

  // the two lanes of a row hold partial sums of the same maximum; then the slices are added in slice order
  l_run += __shfl_xor(l_run, 32);
  if (nk > 0) {
    float* so = reinterpret_cast<float*>(psm + (size_t)wave * 2 * TILE);   // [32 rows][DH], pieces of four channels permuted by row
#pragma unroll
    for (int d = 0; d < CT; ++d)
#pragma unroll
      for (int q4 = 0; q4 < 4; ++q4) {
        const int piece = (d * 8 + q4 * 2 + h) ^ (l32 & (DH / 4 - 1));
        *reinterpret_cast<float4*>(so + l32 * DH + piece * 4) = make_float4(o[d][4 * q4], o[d][4 * q4 + 1], o[d][4 * q4 + 2], o[d][4 * q4 + 3]);
      }
    if (h == 0) {
      sm[wave][l32] = m_run;
      sl[wave][l32] = l_run;
    }
  }
  __syncthreads();
  const int ng = two ? 2 : 1, n_live = min(nsl, n_steps);   // slices that had a step
  for (int t = threadIdx.x; t < ng * 32 * CPT; t += PW * 64) {   // thread -> (group, row, 8 channels)
    const int g = t / (32 * CPT), u = t % (32 * CPT);
    const int r = OUT_XT ? u % 32 : u / CPT, c8 = OUT_XT ? u / 32 : u % CPT;
    if (g * 32 + r >= nrows) continue;
    float M = NEG_BIG;
    for (int i = 0; i < n_live; ++i) M = fmaxf(M, sm[i * ng + g][r]);
    float L = 0.0f, acc[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) acc[e] = 0.0f;
    for (int i = 0; i < n_live; ++i) {
      const int w = i * ng + g;
      const float wgt = __builtin_amdgcn_exp2f(sm[w][r] - M);
      L += sl[w][r] * wgt;
      const float* sp = reinterpret_cast<const float*>(psm + (size_t)w * 2 * TILE) + r * DH;
      const float4 lo = *reinterpret_cast<const float4*>(sp + ((2 * c8) ^ (r & (DH / 4 - 1))) * 4);
      const float4 hi = *reinterpret_cast<const float4*>(sp + ((2 * c8 + 1) ^ (r & (DH / 4 - 1))) * 4);
      const float v[8] = {lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w};
#pragma unroll
      for (int e = 0; e < 8; ++e) acc[e] += v[e] * wgt;
    }
    const float inv = 1.0f / L;
    const int row = row0 + g * 32 + r, col = head * DH + c8 * 8;
    if constexpr (OUT_XT) {
      bf16x8_t o8;
#pragma unroll
      for (int e = 0; e < 8; ++e) o8[e] = (__bf16)(acc[e] * inv);
      *reinterpret_cast<bf16x8_t*>(reinterpret_cast<bf16_t*>(a.out) + xt_index(row, col, a.n_heads * DH)) = o8;
    } else {
      float* op = reinterpret_cast<float*>(a.out) + (size_t)row * a.n_heads * DH + col;
      *reinterpret_cast<float4*>(op) = make_float4(acc[0] * inv, acc[1] * inv, acc[2] * inv, acc[3] * inv);
      *reinterpret_cast<float4*>(op + 4) = make_float4(acc[4] * inv, acc[5] * inv, acc[6] * inv, acc[7] * inv);
    }
  }
}

// Batch rows per workgroup: as many as it takes for one round of workgroups (one per compute unit: 128 KiB of LDS each);
// a workgroup's time hangs on its longest context, not on its rows, so fewer workgroups than that leave the chip idle
// and a second round costs as much as the first.
int prompt_rows(int B, int n_heads) {
  const int blocks = n_heads < 256 ? 256 / n_heads : 1;
  const int R = (B + blocks - 1) / blocks;
  return R < 4 ? 4 : R > PROMPT_ROWS ? PROMPT_ROWS : R;
}

// More than 64 KiB of LDS per workgroup has to be asked for, once per device.
template <int DH, bool OUT_XT>
bool prompt_lds_allowed() {
  static std::atomic<unsigned long long> asked{0};
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) {
    (void)hipGetLastError();
    return false;
  }
  const unsigned long long bit = 1ull << (dev & 63);
  if (asked.load(std::memory_order_relaxed) & bit) return true;
  if (hipFuncSetAttribute(reinterpret_cast<const void*>(attn_prompt_kernel<DH, OUT_XT>), hipFuncAttributeMaxDynamicSharedMemorySize,
                          prompt_lds_bytes<DH>()) != hipSuccess) {
    (void)hipGetLastError();   // not the call's error: another kernel takes the rows
    return false;
  }
  asked.fetch_or(bit, std::memory_order_relaxed);
  return true;
}

// false: the runtime refuses the kernel its LDS, nothing has been enqueued.
template <int DH, bool OUT_XT>
bool launch_prompt(const AttnArgs& a, Pred pred, hipStream_t st) {
  if (!prompt_lds_allowed<DH, OUT_XT>()) return false;
  const int R = prompt_rows(a.B, a.n_heads);
  hipLaunchKernelGGL((attn_prompt_kernel<DH, OUT_XT>), dim3(a.n_heads, (a.B + R - 1) / R), dim3(PW * 64), prompt_lds_bytes<DH>(), st,
                     a, R, pred);
  return true;
}

// Four rows per workgroup measured best at the 7B shape (eight: 300 registers, one wavefront per SIMD, slower).
constexpr int ROWS_PER_GROUP = 4;

template <class T, int DH>
void launch_t(const AttnArgs& a, Pred pred, hipStream_t st) {
  constexpr bool BF16 = std::is_same<T, bf16_t>::value;   // (only bf16 results leave in operand order)
  dim3 block(256);
  const size_t lds = (size_t)a.max_blocks * sizeof(int32_t);
  if (a.row_table) {   // rows share sequences: stream every sequence's K/V once per group of rows
    if constexpr (BF16) {
      if (a.out_xt ? launch_prompt<DH, true>(a, pred, st) : launch_prompt<DH, false>(a, pred, st)) return;
    }
    dim3 grid(a.n_heads, (a.B + ROWS_PER_GROUP - 1) / ROWS_PER_GROUP);
    if constexpr (BF16) {
      if (a.out_xt) {
        hipLaunchKernelGGL((attn_rows_kernel<T, DH, ROWS_PER_GROUP, true>), grid, block, lds, st, a, pred);
        return;
      }
    }
    hipLaunchKernelGGL((attn_rows_kernel<T, DH, ROWS_PER_GROUP, false>), grid, block, lds, st, a, pred);
    return;
  }
  if (a.split_ws && a.split_parts > 1) {
    // the output form only matters to the merge launch; the parts always leave as floats
    dim3 grid(a.n_heads, a.B, a.split_parts);
    hipLaunchKernelGGL((attn_decode_kernel<T, DH, false, true>), grid, block, lds, st, a, pred);
    dim3 gridm(a.n_heads, a.B);
    if (a.out_xt)
      hipLaunchKernelGGL((attn_merge_kernel<DH, true>), gridm, dim3(DH), 0, st, a, pred);
    else
      hipLaunchKernelGGL((attn_merge_kernel<DH, false>), gridm, dim3(DH), 0, st, a, pred);
    return;
  }
  dim3 grid(a.n_heads, a.B);
  if constexpr (BF16) {
    if (a.out_xt) {
      hipLaunchKernelGGL((attn_decode_kernel<T, DH, true, false>), grid, block, lds, st, a, pred);
      return;
    }
  }
  hipLaunchKernelGGL((attn_decode_kernel<T, DH, false, false>), grid, block, lds, st, a, pred);
}

}  // namespace

// One workgroup per (sequence, head) keeps the chip busy from about 256 pairs on.  With at most 64, up to eight
// workgroups share a pair so that about 256 run, as long as every part still has eight blocks (128 positions) of the
// table's width to walk: below that, and at 128 pairs (measured: 28.6 against 29.0 us at 4 x 2048 positions), the second
// launch costs what the idle compute units would have gained.  Measured at the 7B shape, one sequence: 16384
// positions 147 -> 52 us per layer, 4096 positions 41 -> 21 us.
int attn_split_parts(int B, int n_heads, int max_blocks) {
  const long pairs = (long)B * n_heads;
  if (pairs <= 0 || pairs > kAttnSplitMaxPairs) return 1;
  int parts = (int)(256 / pairs);
  if (parts > kAttnMaxSplit) parts = kAttnMaxSplit;
  if (parts > max_blocks / 8) parts = max_blocks / 8;
  return parts < 2 ? 1 : parts;
}

void attention_prepare() {
  prompt_lds_allowed<64, false>();
  prompt_lds_allowed<64, true>();
  prompt_lds_allowed<128, false>();
  prompt_lds_allowed<128, true>();
}

void launch_attention_f32(const AttnArgs& a, const float* w_o, float* parts, Pred pred, hipStream_t st, const SimpleDecision* with) {
  Oproj op{w_o, parts, with ? *with : SimpleDecision{}};
  op.job.n_wg = with ? (with->a.B + a.n_heads - 1) / a.n_heads : 0;
  // Four workgroups share a head's columns, each with the attention to itself: 64 KB of weights are 2 us for one compute unit.
  const dim3 grid(a.n_heads, a.B + op.job.n_wg, w_o ? 4 : 1), block(256);
  const size_t lds = (size_t)a.max_blocks * sizeof(int32_t);
  if (a.head_dim == 64) hipLaunchKernelGGL((attn_f32_kernel<64>), grid, block, lds, st, a, pred, op);
  else hipLaunchKernelGGL((attn_f32_kernel<128>), grid, block, lds, st, a, pred, op);
}

int launch_attention(const AttnArgs& a, int dtype, Pred pred, hipStream_t st) {
  if (a.B == 0) return EE_OK;
  if (a.split_parts > 1 && a.row_table) EE_FAIL(EE_ERR_UNSUPPORTED, "attention: split_parts does not go with row_table");
  if (a.split_parts > kAttnMaxSplit) EE_FAIL(EE_ERR_UNSUPPORTED, "attention: split_parts %d above %d", a.split_parts, kAttnMaxSplit);
  if (a.max_blocks < 1 || a.max_blocks > TABLE_LDS_MAX)
    EE_FAIL(EE_ERR_UNSUPPORTED, "attention: max_blocks %d outside 1..%d", a.max_blocks, TABLE_LDS_MAX);
  if (a.out_pos && a.row_table) EE_FAIL(EE_ERR_UNSUPPORTED, "attention: out_pos does not go with row_table");
  if (dtype == EE_FP32) {
    if (a.head_dim == 64) launch_t<float, 64>(a, pred, st);
    else if (a.head_dim == 128) launch_t<float, 128>(a, pred, st);
    else EE_FAIL(EE_ERR_UNSUPPORTED, "attention: head_dim %d not supported for fp32 (64 or 128)", a.head_dim);
  } else {
    if (a.head_dim == 64) launch_t<bf16_t, 64>(a, pred, st);
    else if (a.head_dim == 128) launch_t<bf16_t, 128>(a, pred, st);
    else EE_FAIL(EE_ERR_UNSUPPORTED, "attention: head_dim %d not supported for bf16 (64 or 128)", a.head_dim);
  }
  return EE_OK;
}

}  // namespace ee
