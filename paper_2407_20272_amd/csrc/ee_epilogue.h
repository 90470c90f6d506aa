// Device-side epilogues shared by the MFMA (bf16) and the plain (fp32) projection kernels.
// Each takes one batch row m and one pair of output rows (f_lo, f_hi) with their finished dot products.
#pragma once

#include "ee_common.h"

namespace ee {

// The control words of an iteration (status, exit layers, the count of accepted sequences, the all-exited flag and
// the batch exit layer) are written by the workgroups that take an exit decision and read by workgroups of other
// compute units, sometimes of the same launch: every access is a relaxed device-scope atomic.
__device__ inline int32_t ctl_load(const int32_t* p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ inline void ctl_store(int32_t* p, int32_t v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }

// Turns the rotary pair (lo, hi) by the angle with this cosine and sine.  Which of the two products is rounded on its own is
// written out, the same for every epilogue: left to the compiler, the block kernel's q and K came out one rounding away from
// what the other kernels and KV filling give (5 of 10 million cached elements differed).
__device__ inline void rotate(float& lo, float& hi, float c, float s) {
  const float a = __builtin_fmaf(lo, c, -(hi * s)), b = __builtin_fmaf(hi, c, lo * s);
  lo = a;
  hi = b;
}

// Rotary embedding (split-half pairing: channel j with j + dh/2, angle = pos * theta^(-2j/dh)) of four consecutive channels
// f_lo0..f_lo0+3 (f_lo0 a multiple of 4) of batch row m and their four rotary partners, and the write of this position's K/V into the paged
// bf16 cache; q goes to a dense buffer.  One look-up of the slot, 8-byte stores into the cache, 16-byte stores into q.  The (cos, sin)
// pairs come from a table that is filled once per call from angles formed in double (long contexts would lose the fraction of the
// angle to float rounding of the frequency).
__device__ inline void epi_qkv4(const QkvEpi& e, int m, int f_lo0, float (&lo)[4], float (&hi)[4]) {
  if (kv_filled(e, m)) return;
  const int d = e.d_model, dh = e.head_dim, half = dh >> 1;
  const int which = f_lo0 / d;  // 0 q, 1 k, 2 v
  const int within = f_lo0 - which * d;
  const int head = within / dh;
  const int j = within - head * dh;  // < dh/2, a multiple of 4
  if (which < 2 && e.rope_theta > 0.0f) {
    const float4 c01 = *reinterpret_cast<const float4*>(e.rope + (size_t)m * half + j);       // (cos, sin) x 2
    const float4 c23 = *reinterpret_cast<const float4*>(e.rope + (size_t)m * half + j + 2);
    const float cs[4] = {c01.x, c01.z, c23.x, c23.z}, sn[4] = {c01.y, c01.w, c23.y, c23.w};
#pragma unroll
    for (int i = 0; i < 4; ++i) rotate(lo[i], hi[i], cs[i], sn[i]);
  }
  if (which == 0) {
    if (e.q) {
      float* q = e.q + (size_t)m * d + head * dh + j;
      *reinterpret_cast<float4*>(q) = make_float4(lo[0], lo[1], lo[2], lo[3]);
      *reinterpret_cast<float4*>(q + half) = make_float4(hi[0], hi[1], hi[2], hi[3]);
    }
    return;
  }
  const int p = e.context_lens[m];
  const bool p_ok = (unsigned)p < (unsigned)(e.max_blocks * 16);
  const int blk = e.block_tables[(size_t)(e.row_table ? safe_row(e.row_table[m], e.table_rows) : m) * e.max_blocks + (p_ok ? p >> 4 : 0)];
  if (!p_ok || (unsigned)blk >= (unsigned)e.num_blocks) return;   // never outside the pools
  const size_t at = (((size_t)blk * e.n_heads + head) * 16 + (p & 15)) * dh + j;
  bf16_t* pool = reinterpret_cast<bf16_t*>(which == 1 ? e.k_pool : e.v_pool);
  typedef bf16_t bf16x4 __attribute__((ext_vector_type(4)));
  *reinterpret_cast<bf16x4*>(pool + at) = bf16x4{(bf16_t)lo[0], (bf16_t)lo[1], (bf16_t)lo[2], (bf16_t)lo[3]};
  *reinterpret_cast<bf16x4*>(pool + at + half) = bf16x4{(bf16_t)hi[0], (bf16_t)hi[1], (bf16_t)hi[2], (bf16_t)hi[3]};
}

// SwiGLU product; f_lo is the gate row f, f_hi the up row f + d_ffn.
template <class T>
__device__ inline void epi_gateup(const GateUpEpi& e, int m, int f, float gate, float up) {
  const float a = gate / (1.0f + expf(-gate)) * up;
  if constexpr (sizeof(T) == 2) {
    reinterpret_cast<bf16_t*>(e.act)[xt_index(m, f, e.d_ffn)] = (bf16_t)a;
  } else {
    reinterpret_cast<float*>(e.act)[(size_t)m * e.d_ffn + f] = a;
  }
}

// SwiGLU products of four consecutive features f0..f0+3 (f0 a multiple of 4), bf16 operand-tile order: one 8-byte store.
__device__ inline void epi_gateup4(const GateUpEpi& e, int m, int f0, const float (&gate)[4], const float (&up)[4]) {
  typedef bf16_t bf16x4 __attribute__((ext_vector_type(4)));
  bf16x4 out;
#pragma unroll
  for (int i = 0; i < 4; ++i) out[i] = (bf16_t)(gate[i] / (1.0f + expf(-gate[i])) * up[i]);
  *reinterpret_cast<bf16x4*>(reinterpret_cast<bf16_t*>(e.act) + xt_index(m, f0, e.d_ffn)) = out;
}

// Running softmax statistics of one row: largest and second largest (unscaled) logit, index of the largest
// (lowest index on ties) and sum of exp(scale * (z - max)).
struct HeadStat {
  float zmax, sum, z2;
  int idx;
};
// exp of a non-positive argument for the softmax sums: the hardware's base-2 exponential (relative error about 1e-7;
// the library routine costs several times the instructions, and an exit head evaluates one per logit and row)
__device__ inline float stat_exp(float x) { return __expf(x); }
constexpr int STAT_NO_INDEX = 0x7fffffff;   // no logit yet, or none that equals the largest: all of them NaN
__device__ inline HeadStat stat_empty() { return {-INFINITY, 0.0f, -INFINITY, STAT_NO_INDEX}; }
__device__ inline HeadStat stat_merge(const HeadStat& a, const HeadStat& b, float scale) {
  HeadStat o;
  if (a.zmax > b.zmax || (a.zmax == b.zmax && a.idx < b.idx)) {
    o.zmax = a.zmax;
    o.idx = a.idx;
    o.z2 = fmaxf(a.z2, b.zmax);
  } else {
    o.zmax = b.zmax;
    o.idx = b.idx;
    o.z2 = fmaxf(b.z2, a.zmax);
  }
  const float wa = a.sum > 0.0f ? a.sum * stat_exp(scale * (a.zmax - o.zmax)) : 0.0f;
  const float wb = b.sum > 0.0f ? b.sum * stat_exp(scale * (b.zmax - o.zmax)) : 0.0f;
  o.sum = wa + wb;
  return o;
}
// Statistics of 32 logits of one row that sit four each in eight neighbouring lanes (lane & 7 = which four):
// two short passes (largest with its index, then the sum of exponentials and the runner-up) instead of 32
// dependent pushes.  z[i] has vocabulary index idx0 + i.  Every one of the eight lanes returns the result.
__device__ inline HeadStat stat_of_8x4(const float (&z)[4], int idx0, float scale) {
  float best = z[0];
  int bi = idx0;
#pragma unroll
  for (int i = 1; i < 4; ++i)
    if (z[i] > best) {   // strict: the lowest index wins among equals
      best = z[i];
      bi = idx0 + i;
    }
#pragma unroll
  for (int x = 1; x < 8; x <<= 1) {
    const float ob = __shfl_xor(best, x);
    const int oi = __shfl_xor(bi, x);
    if (ob > best || (ob == best && oi < bi)) {
      best = ob;
      bi = oi;
    }
  }
  float sum = 0.0f, z2 = -INFINITY;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    sum += stat_exp(scale * (z[i] - best));
    if (idx0 + i != bi) z2 = fmaxf(z2, z[i]);
  }
#pragma unroll
  for (int x = 1; x < 8; x <<= 1) {
    sum += __shfl_xor(sum, x);
    z2 = fmaxf(z2, __shfl_xor(z2, x));
  }
  return {best, sum, z2, bi};
}

__device__ inline float4 stat_pack(const HeadStat& s) { return make_float4(s.zmax, s.sum, s.z2, __int_as_float(s.idx)); }
__device__ inline HeadStat stat_unpack(const float4& v) { return {v.x, v.y, v.z, __float_as_int(v.w)}; }

__device__ inline bool pred_skip(const Pred& p) { return p.flag && ((ctl_load(p.flag) != 0) != (p.run_when != 0)); }

}  // namespace ee
