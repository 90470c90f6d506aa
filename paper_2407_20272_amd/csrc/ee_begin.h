// Start of an iteration, shared by the launches that begin with it.
#pragma once

#include "ee_common.h"

namespace ee {

// ---------------------------------------------------------------------------------------------------
// Status <- False for sequence m (Algorithm 1, initialisation), no confidence yet; row 0: the counters.  One workgroup a row.
// ---------------------------------------------------------------------------------------------------
__device__ inline void init_row(const IterState& s, int m, int B, int n_layers, float* conf_out) {
  if (threadIdx.x == 0) {
    s.status[m] = 0;
    s.exit_layer[m] = n_layers;
    if (m == 0) {
      *s.n_exited = 0;
      *s.done = 0;
      *s.batch_exit_layer = n_layers;
    }
  }
  if (conf_out && (int)threadIdx.x < n_layers) conf_out[(size_t)threadIdx.x * B + m] = __builtin_nanf("");
}

// (cos, sin) of pos * theta^(-2j/dh), the angle formed in double.
__device__ inline float2 rope_turn(int pos, int j, int head_dim, float theta) {
  const double ang = (double)pos * exp2(-2.0 * (double)j / (double)head_dim * log2((double)theta));
  double sn, cs;
  sincos(ang, &sn, &cs);
  return make_float2((float)cs, (float)sn);
}
// The same for every sequence m and channel pair j.
__device__ inline void rope_entry(const int32_t* context_lens, float2* table, int idx, int B, int head_dim, float theta) {
  const int half = head_dim >> 1;
  if (idx >= B * half) return;
  const int m = idx / half, j = idx - m * half;
  table[idx] = rope_turn(context_lens[m], j, head_dim, theta);
}
__device__ inline const float* embed_row_f32(const float* embed, int tok, int vocab, int d) {
  return embed + (size_t)((unsigned)tok < (unsigned)vocab ? tok : 0) * d;   // never outside the table
}
// fp32 path, workgroup wg of 256 threads: the first B take a row each, those behind them the rotary table.
__device__ inline void begin_row_f32(const BeginArgs& a, int wg) {
  const int m = wg, d = a.d;
  if (m >= a.B) {
    if (a.theta > 0.0f) rope_entry(a.context_lens, a.rope, (m - a.B) * 256 + threadIdx.x, a.B, a.head_dim, a.theta);
    return;
  }
  init_row(a.s, m, a.B, a.n_layers, a.conf_out);
  const float* row = embed_row_f32(a.embed_f32, a.tokens[m], a.vocab, d);
  for (int k = threadIdx.x; k < d; k += 256) {
    const float v = row[k];
    a.h[(size_t)m * d + k] = v;
    if (a.snapshot) a.snapshot[(size_t)m * d + k] = v;
  }
}
// bf16 path, rows that are normalised by whoever multiplies them (gemm_small.hip), workgroup wg of 256 threads: as above, from rows of whole 16-byte loads.
__device__ inline void begin_row_small(const BeginArgs& a, int wg) {
  const int m = wg, d = a.d;
  if (m >= a.B) {
    if (a.theta > 0.0f) rope_entry(a.context_lens, a.rope, (m - a.B) * 256 + threadIdx.x, a.B, a.head_dim, a.theta);
    return;
  }
  init_row(a.s, m, a.B, a.n_layers, a.conf_out);
  const int tok = a.tokens[m];
  const bf16_t* row = a.embed + (size_t)((unsigned)tok < (unsigned)a.vocab ? tok : 0) * d;   // never outside the table
  for (int k = threadIdx.x * 8; k < d; k += 256 * 8) {
    const bf16x8 e = *reinterpret_cast<const bf16x8*>(row + k);
    float* h = a.h + (size_t)m * d + k;
    *reinterpret_cast<float4*>(h) = make_float4((float)e[0], (float)e[1], (float)e[2], (float)e[3]);
    *reinterpret_cast<float4*>(h + 4) = make_float4((float)e[4], (float)e[5], (float)e[6], (float)e[7]);
  }
}

}  // namespace ee
