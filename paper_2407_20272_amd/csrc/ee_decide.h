// Exit decision of one layer (Section 3.1), shared by the stand-alone decision kernels and by the QKV projection
// launches that carry the previous layer's decision along.
#pragma once

#include "ee_common.h"
#include "ee_epilogue.h"

namespace ee {

// Section 3.1 status rule for one sequence: an accepted sequence stays accepted (and is not re-checked);
// otherwise the confidence (or the forced exit layer) decides; the last acceptance of the batch raises `done`.
__device__ inline void decide_row(const IterState& s, int m, int B, int layer, float conf, float threshold,
                                  const int32_t* forced_exit_layer, float* conf_out) {
  if (ctl_load(s.status + m) != 0) {
    if (conf_out) conf_out[m] = __builtin_nanf("");
    return;
  }
  if (conf_out) conf_out[m] = conf;
  const bool accepted = forced_exit_layer ? (layer >= forced_exit_layer[m]) : (conf > threshold);
  if (!accepted) return;
  ctl_store(s.status + m, 1);
  ctl_store(s.exit_layer + m, layer);
  const int before = __hip_atomic_fetch_add(s.n_exited, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  if (before + 1 == B) {
    ctl_store(s.batch_exit_layer, layer);
    ctl_store(s.done, 1);
  }
}

// Did layer `layer` run?  It did if the batch has not left, or left at that very layer or later.  The launch that takes the
// layer's decision raises `done` itself, so the live flag alone would tell the workgroups (and wavefronts) that read it late
// to leave out rows accepted at an earlier layer, whose tokens come from this one.  A `done` raised by this launch comes with
// batch_exit_layer == layer or, not yet visible, its initial n_layers; one raised at an earlier layer with that layer's
// number, both visible since an earlier launch.  So every reader of the launch gets the same answer, whenever it reads.
__device__ inline bool layer_ran(const IterState& s, int layer) {
  const int32_t done = ctl_load(s.done), at = ctl_load(s.batch_exit_layer);   // (side by side: behind the exit both are needed)
  return done == 0 || at >= layer;
}
// Had sequence m left at an earlier layer than `layer`?  For a launch that takes layer `layer`'s decision and skips the sequences that have left:
// their status words change under its readers, and wavefronts of one workgroup that disagree do half of its work (half of a block table in LDS,
// say).  The exit layer changes as well, but only from n_layers to `layer`, neither of which is less than it, so that every reader gets the same
// answer here too.
__device__ inline bool left_before(const IterState& s, int m, int layer) { return ctl_load(s.exit_layer + m) < layer; }
// Whether a launch that takes layer `layer`'s decision has nothing to do (layer 0, the final token selection, raises nothing).
__device__ inline bool decision_skip(const Pred& pred, const IterState& s, int layer) {
  return layer > 0 && pred.flag ? !layer_ran(s, layer) : pred_skip(pred);
}

// Confidence and arg max of row m from its softmax statistics, then the status rule.  One thread.
__device__ inline void decide_from_stat(const CombineArgs& a, int m, const HeadStat& s) {
  if (a.argmax_out) a.argmax_out[m] = s.idx == STAT_NO_INDEX ? 0 : s.idx;   // a row of NaN: any token, but one of the vocabulary
  if (a.layer == 0) return;
  float conf = 1.0f / s.sum;                                          // largest softmax probability
  if (a.conf_mode == 1) conf = (1.0f - expf(a.scale * (s.z2 - s.zmax))) / s.sum;  // top-1 minus top-2
  decide_row(a.s, m, a.B, a.layer, conf, a.threshold, a.forced_exit_layer, a.conf_out);
}

// One workgroup of 256 threads merges the per-tile softmax statistics of row m into the confidence and applies
// the status rule.  red: 256 float4 of LDS.  layer == 0: final token selection only.
__device__ inline void combine_row(const CombineArgs& a, int m, float4* red) {
  if (a.left && ctl_load(a.left + m) != 0) return;   // left at an earlier layer: its token and exit layer stand
  HeadStat s = stat_empty();
  for (int i = threadIdx.x; i < a.n_parts; i += blockDim.x)
    s = stat_merge(s, stat_unpack(a.partials[(size_t)m * a.n_parts + i]), a.scale);
  red[threadIdx.x] = stat_pack(s);
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if (threadIdx.x < w)
      red[threadIdx.x] = stat_pack(stat_merge(stat_unpack(red[threadIdx.x]), stat_unpack(red[threadIdx.x + w]), a.scale));
    __syncthreads();
  }
  if (threadIdx.x == 0) decide_from_stat(a, m, stat_unpack(red[0]));
}

// fp32 path: softmax statistics of row m of materialised logits and the decision from them.  One workgroup of 256 threads; red:
// four float4 of LDS.
__device__ inline void decide_row_f32(const float* logits, const float* row_scale, int vocab, CombineArgs a, int m, float4* red) {
  if (a.left && ctl_load(a.left + m) != 0) return;   // left at an earlier layer: its token and exit layer stand
  // largest logit with its index and the runner-up first, the exponentials relative to the wavefront's largest after
  HeadStat s = stat_empty();
  a.scale *= row_scale[m];
  const float* z = logits + (size_t)m * vocab;
  constexpr int AHEAD = 8;   // loads in flight: one at a time a row of 32000 took 53 us, now 24
  auto each = [&](auto take) {
    for (int v0 = threadIdx.x; v0 < vocab; v0 += 256 * AHEAD) {
      float x[AHEAD];
#pragma unroll
      for (int i = 0; i < AHEAD; ++i) x[i] = z[min(v0 + 256 * i, vocab - 1)];
#pragma unroll
      for (int i = 0; i < AHEAD; ++i)
        if (v0 + 256 * i < vocab) take(v0 + 256 * i, x[i]);
    }
  };
  each([&](int v, float x) {
    if (x > s.zmax || s.idx == STAT_NO_INDEX) {   // strict: the lowest index wins among equals
      s.z2 = fmaxf(s.z2, s.zmax);
      s.zmax = x;
      s.idx = v;
    } else {
      s.z2 = fmaxf(s.z2, x);
    }
  });
#pragma unroll
  for (int x = 1; x < 64; x <<= 1) {
    const float ob = __shfl_xor(s.zmax, x), o2 = __shfl_xor(s.z2, x);
    const int oi = __shfl_xor(s.idx, x);
    const bool take = ob > s.zmax || (ob == s.zmax && oi < s.idx);
    s.z2 = fmaxf(fmaxf(s.z2, o2), take ? s.zmax : ob);
    if (take) {
      s.zmax = ob;
      s.idx = oi;
    }
  }
  each([&](int, float x) { s.sum += stat_exp(a.scale * (x - s.zmax)); });
#pragma unroll
  for (int x = 1; x < 64; x <<= 1) s.sum += __shfl_xor(s.sum, x);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = stat_pack(s);
  __syncthreads();
  if (threadIdx.x != 0) return;
#pragma unroll
  for (int w = 1; w < 4; ++w) s = stat_merge(s, stat_unpack(red[w]), a.scale);
  decide_from_stat(a, m, s);
}

// Confidence of row m from one dot product (hidden states similarity, dedicated classifier) and the status rule.
__device__ inline void decide_from_sums(const DecideArgs& a, int m, float dot, float sq_a, float sq_b) {
  float conf;
  if (a.conf_mode == 2) {
    conf = dot / (sqrtf(sq_a) * sqrtf(sq_b));
  } else {
    conf = 1.0f / (1.0f + expf(-(dot * rsqrtf(sq_b / (float)a.d + a.eps) + a.bias[0])));
  }
  decide_row(a.s, m, a.B, a.layer, conf, a.threshold, a.forced_exit_layer, a.conf_out);
}
__device__ inline void decide_from_dot(const DecideArgs& a, int m) {
  decide_from_sums(a, m, a.dots[m], a.conf_mode == 2 ? a.sq_a[m] : 0.0f, a.sq_b[m]);
}

}  // namespace ee
