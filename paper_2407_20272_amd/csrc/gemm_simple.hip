// fp32 projections (plain row-major weights): the small reference-shaped workload runs entirely in float.
// One wavefront computes one pair of output rows for MC batch rows (its row block): lanes stride over the
// contraction, 16 bytes at a time where the operands allow it, and a halving exchange adds the 64 partial sums, so that
// four lanes finish the four batch rows side by side.  A projection of a normalised operand takes the residual rows
// themselves: every wavefront sums the squares of its rows beside the products (the rows are a few kilobytes in L1) and the
// separate normalisation launches are gone.  What bounds this path at small widths is the number of dependent launches, 3 to 4
// us each: one iteration of four layers of width 256 took 65 launches and 217 us, 30
// launches and 110 us in this form, 27 and 100 us with the exit decisions inside the QKV launches.
#include <type_traits>

#include "ee_common.h"
#include "ee_epilogue.h"
#include "ee_decide.h"

namespace ee {
namespace {

constexpr int MC = 4;            // batch rows per wavefront
constexpr int ROW_BLOCKS = 64;   // row blocks side by side in grid.x; grid.y holds the rest (a grid dimension counts less than 2^32 threads)

// Sums of v[0..7] over the wavefront: the lane of bits 5, 4, 3 = i gets sum i in every lane of its eight.
__device__ inline float wave_sums8(float (&v)[8], int lane) {
#pragma unroll
  for (int n = 4, bit = 32; n >= 1; n >>= 1, bit >>= 1) {
    const bool up = (lane & bit) != 0;
#pragma unroll
    for (int i = 0; i < n; ++i) {
      const float keep = up ? v[i + n] : v[i], give = up ? v[i] : v[i + n];
      v[i] = keep + __shfl_xor(give, bit);
    }
  }
  float s = v[0];
#pragma unroll
  for (int x = 4; x >= 1; x >>= 1) s += __shfl_xor(s, x);
  return s;
}
// The same for four sums, lane bits 5, 4.
__device__ inline float wave_sums4(float (&v)[4], int lane) {
#pragma unroll
  for (int n = 2, bit = 32; n >= 1; n >>= 1, bit >>= 1) {
    const bool up = (lane & bit) != 0;
#pragma unroll
    for (int i = 0; i < n; ++i) {
      const float keep = up ? v[i + n] : v[i], give = up ? v[i] : v[i + n];
      v[i] = keep + __shfl_xor(give, bit);
    }
  }
  float s = v[0];
#pragma unroll
  for (int x = 8; x >= 1; x >>= 1) s += __shfl_xor(s, x);
  return s;
}

struct NoFill {};   // (a launch that fills nothing does not carry a kilobyte of layer tables)
struct NoJob {};

template <class Epi, bool NORM, bool VEC, class Fill, class Job>
__global__ __launch_bounds__(256) void gemm_simple_kernel(SimpleShape g, Epi e, Pred pred, Fill fill, Job job) {
  constexpr bool FILL = std::is_same<Fill, SimpleFill>::value;
  int bx = blockIdx.x;
  if constexpr (std::is_same<Job, SimpleDecision>::value) {
    // Leading workgroups: the exit decision of the layer before, one row each.  The projection's own apply the same rule
    // (layer_ran), not the live flag: the projection of the layer after the batch exit layer runs, and what it caches is what KV
    // filling caches there.
    const bool ran = layer_ran(job.a.s, job.a.layer);
    if (bx < job.n_wg) {
      __shared__ float4 red[4];
      if (blockIdx.y == 0 && bx < job.a.B && ran) decide_row_f32(job.logits, job.row_scale, job.vocab, job.a, bx, red);
      return;
    }
    if (!ran) return;
    bx -= job.n_wg;
  } else if (pred_skip(pred)) {
    return;
  }
  // The row blocks of one group of weight rows get ids 8 apart: they run on one XCD at the same time, and all but the first
  // read of a weight row hit its L2.  With the row blocks outermost every block fetched the whole matrix from beyond the L2:
  // LM head of 32000 x 4096 and 32 rows 985 us (rows looped over in the wavefront, the form before: 665), now 570; gate/up
  // of 22016 x 4096 and 64 rows 1370 (1150), now 706.
  const int first = blockIdx.y * ROW_BLOCKS, row_blocks = min(ROW_BLOCKS, (g.M + MC - 1) / MC - first), slot = bx >> 3;
  const int m0 = (first + slot % row_blocks) * MC;
  if constexpr (FILL) {   // one slice of the grid per layer; nothing to do where every row has been cached already
    const int layer = blockIdx.z + 1;
    bool need = false;
    for (int m = m0; m < min(m0 + MC, g.M); ++m) need |= ctl_load(e.fill_from + (size_t)m * e.fill_from_stride) < layer;
    if (!need) return;
    g.w = reinterpret_cast<const float*>(fill.layers.w_qkv[layer - 1]);
    g.gain = reinterpret_cast<const float*>(fill.gains.g[layer - 1]);
    e.layer = layer;
    e.k_pool = reinterpret_cast<char*>(e.k_pool) + (size_t)(layer - 1) * fill.pool_layer_bytes;
    e.v_pool = reinterpret_cast<char*>(e.v_pool) + (size_t)(layer - 1) * fill.pool_layer_bytes;
  }
  const int lane = threadIdx.x & 63;
  const int pair = (slot / row_blocks * 8 + (bx & 7)) * 4 + (threadIdx.x >> 6);
  if (pair >= g.n_rows / 2) return;
  const int s = g.pair_stride;
  const int f_lo = g.row_begin + (pair / s) * 2 * s + pair % s;
  const int f_hi = f_lo + s;
  const float* w_lo = g.w + (size_t)f_lo * g.K;
  const float* w_hi = g.w + (size_t)f_hi * g.K;
  const float* x[MC];
#pragma unroll
  for (int i = 0; i < MC; ++i) x[i] = g.x + (size_t)min(m0 + i, g.M - 1) * g.K;   // rows past the last repeat it, never written
  float sum[2 * MC], sq[MC];   // sum[2 i + hi]
#pragma unroll
  for (int i = 0; i < MC; ++i) sum[2 * i] = sum[2 * i + 1] = sq[i] = 0.0f;
  constexpr int N = VEC ? 4 : 1;
  typedef float vec_t __attribute__((ext_vector_type(N)));
#pragma unroll 2
  for (int k = lane * N; k < g.K; k += 64 * N) {
    const vec_t a = *reinterpret_cast<const vec_t*>(w_lo + k), b = *reinterpret_cast<const vec_t*>(w_hi + k);
    vec_t gn = vec_t(1.0f);
    if constexpr (NORM) gn = *reinterpret_cast<const vec_t*>(g.gain + k);
    vec_t xv[MC];
#pragma unroll
    for (int i = 0; i < MC; ++i) xv[i] = *reinterpret_cast<const vec_t*>(x[i] + k);
#pragma unroll
    for (int i = 0; i < MC; ++i)
#pragma unroll
      for (int j = 0; j < N; ++j) {
        const float v = xv[i][j], u = NORM ? v * gn[j] : v;
        if constexpr (NORM) sq[i] = fmaf(v, v, sq[i]);
        sum[2 * i] = fmaf(a[j], u, sum[2 * i]);
        sum[2 * i + 1] = fmaf(b[j], u, sum[2 * i + 1]);
      }
  }
  static_assert(MC == 4, "eight sums, four squares");
  float r = wave_sums8(sum, lane);      // lane bits 5, 4: batch row, bit 3: lo / hi
  if constexpr (NORM) {
    const float rinv = 1.0f / sqrtf(wave_sums4(sq, lane) / (float)g.K + g.eps);
    if constexpr (std::is_same<Epi, LmEpi>::value) {
      // The logits stay as the sums they are and the decision scales their differences: one rounding of every logit less
      // (confidences are off by 3.2e-7 as with a normalised operand, not 3.7e-7; 37 rows, width 256, logits times 12).
      if (pair == 0 && (lane & 15) == 0 && m0 + (lane >> 4) < g.M) e.row_scale[m0 + (lane >> 4)] = rinv;
    } else {
      r *= rinv;
    }
  }
  const float lo = r, hi = __shfl_xor(r, 8);
  const int m = m0 + (lane >> 4);
  if ((lane & 15) != 0 || m >= g.M) return;
  if constexpr (std::is_same<Epi, QkvEpi>::value) {
    epi_qkv<float>(e, m, f_lo, lo, hi);
  } else if constexpr (std::is_same<Epi, AccEpi>::value) {
    epi_acc(e, m, f_lo, lo);
    epi_acc(e, m, f_hi, hi);
  } else if constexpr (std::is_same<Epi, GateUpEpi>::value) {
    epi_gateup<float>(e, m, f_lo, lo, hi);
  } else {
    e.logits[(size_t)m * e.vocab + f_lo] = lo;
    e.logits[(size_t)m * e.vocab + f_hi] = hi;
  }
}

bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15) == 0; }

template <class Epi, bool NORM, class Fill = NoFill, class Job = NoJob>
void launch(const SimpleShape& g, const Epi& e, Pred pred, hipStream_t st, const Fill& fill = Fill{}, int n_layers = 1, const Job& job = Job{}) {
  const int row_blocks = (g.M + MC - 1) / MC;
  int lead = 0;
  if constexpr (std::is_same<Job, SimpleDecision>::value) lead = job.n_wg;
  const dim3 grid(((g.n_rows / 2 + 3) / 4 + 7) / 8 * 8 * (row_blocks < ROW_BLOCKS ? row_blocks : ROW_BLOCKS) + lead,
                  (row_blocks + ROW_BLOCKS - 1) / ROW_BLOCKS, n_layers);
  // 16-byte loads need rows that keep the alignment and operands that start on it (the library asks no caller for that)
  bool vec = g.K % 4 == 0 && aligned16(g.w) && aligned16(g.x) && aligned16(g.gain);
  if constexpr (std::is_same<Fill, SimpleFill>::value)
    for (int i = 0; i < n_layers; ++i) vec = vec && aligned16(fill.layers.w_qkv[i]) && aligned16(fill.gains.g[i]);
  if (vec)
    hipLaunchKernelGGL((gemm_simple_kernel<Epi, NORM, true, Fill, Job>), grid, dim3(256), 0, st, g, e, pred, fill, job);
  else
    hipLaunchKernelGGL((gemm_simple_kernel<Epi, NORM, false, Fill, Job>), grid, dim3(256), 0, st, g, e, pred, fill, job);
}

}  // namespace

void launch_simple_qkv(const SimpleShape& g, const QkvEpi& e, Pred pred, hipStream_t st, const SimpleDecision* with) {
  if (!with) {
    launch<QkvEpi, true>(g, e, pred, st);
    return;
  }
  SimpleDecision job = *with;
  job.n_wg = (job.a.B + 7) / 8 * 8;   // a multiple of 8: the projection's workgroups keep their XCDs
  launch<QkvEpi, true>(g, e, pred, st, NoFill{}, 1, job);
}
void launch_simple_acc(const SimpleShape& g, const AccEpi& e, Pred pred, hipStream_t st) { launch<AccEpi, false>(g, e, pred, st); }
void launch_simple_gateup(const SimpleShape& g, const GateUpEpi& e, Pred pred, hipStream_t st) {
  launch<GateUpEpi, true>(g, e, pred, st);
}
void launch_simple_lm(const SimpleShape& g, const LmEpi& e, Pred pred, hipStream_t st) { launch<LmEpi, true>(g, e, pred, st); }
void launch_simple_kvfill(const SimpleFill& fill, int n_layers, const SimpleShape& g, const QkvEpi& e, Pred pred, hipStream_t st) {
  launch<QkvEpi, true>(g, e, pred, st, fill, n_layers);
}

}  // namespace ee
