// fp32 projections (plain row-major weights): the small reference-shaped workload runs entirely in float.
// One wavefront computes one pair of output rows for MC batch rows (its row block): lanes stride over the
// contraction, 16 bytes at a time where the operands allow it, and a halving exchange adds the 64 partial sums, so that
// four lanes finish the four batch rows side by side.  A projection of a normalised operand takes the residual rows
// themselves: every wavefront sums the squares of its rows beside the products (the rows are a few kilobytes in L1) and the
// separate normalisation launches are gone.  What bounds this path at small widths is the chain of dependent launches, and in each of
// them the chain of dependent loads (predicate, operands, what the epilogue looks up): a launch took 4 to 5 us for work of well under
// one.  So the launches are few (ee_decode_iteration) and what a launch reads is asked for at once, behind its predicate.
// One iteration of four sequences and four layers of width 256, leaving at layer 3: 65 launches and 217 us with a launch a step, 27
// and 98 us with norms and decisions inside the projections, 19 and 83 us with four launches a layer, 75 us with the operands asked for at once,
// 73 with no second layer-4 projection in KV filling, 18 and 71 us with the start in the first projection's launch, 67 with
// every predicate ahead of the operands.
#include <type_traits>

#include "ee_common.h"
#include "ee_epilogue.h"
#include "ee_decide.h"
#include "ee_begin.h"

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
      const float a = v[i], b = v[i + n], keep = up ? b : a, give = up ? a : b;
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
      const float a = v[i], b = v[i + n], keep = up ? b : a, give = up ? a : b;
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
struct BeginJob {   // the first projection of an iteration: leading workgroups begin it, the others read the embedding rows themselves
  BeginArgs a;
  int n_wg;
};

// What an epilogue reads of batch row m besides the sums.  It is asked for with the first operands: behind the sums it would be a
// chain of dependent loads at the end of a launch that takes a few microseconds.
struct RowOf {
  int pos, block;     // QKV: the row's position and the physical block of it
  bool write;
  float2 turn;        // (cos, sin)
  float lo, hi;       // residual update: what is added to
};
// at: position of the row where the rotary table is not there yet (BEGIN).
template <class Epi, bool BEGIN>
__device__ inline RowOf row_of(const Epi& e, int m, int f_lo, int f_hi, int at) {
  RowOf r{};
  r.write = true;
  if constexpr (std::is_same<Epi, QkvEpi>::value) {
    const int d = e.d_model, dh = e.head_dim, half = dh >> 1, which = f_lo / d, j = (f_lo - which * d) % dh;
    r.write = !kv_filled(e, m);
    if (which < 2 && e.rope_theta > 0.0f) r.turn = BEGIN ? rope_turn(at, j, dh, e.rope_theta) : e.rope[(size_t)m * half + j];
    if (which > 0) {
      r.pos = e.context_lens[m];
      const bool ok = (unsigned)r.pos < (unsigned)(e.max_blocks * 16);
      r.block = e.block_tables[(size_t)(e.row_table ? safe_row(e.row_table[m], e.table_rows) : m) * e.max_blocks + (ok ? r.pos >> 4 : 0)];
      r.write = r.write && ok && (unsigned)r.block < (unsigned)e.num_blocks;   // never outside the pools
    }
  } else if constexpr (std::is_same<Epi, AccEpi>::value) {
    const float* h = (e.h_in ? e.h_in : e.h) + (size_t)m * e.n_out;
    r.lo = h[f_lo];
    r.hi = h[f_hi];
    r.write = !(e.skip && ctl_load(e.skip + m) != 0);
  }
  return r;
}
// Rotary embedding (split-half pairing: channel j with j + dh/2) and the write of this position's K/V into the paged cache; q goes
// to a dense buffer.
__device__ inline void put_qkv(const QkvEpi& e, const RowOf& r, int m, int f_lo, float lo, float hi) {
  const int d = e.d_model, dh = e.head_dim, half = dh >> 1;
  const int which = f_lo / d;  // 0 q, 1 k, 2 v
  const int within = f_lo - which * d, head = within / dh, j = within - head * dh;
  if (!r.write) return;
  if (which < 2 && e.rope_theta > 0.0f) rotate(lo, hi, r.turn.x, r.turn.y);
  float* to;
  if (which == 0) {
    if (!e.q) return;
    to = e.q + (size_t)m * d + head * dh + j;
  } else {
    to = reinterpret_cast<float*>(which == 1 ? e.k_pool : e.v_pool) + (((size_t)r.block * e.n_heads + head) * 16 + (r.pos & 15)) * dh + j;
  }
  to[0] = lo;
  to[half] = hi;
}

// One workgroup (bx of those of a projection) of four wavefronts, a pair of output rows each.  PARTS: the operand comes in parts
// (SimpleShape::parts).  PIECES > 0: the contraction is at most that many times 256, and all of a wavefront's operands are asked for at
// once.  layer: of KV filling.
template <class Epi, bool NORM, bool VEC, bool PARTS, int PIECES, class Fill, class Job = NoJob>
__device__ __forceinline__ void simple_body(SimpleShape g, Epi e, const Fill& fill, int bx, int layer, const Job& job = Job{}) {
  constexpr bool FILL = std::is_same<Fill, SimpleFill>::value, BEGIN = std::is_same<Job, BeginJob>::value;
  // The row blocks of one group of weight rows get ids 8 apart: they run on one XCD at the same time, and all but the first
  // read of a weight row hit its L2.  With the row blocks outermost every block fetched the whole matrix from beyond the L2:
  // LM head of 32000 x 4096 and 32 rows 985 us (rows looped over in the wavefront, the form before: 665), now 570; gate/up
  // of 22016 x 4096 and 64 rows 1370 (1150), now 706.
  const int first = blockIdx.y * ROW_BLOCKS, row_blocks = min(ROW_BLOCKS, (g.M + MC - 1) / MC - first), slot = bx >> 3;
  const int m0 = (first + slot % row_blocks) * MC;
  if constexpr (FILL) {   // one slice of the grid per layer; nothing to do where every row has been cached already
    bool need = false;
    for (int m = m0; m < min(m0 + MC, g.M); ++m) need |= ctl_load(e.fill_from + (size_t)m * e.fill_from_stride) + e.fill_lead < layer;
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
  for (int i = 0; i < MC; ++i) {   // rows past the last repeat it, never written
    const int mi = min(m0 + i, g.M - 1);
    if constexpr (BEGIN) x[i] = embed_row_f32(g.x, job.a.tokens[mi], job.a.vocab, g.K);
    else x[i] = g.x + (size_t)mi * g.K;
  }
  int at = 0;
  if constexpr (BEGIN) at = job.a.context_lens[min(m0 + (lane >> 4), g.M - 1)];   // (ahead of the operands: loads return in order)
  float sum[2 * MC], sq[MC];   // sum[2 i + hi]
#pragma unroll
  for (int i = 0; i < MC; ++i) sum[2 * i] = sum[2 * i + 1] = sq[i] = 0.0f;
  constexpr int N = VEC ? 4 : 1;
  typedef float vec_t __attribute__((ext_vector_type(N)));
  constexpr int PN = PARTS ? 4 : 1;
  struct Piece {
    vec_t a, b, gn, x[MC], p[PN][MC];
  };
  auto load = [&](Piece& v, int k) {
    v.a = *reinterpret_cast<const vec_t*>(w_lo + k);
    v.b = *reinterpret_cast<const vec_t*>(w_hi + k);
    if constexpr (NORM) v.gn = *reinterpret_cast<const vec_t*>(g.gain + k);
#pragma unroll
    for (int i = 0; i < MC; ++i) v.x[i] = *reinterpret_cast<const vec_t*>(x[i] + k);
    if constexpr (PARTS) {   // (four at most: 256 channels, heads of 64 and more)
#pragma unroll
      for (int q = 0; q < PN; ++q)
#pragma unroll
        for (int i = 0; i < MC; ++i)
          v.p[q][i] = *reinterpret_cast<const vec_t*>(g.parts + ((size_t)min(q, g.n_parts - 1) * g.M + min(m0 + i, g.M - 1)) * g.K + k);
    }
  };
  auto multiply = [&](Piece& v, int k) {
    if constexpr (PARTS) {
#pragma unroll
      for (int i = 0; i < MC; ++i) {
        const int m = min(m0 + i, g.M - 1);
        vec_t p = v.p[0][i];
#pragma unroll
        for (int q = 1; q < PN; ++q) p = q < g.n_parts ? p + v.p[q][i] : p;
        if (!(g.left && ctl_load(g.left + m) != 0)) v.x[i] += p;   // (a sequence that has left: its parts may not have been written)
        if (pair == 0 && m0 + i < g.M) *reinterpret_cast<vec_t*>(g.x_out + (size_t)m * g.K + k) = v.x[i];
      }
    }
#pragma unroll
    for (int i = 0; i < MC; ++i)
#pragma unroll
      for (int j = 0; j < N; ++j) {
        const float xv = v.x[i][j], u = NORM ? xv * v.gn[j] : xv;
        if constexpr (NORM) sq[i] = fmaf(xv, xv, sq[i]);
        sum[2 * i] = fmaf(v.a[j], u, sum[2 * i]);
        sum[2 * i + 1] = fmaf(v.b[j], u, sum[2 * i + 1]);
      }
  };
  static_assert(MC == 4, "eight sums, four squares");
  const int m = m0 + (lane >> 4);   // batch row that this lane's sixteen finish
  RowOf row{};
  if constexpr (PIECES > 0) {
    Piece v[PIECES];
#pragma unroll
    for (int c = 0; c < PIECES; ++c) load(v[c], min(c * 64 * N + lane * N, g.K - N));
    row = row_of<Epi, BEGIN>(e, min(m, g.M - 1), f_lo, f_hi, at);
    asm volatile("" ::: "memory");   // the loads above stay above
#pragma unroll
    for (int c = 0; c < PIECES; ++c)
      if (c * 64 * N + lane * N < g.K) multiply(v[c], c * 64 * N + lane * N);
  } else {
#pragma unroll 2
    for (int k = lane * N; k < g.K; k += 64 * N) {
      Piece v;
      load(v, k);
      multiply(v, k);
    }
    row = row_of<Epi, BEGIN>(e, min(m, g.M - 1), f_lo, f_hi, at);
  }
  float r = wave_sums8(sum, lane);      // lane bits 5, 4: batch row, bit 3: lo / hi
  if constexpr (NORM) {
    const float rinv = 1.0f / sqrtf(wave_sums4(sq, lane) / (float)g.K + g.eps);
    if constexpr (std::is_same<Epi, LmEpi>::value) {
      // The logits stay as the sums they are and the decision scales their differences: one rounding of every logit less
      // (confidences are off by 3.2e-7 as with a normalised operand, not 3.7e-7; 37 rows, width 256, logits times 12).
      if (pair == 0 && (lane & 15) == 0 && m < g.M) e.row_scale[m] = rinv;
    } else {
      r *= rinv;
    }
  }
  const float lo = r, hi = __shfl_xor(r, 8);
  if ((lane & 15) != 0 || m >= g.M) return;
  if constexpr (std::is_same<Epi, QkvEpi>::value) {
    put_qkv(e, row, m, f_lo, lo, hi);
  } else if constexpr (std::is_same<Epi, AccEpi>::value) {
    if (row.write) {   // every element of the residual stream has one contributor per launch
      e.h[(size_t)m * e.n_out + f_lo] = row.lo + lo;
      e.h[(size_t)m * e.n_out + f_hi] = row.hi + hi;
    }
  } else if constexpr (std::is_same<Epi, GateUpEpi>::value) {
    epi_gateup<float>(e, m, f_lo, lo, hi);
  } else {
    e.logits[(size_t)m * e.vocab + f_lo] = lo;
    e.logits[(size_t)m * e.vocab + f_hi] = hi;
  }
}

// Every launch looks at its predicate first, and asks for its operands behind it: behind the exit there are four launches a layer with nothing
// to do, and one that had asked for its operands took 3 us instead of 1.7 (a wavefront stays until its loads are back, also where the
// predicate was asked for ahead of them).  Width 256, 24 layers, 4 / 64 sequences that leave at layer 2: 267 / 489 us with the operands first,
// 181 / 319 with the predicate first.
// What the launch was given is fetched ahead of that: behind the branch the compiler would fetch it in a second trip (0.15 us a launch:
// 24 layers that all run, 4 sequences, 404 -> 392 us).
__device__ __forceinline__ void args_first(const SimpleShape& g) {
  asm volatile("" ::"s"(g.w), "s"(g.x), "s"(g.gain), "s"(g.K), "s"(g.M), "s"(g.n_rows), "s"(g.pair_stride));
}

template <class Epi, bool NORM, bool VEC, bool PARTS, int PIECES, class Fill, class Job>
__global__ __launch_bounds__(256) void gemm_simple_kernel(SimpleShape g, Epi e, Pred pred, Fill fill, Job job) {
  int bx = blockIdx.x;
  const int layer = blockIdx.z + 1;
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
    simple_body<Epi, NORM, VEC, PARTS, PIECES>(g, e, fill, bx, layer);
  } else if constexpr (std::is_same<Job, BeginJob>::value) {
    if (bx < job.n_wg) {
      if (blockIdx.y == 0) begin_row_f32(job.a, bx);
      return;
    }
    simple_body<Epi, NORM, VEC, PARTS, PIECES>(g, e, fill, bx - job.n_wg, layer, job);
  } else {
    args_first(g);
    if (pred_skip(pred)) return;
    simple_body<Epi, NORM, VEC, PARTS, PIECES>(g, e, fill, bx, layer);
  }
}

// Two launches in one: the LM head (its workgroups in front) and a projection of the same hidden states that needs no result of it:
// the next layer's QKV, or KV filling of every layer (wgs workgroups each).  In one dimension: as a grid of layers the head's workgroups
// were there once a layer, and all but one of them empty.
template <bool VEC, int PIECES, class Fill>
__global__ __launch_bounds__(256) void gemm_simple_head_kernel(SimpleShape gh, LmEpi eh, Pred ph, SimpleShape g, QkvEpi e, Pred pred, Fill fill, int head_wgs,
                                                               int wgs) {
  args_first(gh);
  args_first(g);
  if ((int)blockIdx.x < head_wgs) {
    if (pred_skip(ph)) return;
    simple_body<LmEpi, true, VEC, false, PIECES>(gh, eh, NoFill{}, blockIdx.x, 0);
    return;
  }
  if (pred_skip(pred)) return;
  const int at = (int)blockIdx.x - head_wgs, layer = at / wgs;
  simple_body<QkvEpi, true, VEC, false, PIECES>(g, e, fill, at - layer * wgs, layer + 1);
}

bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15) == 0; }

// Workgroups of a projection along grid.x: groups of eight side by side, times up to ROW_BLOCKS row blocks.
int workgroups(const SimpleShape& g) {
  const int row_blocks = (g.M + MC - 1) / MC;
  return ((g.n_rows / 2 + 3) / 4 + 7) / 8 * 8 * (row_blocks < ROW_BLOCKS ? row_blocks : ROW_BLOCKS);
}
// 16-byte loads need rows that keep the alignment and operands that start on it (the library asks no caller for that)
bool vectors(const SimpleShape& g) { return g.K % 4 == 0 && aligned16(g.w) && aligned16(g.x) && aligned16(g.gain); }
bool vectors(const SimpleFill& fill, int n_layers) {
  for (int i = 0; i < n_layers; ++i)
    if (!aligned16(fill.layers.w_qkv[i]) || !aligned16(fill.gains.g[i])) return false;
  return true;
}

// Contractions of up to 256 have their operands in registers at once (SHORT: there are no others).  So do those of up to 1024 where the launch
// has no more workgroups than compute units (four layers, four sequences: width 320 87 us in a loop, 81 so; width 640 108 and 103): from there
// on the other wavefronts of a compute unit hide the chain of dependent loads, and 146 registers a lane leave too few of them (four layers,
// 16 / 500 rows of width 512: 266 / 2623 us so, 118 / 1370 in a loop; 64 rows of width 1024 925 and 642).
template <bool SHORT, class Go>
void for_pieces(bool vec, int K, long wgs, Go go) {
  if (vec && K <= 256) return go(std::true_type{}, std::integral_constant<int, 1>{});
  if constexpr (!SHORT) {
    if (vec && K <= 1024 && wgs <= 256) return go(std::true_type{}, std::integral_constant<int, 4>{});
    if (vec) return go(std::true_type{}, std::integral_constant<int, 0>{});
  }
  go(std::false_type{}, std::integral_constant<int, 0>{});
}

template <class Epi, bool NORM, bool PARTS = false, class Fill = NoFill, class Job = NoJob>
void launch(const SimpleShape& g, const Epi& e, Pred pred, hipStream_t st, const Fill& fill = Fill{}, int n_layers = 1, const Job& job = Job{}) {
  const int row_blocks = (g.M + MC - 1) / MC;
  int lead = 0;
  if constexpr (!std::is_same<Job, NoJob>::value) lead = job.n_wg;
  const dim3 grid(workgroups(g) + lead, (row_blocks + ROW_BLOCKS - 1) / ROW_BLOCKS, n_layers);
  bool vec = vectors(g);
  if constexpr (std::is_same<Fill, SimpleFill>::value) vec = vec && vectors(fill, n_layers);
  auto go = [&](auto vec_c, auto pieces_c) {
    hipLaunchKernelGGL((gemm_simple_kernel<Epi, NORM, decltype(vec_c)::value, PARTS, decltype(pieces_c)::value, Fill, Job>), grid, dim3(256), 0, st, g, e,
                       pred, fill, job);
  };
  for_pieces<PARTS || std::is_same<Job, BeginJob>::value>(vec, g.K, (long)grid.x * grid.y * grid.z, go);
}
template <class Fill>
void launch_with_head(const SimpleShape& gh, const LmEpi& eh, Pred ph, const SimpleShape& g, const QkvEpi& e, Pred pred, const Fill& fill, int n_layers,
                      bool vec, hipStream_t st) {
  const int lead = workgroups(gh), wgs = workgroups(g);
  const dim3 grid(lead + wgs * n_layers);   // (both of one group of row blocks: the host sees to that)
  auto go = [&](auto vec_c, auto pieces_c) {
    hipLaunchKernelGGL((gemm_simple_head_kernel<decltype(vec_c)::value, decltype(pieces_c)::value, Fill>), grid, dim3(256), 0, st, gh, eh, ph, g, e, pred,
                       fill, lead, wgs);
  };
  for_pieces<true>(vec && vectors(gh), g.K, grid.x, go);
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
void launch_simple_begin_qkv(const BeginArgs& begin, const SimpleShape& g, const QkvEpi& e, hipStream_t st) {
  const int rope_wgs = begin.theta > 0.0f ? (begin.B * (begin.head_dim / 2) + 255) / 256 : 0;
  launch<QkvEpi, true>(g, e, Pred{nullptr, 0}, st, NoFill{}, 1, BeginJob{begin, (begin.B + rope_wgs + 7) / 8 * 8});
}
void launch_simple_head_qkv(const SimpleShape& gh, const LmEpi& eh, const SimpleShape& g, const QkvEpi& e, Pred pred, hipStream_t st) {
  launch_with_head(gh, eh, pred, g, e, pred, NoFill{}, 1, vectors(g), st);
}
void launch_simple_head_kvfill(const SimpleShape& gh, const LmEpi& eh, Pred ph, const SimpleFill& fill, int n_layers, const SimpleShape& g, const QkvEpi& e,
                               Pred pred, hipStream_t st) {
  launch_with_head(gh, eh, ph, g, e, pred, fill, n_layers, vectors(g) && vectors(fill, n_layers), st);
}
void launch_simple_acc(const SimpleShape& g, const AccEpi& e, Pred pred, hipStream_t st) { launch<AccEpi, false>(g, e, pred, st); }
void launch_simple_gateup(const SimpleShape& g, const GateUpEpi& e, Pred pred, hipStream_t st) {
  if (g.parts) launch<GateUpEpi, true, true>(g, e, pred, st);
  else launch<GateUpEpi, true>(g, e, pred, st);
}
void launch_simple_lm(const SimpleShape& g, const LmEpi& e, Pred pred, hipStream_t st) { launch<LmEpi, true>(g, e, pred, st); }
void launch_simple_kvfill(const SimpleFill& fill, int n_layers, const SimpleShape& g, const QkvEpi& e, Pred pred, hipStream_t st) {
  launch<QkvEpi, true, false>(g, e, pred, st, fill, n_layers);
}

}  // namespace ee
