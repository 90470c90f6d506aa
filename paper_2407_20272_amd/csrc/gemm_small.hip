// bf16 projections of an iteration of up to eight sequences (v_mfma_f32_16x16x32_bf16): a weight streamer whose operand is small
// enough that every workgroup builds it for itself, so that a layer needs no launch for it: QKV, gate/up and the LM head take the
// residual rows and normalise them (the arithmetic of finish_norm_kernel, in its order), the output and down projections add to them.
//   * A wavefront load is 16 output rows x 32 of the contraction (half a packed tile, two contraction steps): a workgroup owns whole
//     contractions of 16 or 32 output rows, its four wavefronts a quarter of each, so nothing is left for another launch to add.
//   * Every wavefront walks its loads, over all of its tiles, as one stream SM_SETS - 1 groups ahead; sums of a tile meet in LDS and one
//     wavefront finishes them while the others go on.  The first weights are asked for before the operand is built.
// 7B shape, two layers: 1 sequence at 1000 positions 246 -> 217 us, 2 sequences of three layers 366 -> 332, 4 sequences 300 -> 275.  One trace of
// the first, both sides: QKV 21.9 -> 19.0, gate/up 31.7 -> 29.5, LM head 43.6 -> 42.3, output 8.4 -> 7.7, two normalisations of 4 to 5 us a layer gone; the
// down projection went 16.7 -> 17.4 (whole contractions in two passes of a workgroup, not eight slices), for the 5 us of the normalisation that
// added its slices.  What bounds it: the weights, 6.2 TB/s in the LM head, and the start of six launches a layer.
#include <type_traits>

#include "ee_common.h"
#include "ee_epilogue.h"
#include "ee_decide.h"
#include "ee_begin.h"

namespace ee {
namespace {

constexpr int NW = 4;        // wavefronts per workgroup
constexpr int SM_U = 4;      // loads of a group
constexpr int SM_SETS = 4;   // groups in registers (6 x 4: 217 -> 224 us, 3 x 4 217, 4 x 3 220, 6 x 2 220, 12 x 2 229, 4 x 8 226; the case above)
constexpr int SM_WGS = 256;  // workgroups: one per compute unit
constexpr int SM_OPERAND = 24576;   // channels of all rows
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

// Operand: RMSNorm of float rows, of embedding rows, float rows (all in LDS), bf16 rows (fetched with the weights: where a workgroup has one 16-row unit,
// as in the down projection of the 7B shape, nothing would be read twice).
enum { X_NORM, X_EMBED, X_F32, X_ROWS };

struct NoJob {};

__host__ __device__ constexpr int x_row_bytes(int K) { return 2 * K + 64; }   // (64: rows start 16 banks apart)
constexpr int lds_bytes(int K, int R, int XM) {
  const int n = (XM == X_ROWS ? 0 : R * x_row_bytes(K)) + 64 + 2 * NW * 2 * R * 16 * 4 + R * 32;
  return n < 4096 ? 4096 : n;   // (a carried decision takes 4096)
}

// Workgroup barrier that leaves global loads in flight.
__device__ inline void meet() {
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

// Sum over the wavefront in the order of __shfl_xor over 32, 16, .. 1 (rows of 16 rotated: what a step leaves repeats twice as often).
__device__ inline float wave_sum(float v) {
  v += __shfl_xor(v, 32);
  v += __shfl_xor(v, 16);
  auto ror = [](float x, auto n) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x120 + decltype(n)::value, 0xf, 0xf, false));
  };
  v += ror(v, std::integral_constant<int, 8>{});
  v += ror(v, std::integral_constant<int, 4>{});
  v += ror(v, std::integral_constant<int, 2>{});
  return v + ror(v, std::integral_constant<int, 1>{});
}

// R: batch rows (columns of the product); NG: groups of 2048 channels that a row has at most; RU: output rows of a unit.  RU = 8: a
// wavefront load is 8 rows x 64 of the contraction, the second 32 as rows 8 to 15 of the first operand against columns 8 to 15 of the
// second, so that both sets of sums come out of one instruction (and two that nobody needs).
template <class Epi, int R, int XM, int NG, int RU, class Job>
__global__ __launch_bounds__(256) void gemm_small_kernel(SmallShape g, Epi e, Pred pred, Job job) {
  extern __shared__ __align__(16) unsigned char sm[];
  constexpr bool QKV = std::is_same<Epi, QkvEpi>::value, ACC = std::is_same<Epi, AccEpi>::value, LM = std::is_same<Epi, LmEpi>::value;
  constexpr bool NORM = XM == X_NORM || XM == X_EMBED;
  int bx = blockIdx.x;
  bool skip = false;
  if constexpr (std::is_same<Job, CombineJob>::value) {   // leading workgroups: the exit decision of the layer before (see gemm_mfma_kernel)
    const bool ran = layer_ran(job.a.s, job.a.layer);
    if (bx < job.n_wg) {
      if (bx < job.a.B && ran) combine_row(job.a, bx, reinterpret_cast<float4*>(sm));
      return;
    }
    skip = !ran;
    bx -= job.n_wg;
  } else if constexpr (XM == X_EMBED) {   // .. or the start of the iteration
    const int lead = gridDim.x - g.wgs;
    if (bx < lead) {
      begin_row_small(job, bx);
      return;
    }
    bx -= lead;
  } else {
    skip = pred_skip(pred);
  }

  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int K = g.K, k_steps = K >> 4, row_bytes = x_row_bytes(K);
  constexpr int FULL = 32 / RU, SPL = RU == 16 ? 2 : 4;   // units of a tile; contraction steps of a load
  static_assert(RU == 16 || (ACC && R <= 8), "columns 8 to 15 are taken");
  // This workgroup's units: whole tiles (two halves, finished together) first, then single halves (or quarters), as even as they come.
  const int per = g.whole / g.wgs, rem = g.whole % g.wgs, most = (2 * g.whole + g.halves + g.wgs - 1) / g.wgs;
  const int tiles = per + (bx < rem ? 1 : 0), tile0 = bx * per + min(bx, rem);
  const int room1 = max(0, most - 2 * (per + 1)), room0 = max(0, most - 2 * per);   // halves behind per + 1 and per tiles
  const int half0 = min(g.halves, bx < rem ? bx * room1 : rem * room1 + (bx - rem) * room0);
  const int halves = min(g.halves - half0, bx < rem ? room1 : room0);
  const int nh = 2 * tiles + halves;
  if (nh == 0) return;
  auto unit_of = [&](int j, int& tile, int& half) {   // of the j-th half
    if (j < 2 * tiles) {
      tile = tile0 + (j >> 1);
      half = j & 1;
    } else {
      const int x = half0 + j - 2 * tiles;
      tile = g.whole + x / FULL;
      half = x % FULL;
    }
  };
  // this wavefront's share of every contraction, in loads
  const int P = (k_steps + SPL - 1) / SPL, p0 = P * wave / NW, p1 = P * (wave + 1) / NW, nc = max(1, (p1 - p0 + SM_U - 1) / SM_U);

  // ---- operand loads -------------------------------------------------------------------------------------
  static_assert(XM == X_ROWS || R * NG <= 16, "all rows in registers");
  float v[R][NG][8];
  bf16x8 gv[NG];
  auto load_rows = [&] {
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
      for (int i = 0; i < NG; ++i) {
        if constexpr (XM == X_EMBED) {
          const int tok = job.tokens[min(r, g.M - 1)];
          const bf16x8 e8 = *reinterpret_cast<const bf16x8*>(job.embed + (size_t)((unsigned)tok < (unsigned)job.vocab ? tok : 0) * K +
                                                             min((i * 256 + (int)threadIdx.x) * 8, K - 8));
#pragma unroll
          for (int x = 0; x < 8; ++x) v[r][i][x] = (float)e8[x];
          continue;
        }
        const float* p = reinterpret_cast<const float*>(g.x) + (size_t)min(r, g.M - 1) * K + min((i * 256 + (int)threadIdx.x) * 8, K - 8);
        const float4 a = *reinterpret_cast<const float4*>(p), b = *reinterpret_cast<const float4*>(p + 4);
        v[r][i][0] = a.x; v[r][i][1] = a.y; v[r][i][2] = a.z; v[r][i][3] = a.w;
        v[r][i][4] = b.x; v[r][i][5] = b.y; v[r][i][6] = b.z; v[r][i][7] = b.w;
      }
  };
  if constexpr (XM != X_ROWS) load_rows();
  if constexpr (NORM) {
#pragma unroll
    for (int i = 0; i < NG; ++i) gv[i] = *reinterpret_cast<const bf16x8*>(g.gain + min((i * 256 + (int)threadIdx.x) * 8, K - 8));
  }
  // what the epilogue looks up: lane -> (result row lane % 16, batch rows lane / 16 + 4 q)
  constexpr int MG = (R + 3) / 4;
  const int r16 = lane & 15, m0 = lane >> 4, row = lane & (RU - 1);
  int pos[MG], block[MG];
  bool write[MG];
  float2 turn[MG];
  float h_in[MG];
#pragma unroll
  for (int q = 0; q < MG; ++q) {
    const int m = m0 + 4 * q, mm = min(m, g.M - 1);
    write[q] = m < g.M;
    if constexpr (QKV) pos[q] = e.context_lens[mm];
    if constexpr (ACC) write[q] = write[q] && !(e.skip && ctl_load(e.skip + mm) != 0);
  }
  auto look = [&](int j) {   // for the unit that starts with half j
    int tile, half;
    unit_of(j, tile, half);
#pragma unroll
    for (int q = 0; q < MG; ++q) {
      const int mm = min(m0 + 4 * q, g.M - 1);
      if constexpr (QKV) {
        const int f0 = packed_row_lo(tile, 0, g.pair_stride);
        if (f0 < 2 * e.d_model && e.rope_theta > 0.0f) turn[q] = XM == X_EMBED ? rope_turn(pos[q], f0 % e.head_dim + r16, e.head_dim, e.rope_theta)
                                : e.rope[(size_t)mm * (e.head_dim >> 1) + f0 % e.head_dim + r16];
      }
      if constexpr (ACC) h_in[q] = e.h[(size_t)mm * e.n_out + tile * 32 + half * RU + row];
    }
  };
  if constexpr (XM != X_EMBED) look(0);
  asm volatile("" ::: "memory");   // all of this is asked for ahead of the weights
  if (skip) return;

  // ---- the stream ----------------------------------------------------------------------------------------
  u32x4 W[SM_SETS][SM_U], X[XM == X_ROWS ? SM_SETS : 1][SM_U];
  // the 8 of the contraction that this lane holds of a load: RU = 16: lane / 16; RU = 8: 4 * (lane / 8 % 2) + lane / 16, of both operands
  const int eight = RU == 16 ? m0 : ((lane >> 3) & 1) * 4 + m0;
  const unsigned lane_off = (unsigned)((eight >> 1) * 1024 + (eight & 1) * 512 + row * 16);
  // a last load that is not full: what is missing of it repeats the last step, against zeros
  const int p_odd = k_steps % SPL ? P - 1 : -1, odd_back = max(0, (eight >> 1) - (k_steps - 1 - (P - 1) * SPL));
  const unsigned lane_odd = lane_off - odd_back * 1024;
  const int col = RU == 16 ? r16 : lane & 7;   // batch row of this lane's column
  const char* xg = reinterpret_cast<const char*>(g.x) + ((size_t)min(col, g.M - 1) * K + eight * 8) * 2;   // (direct operand)
  int ji = 0, ci = 0;
  auto base_of = [&](int j) {
    int tile, half;
    unit_of(min(j, nh - 1), tile, half);
    return reinterpret_cast<const char*>(g.w) + (size_t)tile * k_steps * 1024 + half * (RU * 16);
  };
  const char* from = base_of(0);
  auto issue = [&](u32x4 (&w)[SM_U], u32x4 (&x)[SM_U]) {
#pragma unroll
    for (int u = 0; u < SM_U; ++u) {
      const int p = max(0, min(p0 + ci * SM_U + u, p1 - 1));
      const unsigned off = ji >= nh ? 0u : p == p_odd ? lane_odd : lane_off;   // past the end: 16 bytes, never used
      w[u] = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(from + (size_t)p * (SPL * 1024) + off));
      if constexpr (XM == X_ROWS) x[u] = *reinterpret_cast<const u32x4*>(xg + p * (SPL * 32) - (p == p_odd ? odd_back * 32 : 0));
    }
    if (++ci == nc) {
      ci = 0;
      from = base_of(++ji);
    }
  };
  auto set_x = [&](int s) -> u32x4(&)[SM_U] { return X[XM == X_ROWS ? s : 0]; };
#pragma unroll
  for (int s = 0; s < SM_SETS - 1; ++s) issue(W[s], set_x(s));
  asm volatile("" ::: "memory");

  if constexpr (XM == X_EMBED) look(0);   // (angles: behind the first weights)

  // ---- operand to LDS ------------------------------------------------------------------------------------
  unsigned char* zero16 = sm + (XM == X_ROWS ? 0 : R * row_bytes);
  float* red = reinterpret_cast<float*>(zero16 + 64);              // [2][NW][2][R][16]
  float* sums = red + 2 * NW * 2 * R * 16;                         // [R][8]
  if (threadIdx.x < 4) reinterpret_cast<unsigned*>(zero16)[threadIdx.x] = 0;
  if constexpr (QKV) {
#pragma unroll
    for (int q = 0; q < MG; ++q) {
      const bool ok = (unsigned)pos[q] < (unsigned)(e.max_blocks * 16);
      block[q] = e.block_tables[(size_t)min(m0 + 4 * q, g.M - 1) * e.max_blocks + (ok ? pos[q] >> 4 : 0)];
      write[q] = write[q] && ok;
    }
  }
  if constexpr (XM != X_ROWS) {
    float rinv[R];
    if constexpr (NORM) {
      // the order of finish_norm_kernel: its thread t = (i % 2) * 256 + threadIdx.x owns what v[..][i] and v[..][i + 2] hold
#pragma unroll
      for (int r = 0; r < R; ++r)
#pragma unroll
        for (int i = 0; i < (NG < 2 ? NG : 2); ++i) {
          float ss = 0.0f;
#pragma unroll
          for (int c = i; c < NG; c += 2) {
            float t = ss;
#pragma unroll
            for (int x = 0; x < 8; ++x) t = fmaf(v[r][c][x], v[r][c][x], t);
            if ((c * 256 + (int)threadIdx.x) * 8 < K) ss = t;
          }
          ss = wave_sum(ss);
          if (lane == 0) sums[r * 8 + i * NW + wave] = ss;
        }
      meet();
#pragma unroll
      for (int r = 0; r < R; ++r) {
        float t = 0.0f;
#pragma unroll
        for (int w = 0; w < (NG < 2 ? 4 : 8); ++w) t += sums[r * 8 + w];
        rinv[r] = rsqrtf(t / (float)K + g.eps);
      }
    }
#pragma unroll
    for (int i = 0; i < NG; ++i) {
      const int k0 = (i * 256 + (int)threadIdx.x) * 8;
      if (k0 < K) {
#pragma unroll
        for (int r = 0; r < R; ++r) {
          bf16x8 o;
#pragma unroll
          for (int x = 0; x < 8; ++x) o[x] = NORM ? (bf16_t)(v[r][i][x] * rinv[r] * (float)gv[i][x]) : (bf16_t)v[r][i][x];
          *reinterpret_cast<bf16x8*>(sm + r * row_bytes + k0 * 2) = o;
        }
      }
    }
  }
  meet();

  // ---- multiply ------------------------------------------------------------------------------------------
  const unsigned char* xl = sm + (col < R ? col : 0) * row_bytes + eight * 16;   // column of this lane (past the rows: row 0, unused)
  f32x4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
  int j = 0, c = 0, unit = 0, slot = 0;   // half and group that are multiplied; unit, and half of it
  auto finish = [&](int tile, int half, bool whole) {   // by one wavefront: the sums of a unit, in wavefront order
    const float* s0 = red + (size_t)(unit & 1) * NW * 2 * R * 16;
    auto sum = [&](int hf, int mr, int row) {
      float t = 0.0f;
#pragma unroll
      for (int w = 0; w < NW; ++w) t += s0[((w * 2 + hf) * R + mr) * 16 + row];
      return t;
    };
    if constexpr (LM) {
#pragma unroll
      for (int m8 = 0; m8 < R; m8 += 8) {
        const int ml = m8 + (lane >> 3), part = lane & 7;
        if (ml < R) {
          float z[4];
#pragma unroll
          for (int i = 0; i < 4; ++i) z[i] = sum(part >> 2, ml, (part & 3) * 4 + i);
          const HeadStat st = stat_of_8x4(z, tile * 32 + part * 4, e.scale);
          if (part == 0 && ml < g.M) e.partials[(size_t)ml * e.n_parts + tile] = stat_pack(st);
        }
      }
    } else {
#pragma unroll
      for (int q = 0; q < MG; ++q) {
        const int m = m0 + 4 * q;
        if (m >= g.M) break;
        float lo = sum(0, m, row), hi = whole || RU == 8 ? sum(1, m, row) : 0.0f;
        if (RU == 8) lo += hi;
        if constexpr (ACC) {
          if (write[q] && r16 < RU) e.h[(size_t)m * e.n_out + tile * 32 + half * RU + row] = h_in[q] + lo;
        } else if constexpr (QKV) {
          const int d = e.d_model, dh = e.head_dim, f0 = packed_row_lo(tile, 0, g.pair_stride);
          const int which = f0 / d, head = (f0 - which * d) / dh, ch = f0 % dh + r16 + (half ? dh >> 1 : 0);
          if (which < 2 && e.rope_theta > 0.0f) rotate(lo, hi, turn[q].x, turn[q].y);
          if (which == 0) {
            float* to = e.q + (size_t)m * d + head * dh + ch;
            to[0] = lo;
            to[dh >> 1] = hi;
          } else if (write[q] && (unsigned)block[q] < (unsigned)e.num_blocks) {   // never outside the pools
            bf16_t* to = reinterpret_cast<bf16_t*>(which == 1 ? e.k_pool : e.v_pool) + (((size_t)block[q] * e.n_heads + head) * 16 + (pos[q] & 15)) * dh + ch;
            to[0] = (bf16_t)lo;
            if (whole) to[dh >> 1] = (bf16_t)hi;
          }
        } else {
          reinterpret_cast<bf16_t*>(e.act)[(size_t)m * e.d_ffn + packed_row_lo(tile, r16, g.pair_stride)] = (bf16_t)(lo / (1.0f + expf(-lo)) * hi);
        }
      }
    }
  };
  auto multiply = [&](const u32x4 (&w)[SM_U], const u32x4 (&x)[SM_U]) {
    if (j >= nh) return;
#pragma unroll
    for (int u = 0; u < SM_U; ++u) {
      const int p = p0 + c * SM_U + u;
      bf16x8 b;
      if constexpr (XM == X_ROWS) {
        const bool in = p < p1 && !(p == p_odd && odd_back > 0);
        b = __builtin_bit_cast(bf16x8, in ? x[u] : u32x4{0, 0, 0, 0});
      } else {
        b = *reinterpret_cast<const bf16x8*>(p < p1 ? xl + p * (SPL * 32) : zero16);   // (rows are whole loads: K is a multiple of 64)
      }
      acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, w[u]), b, acc, 0, 0, 0);
    }
    if (++c < nc) return;
    c = 0;
    if constexpr (RU == 16) {
      if (r16 < R) *reinterpret_cast<f32x4*>(red + (((size_t)(unit & 1) * NW + wave) * 2 + slot) * R * 16 + r16 * 16 + m0 * 4) = acc;
    } else {   // rows 0 to 7 of columns 0 to 7, and 8 to 15 of 8 to 15
      if (col < R && r16 >> 3 == m0 >> 1)
        *reinterpret_cast<f32x4*>(red + (((size_t)(unit & 1) * NW + wave) * 2 + (m0 >> 1)) * R * 16 + col * 16 + (m0 & 1) * 4) = acc;
    }
    acc = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    const bool whole = j < 2 * tiles;
    if (whole && slot == 0) {
      slot = 1;
      ++j;
      return;
    }
    meet();   // (two sets of sums: the next but one unit overwrites these behind another meeting)
    int tile, half;
    unit_of(j, tile, half);
    if (wave == (unit & (NW - 1))) finish(tile, whole ? 0 : half, whole);
    ++unit;
    slot = 0;
    if (++j < nh) look(j);
  };
  const int total = nh * nc;
  for (int i = 0; i < total; i += SM_SETS) {
#pragma unroll
    for (int s = 0; s < SM_SETS; ++s) {
      issue(W[(s + SM_SETS - 1) % SM_SETS], set_x((s + SM_SETS - 1) % SM_SETS));
      multiply(W[s], set_x(s));
    }
  }
}

// go(rows, groups of 2048 channels of a row) as constants (gemm_small_takes: eight rows are no wider than 3072).
template <class Go>
void for_shape(int M, int K, Go go) {
  const auto rows = [&](auto ng) {
    if (M == 1) return go(std::integral_constant<int, 1>{}, ng);
    if (M == 2) return go(std::integral_constant<int, 2>{}, ng);
    if constexpr (decltype(ng)::value == 4) return go(std::integral_constant<int, 4>{}, ng);
    else return M <= 4 ? go(std::integral_constant<int, 4>{}, ng) : go(std::integral_constant<int, 8>{}, ng);
  };
  if (K <= 2048) return rows(std::integral_constant<int, 1>{});
  if (K <= 4096) return rows(std::integral_constant<int, 2>{});
  return rows(std::integral_constant<int, 4>{});
}

template <class Epi, int XM, int RU, class Job = NoJob>
void launch(SmallShape g, const Epi& e, Pred pred, hipStream_t st, int lead = 0, const Job& job = Job{}) {
  const int units = g.whole + g.halves;
  g.wgs = units < SM_WGS ? units : SM_WGS;
  for_shape(g.M, XM == X_ROWS ? 0 : g.K, [&](auto r, auto ng) {
    constexpr int R = decltype(r)::value, NG = XM == X_ROWS ? 1 : decltype(ng)::value;   // (that operand passes through no registers)
    // (launch_acc's rule: the output projection takes units of 8 rows up to 2048 channels, never from there to 4096)
    if constexpr (XM != X_F32 || NG != (RU == 8 ? 2 : 1))
      hipLaunchKernelGGL((gemm_small_kernel<Epi, R, XM, NG, RU, Job>), dim3(g.wgs + lead), dim3(256), lds_bytes(g.K, R, XM), st, g, e, pred, job);
  });
}
// Accumulate projections: units of 8 rows where fewer rows then fall to the busiest compute unit (d = 5120: 24 instead of 32).
template <int XM>
void launch_acc(SmallShape g, const AccEpi& e, Pred pred, hipStream_t st) {
  const int d = e.n_out, by16 = (d / 16 + SM_WGS - 1) / SM_WGS * 16, by8 = (d / 8 + SM_WGS - 1) / SM_WGS * 8;
  g.whole = 0;
  g.halves = by8 < by16 ? d / 8 : d / 16;
  if (by8 < by16) launch<AccEpi, XM, 8>(g, e, pred, st);
  else launch<AccEpi, XM, 16>(g, e, pred, st);
}

}  // namespace

// Every workgroup builds the whole operand, so its rows times its channels are what this costs, and launches are what it saves.
// Whole iterations, the other kernels' time over this one's: 1 and 2 rows 1.04 (d = 5120) to 1.4 (1024); 3 and 4 rows 1.09 (4096), 1.00
// (5120), 1.05 (6144); 5 to 8 rows 0.90 (5120), 0.99 to 1.01 (4096), 1.01 (3584), 1.02 (3072), 1.10 (2048), 1.17 (640); 384 and 512 1.00 to 1.03
// without exit checks, 0.98 to 1.00 with checks of 1280 words, 0.93 to 0.96 of 8000 and 0.90 to 0.95 of 32000 (few threads hold all rows, and the
// head is a large part); 9 to 16 rows 0.84 (4096), 0.6 (256).
// The head alone loses where a workgroup has several tiles of short contractions (each an end of its own: a meeting and one wavefront's
// epilogue): 32000 words, exit check of 4 rows, 64 / 256 / 384 / 640 / 1024 / 2048 channels 0.86, 0.92, 1.02, 1.02, 1.10, 1.15, of 1 and 2 rows 0.90, 0.95,
// 1.04, 1.03, 1.13, 1.15, of 8 rows from 384 on 0.97, 0.97, 1.06, 1.13; 8000 words, one tile each, 1.07 and more everywhere.  In an iteration it
// saves no launch of its own: of 3 and 4 rows and 32000 words 0.95 (64 channels), 0.96 (192), 1.00 (256); of 1 and 2 rows 0.99 to 1.05.
bool gemm_small_takes(int B, int d, int head_tiles) {
  const int R = B <= 2 ? B : B <= 4 ? 4 : 8;
  if (R == 4 && d < 256 && head_tiles > SM_WGS) return false;
  return B <= 8 && R * d <= SM_OPERAND && (R < 8 || d >= (head_tiles ? 640 : 384));   // (no more than 64 KiB of LDS)
}
bool gemm_small_takes_check(int B, int d, int head_tiles) {
  if (B > 8 || (B <= 2 ? B : B <= 4 ? 4 : 8) * d > SM_OPERAND) return false;
  return head_tiles <= SM_WGS || d >= (B <= 4 ? 384 : 1024);
}
void launch_small_qkv(const SmallShape& g, const QkvEpi& e, Pred pred, hipStream_t st, const CombineArgs* with_combine) {
  if (!with_combine) {
    launch<QkvEpi, X_NORM, 16>(g, e, pred, st);
    return;
  }
  CombineJob cj{};
  cj.a = *with_combine;
  cj.kind = 1;
  cj.n_wg = (cj.a.B + 7) / 8 * 8;
  launch<QkvEpi, X_NORM, 16>(g, e, pred, st, cj.n_wg, cj);
}
void launch_small_begin_qkv(const BeginArgs& begin, const SmallShape& g, const QkvEpi& e, hipStream_t st) {
  const int rope_wgs = begin.theta > 0.0f ? (begin.B * (begin.head_dim / 2) + 255) / 256 : 0;
  launch<QkvEpi, X_EMBED, 16>(g, e, Pred{nullptr, 0}, st, (begin.B + rope_wgs + 7) / 8 * 8, begin);
}
void launch_small_oproj(const SmallShape& g, const AccEpi& e, Pred pred, hipStream_t st) { launch_acc<X_F32>(g, e, pred, st); }
void launch_small_gateup(const SmallShape& g, const GateUpEpi& e, Pred pred, hipStream_t st) { launch<GateUpEpi, X_NORM, 16>(g, e, pred, st); }
void launch_small_down(const SmallShape& g, const AccEpi& e, Pred pred, hipStream_t st) { launch_acc<X_ROWS>(g, e, pred, st); }
void launch_small_lm(const SmallShape& g, const LmEpi& e, Pred pred, hipStream_t st) { launch<LmEpi, X_NORM, 16>(g, e, pred, st); }

}  // namespace ee
