// bf16 projections of the decode step on the matrix cores (v_mfma_f32_32x32x16_bf16).  Four kernels, by batch size:
//
//   gemm_mfma_kernel   QKV of one or two 32-row batch tiles, output projection of one (of two where blocks gain nothing), weight
//                      tiles that do not come in fours up to 128 rows where blocks gain nothing: a weight streamer.
//                      Every weight byte is fetched from HBM exactly once, straight into registers (1 KiB of
//                      consecutive bytes per wavefront load thanks to the packed tile order), the small activation
//                      operand comes out of L2.  A workgroup of four wavefronts owns one 32-row output tile and splits
//                      the contraction four ways; the partial tiles meet in LDS.
//   gemm_tiled_kernel  LM head and gate/up up to 128 rows, accumulate projections up to 128 rows of a long contraction (8192 on) or,
//                      from 65 rows, onto more than 128 tiles, KV filling, LM heads of more rows where blocks gain nothing: the
//                      four wavefronts own different output tiles over the same contraction range and share the activation
//                      operand through LDS; 128-row chunks.
//   gemm_block_kernel  everything else: blocks of rows x columns, both operands through LDS, brought by wavefronts that do
//                      nothing else.
//   gemm_ring_kernel   LM head at 385-512 rows (gate/up where its blocks fit one round and others do not), where the matrix cores
//                      are what counts: 256 x 256 blocks.
//
// The epilogues (rotary + paged cache write, partial results of the residual updates, SwiGLU, exit-head softmax
// statistics) run on the finished sums, from LDS in the first kernel and from registers in the others.
//
// The second operand is bf16 in operand-tile order: the attention output, the SwiGLU product, or the normalised
// hidden state written by finish_norm_kernel.  (Building the normalised operand on the fly from the float residual
// stream inside the loop was tried and measured slower: twice the L2 traffic per weight byte plus the conversion
// arithmetic cost more than the normalisation launch they replaced.)
#include <type_traits>

#include "ee_common.h"
#include "ee_epilogue.h"
#include "ee_decide.h"

namespace ee {
namespace {

constexpr int NW = 4;  // wavefronts per workgroup
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

struct FillCtl {  // KV filling: one grid.z slice per layer
  FillLayers layers;
  const bf16_t* x_slabs;
  size_t x_slab_elems;
  size_t pool_layer_bytes;
};

struct Lds {
  float red[NW][16][64];
  float zt[32][33];
  float part[8][32];
  int flag;
};

// KV filling: should this workgroup (layer slice `layer`) return at once?  Uniform over the workgroup.  With one
// fill-from layer for the whole batch (Algorithm 1) the predicate word and that layer are fetched together: the
// workgroup waits for one memory round trip, not three, before its first weight load.
__device__ inline bool fill_skip(const Pred& pred, const QkvEpi& e, int M, int layer, int& lds_flag) {
  if (e.fill_from_stride == 0) {
    const int32_t from = ctl_load(e.fill_from);
    const int32_t flag = pred.flag ? ctl_load(pred.flag) : 0;
    if (pred.flag && ((flag != 0) != (pred.run_when != 0))) return true;
    return !(from + e.fill_lead < layer);
  }
  if (pred_skip(pred)) return true;
  if (threadIdx.x == 0) lds_flag = 0;
  __syncthreads();
  int need = 0;
  for (int m = threadIdx.x; m < M; m += blockDim.x) need |= e.fill_from[m] + e.fill_lead < layer;
  if (need) lds_flag = 1;
  __syncthreads();
  const bool any = lds_flag != 0;
  __syncthreads();
  return !any;
}

// Meets the four wavefronts' partial 32x32 tiles in LDS and runs the epilogue on the finished sums.
// Thread t owns result rows r16(a) and r16(a)+16 for a = 2*(t/64), 2*(t/64)+1 in column t%32 (+32*(t%64/32) picks
// the upper row group): the two rows that an epilogue needs together always sit in the same thread.
template <class Epi>
__device__ inline void tile_finish(const f32x16& acc, int nt, int mt_global, const GemmShape& g, const Epi& e, Lds& s,
                                   int wave, int lane, int row_half = -1) {
  __syncthreads();
#pragma unroll
  for (int a = 0; a < 16; ++a) s.red[wave][a][lane] = acc[a];
  __syncthreads();
  const int l2 = threadIdx.x & 63, qq = threadIdx.x >> 6;
  const int m = mt_global * 32 + (l2 & 31);
  float vlo[2], vhi[2];
  int r16[2];
#pragma unroll
  for (int ai = 0; ai < 2; ++ai) {
    const int a = 2 * qq + ai;
    vlo[ai] = s.red[0][a][l2] + s.red[1][a][l2] + s.red[2][a][l2] + s.red[3][a][l2];
    vhi[ai] = s.red[0][a + 8][l2] + s.red[1][a + 8][l2] + s.red[2][a + 8][l2] + s.red[3][a + 8][l2];
    r16[ai] = (a >> 2) * 8 + (l2 >> 5) * 4 + (a & 3);
  }
  if constexpr (std::is_same<Epi, LmEpi>::value) {
#pragma unroll
    for (int ai = 0; ai < 2; ++ai) {
      s.zt[r16[ai]][l2 & 31] = vlo[ai];
      s.zt[r16[ai] + 16][l2 & 31] = vhi[ai];
    }
    __syncthreads();
    {   // eight neighbouring lanes share one batch row: four logits each
      const int ml = threadIdx.x >> 3, part = threadIdx.x & 7;
      float z[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) z[i] = s.zt[part * 4 + i][ml];
      const HeadStat st = stat_of_8x4(z, nt * 32 + part * 4, e.scale);
      const int mm = mt_global * 32 + ml;
      if (part == 0 && mm < g.M) e.partials[(size_t)mm * e.n_parts + (nt - g.tile_begin)] = stat_pack(st);
    }
  } else if constexpr (std::is_same<Epi, AccEpi>::value) {
    // This workgroup summed one slice of the contraction (blockIdx.y): the tile goes to that slice of the partial
    // results with plain stores, transposed through LDS so that a batch row's 32 channels leave as whole 16-byte
    // pieces.  The normalisation launch that follows sums the slices in slice order: no atomics, no dependence on
    // which workgroup finishes first.  (Plain row order of the packed matrix: tile row r is channel nt*32 + r.)
#pragma unroll
    for (int ai = 0; ai < 2; ++ai) {
      s.zt[r16[ai]][l2 & 31] = vlo[ai];
      s.zt[r16[ai] + 16][l2 & 31] = vhi[ai];
    }
    __syncthreads();
    {
      const int mr = threadIdx.x >> 3, c0 = (threadIdx.x & 7) * 4;
      const int mm = mt_global * 32 + mr;
      if (mm < g.M) {
        const float4 v = make_float4(s.zt[c0][mr], s.zt[c0 + 1][mr], s.zt[c0 + 2][mr], s.zt[c0 + 3][mr]);
        *reinterpret_cast<float4*>(e.h + ((size_t)blockIdx.y * e.Mpad + mm) * e.n_out + nt * 32 + c0) = v;
      }
    }
  } else {
    if constexpr (std::is_same<Epi, QkvEpi>::value) {
      // The tile holds, for each of its 32 batch rows, 16 consecutive channels of one head and their 16 rotary
      // partners (half a head further on).  Rotate in registers, stage the tile in LDS, then write whole 16-channel
      // runs (one 16-byte store per thread) instead of single elements scattered over the cache blocks.
      const int d = e.d_model, dh = e.head_dim, hdim = dh >> 1;
      const int f0 = packed_row_lo(nt, 0, g.pair_stride);   // first channel of the tile (uniform)
      const int which = f0 / d;                              // 0 q, 1 k, 2 v
      const int head = (f0 - which * d) / dh;
      const int j0 = f0 - which * d - head * dh;             // < dh/2, a multiple of 16
      const int mcol = l2 & 31;
#pragma unroll
      for (int ai = 0; ai < 2; ++ai) {
        float lo = vlo[ai], hi = vhi[ai];
        if (m < g.M && which < 2 && e.rope_theta > 0.0f) {
          const float2 cs = e.rope[(size_t)m * hdim + j0 + r16[ai]];
          rotate(lo, hi, cs.x, cs.y);
        }
        s.zt[r16[ai]][mcol] = lo;
        s.zt[16 + r16[ai]][mcol] = hi;
      }
      __syncthreads();
      if (which == 0) {
        if (e.q) {   // thread -> (row, run, quarter of the run): four floats
          const int mr = threadIdx.x >> 3, part = threadIdx.x & 7, run = part >> 2, c0 = run * 16 + (part & 3) * 4;
          const int mm = mt_global * 32 + mr;
          if (mm < g.M && !kv_filled(e, mm)) {
            float4 v = make_float4(s.zt[c0][mr], s.zt[c0 + 1][mr], s.zt[c0 + 2][mr], s.zt[c0 + 3][mr]);
            *reinterpret_cast<float4*>(e.q + (size_t)mm * d + head * dh + j0 + run * hdim + (part & 3) * 4) = v;
          }
        }
      } else if (threadIdx.x < 128) {   // thread -> (row, run, half of the run): eight bf16
        const int mr = threadIdx.x >> 2, part = threadIdx.x & 3, run = part >> 1, c0 = run * 16 + (part & 1) * 8;
        const int mm = mt_global * 32 + mr;
        // a workgroup that computed one half of the tile's rows (row_half) holds one of the two runs only
        if (mm < g.M && (row_half < 0 || run == row_half) && !kv_filled(e, mm)) {
          const int p = e.context_lens[mm];
          const bool p_ok = (unsigned)p < (unsigned)(e.max_blocks * 16);
          const int blk = e.block_tables[(size_t)(e.row_table ? safe_row(e.row_table[mm], e.table_rows) : mm) * e.max_blocks + (p_ok ? p >> 4 : 0)];
          const size_t at = (((size_t)blk * e.n_heads + head) * 16 + (p & 15)) * dh + j0 + run * hdim + (part & 1) * 8;
          bf16x8 v;
#pragma unroll
          for (int i = 0; i < 8; ++i) v[i] = (bf16_t)s.zt[c0 + i][mr];
          bf16_t* pool = reinterpret_cast<bf16_t*>(which == 1 ? e.k_pool : e.v_pool);
          if (p_ok && (unsigned)blk < (unsigned)e.num_blocks) *reinterpret_cast<bf16x8*>(pool + at) = v;
        }
      }
    } else {
      if (m < g.M) {
#pragma unroll
        for (int ai = 0; ai < 2; ++ai) {
          const int f_lo = packed_row_lo(nt, r16[ai], g.pair_stride);
          epi_gateup<bf16_t>(e, m, f_lo, vlo[ai], vhi[ai]);
        }
      }
    }
  }
}

// Lane of an activation tile (row lane % 32) that this lane fetches for batch tile mt: the lanes of rows that no sequence has
// fetch what row 0's lane does, the same bytes, instead of padding (their result columns are never written): a compute unit takes
// in only so many bytes at a time, and a tile of 32 rows is as many as a weight tile.  7B shape, two layers at 1 / 33 / 47 rows
// 241.5 -> 237.7, 311.8 -> 302.5, 334 -> 327 us; KV filling of two layers at 33 rows 48.7 -> 46.1.
__device__ inline int x_lane(int lane, int mt, int M) { return mt * 32 + (lane & 31) < M ? lane : lane & 32; }

// ---------------------------------------------------------------------------------------------------------
// Main loop 1: bf16 operand tiles on both sides
// ---------------------------------------------------------------------------------------------------------
template <int MT, int NT, int U>
struct Frag {
  u32x4 w[NT][U];
  u32x4 x[MT][U];
};

template <int MT, int NT, int U>
__device__ inline void frag_load(Frag<MT, NT, U>& f, const u32x4* const (&wp)[NT], const u32x4* const (&xp)[MT], int ks) {
#pragma unroll
  for (int u = 0; u < U; ++u)
#pragma unroll
    for (int t = 0; t < NT; ++t) f.w[t][u] = __builtin_nontemporal_load(wp[t] + (size_t)(ks + u) * 64);
#pragma unroll
  for (int mt = 0; mt < MT; ++mt)
#pragma unroll
    for (int u = 0; u < U; ++u) f.x[mt][u] = xp[mt][(size_t)(ks + u) * 64];
}

// Last, partial group: steps past ks1 re-read the last valid weight tile against a zero activation tile.
template <int MT, int NT, int U>
__device__ inline void frag_load_tail(Frag<MT, NT, U>& f, const u32x4* const (&wp)[NT], const u32x4* const (&xp)[MT], int ks, int ks1) {
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const bool ok = ks + u < ks1;
    const int kk = ok ? ks + u : ks1 - 1;
#pragma unroll
    for (int t = 0; t < NT; ++t) f.w[t][u] = __builtin_nontemporal_load(wp[t] + (size_t)kk * 64);
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
      u32x4 v = xp[mt][(size_t)kk * 64];
      f.x[mt][u] = ok ? v : u32x4{0, 0, 0, 0};
    }
  }
}

template <int MT, int NT, int U>
__device__ inline void frag_mma(const Frag<MT, NT, U>& f, f32x16 (&acc)[NT][MT]) {
#pragma unroll
  for (int u = 0; u < U; ++u)
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
      for (int t = 0; t < NT; ++t)
        acc[t][mt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, f.w[t][u]),
                                                             __builtin_bit_cast(bf16x8, f.x[mt][u]), acc[t][mt], 0, 0, 0);
}

// NT = 2: a workgroup streams two output tiles, so the activation operand, which otherwise costs a compute unit as many
// bytes from L2 as the weights do from memory at 64 rows (half as many at 32), is fetched once for both: two neighbouring
// tiles, or, with one batch tile (QKV), a whole Q/K tile and half a V tile (g.split_tiles = 2 x as many whole tiles).
template <int MT, int NT, int U, class Epi, bool FILL>
__global__ __launch_bounds__(256) void gemm_mfma_kernel(GemmShape g, Epi e, Pred pred, FillCtl fc, CombineJob cj) {
  __shared__ Lds s;

  int bx = blockIdx.x;
  if constexpr (std::is_same<Epi, QkvEpi>::value && !FILL) {
    // Leading workgroups: the exit decision of the previous layer, one row each.  The projection's own workgroups apply
    // the SAME rule (layer_ran) instead of the live flag, so every workgroup of the launch takes the same branch whatever
    // the interleaving: the projection of the layer after the batch exit layer always runs (what it caches is what KV
    // filling caches there anyway), and a tile that two workgroups share is never left half done.
    if (cj.n_wg) {
      const IterState& cs = cj.kind == 1 ? cj.a.s : cj.d.s;
      const bool ran = layer_ran(cs, cj.kind == 1 ? cj.a.layer : cj.d.layer);
      if (bx < cj.n_wg) {
        if (cj.kind == 1) {
          if (bx < cj.a.B && ran) combine_row(cj.a, bx, reinterpret_cast<float4*>(&s.red[0][0][0]));
        } else if (bx == 0 && ran) {
          for (int m = threadIdx.x; m < cj.d.B; m += blockDim.x) decide_from_dot(cj.d, m);
        }
        return;
      }
      if (!ran) return;
      bx -= cj.n_wg;
    } else if (pred_skip(pred)) {
      return;
    }
  } else if constexpr (!FILL) {
    if (pred_skip(pred)) return;
  }
  if constexpr (FILL) {
    const int layer = (int)gridDim.z - (int)blockIdx.z;   // deepest layer first: the slices that have work start first
    if (fill_skip(pred, e, g.M, layer, s.flag)) return;
    g.w = fc.layers.w_qkv[layer - 1];
    g.x = fc.x_slabs + (size_t)(layer - 1) * fc.x_slab_elems;
    e.layer = layer;
    e.k_pool = reinterpret_cast<char*>(e.k_pool) + (size_t)(layer - 1) * fc.pool_layer_bytes;
    e.v_pool = reinterpret_cast<char*>(e.v_pool) + (size_t)(layer - 1) * fc.pool_layer_bytes;
  }

  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  // Tiles that two workgroups share come first in the grid (two consecutive block indices per tile): each computes
  // 16 of the tile's 32 output rows, i.e. one of its two 16-channel runs, over the whole contraction, from the half
  // of every weight tile that holds those rows (two 256-byte pieces of each kilobyte).  Both halves are complete
  // results: the workgroups share nothing and never meet.  With 384 tiles on 256 compute units this turns two rounds
  // of workgroups into one and a half.  Only tiles without a rotation may be split (V: the host sees to that).
  int nt[NT], rhalf[NT];   // this workgroup's tiles; rhalf: which half of the tile's rows, -1 = all
  if constexpr (NT == 1) {
    const bool half_tile = bx < 2 * g.split_tiles;
    int tl = half_tile ? bx >> 1 : bx - 2 * g.split_tiles;   // tile within its class (halved / whole)
    rhalf[0] = half_tile ? bx & 1 : -1;
    if constexpr (std::is_same<Epi, QkvEpi>::value) {
      // Four consecutive tiles hold the 128 channels of one head (or two heads of 64): each writes 32-byte runs of
      // the same cache lines of the paged cache (64-byte runs of q).  Workgroup ids congruent modulo 8 run on the
      // same XCD behind the same L2, so the four tiles of a head get ids 8 apart: their partial lines meet in that
      // L2 before they go to memory.  Only whole groups are rearranged (32 whole tiles = 8 heads x 4 tiles; 64 half
      // tiles = 8 heads x 4 tiles x 2 halves, both halves of a tile on one XCD as well).
      if (half_tile) {
        if (bx < ((2 * g.split_tiles) & ~63)) {
          const int q = (bx >> 3) & 7;
          tl = (((bx >> 6) << 3) + (bx & 7)) * 4 + (q >> 1);
          rhalf[0] = q & 1;
        }
      } else if (tl < ((g.n_tiles - g.split_tiles) & ~31)) {
        tl = (tl & ~31) + ((tl & 7) << 2) + ((tl >> 3) & 3);
      }
    }
    nt[0] = half_tile ? g.tile_begin + g.n_tiles - g.split_tiles + tl : g.tile_begin + tl;
  } else if (g.split_tiles) {   // a whole tile and half of one of the last split_tiles (grid: 2 * split_tiles = the others)
    int tl = bx, hl = bx >> 1;
    rhalf[0] = -1;
    rhalf[1] = bx & 1;
    if (bx < ((2 * g.split_tiles) & ~63)) {   // heads stay on one XCD, as above
      const int q = (bx >> 3) & 7;
      tl = (bx & ~31) + ((bx & 7) << 2) + ((bx >> 3) & 3);
      hl = (((bx >> 6) << 3) + (bx & 7)) * 4 + (q >> 1);
      rhalf[1] = q & 1;
    }
    nt[0] = g.tile_begin + tl;
    nt[1] = g.tile_begin + 2 * g.split_tiles + hl;
  } else {
    int pr = bx;   // two neighbouring tiles; the two pairs of a head get ids 8 apart
    if (std::is_same<Epi, QkvEpi>::value && bx < ((g.n_tiles >> 1) & ~15)) pr = (bx & ~15) + ((bx & 7) << 1) + ((bx >> 3) & 1);
    nt[0] = g.tile_begin + 2 * pr;
    nt[1] = nt[0] + 1;
    rhalf[0] = rhalf[1] = -1;
  }
  const int k_steps = g.K >> 4;
  const int chunks = gridDim.y * NW;
  const int c = blockIdx.y * NW + wave;
  const int ks0 = (int)((long)k_steps * c / chunks);
  const int ks1 = (int)((long)k_steps * (c + 1) / chunks);
  const int m_tiles = (g.M + 31) >> 5;
  const size_t x_tile_stride = (size_t)k_steps * 64;

  // Lane l of a weight tile holds row l % 32.  In a halved tile the lanes of the other 16 rows fetch what their
  // partner lanes fetch (the same bytes, no further memory traffic): their result rows are duplicates, never written.
  const u32x4* wp[NT];
#pragma unroll
  for (int t = 0; t < NT; ++t)
    wp[t] = reinterpret_cast<const u32x4*>(g.w) + (size_t)nt[t] * k_steps * 64 + (rhalf[t] >= 0 ? ((lane & ~16) | (rhalf[t] << 4)) : lane);

  for (int mt0 = 0; mt0 < m_tiles; mt0 += MT) {
    const u32x4* xp[MT];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) xp[mt] = reinterpret_cast<const u32x4*>(g.x) + (size_t)(mt0 + mt) * x_tile_stride + x_lane(lane, mt0 + mt, g.M);
    f32x16 acc[NT][MT];
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
      for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[t][mt][i] = 0.0f;

    // double-buffered stream over this wavefront's share of the contraction
    Frag<MT, NT, U> A, B;
    const int n = (ks1 - ks0) / U;
    int k = ks0;
    if (n > 0) frag_load(A, wp, xp, k);
    int i = 0;
    // (An unconditional steady-state loop with counted waits that keeps a whole group in flight behind the one
    // being multiplied was measured too: no faster in the decode step, so the simpler loop stays.)
    for (; i + 2 <= n; i += 2) {
      frag_load(B, wp, xp, k + U);
      frag_mma(A, acc);
      if (i + 2 < n) frag_load(A, wp, xp, k + 2 * U);
      frag_mma(B, acc);
      k += 2 * U;
    }
    if (i < n) {
      frag_mma(A, acc);
      k += U;
    }
    if (k < ks1) {
      frag_load_tail(A, wp, xp, k, ks1);
      frag_mma(A, acc);
    }
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) tile_finish(acc[t][mt], nt[t], mt0 + mt, g, e, s, wave, lane, rhalf[t]);
  }
}

// ---------------------------------------------------------------------------------------------------------
// Main loop 2 (LM head, gate/up and long accumulate projections up to four 32-row batch tiles, KV filling): the four
// wavefronts of a workgroup own four different 32-row output tiles over the SAME contraction range, so the activation
// operand is fetched from L2 once per workgroup, staged in LDS and read by all four; weights still go straight from HBM to registers, each byte
// once per batch chunk of MT*32 rows.  Groups of UT contraction steps: while group g is multiplied, the loads
// of groups g+1 and g+2 are in flight (three rotating weight register sets, two activation register sets that
// drain into two LDS stages).  Every wavefront finishes its own tiles, so the epilogue runs from registers.
// ---------------------------------------------------------------------------------------------------------
constexpr int UT = 4;
__device__ u32x4 k_zero_tile[64];   // one operand tile of zeros, never written (activation rows past the contraction range; not const: it must live in the same address space as the operands)

// Exit-head epilogue of NT neighbouring 32-column tiles of one batch tile, from registers: the statistics of all their logits
// of a row as one record in the first tile's place (the others' are empty).  Accumulators as in finish_from_registers below.
// Nothing hides this work (one or two wavefronts per SIMD, all in the same phase), so it is as few instructions as it can
// be: largest and runner-up as a maximum and a median of three, the row's largest settled between its two lanes before the
// exponentials, so that merging them takes none.  The statistics were about 20 us of the ring kernel's 120 at 500 rows; exit
// check 128.8 -> 125.1 us there, 160 -> 148 at 300 rows (tiled kernel, two tiles), 99 -> 93 for 256 compacted rows.
template <int NT, class Get>
__device__ inline void finish_lm(Get acc, int nt, int mtile, int M_eff, const GemmShape& g, const LmEpi& e, int lane) {
  constexpr int N = NT * 16;
  const int half = lane >> 5, m = mtile * 32 + (lane & 31);
  float m1[NT], m2[NT];
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    m1[t] = acc(t, 0);
    m2[t] = -INFINITY;
#pragma unroll
    for (int a = 1; a < 16; ++a) {
      const float z = acc(t, a);
      m2[t] = __builtin_amdgcn_fmed3f(m1[t], m2[t], z);
      m1[t] = fmaxf(m1[t], z);
    }
  }
  float lane_best = m1[0], z2 = m2[0];
#pragma unroll
  for (int t = 1; t < NT; ++t) {
    z2 = fmaxf(fminf(lane_best, m1[t]), fmaxf(z2, m2[t]));
    lane_best = fmaxf(lane_best, m1[t]);
  }
  const float other = __shfl_xor(lane_best, 32);
  z2 = fmaxf(fminf(lane_best, other), fmaxf(z2, __shfl_xor(z2, 32)));
  const float best = fmaxf(lane_best, other);
  // number of the lane's first logit (they are in vocabulary order) that is the row's largest
  int at = N;
#pragma unroll
  for (int i = N - 1; i >= 0; --i) at = acc(i >> 4, i & 15) == best ? i : at;
  int idx = at < N ? (nt + (at >> 4)) * 32 + ((at >> 3) & 1) * 16 + ((at >> 2) & 1) * 8 + half * 4 + (at & 3) : STAT_NO_INDEX;
  idx = min(idx, __shfl_xor(idx, 32));
  const float c = e.scale * 1.4426950408889634f;
  float sum[2] = {0.0f, 0.0f};
#pragma unroll
  for (int i = 0; i < N; ++i) sum[i & 1] += __builtin_amdgcn_exp2f(c * (acc(i >> 4, i & 15) - best));
  float total = sum[0] + sum[1];
  total += __shfl_xor(total, 32);
  if (half == 0 && m < M_eff) {
    float4* rec = e.partials + (size_t)(e.perm ? e.perm[m] : m) * e.n_parts + (nt - g.tile_begin);
    rec[0] = stat_pack(HeadStat{best, total, z2, idx});
#pragma unroll
    for (int t = 1; t < NT; ++t) rec[t] = stat_pack(stat_empty());
  }
}

// Epilogue of one finished 32 x 32 result tile held in a wavefront's registers (tiled, block and ring kernels): accumulator a
// (< 8) of a lane is result row r16 = (a/4)*8 + (lane/32)*4 + a%4 of column lane%32, accumulator a+8 is row r16+16 (its
// partner row in the packed order).  nt: packed weight tile, mtile: 32-row batch tile, M_eff: valid rows, ksl: the
// contraction slice this workgroup summed (accumulate projections).
template <class Epi>
__device__ inline void finish_from_registers(const f32x16& acc, int nt, int mtile, int M_eff, int ksl, const GemmShape& g,
                                             const Epi& e, int lane) {
  const int half = lane >> 5, ml = lane & 31;
  const int m = mtile * 32 + ml;
  if constexpr (std::is_same<Epi, AccEpi>::value) {
    // this workgroup's contraction slice (ksl) of the partial results, plain 16-byte stores: a lane holds, for its
    // batch row, two runs of four consecutive channels and the two runs 16 channels further on
    if (m < M_eff) {
      float* row = e.h + ((size_t)ksl * e.Mpad + m) * e.n_out + nt * 32 + half * 4;
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        *reinterpret_cast<float4*>(row + q * 8) = make_float4(acc[4 * q], acc[4 * q + 1], acc[4 * q + 2], acc[4 * q + 3]);
        *reinterpret_cast<float4*>(row + q * 8 + 16) =
            make_float4(acc[4 * q + 8], acc[4 * q + 9], acc[4 * q + 10], acc[4 * q + 11]);
      }
    }
  } else {
    if (m < M_eff) {
      // this lane holds two runs of four consecutive output rows (and their partners 16 rows on) of its batch row
#pragma unroll
      for (int run = 0; run < 2; ++run) {
        const int f_lo0 = packed_row_lo(nt, run * 8 + half * 4, g.pair_stride);
        float lo[4], hi[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          lo[i] = acc[run * 4 + i];
          hi[i] = acc[run * 4 + i + 8];
        }
        if constexpr (std::is_same<Epi, QkvEpi>::value) {
          epi_qkv4(e, m, f_lo0, lo, hi);
        } else {
          epi_gateup4(e, m, f_lo0, lo, hi);
        }
      }
    }
  }
}

// 16 bytes of a packed weight tile: streamed past the caches (nt) when one workgroup reads it, kept for the others when
// several do.
template <bool KEEP>
__device__ inline u32x4 weight_load(const u32x4* p) {
  if constexpr (KEEP) return *p;
  else return __builtin_nontemporal_load(p);
}

template <int MT>
struct TiledLds {
  u32x4 b[2][UT][MT][64];
  int flag;
};

template <int MT, int NTW, class Epi, bool FILL>
__global__ __launch_bounds__(256) void gemm_tiled_kernel(GemmShape g, Epi e, Pred pred, FillCtl fc) {
  __shared__ TiledLds<MT> s;
  constexpr int XR = UT * MT / NW;   // activation tiles each wavefront stages per group
  static_assert(UT * MT % NW == 0, "stage must split evenly over the wavefronts");

  if constexpr (!FILL) {
    if (pred_skip(pred)) return;
  } else {
    const int layer = (int)gridDim.z - (int)blockIdx.z;   // deepest layer first: the slices that have work start first
    if (fill_skip(pred, e, g.M, layer, s.flag)) return;
    g.w = fc.layers.w_qkv[layer - 1];
    g.x = fc.x_slabs + (size_t)(layer - 1) * fc.x_slab_elems;
    e.layer = layer;
    e.k_pool = reinterpret_cast<char*>(e.k_pool) + (size_t)(layer - 1) * fc.pool_layer_bytes;
    e.v_pool = reinterpret_cast<char*>(e.v_pool) + (size_t)(layer - 1) * fc.pool_layer_bytes;
  }

  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int m_tiles = (g.M + 31) >> 5;
  const int chunks = (m_tiles + MT - 1) / MT;   // the last chunk may be short: its missing tiles re-read its last
                                                // valid one, and their rows are never written
  // One-dimensional grid.  Workgroup ids that are congruent modulo 8 run on the same XCD and share its L2, so
  // the workgroups that stream the SAME weight tiles (the batch chunks and contraction slices of one tile group)
  // get consecutive ids of one residue class: they start together on one XCD, and all but the first read of a
  // weight tile hit that L2 instead of going out to memory once per chunk.
  const int ny = g.grid_y;                      // chunks * contraction slices
  const int ksplit = ny / chunks;
  const int slot = (int)blockIdx.x >> 3;
  const int bx = (slot / ny) * 8 + ((int)blockIdx.x & 7), by = slot % ny;
  // Which output tiles this workgroup owns.  Even split: four per workgroup.  Uneven split (g.even_wgs > 0, one
  // chunk, no contraction slices): the tiles are dealt out over exactly g.even_wgs workgroups, n_tiles / even_wgs
  // or one more each, and a wavefront beyond its workgroup's count owns none: it still stages its share of the
  // activation operand, but streams no weights.  A compute unit sustains only so many bytes per second from beyond
  // its L2, so the launch is as fast as its most loaded compute unit: 688 tiles as 172 x 4 keep a third of the chip
  // idle while 172 units stream four tiles each; as 176 x 3 + 80 x 2 nobody streams more than three.
  int my_tiles = NW, tile0 = bx * NW * NTW;
  if (g.even_wgs > 0) {
    if (bx >= g.even_wgs) return;
    const int base = g.n_tiles / g.even_wgs, rem = g.n_tiles % g.even_wgs;
    my_tiles = base + (bx < rem ? 1 : 0);
    tile0 = bx * base + min(bx, rem);
  } else if (tile0 >= g.n_tiles) {
    return;                                     // the group count is padded to a multiple of 8
  }
  const bool active = wave < my_tiles;
  const int chunk = by / ksplit, ksl = by % ksplit;
  // this wavefront's NTW consecutive output tiles (a wavefront without tiles points at the workgroup's first: never loaded)
  const int nt0 = g.tile_begin + tile0 + (active ? wave : 0) * NTW;
  const int k_steps = g.K >> 4;
  const int ks0 = (int)((long)k_steps * ksl / ksplit);
  const int ks1 = (int)((long)k_steps * (ksl + 1) / ksplit);
  const size_t x_tile_stride = (size_t)k_steps * 64;
  const size_t w_tile_stride = (size_t)k_steps * 64;
  const u32x4* wp = reinterpret_cast<const u32x4*>(g.w) + (size_t)nt0 * k_steps * 64 + lane;
  const u32x4* xp = reinterpret_cast<const u32x4*>(g.x) + (size_t)(chunk * MT) * x_tile_stride + lane;
  const int mt_last = min(MT, m_tiles - chunk * MT) - 1;   // last batch tile of this chunk that exists
  // One or two batch tiles: every wavefront stages pieces of one of them, the rows that exist (x_lane).  (With four that form is
  // slower, also where every row exists: 97 rows of the 13B shape, one layer, 317 -> 331 us; KV filling at 65 rows 51.8 -> 54.7.)
  const int x_mt = MT <= 2 ? min(wave % MT, mt_last) : 0;
  if constexpr (MT <= 2) xp += (size_t)x_mt * x_tile_stride + (x_lane(lane, chunk * MT + x_mt, g.M) - lane);

  f32x16 acc[NTW][MT];
#pragma unroll
  for (int t = 0; t < NTW; ++t)
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
      for (int i = 0; i < 16; ++i) acc[t][mt][i] = 0.0f;

  // Everything in the loop is unconditional (a conditional load would force the compiler to wait for every
  // outstanding load where the branches meet): the group count is rounded up to the rotation period and
  // groups past the end load a clamped weight tile against zero activations.
  const int n = (ks1 - ks0 + UT - 1) / UT;
  // The main loop exists in three forms, chosen once per wavefront: without a weight stream, with one that nobody else
  // reads, with one that the other row chunks read too.  All take the same barriers.
  auto main_loop = [&](auto streams_c, auto keep_c) {
    constexpr bool STREAMS = decltype(streams_c)::value;
    constexpr bool KEEP = decltype(keep_c)::value;
    u32x4 W[4][NTW][UT], X[2][XR];
    auto gload = [&](int grp, u32x4 (&wr)[NTW][UT], u32x4 (&xr)[XR]) {
      const int kbase = ks0 + grp * UT;
      if constexpr (STREAMS) {
#pragma unroll
        for (int u = 0; u < UT; ++u) {
          const int kk = kbase + u < ks1 ? kbase + u : ks1 - 1;
#pragma unroll
          for (int t = 0; t < NTW; ++t) wr[t][u] = weight_load<KEEP>(wp + t * w_tile_stride + (size_t)kk * 64);
        }
      }
#pragma unroll
      for (int j = 0; j < XR; ++j) {
        const int t = wave + NW * j, u = t / MT, mt = MT <= 2 ? 0 : t % MT;
        // past the end: a tile of zeros, chosen by address (a select on the loaded value would sit right behind
        // the load and make the wavefront wait for everything it has in flight)
        const bool ok = kbase + u < ks1;
        const u32x4* src = ok ? xp + min(mt, mt_last) * x_tile_stride + (size_t)(kbase + u) * 64 : k_zero_tile + lane;
        xr[j] = *src;
      }
    };
    // One group: drain its activation registers into LDS stage XS, start the loads of group grp+2 into the
    // registers just freed and an idle weight set, multiply group grp.
    auto step = [&](int grp, const u32x4 (&wcur)[NTW][UT], u32x4 (&wnext2)[NTW][UT], u32x4 (&xs)[XR], int XS) {
      // keeps the LDS stores below from being hoisted into the previous group, ahead of its loads: there they would
      // wait for loads that were only just issued
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int j = 0; j < XR; ++j) {
        const int t = wave + NW * j;
        s.b[XS][t / MT][t % MT][lane] = xs[j];
      }
      __syncthreads();
      gload(grp + 2, wnext2, xs);
      if constexpr (STREAMS) {
        // the LDS reads of contraction step u+1 are issued before the multiplies of step u
        u32x4 bf[2][MT];
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) bf[0][mt] = s.b[XS][0][mt][lane];
#pragma unroll
        for (int u = 0; u < UT; ++u) {
          if (u + 1 < UT) {
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) bf[(u + 1) & 1][mt] = s.b[XS][u + 1][mt][lane];
          }
#pragma unroll
          for (int mt = 0; mt < MT; ++mt)
#pragma unroll
            for (int t = 0; t < NTW; ++t)
              acc[t][mt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, wcur[t][u]),
                                                                   __builtin_bit_cast(bf16x8, bf[u & 1][mt]), acc[t][mt], 0, 0, 0);
        }
        if constexpr (MT >= 4) {
          // Order of the group, spelled out for the scheduler: the first step's fragments, then one fragment read
          // of the next step behind every NTW multiplies, the last step's multiplies.  Left alone it issues each
          // read right in front of the multiplies that use it and the matrix cores wait out every LDS round trip.
          __builtin_amdgcn_sched_group_barrier(0x100, MT, 0);
#pragma unroll
          for (int i = 0; i < (UT - 1) * MT; ++i) {
            __builtin_amdgcn_sched_group_barrier(0x008, NTW, 0);
            __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
          }
          __builtin_amdgcn_sched_group_barrier(0x008, MT * NTW, 0);
        }
      }
    };

    gload(0, W[0], X[0]);
    gload(1, W[1], X[1]);
    for (int gi = 0; gi < n; gi += 4) {
      step(gi, W[0], W[2], X[0], 0);
      step(gi + 1, W[1], W[3], X[1], 1);
      step(gi + 2, W[2], W[0], X[0], 0);
      step(gi + 3, W[3], W[1], X[1], 1);
    }
    __syncthreads();
  };
  if (!active) {
    main_loop(std::false_type{}, std::false_type{});
    return;       // nothing to finish; the epilogues below take no workgroup barrier
  }
  if (FILL && g.keep)   // (nothing else is launched with it)
    main_loop(std::true_type{}, std::integral_constant<bool, FILL>{});
  else
    main_loop(std::true_type{}, std::false_type{});

  // every wavefront finishes its own tiles from registers
  if constexpr (std::is_same<Epi, LmEpi>::value) {
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
      finish_lm<NTW>([&](int t, int a) { return acc[t][mt][a]; }, nt0, chunk * MT + mt, g.M, g, e, lane);
  } else {
#pragma unroll
    for (int t = 0; t < NTW; ++t)
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) finish_from_registers(acc[t][mt], nt0 + t, chunk * MT + mt, g.M, ksl, g, e, lane);
  }
}

// ---------------------------------------------------------------------------------------------------------
// Main loop 3 (LM head, and now and then gate/up, at 385 to 512 rows, where the matrix cores are what counts): one workgroup owns a
// 256-row x 256-column block of the result (eight batch tiles x eight weight tiles).  Wavefront w owns two weight
// tiles (64 columns) against all eight batch tiles, 16 accumulator tiles = all 256 accumulation registers:
//   * its weight fragments come straight from HBM into registers, RING_D contraction steps ahead (nobody else in
//     the workgroup needs them, so they never touch LDS);
//   * the activation fragments of a step (8 KiB, needed by all four wavefronts) land in a ring of RING_D + 1 LDS
//     slots through direct-to-LDS loads, two tiles per wavefront, just as far ahead: a wavefront's loads complete
//     in order, so a fragment from L2 queued behind a weight tile from HBM is ready no sooner than that tile and must
//     have been asked for as early;
//   * one bare barrier per contraction step (a fence would wait for every load in flight): at step s every
//     wavefront has waited for its own two tiles of step s+1, and the slot of step s-1, whose fragments everybody
//     has multiplied, takes step s+RING_D.
// Per compute unit and step: 16 KiB from memory, 8 KiB written to and 32 KiB read from LDS, 64 MFMAs.  Every weight
// byte leaves HBM once: the two row blocks of a column block run on one XCD and meet in its L2.
// ---------------------------------------------------------------------------------------------------------
constexpr int RING_D = 15;
constexpr int RING_LDS_BYTES = (RING_D + 1) * 8 * 1024;
typedef __attribute__((address_space(3))) void* lds_void_ptr;
typedef __attribute__((address_space(1))) const void* global_void_ptr;
template <int N>
__device__ inline void wait_loads_but() { asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory"); }

template <class Epi>
__global__ __launch_bounds__(256) void gemm_ring_kernel(GemmShape g, Epi e, Pred pred) {
  extern __shared__ u32x4 ring[];   // [RING_D + 1][8 batch tiles][64 lanes]
  if (pred_skip(pred)) return;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int m_tiles = (g.M + 31) >> 5;
  const int row_blocks = (m_tiles + 7) >> 3, col_blocks = g.n_tiles >> 3;
  // ids congruent modulo 8 share an XCD: the row blocks of one column block get consecutive ids of one class
  const int xcd = (int)blockIdx.x & 7, j = (int)blockIdx.x >> 3;
  const int bm = j % row_blocks, bn = (j / row_blocks) * 8 + xcd;
  if (bn >= col_blocks) return;
  const int k_steps = g.K >> 4;     // a multiple of RING_D + 1 (the host checks)
  const int nt0 = g.tile_begin + bn * 8 + wave * 2;
  const u32x4* wsrc[2];
  const u32x4* xsrc[2];
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    wsrc[i] = reinterpret_cast<const u32x4*>(g.w) + (size_t)(nt0 + i) * k_steps * 64 + lane;
    xsrc[i] = reinterpret_cast<const u32x4*>(g.x) + (size_t)min(bm * 8 + wave * 2 + i, m_tiles - 1) * k_steps * 64 + lane;
  }
  // Exactly four loads per wavefront and step, in this order; steps past the end repeat the last one (never used).
  auto issue = [&](int s, u32x4 (&wr)[2], int slot) {
    const int ss = s < k_steps ? s : k_steps - 1;
#pragma unroll
    for (int i = 0; i < 2; ++i) wr[i] = __builtin_nontemporal_load(wsrc[i] + (size_t)ss * 64);
#pragma unroll
    for (int i = 0; i < 2; ++i)
      __builtin_amdgcn_global_load_lds((global_void_ptr)(xsrc[i] + (size_t)ss * 64),
                                       (lds_void_ptr)(ring + ((size_t)slot * 8 + wave * 2 + i) * 64), 16, 0, 0);
  };
  auto read_x = [&](u32x4 (&f)[8], int slot) {
    const u32x4* sp = ring + (size_t)slot * 8 * 64 + lane;
#pragma unroll
    for (int b = 0; b < 8; ++b) f[b] = sp[b * 64];
  };
  f32x16 acc[2][8];
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int b = 0; b < 8; ++b)
#pragma unroll
      for (int i = 0; i < 16; ++i) acc[a][b][i] = 0.0f;

  u32x4 wr[RING_D + 1][2];
  u32x4 f[2][8];
#pragma unroll
  for (int q = 0; q < RING_D; ++q) {
    issue(q, wr[q], q);
    asm volatile("" ::: "memory");      // the counted waits rely on the loads of a step staying together, in step order
  }
  wait_loads_but<(RING_D - 1) * 4>();   // step 0 has landed; the loop's own waits take it from there
  __builtin_amdgcn_s_barrier();
  read_x(f[0], 0);
  // q = s % (RING_D + 1): step s lives in register set / ring slot q
  auto step = [&](int s, const u32x4 (&wcur)[2], u32x4 (&wnew)[2], const u32x4 (&fcur)[8], u32x4 (&fnext)[8], int q) {
    // loads issued after this wavefront's activation tiles of step s+1: the RING_D - 2 steps s-13 .. s-1
    wait_loads_but<(RING_D - 2) * 4>();
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
    issue(s + RING_D, wnew, (q + RING_D) % (RING_D + 1));
    read_x(fnext, (q + 1) % (RING_D + 1));
#pragma unroll
    for (int b = 0; b < 8; ++b)
#pragma unroll
      for (int a = 0; a < 2; ++a)
        acc[a][b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, wcur[a]),
                                                            __builtin_bit_cast(bf16x8, fcur[b]), acc[a][b], 0, 0, 0);
    // the multiplies start at once; one load, then one fragment read, goes out behind each of the first twelve
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
      __builtin_amdgcn_sched_group_barrier(0x010, 1, 0);
    }
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
      __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
    }
    __builtin_amdgcn_sched_group_barrier(0x008, 4, 0);
    __builtin_amdgcn_sched_barrier(0);
  };
  static_assert(RING_D == 15, "the loop below is unrolled for sixteen register sets");
  for (int s = 0; s < k_steps; s += 16) {
#define EE_RING_STEP(i) step(s + i, wr[i], wr[(i + 15) % 16], f[i & 1], f[(i + 1) & 1], i)
    EE_RING_STEP(0); EE_RING_STEP(1); EE_RING_STEP(2); EE_RING_STEP(3);
    EE_RING_STEP(4); EE_RING_STEP(5); EE_RING_STEP(6); EE_RING_STEP(7);
    EE_RING_STEP(8); EE_RING_STEP(9); EE_RING_STEP(10); EE_RING_STEP(11);
    EE_RING_STEP(12); EE_RING_STEP(13); EE_RING_STEP(14); EE_RING_STEP(15);
#undef EE_RING_STEP
  }
  wait_loads_but<0>();   // the repeated loads past the end still target LDS and registers
#pragma unroll
  for (int b = 0; b < 8; ++b) {
    if (bm * 8 + b >= m_tiles) continue;
    if constexpr (std::is_same<Epi, LmEpi>::value) {
      finish_lm<2>([&](int t, int a) { return acc[t][b][a]; }, nt0, bm * 8 + b, g.M, g, e, lane);
    } else {
#pragma unroll
      for (int a = 0; a < 2; ++a) finish_from_registers(acc[a][b], nt0 + a, bm * 8 + b, g.M, 0, g, e, lane);
    }
  }
}

// ---------------------------------------------------------------------------------------------------------
// Main loop 4: one workgroup owns a block of MT batch tiles x NT weight tiles; both operands land in a ring of DS stages of two
// contraction steps in LDS through direct-to-LDS loads, and every wavefront of WM x WN multiplies its part of the block.
//   * What bounds it is how fast a compute unit takes its operands in: loads that miss L2 come at 31 GB/s a compute unit, shared
//     or not, hits at 75 to 120, whatever is in flight beyond 32 KiB (so two or three stages are enough), and the order, the
//     layout and the cache policy of the loads change little.  A block of 128 x 192 needs 10 KiB a step: 48 us over 256 steps
//     with nothing but the loads; 256 x 192 14 KiB, 67 us.
//   * A wavefront that issues such a load waits at it until the memory pipeline accepts it, and multiplies nothing meanwhile:
//     with the loads in the multiplying wavefronts the same blocks took 77 and 115 us, loads and multiplies one after the
//     other.  So two wavefronts do nothing but load.  They are as fast as their address arithmetic: one bound register pair and a
//     scalar offset (buffer loads), with 64-bit pointers and a select per load two of them reached 35 GB/s.
//   * One barrier a stage: past it the next stage has landed (the loaders waited for it), and the fragments of this stage's last
//     step are in registers, so its slot can be loaded again.
// 512 rows of the 7B shape, before (tiled and ring kernels) and now: QKV 76 -> 59 us (128 x 192 blocks, 0.87 PFLOP/s, matrix
// cores busy 35 % of the time), gate/up 107 -> 82 (256 x 192, 1.12, 52 %), down 58 -> 56 (128 x 128 in two slices, 0.83).  Tried: a wavefront
// that touches this workgroup's share of the shared weight lines ahead of the loaders: 10 to 17 % faster without multiplies, 0 to
// 30 % slower with them; weights past the caches: up to a third slower; four multiplying wavefronts of 128 x 96 instead of eight
// of 64 x 96: 92 -> 97 us.
// ---------------------------------------------------------------------------------------------------------
constexpr int BLOCK_U = 2, BLOCK_NL = 2;   // contraction steps a stage, loaders
struct BlockGrid {
  int row_blocks, col_blocks, ksplit;
};

#if defined(__HIP_DEVICE_COMPILE__)
typedef __amdgpu_buffer_rsrc_t buffer_t;
__device__ inline buffer_t buffer_at(const char* p) { return __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(p), 0, 0x7fffffff, 0x00020000); }
__device__ inline void buffer_to_lds(buffer_t b, lds_void_ptr to, int lane_off, int off) {
  // (cached, also weights that one workgroup reads: past the caches, as the other kernels load them, these loads are up to a third slower)
  __builtin_amdgcn_raw_ptr_buffer_load_lds(b, to, 16, lane_off, off, 0, 0);
}
#else   // (the host pass knows neither the type nor the instruction)
typedef int buffer_t;
__device__ inline buffer_t buffer_at(const char*) { return 0; }
__device__ inline void buffer_to_lds(buffer_t, lds_void_ptr, int, int) {}
#endif

// QKV epilogue of a block's wavefront: NTW neighbouring output tiles x MTW batch tiles.  Where a batch row's K and V go is
// looked up while the first operands are on their way (slot: element of the layer's pool at head 0, channel 0; -1: nowhere),
// and the rotary pairs of one batch tile are fetched while the one before is stored: looked up tile by tile, as the other
// kernels do, each tile waits for a chain of dependent loads behind the stores of the last.
__device__ inline long kv_slot(const QkvEpi& e, int m, int M) {
  if (m >= M || kv_filled(e, m)) return -1;
  const int p = e.context_lens[m];
  if ((unsigned)p >= (unsigned)(e.max_blocks * 16)) return -1;
  const int blk = e.block_tables[(size_t)(e.row_table ? safe_row(e.row_table[m], e.table_rows) : m) * e.max_blocks + (p >> 4)];
  if ((unsigned)blk >= (unsigned)e.num_blocks) return -1;   // never outside the pools
  return ((long)blk * e.n_heads * 16 + (p & 15)) * e.head_dim;
}
template <int MTW, int NTW>
__device__ inline void finish_qkv(const f32x16 (&acc)[NTW][MTW], int nt0, int n_tiles, int mtile0, const long (&slot)[MTW], const GemmShape& g,
                                  const QkvEpi& e, int lane) {
  const int d = e.d_model, dh = e.head_dim, hdim = dh >> 1, sub = (lane >> 5) * 4;
  typedef bf16_t bf16x4 __attribute__((ext_vector_type(4)));
  float4 cs[2][NTW][2][2];
  auto fetch = [&](int mt, float4 (&c)[NTW][2][2]) {
    const int m = min((mtile0 + mt) * 32 + (lane & 31), g.M - 1);
#pragma unroll
    for (int t = 0; t < NTW; ++t) {
      const int f0 = packed_row_lo(nt0 + t, 0, g.pair_stride), j0 = f0 % dh;
      if (nt0 + t < n_tiles && f0 < 2 * d && e.rope_theta > 0.0f) {
        const float2* src = e.rope + (size_t)m * hdim + j0 + sub;
#pragma unroll
        for (int run = 0; run < 2; ++run) {
          c[t][run][0] = *reinterpret_cast<const float4*>(src + run * 8);
          c[t][run][1] = *reinterpret_cast<const float4*>(src + run * 8 + 2);
        }
      }
    }
  };
  fetch(0, cs[0]);
#pragma unroll
  for (int mt = 0; mt < MTW; ++mt) {
    if (mt + 1 < MTW) fetch(mt + 1, cs[(mt + 1) & 1]);
    const int m = (mtile0 + mt) * 32 + (lane & 31);
#pragma unroll
    for (int t = 0; t < NTW; ++t) {
      if (nt0 + t >= n_tiles) break;
      const int f0 = packed_row_lo(nt0 + t, 0, g.pair_stride);   // all of this is the same for the whole wavefront
      const int which = f0 / d, within = f0 - which * d, head = within / dh, j = within - head * dh + sub;
      const bool turn = which < 2 && e.rope_theta > 0.0f;
#pragma unroll
      for (int run = 0; run < 2; ++run) {
        const float4 c01 = cs[mt & 1][t][run][0], c23 = cs[mt & 1][t][run][1];
        const float co[4] = {c01.x, c01.z, c23.x, c23.z}, si[4] = {c01.y, c01.w, c23.y, c23.w};
        float lo[4], hi[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const float a = acc[t][mt][run * 4 + i], b = acc[t][mt][run * 4 + i + 8];
          lo[i] = a;
          hi[i] = b;
          rotate(lo[i], hi[i], co[i], si[i]);
          lo[i] = turn ? lo[i] : a;
          hi[i] = turn ? hi[i] : b;
        }
        if (which == 0) {
          if (m < g.M && e.q) {
            float* q = e.q + (size_t)m * d + head * dh + j + run * 8;
            *reinterpret_cast<float4*>(q) = make_float4(lo[0], lo[1], lo[2], lo[3]);
            *reinterpret_cast<float4*>(q + hdim) = make_float4(hi[0], hi[1], hi[2], hi[3]);
          }
        } else if (slot[mt] >= 0) {
          bf16_t* at = reinterpret_cast<bf16_t*>(which == 1 ? e.k_pool : e.v_pool) + slot[mt] + (long)head * 16 * dh + j + run * 8;
          *reinterpret_cast<bf16x4*>(at) = bf16x4{(bf16_t)lo[0], (bf16_t)lo[1], (bf16_t)lo[2], (bf16_t)lo[3]};
          *reinterpret_cast<bf16x4*>(at + hdim) = bf16x4{(bf16_t)hi[0], (bf16_t)hi[1], (bf16_t)hi[2], (bf16_t)hi[3]};
        }
      }
    }
  }
}

template <int MT, int NT, int WM, int WN, int DS, bool COMPACTED, class Epi>
__device__ __forceinline__ void block_body(u32x4* ring, const GemmShape& g, const Epi& e, int ksplit, int bm, int bn, int ksl, int M_eff) {
  constexpr int U = BLOCK_U, NL = BLOCK_NL, P = MT + NT, CW = WM * WN, T = U * P / NL, MTW = MT / WM, NTW = NT / WN;
  static_assert(U == 2 && U * P % NL == 0 && MT % WM == 0 && NT % WN == 0 && DS > 2 && (DS - 1) * T < 64, "");
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int m_tiles = (g.M + 31) >> 5, k_steps = g.K >> 4;
  const int ks0 = (int)((long)k_steps * ksl / ksplit), n = (int)((long)k_steps * (ksl + 1) / ksplit) - ks0;
  const int stages = n / U;   // whole ones; the step that an odd contraction leaves over follows

  if (wave >= CW) {   // a loader: its share of the pieces of every stage
    const int lw = wave - CW;
    const size_t tile_bytes = (size_t)k_steps * 1024;
    const buffer_t wsrc = buffer_at(reinterpret_cast<const char*>(g.w) + (g.tile_begin + (size_t)bn * NT) * tile_bytes + (size_t)ks0 * 1024);
    const buffer_t xsrc = buffer_at(reinterpret_cast<const char*>(g.x) + (size_t)bm * MT * tile_bytes + (size_t)ks0 * 1024);
    int off[T];
#pragma unroll
    for (int i = 0; i < T; ++i) {
      const int t = (i * NL + lw) % P;
      off[i] = (int)((t < MT ? min(t, m_tiles - 1 - bm * MT) : min(t - MT, g.n_tiles - 1 - bn * NT)) * tile_bytes) + lane * 16;
    }
    auto issue = [&](int s, int slot) {
#pragma unroll
      for (int i = 0; i < T; ++i) {
        const int piece = i * NL + lw;
        buffer_to_lds(piece % P < MT ? xsrc : wsrc, (lds_void_ptr)(ring + ((size_t)slot * U * P + piece) * 64), off[i],
                      min(s * U + piece / P, n - 1) * 1024);
      }
    };
#pragma unroll
    for (int s = 0; s < DS; ++s) {
      issue(s, s);
      asm volatile("" ::: "memory");
    }
    wait_loads_but<(DS - 1) * T>();
    __builtin_amdgcn_s_barrier();
    int slot = 0;
    for (int s = 0; s < stages; ++s) {
      wait_loads_but<(DS - 2) * T>();
      __builtin_amdgcn_s_barrier();
      asm volatile("" ::: "memory");
      issue(s + DS, slot);
      slot = slot + 1 == DS ? 0 : slot + 1;
    }
    wait_loads_but<0>();   // (the loads past the end still target LDS)
    return;
  }
  const int wm = wave % WM, wn = wave / WM;
  u32x4 fx[2][MTW], fw[2][NTW];
  auto read = [&](int slot, int u, int b) {
    const u32x4* sp = ring + (size_t)(slot * U + u) * P * 64 + lane;
#pragma unroll
    for (int t = 0; t < MTW; ++t) fx[b][t] = sp[(wm * MTW + t) * 64];
#pragma unroll
    for (int t = 0; t < NTW; ++t) fw[b][t] = sp[(MT + wn * NTW + t) * 64];
  };
  long kv_at[MTW];
  if constexpr (std::is_same<Epi, QkvEpi>::value) {
#pragma unroll
    for (int mt = 0; mt < MTW; ++mt) kv_at[mt] = kv_slot(e, (bm * MT + wm * MTW + mt) * 32 + (lane & 31), g.M);
  }
  f32x16 acc[NTW][MTW];
#pragma unroll
  for (int t = 0; t < NTW; ++t)
#pragma unroll
    for (int mt = 0; mt < MTW; ++mt)
#pragma unroll
      for (int i = 0; i < 16; ++i) acc[t][mt][i] = 0.0f;
  // 64 x 64 blocks stand in for the streaming kernel and add as it does: a slice in four parts, the parts' sums one after the other.
  constexpr bool PARTS = MT == 2 && NT == 2;
  f32x16 sum[PARTS ? NTW : 1][PARTS ? MTW : 1] = {};
  const int per = 4 * ksplit;   // (a slice has four steps at least: no part is empty)
  int end = k_steps * (4 * ksl + 1) / per - ks0;
  const int end2 = k_steps * (4 * ksl + 2) / per - ks0, end3 = k_steps * (4 * ksl + 3) / per - ks0;
  auto add_part = [&]() {
#pragma unroll
    for (int t = 0; t < NTW; ++t)
#pragma unroll
      for (int mt = 0; mt < MTW; ++mt)
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          sum[t][mt][i] += acc[t][mt][i];
          acc[t][mt][i] = 0.0f;
        }
    end = end < end2 ? end2 : end < end3 ? end3 : -1;
  };
  auto multiply = [&](int b) {
#pragma unroll
    for (int t = 0; t < NTW; ++t)
#pragma unroll
      for (int mt = 0; mt < MTW; ++mt)
        acc[t][mt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, fw[b][t]),
                                                             __builtin_bit_cast(bf16x8, fx[b][mt]), acc[t][mt], 0, 0, 0);
  };
  auto all_meet = [&]() {
    // the loaders' pieces of the next stage have landed; this wavefront's fragments of the present one are in registers
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
  };

  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
  read(0, 0, 0);
  int slot = 0;
  for (int s = 0; s < stages; ++s) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      constexpr int NM = MTW * NTW, RPM = MTW + NTW > 2 * NM ? 3 : 2;
      if constexpr (PARTS)
        if (s * U + u == end) add_part();
      __builtin_amdgcn_sched_barrier(0);
      if (u == U - 1) {
        all_meet();
        slot = slot + 1 == DS ? 0 : slot + 1;
        read(slot, 0, (u + 1) & 1);
      } else {
        read(slot, u + 1, (u + 1) & 1);
      }
      multiply(u & 1);
      // fragment reads go out behind the first multiplies
#pragma unroll
      for (int i = 0; i < NM; ++i) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        __builtin_amdgcn_sched_group_barrier(0x100, RPM, 0);
      }
    }
  }
  if constexpr (PARTS)
    if (n % U)
      if (n - 1 == end) add_part();
  if (n % U) multiply(0);   // the first step of the next stage, which has landed and been read
  if constexpr (PARTS) {
    add_part();
#pragma unroll
    for (int t = 0; t < NTW; ++t)
#pragma unroll
      for (int mt = 0; mt < MTW; ++mt) acc[t][mt] = sum[t][mt];
  }
  if constexpr (std::is_same<Epi, QkvEpi>::value) {
    finish_qkv<MTW, NTW>(acc, g.tile_begin + bn * NT + wn * NTW, g.tile_begin + g.n_tiles, bm * MT + wm * MTW, kv_at, g, e, lane);
  } else {
#pragma unroll
    for (int mt = 0; mt < MTW; ++mt) {
      const int mtile = bm * MT + wm * MTW + mt, nt0 = bn * NT + wn * NTW;
      if (mtile >= m_tiles) continue;
      if constexpr (std::is_same<Epi, LmEpi>::value) {
        // (compacted rows: a record a tile, so that a confidence does not hang on whether the block or half of it is worked on)
        if (!COMPACTED && nt0 + NTW <= g.n_tiles) {
          finish_lm<NTW>([&](int t, int a) { return acc[t][mt][a]; }, g.tile_begin + nt0, mtile, M_eff, g, e, lane);
        } else {
#pragma unroll
          for (int t = 0; t < NTW; ++t)
            if (nt0 + t < g.n_tiles) finish_lm<1>([&](int, int a) { return acc[t][mt][a]; }, g.tile_begin + nt0 + t, mtile, M_eff, g, e, lane);
        }
      } else {
#pragma unroll
        for (int t = 0; t < NTW; ++t)
          if (nt0 + t < g.n_tiles) finish_from_registers(acc[t][mt], g.tile_begin + nt0 + t, mtile, M_eff, ksl, g, e, lane);
      }
    }
  }
}

template <int MT, int NT, int WM, int WN, int DS, bool HALVES, class Epi>
__global__ __launch_bounds__((WM * WN + BLOCK_NL) * 64) void gemm_block_kernel(GemmShape g, Epi e, Pred pred, BlockGrid bg) {
  __shared__ u32x4 ring[DS * BLOCK_U * (MT + NT) * 64];   // [stage][step][tile][lane]
  if (pred_skip(pred)) return;
  // Ids congruent modulo 8 share an XCD: the row blocks of a column block run on one, neighbouring column blocks too.
  const int xcd = (int)blockIdx.x & 7, j = (int)blockIdx.x >> 3, nq = bg.col_blocks * bg.ksplit, per = (nq + 7) >> 3;
  int bm = HALVES ? j / per : j % bg.row_blocks;
  const int q = nq * xcd / 8 + (HALVES ? j % per : j / bg.row_blocks);
  if (q >= nq * (xcd + 1) / 8) return;
  int bn = q / bg.ksplit;
  const int ksl = q % bg.ksplit;
  if constexpr (HALVES) {
    // compacted operand: only the first *n_rows_dev rows hold sequences that are still active
    const int M_eff = g.n_rows_dev[0], active = (M_eff + MT * 32 - 1) / (MT * 32);
    if constexpr (MT == 8) {
      // the only row block (the host sees to that): its upper half is left out once it is empty
      if (M_eff > MT * 16)
        block_body<MT, NT, WM, WN, DS, HALVES>(ring, g, e, bg.ksplit, 0, bn, ksl, M_eff);
      else if (M_eff > 0)
        block_body<MT / 2, NT, WM, WN, DS, HALVES>(ring, g, e, bg.ksplit, 0, bn, ksl, M_eff);
    } else if (active * 2 <= bg.row_blocks) {
      // half of the row blocks are without work: two workgroups share a column block (7B shape, 128 rows active of 256: gate/up
      // 63 -> 48 us)
      constexpr int HM = NT / 2 % WN ? WM * WN : WM, HN = WM * WN / HM;   // wavefronts, rows x columns
      if (active == 0 || bm >= 2 * active) return;
      bn = bn * 2 + bm / active;
      if (bn * (NT / 2) >= g.n_tiles) return;
      block_body<MT, NT / 2, HM, HN, DS, HALVES>(ring, g, e, bg.ksplit, bm % active, bn, ksl, M_eff);
    } else if (bm < active) {
      block_body<MT, NT, WM, WN, DS, HALVES>(ring, g, e, bg.ksplit, bm, bn, ksl, M_eff);
    }
  } else {
    block_body<MT, NT, WM, WN, DS, HALVES>(ring, g, e, bg.ksplit, bm, bn, ksl, g.M);
  }
}

// Which shapes the ring kernel serves: 385 to 512 rows (two row blocks, the second at least half full: below that blocks of
// 128 rows waste less; above, the workgroups no longer fit the chip in one round), whole blocks of eight weight tiles, a
// contraction of whole groups of sixteen steps.
bool ring_serves(int M, int n_tiles, int K) {
  return M > 384 && M <= 512 && n_tiles % 8 == 0 && (K >> 4) % (RING_D + 1) == 0 && (K & 15) == 0;
}

// From three batch tiles on, the tiled kernel (128-row chunks, the last one padded) beats re-streaming the weights
// once per pass of the streaming kernel.
bool tiled(int M, int n_tiles) { return (M + 31) / 32 >= 3 && n_tiles % NW == 0; }

// Time of a projection in blocks of mt batch tiles x nt weight tiles over `steps` contraction steps, in ns: the blocks go round
// by round over 256 compute units, and a step takes a compute unit what its operands take to come in (22 ns a KiB of weights,
// 14 ns a KiB of activations: fitted to the kernel without multiplies, 128 x 192 blocks 48 us over 256 steps, 256 x 96 44,
// 128 x 96 31) or what its multiplies take (7 ns a tile: 256 x 192 blocks 80 to 92 us, from card to card).  Start, first loads and epilogue of a
// round: 5 us.
constexpr long block_cost(int m_tiles, int n_tiles, int steps, int mt, int nt, int slices = 1) {
  const long blocks = (long)((m_tiles + mt - 1) / mt) * ((n_tiles + nt - 1) / nt) * slices, in = 22 * nt + 14 * mt, mul = 7 * mt * nt;
  return (blocks + 255) / 256 * (5000 + steps * (in > mul ? in : mul));
}
// The cheapest of a kernel's block shapes for a projection.
struct BlockShape {
  int mt, nt;
};
template <int N>
BlockShape pick_block(const BlockShape (&shapes)[N], int m_tiles, int n_tiles, int steps, int slices = 1) {
  BlockShape best{0, 0};
  long best_cost = 0;
  for (const BlockShape& b : shapes) {
    const long c = block_cost(m_tiles, n_tiles, steps, b.mt, b.nt, slices);
    if (best.mt == 0 || c < best_cost) {
      best = b;
      best_cost = c;
    }
  }
  return best;
}
constexpr BlockShape kQkvBlocks[] = {{2, 3}, {4, 2}, {4, 3}, {4, 4}, {4, 6}}, kGateUpBlocks[] = {{4, 3}, {4, 4}, {4, 6}, {8, 4}, {8, 6}},
                     kLmBlocks[] = {{4, 4}, {4, 8}}, kAccBlocks[] = {{4, 2}, {4, 4}, {8, 4}};
// Of a compacted operand, those that come in halves: 128-row blocks in halves of their columns; 256-row blocks in halves of their
// rows, of gate/up up to 256 rows, where 128-row blocks may need a second round (13B shape, gate/up of 256 rows, all of them active:
// 98 us in the tiled kernel, 117 in 128 x 192 blocks, 91 in 256 x 128; three layers of 140 to 256 rows with exits of their own 2.5 to
// 10 % faster than without).
constexpr BlockShape kAccHalves[] = {{4, 2}, {4, 4}}, kGateUpHalves[] = {{4, 4}, {4, 6}}, kGateUpHalves256[] = {{4, 4}, {4, 6}, {8, 4}, {8, 6}};

// Which kernel an accumulate projection (output or down projection) of M rows onto n_tiles packed tiles over a
// contraction of K runs in, and how many contraction slices it writes.  Every slice is one more partial result for
// the normalisation launch to read, so the count stays as small as filling the chip allows.
struct AccPlan {
  int kind;     // 0: streaming kernel, 1: block kernel, 2: tiled kernel, one chunk of up to four tiles,
                // 3: streaming kernel, two output tiles per workgroup
  int ksplit;
  BlockShape block;
  long cost;    // of a plan for the block kernel
};
// Slices hold at least 64 contraction steps; the normalisation launch adds at most eight, of 129 to 512 rows more than four only of a
// long contraction that 128 x 64 blocks in as many slices sum in one round.
int acc_slices_most(int m_tiles, int n_tiles, int K) {
  const int by_k = K / 1024 < 1 ? 1 : K / 1024, round = 256 / ((m_tiles + 3) / 4 * ((n_tiles + 1) / 2));
  const int by_m = m_tiles <= 4 ? 8 : m_tiles > 16 ? (64 / m_tiles < 1 ? 1 : 64 / m_tiles) : K < 8192 || round < 4 ? 4 : round > 8 ? 8 : round;
  return by_k < by_m ? by_k : by_m;
}
AccPlan acc_plan(int M, int n_tiles, int K, bool compacted = false) {
  const int m_tiles = (M + 31) / 32, k_steps = K / 16, most = acc_slices_most(m_tiles, n_tiles, K);
  AccPlan p{0, 1, {0, 0}, 0};
  // (One row chunk: more than 128 tiles or 512 steps stay with the tiled kernel, bound by the weight stream either way: 13B output
  // projection at 128 rows 19.1 against 19.6 us in blocks, down projection 35.9 against 40.0.)
  const bool one_chunk = m_tiles <= 4 && n_tiles % NW == 0 && (k_steps >= 512 || (m_tiles >= 3 && n_tiles > 128));
  if (m_tiles >= 3 && !one_chunk) {
    // A slice costs its partial result's way out and back in: 8 bytes an element at 5 TB/s.  (7B shape, down projection at 192 / 256 /
    // 384 / 512 rows 35 -> 32, 36.5 -> 35, 56 -> 49, 58 -> 56 us, output projection at 128 / 512 rows 15.6 -> 13.6, 26.3 -> 25.2.)
    const auto in_slices = [&](int ks) {   // the cheapest blocks of that many slices, and their cost
      AccPlan q{1, ks, pick_block(kAccBlocks, m_tiles, n_tiles, (k_steps + ks - 1) / ks, ks)};
      q.cost = block_cost(m_tiles, n_tiles, (k_steps + ks - 1) / ks, q.block.mt, q.block.nt, ks) + (long)ks * m_tiles * n_tiles * 1024 * 8 / 5000;
      return q;
    };
    for (int ks = 1; ks <= most; ++ks) {
      const AccPlan q = in_slices(ks);
      if (ks == 1 || q.cost < p.cost) p = q;
    }
    // No more than 128 x 128 blocks fill the chip with, unless more are a tenth cheaper: the rule is no finer than that (7B shape, down
    // projection: it finds four slices 7 % cheaper than two; a whole call is 1.7 / 1.2 / 0.9 % faster with two at 288 / 416 / 448 rows,
    // as fast at 480, 0.7 % slower at 512), and the sums stay those of the tiled kernel, which sliced like this.
    const int fill = 256 / ((m_tiles + 3) / 4 * ((n_tiles + 3) / 4));
    if (p.ksplit > fill) {
      const AccPlan q = in_slices(fill < 1 ? 1 : fill);
      if (p.cost * 10 >= q.cost * 9) p = q;
    }
    if (compacted) p.block = pick_block(kAccHalves, m_tiles, n_tiles, k_steps / p.ksplit, p.ksplit);
    return p;
  }
  if (one_chunk) {
    p.kind = 2;
    p.ksplit = 256 / (n_tiles / NW);
  } else if ((m_tiles == 1 || (m_tiles == 2 && n_tiles > 212)) && n_tiles % 2 == 0 && n_tiles > 128 && n_tiles < 256 && k_steps / 64 >= 512 / n_tiles) {
    // One tile per workgroup would need two slices and a second round of workgroups for the remainder: two tiles and up to
    // three slices fit one round (13B output projection, 160 tiles: 16.1 -> 13.8 us at 32 rows).  At 128 tiles two slices fill the
    // chip exactly, and four of two tiles cost the normalisation more than they gain (12.6 against 13.0).
    p.kind = 3;
    p.ksplit = 512 / n_tiles;
  } else if (m_tiles == 2 && n_tiles >= 128 && k_steps >= 4) {
    // 64 x 64 blocks: 7B output projection 12.9 -> 9.1 us at 64 rows (its four wavefronts no longer fetch an operand each).  A whole
    // iteration against the form above or, at 128 and 256 tiles, below: 136 to 200 tiles 2.4 to 4.4 % faster at 64 rows, 2 to 3 % at
    // 36 to 40, 212 tiles 1 and 0 %, 256 tiles 3 and 2.5 %; 216 to 248 tiles, where that form's pairs fill the chip as well, 1 to 1.5 %
    // slower at 36 rows and no faster at 64: they keep it.  (Adding a slice in four parts, as that kernel does, costs nothing.)
    p.kind = 1;
    p.block = {2, 2};
    p.ksplit = 512 / n_tiles;
  } else {
    // streaming kernel (its four wavefronts already split the slice four ways): enough workgroups for every
    // compute unit, no more
    p.ksplit = (256 + n_tiles - 1) / n_tiles;
  }
  if (p.ksplit > most) p.ksplit = most;
  if (p.ksplit < 1) p.ksplit = 1;
  return p;
}

// The ring kernel needs 128 KiB of dynamic LDS: asked for once per process (the attribute belongs to the function,
// not to a launch), at the first launch that wants it or by gemm_bf16_prepare().
template <class Epi>
bool ring_allowed() {
  static int ok = -1;
  if (ok < 0) {
    ok = hipFuncSetAttribute(reinterpret_cast<const void*>(gemm_ring_kernel<Epi>), hipFuncAttributeMaxDynamicSharedMemorySize,
                             RING_LDS_BYTES) == hipSuccess;
    if (!ok) (void)hipGetLastError();   // not the call's error: another kernel takes the shape
  }
  return ok > 0;
}

// Wavefronts that multiply (rows x columns of the block) and stages of each block shape.  Two workgroups share a compute unit where
// LDS (2 * DS * (MT + NT) KiB of 160) and registers allow: not with eight batch or weight tiles, nor in 128 x 192 blocks of QKV (206
// registers).
template <int MT, int NT, int WM, int WN, int DS, class Epi>
void launch_block(const GemmShape& g, const Epi& e, Pred pred, int ksplit, hipStream_t st) {
  const BlockGrid bg{((g.M + 31) / 32 + MT - 1) / MT, (g.n_tiles + NT - 1) / NT, ksplit};
  const dim3 grid((bg.col_blocks * ksplit + 7) / 8 * 8 * bg.row_blocks), block((WM * WN + BLOCK_NL) * 64);
  if constexpr ((MT == 4 && NT % 2 == 0 && !std::is_same<Epi, QkvEpi>::value) || (MT == 8 && std::is_same<Epi, GateUpEpi>::value)) {
    if (g.n_rows_dev) {
      hipLaunchKernelGGL((gemm_block_kernel<MT, NT, WM, WN, DS, true, Epi>), grid, block, 0, st, g, e, pred, bg);
      return;
    }
  }
  hipLaunchKernelGGL((gemm_block_kernel<MT, NT, WM, WN, DS, false, Epi>), grid, block, 0, st, g, e, pred, bg);
}
template <class Epi>
void launch_blocks(BlockShape b, const GemmShape& g, const Epi& e, Pred pred, int ksplit, hipStream_t st) {
  constexpr bool QKV = std::is_same<Epi, QkvEpi>::value, ACC = std::is_same<Epi, AccEpi>::value, GATE = std::is_same<Epi, GateUpEpi>::value,
                 LM = std::is_same<Epi, LmEpi>::value;
  switch (b.mt * 16 + b.nt) {
    case 0x22: if constexpr (ACC) launch_block<2, 2, 2, 1, 8>(g, e, pred, ksplit, st); break;
    case 0x23: if constexpr (QKV) launch_block<2, 3, 2, 1, 8>(g, e, pred, ksplit, st); break;
    case 0x42: if constexpr (QKV || ACC) launch_block<4, 2, 4, 1, 6>(g, e, pred, ksplit, st); break;
    case 0x43: if constexpr (QKV || GATE) launch_block<4, 3, 4, 1, 5>(g, e, pred, ksplit, st); break;
    case 0x44: launch_block<4, 4, 2, 2, 5>(g, e, pred, ksplit, st); break;
    case 0x46: if constexpr (QKV || GATE) launch_block<4, 6, 2, 2, 4>(g, e, pred, ksplit, st); break;
    case 0x48: if constexpr (LM) launch_block<4, 8, 2, 2, 5>(g, e, pred, ksplit, st); break;
    case 0x84: if constexpr (GATE || ACC) launch_block<8, 4, 2, 2, 5>(g, e, pred, ksplit, st); break;
    case 0x86: if constexpr (GATE) launch_block<8, 6, 4, 2, 5>(g, e, pred, ksplit, st); break;
  }
}

template <class Epi, bool FILL>
void launch(const GemmShape& g, const Epi& e, Pred pred, const FillCtl& fc, int nz, hipStream_t st,
            const CombineJob& cj = CombineJob{}) {
  dim3 block(256);
  const int m_tiles = (g.M + 31) / 32;
  constexpr bool ACC = std::is_same<Epi, AccEpi>::value, LM = std::is_same<Epi, LmEpi>::value;
  const AccPlan ap = ACC ? acc_plan(g.M, g.n_tiles, g.K, g.n_rows_dev != nullptr) : AccPlan{0, 1, {0, 0}, 0};
  const int k_steps = g.K >> 4;
  if constexpr (!FILL) {
    // Block kernel: QKV from three batch tiles on (at two the streaming kernel, which carries the exit decision), accumulate
    // projections by acc_plan, gate/up and the LM head from five (three where the tiled kernel does not take their tiles, below).
    // (7B shape, us: QKV at 128 / 192 / 256 / 384 / 512 rows 39 -> 34, 47 -> 38, 49 -> 42, 74 -> 58, 76 -> 59; gate/up at 192 / 256 / 384 /
    // 512 74 -> 58, 76 -> 62, 95 -> 81, 107 -> 82; LM head at 192 / 350 / 384 80 -> 77, 129 -> 116, 129 -> 116; at 128 rows and fewer
    // gate/up and the LM head are bound by the weight stream either way: 44 against 43 to 46 us, 47 against 51.)
    if constexpr (ACC) {
      if (ap.kind == 1) {
        launch_blocks(ap.block, g, e, pred, ap.ksplit, st);
        return;
      }
    } else if constexpr (std::is_same<Epi, QkvEpi>::value) {
      if (m_tiles >= 3) {
        launch_blocks(pick_block(kQkvBlocks, m_tiles, g.n_tiles, k_steps), g, e, pred, 1, st);
        return;
      }
    } else {
      // If the runtime refused the ring its 128 KiB of dynamic LDS, another kernel serves the shape.  (Only what is asked for can be
      // refused: the blocks' LDS, up to 140 KiB, is static.)
      const bool ring = !g.n_rows_dev && ring_serves(g.M, g.n_tiles, g.K) && ring_allowed<Epi>();
      // Three or four batch tiles, weight tiles that the tiled kernel does not take: blocks where one workgroup a tile no longer
      // fits one round (331 tiles, exit check: K of 704 / 2048 / 4096 2 to 6 / 7 to 13 / 16 to 32 us faster than in the streaming
      // kernel).  Fewer tiles leave compute units idle in either, but the streaming kernel's wavefronts split the contraction four
      // ways (128 rows, 50 tiles: K of 2048 / 4096 24.1 / 35.5 us a check in blocks, 22.3 / 26.9), unless three batch tiles, which it
      // takes one after the other, cost it more: up to 48 steps (78 tiles of 44 steps 18.6 -> 17.4) or from 129 tiles on.
      const bool blocks = m_tiles >= 5 || (m_tiles >= 3 && g.n_tiles % NW && (g.n_tiles > 256 || (m_tiles == 3 && (k_steps <= 48 || g.n_tiles > 128))));
      if constexpr (std::is_same<Epi, GateUpEpi>::value) {
        const BlockShape b = !g.n_rows_dev   ? pick_block(kGateUpBlocks, m_tiles, g.n_tiles, k_steps)
                             : m_tiles <= 8 ? pick_block(kGateUpHalves256, m_tiles, g.n_tiles, k_steps)
                                            : pick_block(kGateUpHalves, m_tiles, g.n_tiles, k_steps);
        // The ring kernel where its 256 x 256 blocks fit one round and 256 x 192 ones do not (776 to 1024 tiles; 1544 to 2048 in two
        // rounds against three).  A whole iteration of 400 to 512 rows, 776 to 1024 tiles, in blocks and in the ring: K of 1024 480 to
        // 568 -> 454 to 526 us, 2048 408 to 469 -> 382 to 451, 4096 722 to 833 -> 707 to 814, 5120 (13B shape, 864 tiles, 512 rows) 1020
        // -> 995; K of 256 299 to 335 -> 302 to 331.  1544 to 2048 tiles: K of 1024 396 to 463 -> 369 to 419, 4096 1054 to 1226 -> 1025 to 1198.
        const long ring_cost = block_cost(m_tiles, g.n_tiles, k_steps, 8, 8);
        if (blocks && !(ring && ring_cost < block_cost(m_tiles, g.n_tiles, k_steps, b.mt, b.nt))) {
          launch_blocks(b, g, e, pred, 1, st);
          return;
        }
      } else if (blocks && (g.n_rows_dev || !ring_serves(g.M, g.n_tiles, g.K))) {
        // 128 x 256 blocks are what the tiled kernel has with two tiles per wavefront: they pay from 192 steps on (140 to 192 rows, 1000
        // tiles: 128 steps 39.4 -> 41.8 us, 256 steps 76 to 74 -> 66 to 70; 320 to 384 rows: 124 to 126 -> 114 to 118), not where that
        // kernel's two 128-row chunks are nearly full (200 to 256 rows: 73 to 76 both ways).
        const BlockShape b = pick_block(kLmBlocks, m_tiles, g.n_tiles, k_steps);
        if (g.n_rows_dev || b.nt < 8 || (k_steps >= 192 && (m_tiles < 7 || m_tiles > 8)) || g.n_tiles % (2 * NW)) {
          launch_blocks(b, g, e, pred, 1, st);
          return;
        }
      }
      if (ring) {
        const int row_blocks = (m_tiles + 7) / 8, col_blocks = g.n_tiles / 8;
        dim3 gridr((col_blocks + 7) / 8 * 8 * row_blocks, 1, 1);
        hipLaunchKernelGGL((gemm_ring_kernel<Epi>), gridr, block, RING_LDS_BYTES, st, g, e, pred);
        return;
      }
    }
  }
  // Tiled kernel: KV filling, gate/up and the LM head at three and four batch tiles, the LM head where block_cost leaves it.  Batch
  // chunks of 4 tiles (128 rows) measured faster than 8 at batch 256 and 512: twice the workgroups, each with half the accumulators,
  // keeps more loads in flight; the second chunk's weight reads mostly hit the caches.
  if constexpr (FILL || LM || std::is_same<Epi, GateUpEpi>::value) {
    if (tiled(g.M, g.n_tiles)) {
      const int chunks = (m_tiles + 3) / 4, groups = g.n_tiles / NW;
      // Weights that three row chunks and more read are loaded to stay in the L2 that the chunks share, instead of past it.
      GemmShape g4 = g;
      g4.grid_y = chunks;
      g4.keep = FILL && chunks >= 3;
      if constexpr (LM) {
        // Two output tiles per wavefront (each LDS operand read feeds two MFMAs, half the workgroups): 161 -> 153 us at 512
        // rows.
        if (g.n_tiles % (2 * NW) == 0 && chunks >= 2) {
          const int groups2 = g.n_tiles / (2 * NW);
          dim3 grid2((groups2 + 7) / 8 * 8 * chunks, 1, nz);
          hipLaunchKernelGGL((gemm_tiled_kernel<4, 2, Epi, FILL>), grid2, block, 0, st, g4, e, pred, fc);
          return;
        }
      }
      dim3 grid((groups + 7) / 8 * 8 * chunks, 1, nz);
      hipLaunchKernelGGL((gemm_tiled_kernel<4, 1, Epi, FILL>), grid, block, 0, st, g4, e, pred, fc);
      return;
    }
  }
  // One or two batch tiles: the tiled kernel still wins where enough output tiles keep the chip busy with four
  // tiles per workgroup (its four wavefronts share every activation tile through LDS, a quarter of the L2 reads
  // of the streaming kernel): LM head, gate/up and the down projection (measured at 32 rows: 47.0 -> 44.0,
  // 34.6 -> 33.2, 21.8 -> 20.8 us; at 64 rows: 62.8 -> 43.5, 44.4 -> 38.3, 27.5 -> 25.4).  QKV and the output
  // projection have too few tiles for that and stay with the streaming kernel.
  // KV filling takes the same route: one launch covers many layers, so there are always enough workgroups, and the
  // four tiles of a workgroup are the 128 channels of one head, whose cache lines then leave from one L2.
  if constexpr (FILL || !std::is_same<Epi, QkvEpi>::value) {
    const bool small_tiled = ACC ? ap.kind == 2 : (m_tiles <= 2 && g.n_tiles % NW == 0 && g.split_tiles == 0);
    if (small_tiled) {
      const int groups = g.n_tiles / NW;
      GemmShape gs = g;
      gs.grid_y = ap.ksplit;   // one chunk
      dim3 grid1((groups + 7) / 8 * 8 * ap.ksplit, 1, nz);
      // Fewer groups of four than compute units, more tiles than compute units: deal the tiles out over all 256
      // units instead (two to four each), so that no unit streams more than its share.
      if (!ACC && !FILL && groups < 256 && g.n_tiles > 256) {
        gs.even_wgs = 256;
        grid1 = dim3(256, 1, nz);
      }
      if (m_tiles == 1)
        hipLaunchKernelGGL((gemm_tiled_kernel<1, 1, Epi, FILL>), grid1, block, 0, st, gs, e, pred, fc);
      else if (!ACC || m_tiles == 2)
        hipLaunchKernelGGL((gemm_tiled_kernel<2, 1, Epi, FILL>), grid1, block, 0, st, gs, e, pred, fc);
      else if constexpr (ACC)
        hipLaunchKernelGGL((gemm_tiled_kernel<4, 1, Epi, FILL>), grid1, block, 0, st, gs, e, pred, fc);
      return;
    }
  }
  // Streaming kernel.  Two tiles per workgroup where they fill the chip in one round.
  // QKV, two batch tiles: pairs on 129 to 256 workgroups (264 tiles: 24.4 -> 22.6 us, 384: 34 -> 31, 480: 45 -> 38; 64 x 64 blocks:
  // as fast, 38.3 against 37.8).  One batch tile: up to 384 tiles 2 * split_tiles whole tiles with a half each (294 tiles: 20.5 -> 19.0,
  // 384: 24.2 -> 22.7), beyond pairs (480: 39 -> 31); at 288 tiles and fewer the idle compute units cost more than the shared operand
  // saves (pairs of 288: 19.1 -> 20.3, of 264: 17.4 -> 19.6).
  // Gate/up whose tiles do not divide by four: two batch tiles only (258 to 506 tiles: 16.1 -> 15.9, 17.5 -> 16.5, 18.1 -> 17.4,
  // 19.7 -> 19.6; one: 12.5 -> 13.4, 13.9 -> 14.5, 14.4 -> 14.9, 15.8 -> 17.7).  The LM head gains at neither (16 rows: 12.7 to 15.4 ->
  // 14.0 to 18.1, 64 rows: 16.8 to 19.9 -> 17.0 to 20.9): its statistics follow each tile.
  if constexpr (!FILL) {   // (KV filling has whole groups of four tiles)
    if constexpr (!LM) {
      constexpr bool QKV = std::is_same<Epi, QkvEpi>::value, GATE = std::is_same<Epi, GateUpEpi>::value;
      const bool one_half = QKV && m_tiles == 1 && 3 * g.split_tiles == g.n_tiles && g.split_tiles > 96 && g.split_tiles <= 128;
      const bool pairs = m_tiles <= 2 && g.n_tiles % 2 == 0 && g.n_tiles > (m_tiles == 1 ? 384 : 256) && g.n_tiles <= 512;
      if (ACC ? ap.kind == 3 : one_half || (pairs && (QKV || m_tiles == 2))) {
        GemmShape g2 = g;
        if (!one_half) g2.split_tiles = 0;
        const dim3 grid2((one_half ? 2 * g.split_tiles : g.n_tiles / 2) + cj.n_wg, ACC ? ap.ksplit : 1, nz);
        if constexpr (!GATE) {
          if (m_tiles == 1) {
            hipLaunchKernelGGL((gemm_mfma_kernel<1, 2, 4, Epi, FILL>), grid2, block, 0, st, g2, e, pred, fc, cj);
            return;
          }
        }
        hipLaunchKernelGGL((gemm_mfma_kernel<2, 2, 4, Epi, FILL>), grid2, block, 0, st, g2, e, pred, fc, cj);
        return;
      }
    }
    // split tiles take two workgroups each (one batch tile only); the workgroups of a combine job come first
    dim3 grid(g.n_tiles + g.split_tiles + cj.n_wg, ACC ? ap.ksplit : 1, nz);
    if constexpr (LM || std::is_same<Epi, GateUpEpi>::value) {
      if (m_tiles == 4) {
        hipLaunchKernelGGL((gemm_mfma_kernel<4, 1, 2, Epi, FILL>), grid, block, 0, st, g, e, pred, fc, cj);
        return;
      }
    }
    if (m_tiles == 2)
      hipLaunchKernelGGL((gemm_mfma_kernel<2, 1, 4, Epi, FILL>), grid, block, 0, st, g, e, pred, fc, cj);
    else
      hipLaunchKernelGGL((gemm_mfma_kernel<1, 1, 8, Epi, FILL>), grid, block, 0, st, g, e, pred, fc, cj);
  }
}

}  // namespace

bool gemm_bf16_takes_compacted(int n_tiles) { return n_tiles % NW == 0; }

void gemm_bf16_prepare() {
  ring_allowed<LmEpi>();
  ring_allowed<GateUpEpi>();
}

int gemm_acc_slices(int M, int n_tiles, int K) { return acc_plan(M, n_tiles, K).ksplit; }

// (the most that the plan may write at M rows or, where fewer rows come in more slices, at fewer)
size_t gemm_acc_rows(int M, int n_tiles, int K) {
  const int m = (M + 31) / 32;
  int tiles = m;
  for (int i = 1; i <= 16 && i <= m; ++i)
    if (tiles < i * acc_slices_most(i, n_tiles, K)) tiles = i * acc_slices_most(i, n_tiles, K);
  const int wide = K / 1024 * m < 64 ? K / 1024 * m : 64;   // more than 512 rows: up to 64 tiles in all
  if (m > 16 && tiles < wide) tiles = wide;
  return (size_t)tiles * 32;
}

bool gemm_qkv_carries_combine(int M) { return (M + 31) / 32 <= 2; }   // the streaming kernel serves these batches

void launch_gemm_qkv_bf16(const GemmShape& g, const QkvEpi& e, Pred pred, hipStream_t st, const CombineArgs* with_combine,
                          const DecideArgs* with_decide) {
  FillCtl fc{};
  CombineJob cj{};
  if (with_combine) {
    cj.a = *with_combine;
    cj.kind = 1;
    cj.n_wg = (with_combine->B + 7) / 8 * 8;   // a multiple of 8: the tiles keep their XCDs
  } else if (with_decide) {
    cj.d = *with_decide;
    cj.kind = 2;
    cj.n_wg = 8;
  }
  launch<QkvEpi, false>(g, e, pred, fc, 1, st, cj);
}
void launch_gemm_acc_bf16(const GemmShape& g, const AccEpi& e, Pred pred, hipStream_t st) {
  FillCtl fc{};
  launch<AccEpi, false>(g, e, pred, fc, 1, st);
}
void launch_gemm_gateup_bf16(const GemmShape& g, const GateUpEpi& e, Pred pred, hipStream_t st) {
  FillCtl fc{};
  launch<GateUpEpi, false>(g, e, pred, fc, 1, st);
}
void launch_gemm_lm_bf16(const GemmShape& g, const LmEpi& e, Pred pred, hipStream_t st) {
  FillCtl fc{};
  launch<LmEpi, false>(g, e, pred, fc, 1, st);
}
void launch_gemm_kvfill_bf16(const FillLayers& fl, int n_layers, const bf16_t* x_slabs, size_t x_slab_elems,
                             size_t pool_layer_elems, const GemmShape& g, const QkvEpi& e, Pred pred, hipStream_t st) {
  FillCtl fc{};
  fc.layers = fl;
  fc.x_slabs = x_slabs;
  fc.x_slab_elems = x_slab_elems;
  fc.pool_layer_bytes = pool_layer_elems * sizeof(bf16_t);
  launch<QkvEpi, true>(g, e, pred, fc, n_layers, st);
}

}  // namespace ee
