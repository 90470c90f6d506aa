"""Attention of the float path beside the exit decision that shares its launch, without a GPU: the kernel's source is built for the host
with stand-ins for the device built-ins (a lane is a coroutine, a shuffle an exchange, LDS a static array), and its workgroup runs while the
decision's stores become visible at any point, in any part.

One wavefront may see a sequence as left where the next one still sees it stay, if they look at a word that the launch writes.  The
workgroup then walks a block table that only some of its wavefronts have filled, and the cache is read wherever the leftovers of LDS point."""
import os
import re
import subprocess

import pytest

from paper_2407_20272_amd import build

RUNTIME = r"""
#pragma once
#include <math.h>
#include <stddef.h>
#include <stdint.h>
#include <string.h>
#define __global__
#define __device__
#define __host__
#define __shared__ static
#define __forceinline__ inline
#define __launch_bounds__(...)
#define __align__(n) __attribute__((aligned(n)))
#define __hip_atomic_load(p, order, scope) emu::load(p)
#define __hip_atomic_store(p, v, order, scope) emu::store(p, v)
#define __hip_atomic_fetch_add(p, v, order, scope) emu::add(p, v)
#define __builtin_nontemporal_load(p) emu::fetch(p)
#define __builtin_amdgcn_readfirstlane(x) (x)
#define __builtin_amdgcn_exp2f(x) exp2f(x)
#define __builtin_amdgcn_sched_barrier(x) ((void)0)
#define __builtin_amdgcn_update_dpp(old, v, ctrl, rows, banks, bound) \
  emu::swap(v, (ctrl) == 0xB1 ? 1 : (ctrl) == 0x4E ? 2 : (ctrl) == 0x141 ? 7 : 15)
#define __shfl_xor(v, x) emu::swap(v, x)
#define __syncthreads() emu::meet()
#define threadIdx (*emu::tid)
struct dim3 { unsigned x, y, z; };
struct uint4 { unsigned x, y, z, w; };
struct float2 { float x, y; };
struct __attribute__((aligned(16))) float4 { float x, y, z, w; };
typedef void* hipStream_t;
typedef int hipError_t;
inline uint4 make_uint4(unsigned x, unsigned y, unsigned z, unsigned w) { return {x, y, z, w}; }
inline float2 make_float2(float x, float y) { return {x, y}; }
inline float4 make_float4(float x, float y, float z, float w) { return {x, y, z, w}; }
inline int min(int a, int b) { return a < b ? a : b; }
inline int max(int a, int b) { return a > b ? a : b; }
inline int __float_as_int(float x) { int i; memcpy(&i, &x, 4); return i; }
inline float __int_as_float(int i) { float x; memcpy(&x, &i, 4); return x; }
inline float __uint_as_float(unsigned i) { float x; memcpy(&x, &i, 4); return x; }
inline float rsqrtf(float x) { return 1 / sqrtf(x); }
#define __expf expf
static dim3 blockIdx, gridDim, blockDim = {256, 1, 1};
namespace emu {
extern dim3* tid;
int32_t load(const int32_t* p);
void store(int32_t* p, int32_t v);
int32_t add(int32_t* p, int32_t v);
unsigned exchange(unsigned v, int x);
void meet();
const void* within(const void* p);
template <class T> T swap(T v, int x) { unsigned u; memcpy(&u, &v, 4); u = exchange(u, x); memcpy(&v, &u, 4); return v; }
template <class T> T fetch(const T* p) { return *(const T*)within(p); }
}
"""

PROGRAM = r"""
#include <stdio.h>
#include <stdlib.h>
#include <ucontext.h>
#include <vector>
#include "attention_source.h"
namespace ee { namespace { int32_t tbl[16384]; } }

constexpr int H = 2, DH = 64, D = H * DH, B = 2, BLOCKS = 256, N_LAYERS = 3;
alignas(16) static float k_pool[BLOCKS * H * 16 * DH], v_pool[BLOCKS * H * 16 * DH], q[B * D], w_o[D * D], ao[B * D], parts[H * B * D];
static int32_t status[B], exit_layer[B], n_exited, done, batch_exit_layer, lens[B], tables[B * 256];
static const ee::IterState state = {status, exit_layer, &n_exited, &done, &batch_exit_layer};

// ---- a workgroup: 256 coroutines, wavefronts one after the other in a given order ----
namespace emu {
struct Lane { ucontext_t c; dim3 id; bool at_barrier, over; };
static Lane lanes[256];
static ucontext_t here;
static unsigned slots[4][2][64], turn[256];
static int cur, outside;
dim3* tid;
static ee::AttnArgs args; static ee::Oproj op; static ee::Pred pred;
static unsigned visible = ~0u;                                   // which of the decision's words are

static int bit(const int32_t* p) {
  return p == &n_exited ? 0 : p == &done ? 1 : p == &batch_exit_layer ? 2 : p >= status && p < status + B ? 3 : 4;
}
int32_t load(const int32_t* p) { return *p; }
void store(int32_t* p, int32_t v) { if (visible >> bit(p) & 1) *p = v; }
int32_t add(int32_t* p, int32_t v) { int32_t o = *p; store(p, o + v); return o; }
static void leave() { swapcontext(&lanes[cur].c, &here); }
unsigned exchange(unsigned v, int x) {                           // two sets: a lane may be one exchange ahead of another
  const int t = cur, wave = t >> 6, set = turn[t]++ & 1;
  slots[wave][set][t & 63] = v;
  leave();
  return slots[wave][set][(t & 63) ^ x];
}
void meet() { lanes[cur].at_barrier = true; leave(); }
const void* within(const void* p) {
  static const char zeros[64] = {};
  const char* c = (const char*)p;
  auto in = [&](const void* a, size_t n) { return c >= (const char*)a && c + 16 <= (const char*)a + n; };
  if (in(k_pool, sizeof k_pool) || in(v_pool, sizeof v_pool) || in(&ee::k_zero16, 16)) return p;
  ++outside;
  return zeros;
}
static void body() {
  ee::attn_f32_kernel<DH>(args, pred, op);
  lanes[cur].over = true;
  leave();
}
template <class Before>
static void workgroup(const int (&order)[4], Before before) {    // before(k): ahead of the k-th wavefront's first instruction
  static std::vector<char> stacks(256 * 65536);
  for (int t = 0; t < 256; ++t) {
    lanes[t] = Lane{};
    lanes[t].id = {(unsigned)t, 0, 0};
    turn[t] = 0;
    getcontext(&lanes[t].c);
    lanes[t].c.uc_stack.ss_sp = &stacks[(size_t)t * 65536];
    lanes[t].c.uc_stack.ss_size = 65536;
    lanes[t].c.uc_link = nullptr;
    makecontext(&lanes[t].c, body, 0);
  }
  for (bool first = true;; first = false) {
    bool any = false;
    for (int k = 0; k < 4; ++k) {
      if (first) before(k);
      for (bool again = true; again;) {                          // a step of all 64 lanes, until the wavefront waits or is over
        again = false;
        for (int l = 0; l < 64; ++l) {
          cur = order[k] * 64 + l;
          if (lanes[cur].at_barrier || lanes[cur].over) continue;
          tid = &lanes[cur].id;
          swapcontext(&here, &lanes[cur].c);
          again = true;
        }
      }
    }
    for (Lane& l : lanes)
      if (!l.over) l.at_barrier = false, any = true;
    if (!any) return;
  }
}
}

int main(int argc, char** argv) {
  const int max_blocks = atoi(argv[1]), ctx = atoi(argv[2]), oproj = atoi(argv[3]);
  unsigned seed = 1;
  auto rnd = [&] { seed = seed * 1664525u + 1013904223u; return (float)(seed >> 8) / (1 << 24) - 0.5f; };
  for (float* p : {k_pool, v_pool}) for (int i = 0; i < BLOCKS * H * 16 * DH; ++i) p[i] = rnd();
  for (float& x : q) x = rnd();
  for (float& x : w_o) x = rnd();
  for (int b = 0; b < B; ++b) {
    lens[b] = ctx - b;
    for (int i = 0; i < max_blocks; ++i) tables[b * max_blocks + i] = (i * 37 + b * 5) % BLOCKS;
  }
  const int layer = 2;                                           // the decision that shares the launch
  ee::CombineArgs ca{};
  ca.B = B; ca.layer = layer; ca.s = state; ca.left = status;
  emu::args = ee::AttnArgs{q, k_pool, v_pool, lens, tables, max_blocks, B, H, DH, ao, 0, status, nullptr, nullptr, BLOCKS, nullptr, 1};
  emu::op = ee::Oproj{oproj ? w_o : nullptr, parts, ee::SimpleDecision{ca, nullptr, nullptr, 0, 1}};
  gridDim = {H, B + 1, oproj ? 4u : 1u};
  auto fresh = [&](int others) {                                 // others: the other sequence left at this layer already, or before
    for (int b = 0; b < B; ++b) status[b] = 0, exit_layer[b] = N_LAYERS;
    n_exited = done = 0;
    batch_exit_layer = N_LAYERS;
    if (others) status[0] = 1, exit_layer[0] = others, n_exited = 1;
    for (int32_t& x : ee::tbl) x = 1 << 26;                      // what an earlier workgroup left
    memset(ao, 0xff, sizeof ao);
    memset(parts, 0xff, sizeof parts);
  };
  int runs = 0, wrong = 0, idle = 0;
  std::vector<char> want(sizeof ao + sizeof parts), got(want);
  auto keep = [&](std::vector<char>& v) { memcpy(v.data(), ao, sizeof ao); memcpy(v.data() + sizeof ao, parts, sizeof parts); };
  const int orders[2][4] = {{0, 1, 2, 3}, {3, 1, 2, 0}};
  blockIdx = {1, 2, oproj ? 2u : 0u};                            // head 1, sequence 1, one of the four that share a head's columns
  fresh(0);
  emu::workgroup(orders[0], [](int) {});
  keep(want);
  if (!memcmp(want.data(), std::vector<char>(want.size(), 0xff).data(), want.size())) return printf("nothing was written\n"), 1;
  for (int others : {0, 1, 2})
    for (auto& order : orders)
      for (int when = 0; when < 4; ++when)
        for (unsigned visible = 0; visible < 32; ++visible) {
          const int words = __builtin_popcount(visible);         // none, one, all but one, all
          if (words > 1 && words < 4) continue;
          fresh(others);
          emu::workgroup(order, [&](int k) {
            if (k != when) return;
            emu::visible = visible;
            ee::decide_row(state, 1, B, layer, 1.0f, 0.5f, nullptr, nullptr);
            emu::visible = ~0u;
          });
          keep(got);
          ++runs;
          wrong += got != want;
        }
  // a sequence that left at an earlier layer is not attended, however late the launch's own decision about the other comes
  for (int when = 0; when < 4; ++when) {
    fresh(0);
    status[1] = 1, exit_layer[1] = 1, n_exited = 1;
    emu::workgroup(orders[when % 2], [&](int k) { if (k == when) ee::decide_row(state, 0, B, layer, 1.0f, 0.5f, nullptr, nullptr); });
    for (float x : parts) idle += x == x;
    for (float x : ao) idle += x == x;
  }
  printf("%d runs, %d with other results, %d loads outside the pools, %d values of a sequence that had left\n", runs, wrong, emu::outside, idle);
  return wrong || emu::outside || idle;
}
"""

def kernels_of(name, end):
    """A source file up to where its kernels end, for a compiler that knows neither LDS nor the GPU's registers."""
    with open(os.path.join(build.CSRC, name)) as f:
        source = f.read()
    assert source.count(end) == 1
    source = re.sub(r'asm volatile\("" ::"s"[^;]*;', ";", source[:source.index(end)].replace("extern __shared__", "extern"))
    return source + "\n}}\n"


def build_for_host(d, program):
    (d / "hip").mkdir()
    (d / "hip" / "hip_runtime.h").write_text(RUNTIME)
    (d / "attention_source.h").write_text(kernels_of("attention.hip", "// Second launch of the split form"))
    (d / "projections_source.h").write_text(kernels_of("gemm_simple.hip", "bool aligned16("))
    (d / "program.cpp").write_text(program)
    clang = os.path.join(os.path.dirname(os.path.realpath(build._hipcc())), "..", "llvm", "bin", "clang++")
    subprocess.run([clang if os.path.exists(clang) else "/opt/rocm/llvm/bin/clang++", "-x", "c++", "-std=c++17", "-O1", "-Wno-everything", "-I" + str(d),
                    "-I" + os.path.join(build.ROOT, "include"), "-I" + build.CSRC, str(d / "program.cpp"), "-o", str(d / "program")],
                   check=True, capture_output=True, text=True)
    return str(d / "program")


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    return build_for_host(tmp_path_factory.mktemp("host_float_attention"), PROGRAM)


@pytest.mark.parametrize("max_blocks,ctx,oproj", [
    (15, 200, 1),    # a table that one wavefront fills, the output projection inside
    (15, 200, 0),
    (70, 1100, 0),   # a table of two wavefronts
    (3, 17, 1),      # fewer blocks than wavefronts
])
def test_wavefronts_agree_while_the_launch_decides(program, max_blocks, ctx, oproj):
    out = subprocess.run([program, str(max_blocks), str(ctx), str(oproj)], capture_output=True, text=True, timeout=120)
    assert out.returncode == 0, out.stdout + out.stderr

IN_VAIN = r"""
#include <stdio.h>
#include <stdlib.h>
#include "attention_source.h"
#include "projections_source.h"
namespace ee { namespace { int32_t tbl[16384]; } }
namespace emu {
static dim3 one;
dim3* tid = &one;
static int32_t words[2] = {1, 1};                                // the batch has left, at layer 1
int32_t load(const int32_t* p) { return *p; }
void store(int32_t*, int32_t) { abort(); }
int32_t add(int32_t*, int32_t) { abort(); }
unsigned exchange(unsigned, int) { abort(); }
void meet() { abort(); }
const void* within(const void*) { abort(); }
}
using namespace ee;
template <class Epi, bool NORM, bool PARTS>
static void projection(Epi e) {
  SimpleShape g{};                                               // an operand that is looked at is a null pointer
  g.K = 256, g.M = 4, g.n_rows = 64, g.pair_stride = 1;
  const Pred pred{&emu::words[0], 0};
  gemm_simple_kernel<Epi, NORM, true, PARTS, 1>(g, e, pred, NoFill{}, NoJob{});
  if (!PARTS) gemm_simple_kernel<Epi, NORM, true, false, 0>(g, e, pred, NoFill{}, NoJob{}), gemm_simple_kernel<Epi, NORM, true, false, 4>(g, e, pred, NoFill{}, NoJob{});
  gemm_simple_kernel<Epi, NORM, false, PARTS, 0>(g, e, pred, NoFill{}, NoJob{});
}
int main() {
  gridDim = {4, 4, 4};
  QkvEpi qkv{};
  qkv.n_heads = 4, qkv.head_dim = 64, qkv.d_model = 256, qkv.max_blocks = 15, qkv.rope_theta = 1;
  projection<QkvEpi, true, false>(qkv);
  projection<AccEpi, false, false>(AccEpi{});
  projection<GateUpEpi, true, false>(GateUpEpi{});
  projection<GateUpEpi, true, true>(GateUpEpi{});
  projection<LmEpi, true, false>(LmEpi{});
  AttnArgs a{};
  a.max_blocks = 15, a.B = 4, a.n_heads = 4, a.head_dim = 64, a.num_blocks = 64;
  attn_f32_kernel<64>(a, Pred{&emu::words[0], 0}, Oproj{});
  Oproj op{};
  op.job.n_wg = 1, op.job.a.layer = 2, op.job.a.s.done = &emu::words[0], op.job.a.s.batch_exit_layer = &emu::words[1];
  blockIdx = {0, 1, 0};
  attn_f32_kernel<64>(a, Pred{}, op);
  puts("nothing was looked at");
}
"""


def test_launches_behind_the_exit_look_at_nothing(tmp_path):
    """The layers of a batch that has left are launches in vain: they return on the predicate and ask for no operand first (every pointer of
    theirs is null here)."""
    out = subprocess.run([build_for_host(tmp_path, IN_VAIN)], capture_output=True, text=True, timeout=60)
    assert out.returncode == 0 and out.stdout == "nothing was looked at\n", out
