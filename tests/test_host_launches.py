"""What the host side enqueues when the runtime refuses something, without a GPU: a small C program brings its own
hipLaunchKernel, hipFuncSetAttribute, .. (a program's symbols come before those of the libraries it loads), calls the library with
made-up device pointers, which the host never follows, and prints every launch, with the kernel's name."""
import ctypes
import os
import subprocess

import pytest

from paper_2407_20272_amd import binding as B
from paper_2407_20272_amd import build

PROGRAM = r"""
#include <stdio.h>
#include <stdlib.h>
#include <string.h>
#include "ee_decode.h"

typedef struct { unsigned x, y, z; } dim;
static int refuse, pending;
static dim grid, block;
static size_t lds;

int hipGetDevice(int* d) { *d = 0; return 0; }
int hipGetLastError(void) { int e = pending; pending = 0; return e; }
int hipFuncSetAttribute(const void* f, int attr, int value) {
  (void)f; (void)attr;
  printf("attribute %d\n", value);
  if (refuse && value > 65536) return pending = 1;   /* like the runtime: the error also waits for hipGetLastError */
  return 0;
}
int __hipPushCallConfiguration(dim g, dim b, size_t s, void* st) { (void)st; grid = g; block = b; lds = s; return 0; }
int __hipPopCallConfiguration(dim* g, dim* b, size_t* s, void** st) { *g = grid; *b = block; *s = lds; *st = 0; return 0; }
int hipGetSymbolAddress(void** p, const void* s) { (void)s; *p = (void*)0x20000; return 0; }
static struct { const void* f; const char* name; } kernels[4096];
static int n_kernels;
void __hipRegisterFunction(void** modules, const void* f, char* device, const char* name, unsigned limit, void* tid, void* bid, void* bd, void* gd,
                           int* size) {
  (void)modules; (void)device; (void)limit; (void)tid; (void)bid; (void)bd; (void)gd; (void)size;
  kernels[n_kernels].f = f;
  kernels[n_kernels++].name = name;
}
int hipLaunchKernel(const void* f, dim g, dim b, void** args, size_t s, void* st) {
  (void)args; (void)st;
  printf("launch %u %u %u %u %zu", g.x, g.y, g.z, b.x, s);
  for (int i = 0; i < n_kernels; ++i)
    if (kernels[i].f == f) printf(" %s", kernels[i].name);
  printf("\n");
  return 0;
}

int hipEventCreate(void** e) { static char event; *e = &event; return 0; }
int hipEventRecord(void* e, void* st) { (void)e; (void)st; return 0; }
int hipEventSynchronize(void* e) { (void)e; return 0; }
int hipEventElapsedTime(float* ms, void* a, void* b) { (void)a; (void)b; *ms = 0; return 0; }

int main(int argc, char** argv) {
  void* p = (void*)0x10000;                          /* any aligned address */
  const int B = atoi(argv[3]);
  refuse = atoi(argv[2]);
  ee_layer_weights w[2] = {{p, p, p, p, p, p}, {p, p, p, p, p, p}};
  ee_model m = {{2, 256, 2, 128, 512, 1024, EE_BF16, 1e-5f, 1e4f, 1, 1.0f, 0}, p, p, p, w, 0, 0};
  ee_kv_cache c = {p, p, 64, 16};
  ee_batch b = {B, p, p, p, 20, 300, p};
  if (!strcmp(argv[1], "check_fp32")) {
    m.desc.dtype = EE_FP32;
    m.desc.vocab = 32000;
  }
  if (argc > 4) {                                    /* heads of 128, features, vocabulary */
    m.desc.n_heads = atoi(argv[4]);
    m.desc.d_model = m.desc.n_heads * 128;
    m.desc.d_ffn = atoi(argv[5]);
    m.desc.vocab = atoi(argv[6]);
  }
  if (!strcmp(argv[1], "float")) {                   /* heads of 64, 15 blocks a sequence */
    m.desc.dtype = EE_FP32;
    m.desc.head_dim = 64;
    m.desc.d_model = m.desc.n_heads * 64;
    b = (ee_batch){B, p, p, p, 15, 200, 0};
  }
  const size_t n = ee_workspace_bytes(&m.desc, B, 300);
  const float never[2] = {2, 2};
  int rc;
  ee_profile_enable(1);
  if (!strcmp(argv[1], "init"))
    rc = ee_noalloc_init();
  else if (!strcmp(argv[1], "iteration"))
    rc = ee_decode_iteration(&m, &c, &b, 0, 0, EE_EXIT_NONE, p, p, p, 0, 0, p, n, 0);
  else if (!strcmp(argv[1], "float"))
    rc = ee_decode_iteration(&m, &c, &b, never, 0, EE_EXIT_BATCH, p, p, p, 0, 0, p, n, 0);
  else if (!strcmp(argv[1], "per_sequence") || !strcmp(argv[1], "no_checks")) {
    b.row_table = 0;
    rc = ee_decode_iteration(&m, &c, &b, never, 0, argv[1][0] == 'n' ? EE_EXIT_NONE : EE_EXIT_PER_SEQUENCE, p, p, p, 0, 0, p, n, 0);
  } else if (!strcmp(argv[1], "attention"))
    rc = ee_paged_attention_decode(&m.desc, &c, 1, p, &b, p, 0, 0, 0);
  else
    rc = ee_exit_check(&m, 1, p, B, 0.5f, 0, p, p, p, p, p, 0, 0, p, n, 0);
  printf("rc %d %s\n", rc, rc ? ee_last_error() : "");
  static int32_t cls[1000], layer[1000];
  static float ms[1000];
  const int records = ee_profile_read(cls, layer, ms, 1000);
  for (int i = 0; i < records; ++i) printf("record %d\n", cls[i]);
  fflush(stdout);
  _Exit(argc < 0);
}
"""


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    B.lib()
    d = tmp_path_factory.mktemp("host_launches")
    src, exe = d / "program.c", d / "program"
    src.write_text(PROGRAM)
    subprocess.run(["gcc", "-O1", "-rdynamic", "-I" + os.path.join(build.ROOT, "include"), str(src), "-o", str(exe), B.LIB_PATH,
                    "-Wl,-rpath-link,/opt/rocm/lib"], check=True, capture_output=True, text=True)

    def run(*args):
        out = subprocess.run([str(exe), *map(str, args)], check=True, capture_output=True, text=True, timeout=60).stdout.split("\n")
        run.attributes = [int(line.split()[1]) for line in out if line.startswith("attribute")]
        launches = [tuple(int(x) for x in line.split()[1:6]) for line in out if line.startswith("launch")]
        run.records = [int(line.split()[1]) for line in out if line.startswith("record")]
        run.names = [line.split()[6] for line in out if line.startswith("launch")]
        return launches, [line for line in out if line.startswith("rc")][0]

    return run


@pytest.mark.parametrize("call,refused_before", [("attention", 0), ("iteration", 2)])
def test_prompt_attention_without_its_lds(program, call, refused_before):
    """128 KiB of LDS refused: the call succeeds all the same, and four rows a workgroup over a block table in LDS take the
    place of the matrix-core kernel; nothing else in the sequence of launches changes."""
    rows = 30
    want, rc = program(call, 0, rows)
    assert rc.strip() == "rc 0"
    prompt = [i for i, x in enumerate(want) if x[3:] == (512, 131072)]
    assert prompt[0] == refused_before and len(prompt) == (1 if call == "attention" else 2)
    got, rc = program(call, 1, rows)
    assert rc.strip() == "rc 0"
    for i in prompt:
        want[i] = (2, (rows + 3) // 4, 1, 256, 20 * 4)
    assert got == want


def test_exit_check_without_the_lds_of_the_ring_kernel(program):
    """385 to 512 rows with 128 KiB of LDS refused: the tiled kernel's blocks of 128 rows, and no error left behind."""
    want, rc = program("check", 0, 450)
    assert rc.strip() == "rc 0" and [x[3:] for x in want] == [(512, 0), (256, 131072), (256, 0)]
    got, rc = program("check", 1, 450)
    assert rc.strip() == "rc 0"
    assert got == [want[0], (8 * 4, 1, 1, 256, 0), want[2]]


def test_set_up_before_a_graph_capture_asks_for_every_lds_size(program):
    """ee_noalloc_init: two ring kernels, prompt attention with heads of 64 and 128 in both output orders."""
    launches, rc = program("init", 0, 1)
    assert rc.strip() == "rc 0" and not launches
    assert sorted(program.attributes) == [65536, 65536, 131072, 131072, 131072, 131072]


@pytest.mark.parametrize("rows", [1, 4, 255, 257, 20000, 300000])
def test_float_head_grid_covers_every_row_within_the_limits(program, rows):
    """Eight weight rows a workgroup, padded to the eight XCDs, times up to 64 row blocks of four in x, the rest in y: a dimension
    holds less than 2^32 threads and 65536 workgroups in y."""
    launches, rc = program("check_fp32", 0, rows)
    assert rc.strip() == "rc 0"
    (x, y, z, threads, _), decide = launches
    blocks = (rows + 3) // 4
    assert (x, z, threads) == (4000 * min(blocks, 64), 1, 256) and (y - 1) * 64 < blocks <= y * 64
    assert x * threads < 2 ** 32 and y < 65536 and decide[:4] == (rows, 1, 1, 256)


STREAMING, BLOCKS = 256, 384   # threads: four wavefronts a tile; four that multiply and two that load


@pytest.mark.parametrize("rows,heads,tiles,threads", [
    (128, 32, 50, STREAMING), (128, 16, 201, STREAMING), (97, 3, 255, STREAMING),   # four batch tiles: one round of tiles ...
    (128, 16, 257, BLOCKS), (97, 3, 331, BLOCKS),                                   # ... or more
    (96, 32, 50, STREAMING), (65, 8, 127, STREAMING),                               # three: a long contraction of few tiles ...
    (96, 6, 50, BLOCKS), (65, 8, 129, BLOCKS),                                      # ... 48 steps, or more tiles
])
def test_lm_head_of_tiles_that_do_not_come_in_fours(program, rows, heads, tiles, threads):
    """65 to 128 rows: the streaming kernel's four wavefronts split the contraction of a tile; a block's do not."""
    launches, rc = program("check", 0, rows, heads, 512, 32 * tiles)
    assert rc.strip() == "rc 0" and launches[1][3] == threads
    if threads == STREAMING:
        assert launches[1][:3] == (tiles, 1, 1)


@pytest.mark.parametrize("heads,rows,pairs", [(53, 64, False), (54, 64, True), (55, 33, True), (62, 64, True), (64, 64, False), (51, 32, True)])
def test_output_projection_of_two_batch_tiles(program, heads, rows, pairs):
    """33 to 64 rows: two tiles a workgroup in two slices where that fills the chip (214 to 254 tiles), else 64 x 64 blocks of two
    wavefronts that multiply and two that load."""
    launches, rc = program("iteration", 0, rows, heads, 512, 1024)
    assert rc.strip() == "rc 0"
    tiles = 4 * heads
    assert ((tiles // 2, 2, 1, 256, 0) in launches) == pairs
    assert ((tiles + 7) // 8 * 8, 1, 1, 256, 0) in launches or pairs   # (a workgroup for each XCD's last block)


@pytest.fixture(scope="module")
def slices():
    """(contraction slices of M rows onto n tiles over K, rows of partial results set aside for up to M rows)"""
    f, g = B.lib()._ZN2ee15gemm_acc_slicesEiii, B.lib()._ZN2ee13gemm_acc_rowsEiii
    f.restype, g.restype = ctypes.c_int, ctypes.c_size_t
    return f, g


@pytest.mark.parametrize("tiles,K", [(4, 16), (8, 16384), (20, 1008), (32, 5632), (32, 16384), (64, 28672), (96, 8192), (128, 4096), (128, 11008),
                                     (160, 13824), (206, 6592), (256, 28672)])
def test_workspace_covers_the_slices_of_every_smaller_batch(slices, tiles, K):
    need = most = 0
    for rows in list(range(1, 700)) + [1000, 1024, 2047, 2048, 2049, 5000]:
        k = slices[0](rows, tiles, K)
        assert 1 <= k <= 8 and k <= max(1, K // 1024)
        need = max(need, k * ((rows + 31) // 32 * 32))
        set_aside = slices[1](rows, tiles, K)
        assert set_aside >= need and set_aside >= most
        most = set_aside


@pytest.mark.parametrize("rows,tiles,K,want", [(250, 32, 16384, 8), (300, 32, 16384, 5), (160, 8, 8192, 8), (512, 16, 11008, 8),
                                                   (300, 48, 6080, 3), (250, 64, 11008, 4), (512, 128, 11008, 2), (384, 128, 11008, 4), (512, 160, 13824, 3)])
def test_long_contractions_of_narrow_models_come_in_more_slices(slices, rows, tiles, K, want):
    """More than 128 rows: as many slices as 128 x 64 blocks fill the chip with in one round, from four to eight, where the contraction
    is long; the cheapest up to four where it is not."""
    assert slices[0](rows, tiles, K) == want


@pytest.mark.parametrize("rows,tiles,blocks,threads", [
    (256, 768, 2 * 128, 384), (256, 772, 200, 384), (200, 864, 216, 384), (129, 1024, 256, 384),   # 128 x 192 as long as they fit one round; 256 x 128
    (256, 1036, 176, 640), (129, 1536, 256, 640),                                                  # 256 x 192
    (257, 864, 3 * 144, 384),                                                                      # more rows: 128-row blocks
])
def test_gate_up_of_a_compacted_operand(program, rows, tiles, blocks, threads):
    launches, rc = program("per_sequence", 0, rows, 1, 16 * tiles, 4096)
    assert rc.strip() == "rc 0"
    assert launches.count((blocks, 1, 1, threads, 0)) == 2


@pytest.mark.parametrize("rows,heads,tiles,ring", [(385, 2, 776, True), (512, 2, 1024, True), (400, 4, 1544, True), (512, 2, 768, False), (384, 2, 776, False),
                                                   (513, 2, 776, False), (450, 2, 778, False)])
def test_gate_up_in_the_ring_kernel(program, rows, heads, tiles, ring):
    """385 to 512 rows, weight tiles in whole blocks of eight whose blocks take fewer rounds than others; without its 128 KiB the
    block kernel takes the shape."""
    want = ((tiles // 8 + 7) // 8 * 8 * 2, 1, 1, 256, 131072)
    launches, rc = program("iteration", 0, rows, heads, 16 * tiles, 1024)
    assert rc.strip() == "rc 0" and launches.count(want) == (2 if ring else 0)
    launches, rc = program("iteration", 1, rows, heads, 16 * tiles, 1024)
    assert rc.strip() == "rc 0" and want not in launches


@pytest.mark.parametrize("rows,heads,vocab,small", [
    (1, 3, 32000, True), (2, 3, 8192, True), (2, 2, 32000, False), (4, 2, 8224, False), (4, 3, 32000, True), (8, 8, 32000, True), (8, 8, 8224, True), (8, 7, 8224, False),
    (8, 7, 8192, True), (5, 25, 8192, False)])
def test_exit_check_of_up_to_eight_rows_without_a_launch_for_its_operand(program, rows, heads, vocab, small):
    """Where several tiles a workgroup and short contractions (heads of 128) do not make it the slower one."""
    launches, rc = program("check", 0, rows, heads, 512, vocab)
    assert rc.strip() == "rc 0"
    assert any("gemm_small_kernel" in n for n in program.names) == small and len(launches) == (2 if small else 3)


@pytest.mark.parametrize("call,rows,heads,vocab,small", [
    ("per_sequence", 8, 5, 1024, True), ("per_sequence", 8, 4, 1024, False), ("per_sequence", 5, 3, 1024, False), ("per_sequence", 4, 1, 8192, True),
    ("per_sequence", 4, 1, 8224, False), ("per_sequence", 4, 2, 8224, True), ("per_sequence", 3, 3, 32000, True), ("per_sequence", 2, 1, 32000, True),
    ("per_sequence", 8, 25, 1024, False), ("no_checks", 8, 3, 32000, True), ("no_checks", 8, 2, 1024, False), ("no_checks", 4, 1, 32000, True)])
def test_iteration_of_up_to_eight_rows_in_projections_that_normalise(program, call, rows, heads, vocab, small):
    _, rc = program(call, 0, rows, heads, 512, vocab)
    assert rc.strip() == "rc 0"
    assert any("gemm_small_kernel" in n for n in program.names) == small


FOUR_PIECES = "ELi4E"   # gemm_simple_kernel<.., PIECES = 4, ..>


@pytest.mark.parametrize("heads,rows,launches", [(1, 1, 10), (4, 16, 10), (4, 17, 12), (4, 64, 12), (4, 65, 16), (5, 1, 15), (5, 16, 15), (8, 4, 15)])
def test_float_layers_in_four_launches_up_to_width_256(program, heads, rows, launches):
    """Two layers of four launches and two behind them; five a layer above 64 (sequence, head) pairs; wider models and more rows keep the
    launches that are faster there."""
    _, rc = program("float", 0, rows, heads, 256 * heads, 512)
    assert rc.strip() == "rc 0"
    assert len(program.names) == launches
    assert any("attn_f32_kernel" in n for n in program.names) == (launches <= 12)


@pytest.mark.parametrize("rows,heads,ffn,vocab", [(4, 5, 1280, 512), (16, 8, 2048, 512), (4, 8, 1024, 32000), (64, 4, 1024, 512), (500, 16, 4096, 8000)])
def test_float_contractions_of_four_pieces_where_a_launch_leaves_the_chip_idle(program, rows, heads, ffn, vocab):
    """All operands of a contraction of 257 to 1024 at once only where there are no more workgroups than compute units."""
    launches, rc = program("float", 0, rows, heads, ffn, vocab)
    assert rc.strip() == "rc 0"
    for (x, y, z, _, _), name in zip(launches, program.names):
        if FOUR_PIECES in name:
            assert x * y * z <= 256, name


@pytest.mark.parametrize("rows,vocab", [(1, 512), (64, 32000)])
def test_float_head_beside_kv_filling_is_there_once(program, rows, vocab):
    """Not once a layer: the head's workgroups, then those of each of the two layers."""
    launches, rc = program("float", 0, rows, 4, 1024, vocab)
    assert rc.strip() == "rc 0"
    blocks = (rows + 3) // 4
    head, fill = -(-vocab // 8 // 8) * 8 * blocks, 64 * blocks
    assert launches[-2][:3] == (head + 2 * fill, 1, 1)


@pytest.mark.parametrize("call,rows,heads,begins", [("float", 4, 4, False), ("float", 4, 5, True), ("no_checks", 8, 9, False), ("no_checks", 9, 9, True)])
def test_records_of_launches_that_are_made(program, call, rows, heads, begins):
    """Where the start of the iteration is inside the first QKV launch there is no record of a start.  (More than 64 pairs: no merge launch, one record each.)"""
    launches, rc = program(call, 0, rows, heads, 256 * heads, 512)
    assert rc.strip() == "rc 0"
    assert program.records.count(B.KERNEL_CLASSES.index("other")) == (1 if begins else 0) and len(program.records) == len(launches)
