"""Per-entry-point parity on the GPU: ee_paged_attention_decode, ee_exit_check, ee_kv_fill against the CPU oracle
on seeded tensors, at sizes that span several tiles and ragged tails, plus the degenerate cases."""
import math
import os
import subprocess
import sys

import pytest
import torch

from oracle import ee_oracle as O
from paper_2407_20272_amd import binding as B
from paper_2407_20272_amd import workloads as W
from gpu_harness import F64, HipRun, assert_close_scaled, conf_tolerance, tol_of

pytestmark = pytest.mark.gpu
TINY, L7B = W.CONFIGS[0], W.CONFIGS[1]


def cfg_of(dtype, head_dim, n_heads, **kw):
    base = dict(dtype=dtype, head_dim=head_dim, n_heads=n_heads, d_model=head_dim * n_heads, n_layers=2, d_ffn=256,
                vocab=512, weight_std=0.05)
    base.update(kw)
    return W.reduced(TINY, **base)


# ------------------------------------------------------------------------------------------------------
# paged decode attention
# ------------------------------------------------------------------------------------------------------
def poison_unwritten_slots(cache, bt, n_pos):
    """NaN in every cache slot that holds no position of any sequence (sequence b owns positions 0..n_pos[b]-1)."""
    nb = cache.k.shape[1]
    valid = torch.zeros(nb, 16, dtype=torch.bool)
    for b in range(len(n_pos)):
        for p_ in range(int(n_pos[b])):
            blk, off = W.slot_of(bt, b, p_, 16)
            valid[blk, off] = True
    mask = (~valid).cuda()[None, :, None, :, None].expand_as(cache.k)
    cache.k[mask] = float("nan")
    cache.v[mask] = float("nan")


class RawWorkspace:
    """A bare device buffer with the two attributes the binding reads from a workspace."""

    def __init__(self, n_bytes):
        self.buf = torch.empty(max(n_bytes, 16), dtype=torch.uint8, device="cuda")
        self.bytes = n_bytes


def run_attention(cfg, lens, seed, shuffled=True, sample=None, poison=False, ws_bytes=None):
    lens = torch.tensor(lens, dtype=torch.int32)
    cfg = cfg.with_(batch=len(lens), shuffled_blocks=shuffled)
    max_ctx = int(lens.max()) + 1
    Ks, Vs = W.make_dense_kv(cfg, lens + 1, max_ctx, seed=seed, device="cuda")      # positions 0..len inclusive
    bt, nb = W.make_block_tables(lens, 1, 16, shuffled, seed, spare_blocks=1)
    cache = B.PagedKV(cfg, nb)
    for i in range(cfg.n_layers):
        cache.k[i] = W.dense_to_paged(Ks[i], bt, nb, 16)
        cache.v[i] = W.dense_to_paged(Vs[i], bt, nb, 16)
    if poison:
        poison_unwritten_slots(cache, bt, lens + 1)
    g = torch.Generator().manual_seed(seed)
    q = torch.randn(cfg.batch, cfg.n_heads, cfg.head_dim, generator=g) * 1.5
    out = torch.zeros(cfg.batch, cfg.n_heads, cfg.head_dim, device="cuda")
    batch = B.make_batch(None, lens.cuda(), bt.cuda(), max_ctx)
    layer = cfg.n_layers
    ws = None if ws_bytes is None else RawWorkspace(ws_bytes)
    if ws is not None:
        ws.buf.fill_(0xFF)           # NaN patterns: a part that is not written would show
    B.ee_paged_attention_decode(B.make_desc(cfg), cache, layer, q.cuda(), batch, out, ws)
    torch.cuda.synchronize()
    out = out.cpu()
    rows = range(cfg.batch) if sample is None else sample
    Kc, Vc = Ks[layer - 1].cpu(), Vs[layer - 1].cpu()
    for b in rows:
        n = int(lens[b]) + 1
        want = O.attention_decode(q[b].to(F64), Kc[b, :n], Vc[b, :n])
        assert_close_scaled(out[b], want, tol_of(cfg), f"attention sequence {b} (len {n})")


@pytest.mark.parametrize("dtype,dh", [("fp32", 64), ("fp32", 128), ("bf16", 64), ("bf16", 128)])
def test_attention_ragged_lengths(dtype, dh):
    cfg = cfg_of(dtype, dh, 3)
    run_attention(cfg, [0, 1, 14, 15, 16, 17, 31, 32, 63, 64, 65, 100, 257, 5], seed=11)


@pytest.mark.parametrize("dtype,dh", [("fp32", 64), ("bf16", 64), ("bf16", 128)])
def test_attention_ignores_what_unwritten_slots_hold(dtype, dh):
    """Slots after a sequence's last position (and blocks nobody owns) hold NaN: no result may change."""
    cfg = cfg_of(dtype, dh, 2)
    run_attention(cfg, [0, 1, 14, 15, 16, 17, 31, 32, 63, 64, 65, 100, 257, 5], seed=12, poison=True)


@pytest.mark.parametrize("dtype,dh,heads", [("fp32", 64, 2), ("bf16", 64, 8), ("bf16", 128, 3)])
def test_attention_context_split_among_workgroups(dtype, dh, heads):
    """Few (sequence, head) pairs and a wide block table: with a workspace up to eight workgroups share a pair, each
    over a contiguous part of the context (parts of a short sequence are empty), and a second launch merges them.
    Unowned slots hold NaN.  A workspace that is too small is not an error: the call runs one workgroup per pair."""
    cfg = cfg_of(dtype, dh, heads)
    lens = [0, 5, 130, 700, 2049]
    need = len(lens) * heads * 8 * (dh + 2) * 4
    run_attention(cfg, lens, seed=15, poison=True, ws_bytes=need)
    run_attention(cfg, lens, seed=16, poison=True, ws_bytes=need // 16)
    run_attention(cfg, [4000], seed=17, ws_bytes=heads * 8 * (dh + 2) * 4)          # one sequence, every part full


def test_attention_rows_sharing_one_block_table():
    """Several batch rows at consecutive positions of ONE sequence (row_table): each attends positions 0..its own."""
    cfg = cfg_of("bf16", 128, 2).with_(batch=1, shuffled_blocks=True)
    L = 70                                                      # the sequence holds positions 0..L
    lens1 = torch.tensor([L], dtype=torch.int32)
    Ks, Vs = W.make_dense_kv(cfg, lens1 + 1, L + 1, seed=14, device="cuda")
    bt, nb = W.make_block_tables(lens1, 1, 16, True, 14, spare_blocks=1)
    cache = B.PagedKV(cfg, nb)
    for i in range(cfg.n_layers):
        cache.k[i] = W.dense_to_paged(Ks[i], bt, nb, 16)
        cache.v[i] = W.dense_to_paged(Vs[i], bt, nb, 16)
    pos = torch.tensor([0, 15, 16, 17, 40, 69, 70], dtype=torch.int32)          # rows of the one sequence
    R = len(pos)
    q = torch.randn(R, cfg.n_heads, cfg.head_dim, generator=torch.Generator().manual_seed(14)) * 1.5
    out = torch.zeros(R, cfg.n_heads, cfg.head_dim, device="cuda")
    batch = B.make_batch(None, pos.cuda(), bt.cuda(), L + 1, torch.zeros(R, dtype=torch.int32).cuda())
    B.ee_paged_attention_decode(B.make_desc(cfg), cache, 2, q.cuda(), batch, out)
    torch.cuda.synchronize()
    Kc, Vc = Ks[1].cpu(), Vs[1].cpu()
    for r in range(R):
        n = int(pos[r]) + 1
        want = O.attention_decode(q[r].to(F64), Kc[0, :n], Vc[0, :n])
        assert_close_scaled(out[r].cpu(), want, tol_of(cfg), f"row {r} at position {n - 1}")


@pytest.mark.parametrize("dh", [64, 128])
def test_attention_rows_of_several_sequences_across_row_groups(dh):
    """Rows of three sequences in one call (row_table), runs of 20, 5 and 17 rows: the row groups of the
    matrix-core kernel straddle the runs, the last group is ragged, block counts are odd and even."""
    cfg = cfg_of("bf16", dh, 2).with_(batch=3, shuffled_blocks=True)
    lens = torch.tensor([69, 4, 199], dtype=torch.int32)        # last cached position of each sequence
    Lmax = int(lens.max()) + 1
    Ks, Vs = W.make_dense_kv(cfg, lens + 1, Lmax, seed=15, device="cuda")
    bt, nb = W.make_block_tables(lens, 1, 16, True, 15, spare_blocks=2)
    cache = B.PagedKV(cfg, nb)
    for i in range(cfg.n_layers):
        cache.k[i] = W.dense_to_paged(Ks[i], bt, nb, 16)
        cache.v[i] = W.dense_to_paged(Vs[i], bt, nb, 16)
    poison_unwritten_slots(cache, bt, lens + 1)   # what lies after a sequence's last position must not matter
    rows = [(0, p) for p in range(50, 70)] + [(1, p) for p in range(0, 5)] + [(2, p) for p in range(183, 200)]
    R = len(rows)
    pos = torch.tensor([p for _, p in rows], dtype=torch.int32)
    seq = torch.tensor([s_ for s_, _ in rows], dtype=torch.int32)
    q = torch.randn(R, cfg.n_heads, cfg.head_dim, generator=torch.Generator().manual_seed(15)) * 1.5
    out = torch.zeros(R, cfg.n_heads, cfg.head_dim, device="cuda")
    batch = B.make_batch(None, pos.cuda(), bt.cuda(), Lmax, seq.cuda())
    B.ee_paged_attention_decode(B.make_desc(cfg), cache, 1, q.cuda(), batch, out)
    torch.cuda.synchronize()
    Kc, Vc = Ks[0].cpu(), Vs[0].cpu()
    for r, (s_, p_) in enumerate(rows):
        want = O.attention_decode(q[r].to(F64), Kc[s_, :p_ + 1], Vc[s_, :p_ + 1])
        assert_close_scaled(out[r].cpu(), want, tol_of(cfg), f"row {r}: sequence {s_} at position {p_}")


@pytest.mark.parametrize("dh,n_heads,runs", [
    (128, 2, [(1, 0), (3, 31), (1, 40), (2, 15)]),                    # four rows a workgroup, runs of one to three rows
    (128, 40, [(33, 0), (64, 95), (5, 17), (90, 500)]),               # six blocks of rows: one group of 32, runs straddle them
    (64, 40, [(200, 0), (1, 300), (120, 33), (59, 130)]),             # two groups of 32, a last block of few rows
    (128, 32, [(250, 4200), (262, 0)]),                               # two groups, more steps per slice than one look-up of ids
    (64, 2, [(7, 8300)]),                                             # one group, likewise
])
def test_attention_prompt_rows_run_structure(dh, n_heads, runs):
    """Prompt rows as (rows, first position) per sequence, consecutive positions, NaN behind every sequence's end: group
    sizes, runs that straddle groups and workgroups, odd block counts, long slices.  q and the probabilities are carried
    with 16 significant bits or more (bf16 head + remainder), so a score of magnitude 8 is off by at most 8 * 2^-17 and a
    result by about as much: 6e-5 at worst, averaged well below over a row; asserted on the 2-norm at 2e-5."""
    cfg = cfg_of("bf16", dh, n_heads, n_layers=1).with_(batch=len(runs), shuffled_blocks=True)
    lens = torch.tensor([b + n - 1 for n, b in runs], dtype=torch.int32)
    Lmax = int(lens.max()) + 1
    Ks, Vs = W.make_dense_kv(cfg, lens + 1, Lmax, seed=18, device="cuda")
    bt, nb = W.make_block_tables(lens, 1, 16, True, 18, spare_blocks=2)
    cache = B.PagedKV(cfg, nb)
    cache.k[0] = W.dense_to_paged(Ks[0], bt, nb, 16)
    cache.v[0] = W.dense_to_paged(Vs[0], bt, nb, 16)
    poison_unwritten_slots(cache, bt, lens + 1)
    rows = [(s, b + i) for s, (n, b) in enumerate(runs) for i in range(n)]
    pos = torch.tensor([p for _, p in rows], dtype=torch.int32)
    seq = torch.tensor([s for s, _ in rows], dtype=torch.int32)
    q = torch.randn(len(rows), n_heads, dh, generator=torch.Generator().manual_seed(18)) * 1.3
    out = torch.zeros(len(rows), n_heads, dh, device="cuda")
    batch = B.make_batch(None, pos.cuda(), bt.cuda(), Lmax, seq.cuda())
    B.ee_paged_attention_decode(B.make_desc(cfg), cache, 1, q.cuda(), batch, out)
    torch.cuda.synchronize()
    want = torch.empty(len(rows), n_heads, dh, dtype=F64)
    for s, (n, b) in enumerate(runs):   # every head a plain 2-D product in float64
        mask = torch.arange(b + n)[None, :] > torch.arange(b, b + n)[:, None]
        at = [r for r, (t, _) in enumerate(rows) if t == s]
        for h in range(n_heads):
            K, V = Ks[0][s, :b + n, h].cpu().to(F64), Vs[0][s, :b + n, h].cpu().to(F64)
            z = (q[at, h].to(F64) @ K.T / math.sqrt(dh)).masked_fill(mask, -math.inf)
            want[at, h] = z.softmax(-1) @ V
    err = ((out.cpu().to(F64) - want).flatten(1).norm(dim=1) / want.flatten(1).norm(dim=1)).max().item()
    assert err <= 2e-5, f"relative error of a row: {err}"


@pytest.mark.parametrize("dh,n_heads,runs,bad_seq,bad_pos", [
    (128, 2, [(3, 20), (1, 40), (2, 15), (4, 61)], 1, 7),                          # four rows a workgroup
    (64, 40, [(20, 0), (0, 0), (30, 70), (60, 5)], 2, 80),                          # one group of 32, runs straddle workgroups
    (128, 40, [(40, 300), (20, None), (50, 64), (100, 0)], 0, 0),                   # two groups, a run of no positions between
    (64, 32, [(250, 90), (6, None), (240, 0)], 2, 239),                             # two groups, the last position of a prompt
])
@pytest.mark.parametrize("value", [float("inf"), float("nan")])
def test_attention_prompt_rows_beside_a_sequence_that_is_not_finite(dh, n_heads, runs, bad_seq, bad_pos, value):
    """One cached V of one sequence is Inf or NaN: rows that do not attend that position (other sequences' rows in the same
    group of 32, and the sequence's own earlier ones) keep their results, within the bound of the test above; rows that attend
    it show it in that channel.  A run of garbage (negative) contexts in the middle has no result and no steps."""
    cfg = cfg_of("bf16", dh, n_heads, n_layers=1).with_(batch=len(runs), shuffled_blocks=True)
    lens = torch.tensor([0 if b is None else max(b + n - 1, 0) for n, b in runs], dtype=torch.int32)
    Lmax = int(lens.max()) + 1
    Ks, Vs = W.make_dense_kv(cfg, lens + 1, Lmax, seed=28, device="cuda")
    Vs[0][bad_seq, bad_pos, n_heads - 1, 5] = value
    bt, nb = W.make_block_tables(lens, 1, 16, True, 28, spare_blocks=2)
    cache = B.PagedKV(cfg, nb)
    cache.k[0] = W.dense_to_paged(Ks[0], bt, nb, 16)
    cache.v[0] = W.dense_to_paged(Vs[0], bt, nb, 16)
    poison_unwritten_slots(cache, bt, lens + 1)
    rows = [(s, -5 if b is None else b + i) for s, (n, b) in enumerate(runs) for i in range(n)]
    seq, pos = (torch.tensor(x, dtype=torch.int32) for x in zip(*rows))
    q = torch.randn(len(rows), n_heads, dh, generator=torch.Generator().manual_seed(28)) * 1.3
    out = torch.zeros(len(rows), n_heads, dh, device="cuda")
    batch = B.make_batch(None, pos.cuda(), bt.cuda(), Lmax, seq.cuda())
    B.ee_paged_attention_decode(B.make_desc(cfg), cache, 1, q.cuda(), batch, out)
    torch.cuda.synchronize()
    out = out.cpu().to(F64)
    for r, (s, p) in enumerate(rows):
        if p < 0:
            continue
        K, V = (x[0][s, :p + 1].cpu().to(F64).permute(1, 0, 2) for x in (Ks, Vs))     # [head][position][channel]
        w = (K @ q[r].to(F64)[:, :, None] / math.sqrt(dh)).softmax(1)
        want = (w * V).sum(1)
        if s == bad_seq and p >= bad_pos:
            assert not math.isfinite(float(out[r, n_heads - 1, 5]))
            want[n_heads - 1, 5] = out[r, n_heads - 1, 5] = 0.0
        err = ((out[r] - want).norm() / want.norm()).item()
        assert err <= 2e-5, f"row {r} (sequence {s}, position {p}): relative error {err}"


def test_attention_prompt_rows_without_the_lds_of_the_matrix_core_kernel(tmp_path):
    """The runtime refuses 128 KiB of LDS (a library loaded first into the process answers hipFuncSetAttribute so): the rows
    take another kernel, within the same bound."""
    src, so = tmp_path / "refuse.c", tmp_path / "refuse.so"
    src.write_text("int refused; int hipFuncSetAttribute(const void* f, int a, int v) { (void)f; (void)a; (void)v; ++refused; return 1; }\n")
    subprocess.run(["gcc", "-shared", "-fPIC", str(src), "-o", str(so)], check=True)
    code = ("import ctypes, sys; L = ctypes.CDLL(sys.argv[1], ctypes.RTLD_GLOBAL); sys.path[:0] = sys.argv[2:]; import test_gpu_kernels as T\n"
            "T.test_attention_prompt_rows_run_structure(128, 2, [(1, 0), (3, 31), (1, 40), (2, 15)])\n"
            "T.test_attention_prompt_rows_run_structure(64, 3, [(7, 300), (20, 5)])\n"
            "assert ctypes.c_int.in_dll(L, 'refused').value >= 2\n")
    here = os.path.dirname(os.path.abspath(__file__))
    subprocess.run([sys.executable, "-c", code, str(so), here, os.path.dirname(here)], check=True, timeout=100)


def test_attention_prompt_rows_beside_a_negative_context():
    """A sequence whose context lengths are garbage (negative) has no result, but its neighbours keep theirs."""
    cfg = cfg_of("bf16", 64, 2, n_layers=1).with_(batch=3, shuffled_blocks=True)
    lens = torch.tensor([40, 16, 70], dtype=torch.int32)
    Ks, Vs = W.make_dense_kv(cfg, lens + 1, 71, seed=19, device="cuda")
    bt, nb = W.make_block_tables(lens, 1, 16, True, 19, spare_blocks=1)
    cache = B.PagedKV(cfg, nb)
    cache.k[0], cache.v[0] = W.dense_to_paged(Ks[0], bt, nb, 16), W.dense_to_paged(Vs[0], bt, nb, 16)
    seq = torch.tensor([0] * 3 + [1] * 5 + [2] * 4, dtype=torch.int32)
    pos = torch.tensor([38, 39, 40] + [-100, -1, -2 ** 31, -33, -7] + [67, 68, 69, 70], dtype=torch.int32)
    q = torch.randn(12, 2, 64, generator=torch.Generator().manual_seed(19))
    out = torch.zeros(12, 2, 64, device="cuda")
    batch = B.make_batch(None, pos.cuda(), bt.cuda(), 71, seq.cuda())
    B.ee_paged_attention_decode(B.make_desc(cfg), cache, 1, q.cuda(), batch, out)
    torch.cuda.synchronize()
    for r in (0, 1, 2, 8, 9, 10, 11):
        s_, n = int(seq[r]), int(pos[r]) + 1
        want = O.attention_decode(q[r].to(F64), Ks[0][s_, :n].cpu(), Vs[0][s_, :n].cpu())
        assert_close_scaled(out[r].cpu(), want, tol_of(cfg), f"row {r}")


def test_attention_single_sequence_and_sequential_blocks():
    run_attention(cfg_of("bf16", 128, 2), [300], seed=12, shuffled=False)
    run_attention(cfg_of("fp32", 64, 4), [47], seed=13, shuffled=False)


def test_attention_llama7b_shape_sampled():
    """Full width of the 7B-shaped workload (32 heads x 128, batch 32, context 512..640), sampled sequences."""
    cfg = W.reduced(L7B, n_layers=1)
    g = torch.Generator().manual_seed(5)
    lens = torch.randint(512, 640, (32,), generator=g).tolist()
    run_attention(cfg, lens, seed=14, sample=[0, 7, 31])


def test_attention_long_ragged_batch():
    """Ragged lengths 128..2048 over shuffled block tables (the shape of the batch-256 workload, fewer heads)."""
    cfg = cfg_of("bf16", 128, 4, n_layers=1)
    g = torch.Generator().manual_seed(6)
    lens = torch.randint(128, 2049, (48,), generator=g).tolist()
    run_attention(cfg, lens, seed=15, sample=[0, 1, 2, 47])


def test_attention_very_long_context():
    """20000 cached tokens (1251 blocks of the table in LDS), one short sequence beside it."""
    run_attention(cfg_of("bf16", 128, 2), [20000, 7], seed=15)


def test_attention_uniform_values_give_their_mean():
    """All keys equal -> uniform weights -> output = mean of V (a closed form, independent of the oracle)."""
    cfg = cfg_of("fp32", 64, 2).with_(batch=1)
    lens = torch.tensor([36], dtype=torch.int32)
    bt, nb = W.make_block_tables(lens, 1, 16, True, 3)
    cache = B.PagedKV(cfg, nb)
    v = torch.randn(1, 37, 2, 64)
    cache.k.fill_(0.25)
    cache.v[0] = W.dense_to_paged(v.cuda(), bt, nb, 16)
    out = torch.zeros(1, 2, 64, device="cuda")
    q = torch.randn(1, 2, 64).cuda()
    B.ee_paged_attention_decode(B.make_desc(cfg), cache, 1, q, B.make_batch(None, lens.cuda(), bt.cuda(), 37), out)
    torch.cuda.synchronize()
    torch.testing.assert_close(out.cpu()[0], v[0].mean(0), rtol=1e-5, atol=1e-6)


# ------------------------------------------------------------------------------------------------------
# exit check
# ------------------------------------------------------------------------------------------------------
def run_exit_check(cfg, seed, layer, threshold, hidden_scale=1.0, forced=None, pre_status=None):
    w = W.make_weights(cfg, seed=seed, gain_jitter=0.2)
    m = O.model_from_config(cfg, w)
    model = B.DeviceModel(cfg, w)
    ws = B.Workspace(model.desc, cfg.batch, 16)
    Bsz, n = cfg.batch, cfg.n_layers
    g = torch.Generator().manual_seed(seed)
    hidden = torch.randn(Bsz, cfg.d_model, generator=g) * hidden_scale
    status0 = torch.zeros(Bsz, dtype=torch.int32) if pre_status is None else pre_status.clone()
    exit0 = torch.where(status0 > 0, torch.ones_like(status0), torch.full_like(status0, n))
    status, exit_layer = status0.cuda(), exit0.cuda()
    n_exited = torch.tensor([int(status0.sum())], dtype=torch.int32, device="cuda")
    done = torch.zeros(1, dtype=torch.int32, device="cuda")
    L = torch.full((1,), n, dtype=torch.int32, device="cuda")
    argmax = torch.zeros(Bsz, dtype=torch.int32, device="cuda")
    conf = torch.zeros(Bsz, dtype=torch.float32, device="cuda")
    f = None if forced is None else forced.cuda()
    B.ee_exit_check(model, layer, hidden.cuda(), threshold, f, status, exit_layer, n_exited, done, L, argmax, conf, ws)
    torch.cuda.synchronize()
    # oracle
    rows = [b for b in range(Bsz) if not status0[b]]
    c, am_active = O.exit_check(m, layer, hidden.to(F64), rows)
    _, am_all = O.exit_check(m, layer, hidden.to(F64), list(range(Bsz)))
    st, el = [bool(x) for x in status0], exit0.tolist()
    cd = {b: float(c[r]) for r, b in enumerate(rows)}
    if forced is not None:
        cd = {b: (math.inf if layer >= int(forced[b]) else -math.inf) for b in rows}
    O.update_status(st, el, layer, cd, threshold)
    tol = tol_of(cfg)
    conf = conf.cpu()
    near = 0
    zabs = O.head_logits(m, hidden.to(F64)).abs().amax(-1)
    scale = cfg.logit_scale * layer
    for r, b in enumerate(rows):
        assert abs(float(conf[b]) - float(c[r])) <= conf_tolerance(cfg, float(c[r]), scale, float(zabs[b])), \
            (b, float(conf[b]), float(c[r]))
    for b in range(Bsz):
        if status0[b]:
            assert math.isnan(float(conf[b]))
    got_st = status.cpu().tolist()
    for b in range(Bsz):
        if bool(got_st[b]) != st[b]:
            assert forced is None and abs(cd[b] - threshold) <= conf_tolerance(cfg, cd[b], scale, float(zabs[b])), (b, cd[b])
            near += 1
            st[b] = bool(got_st[b])
            el[b] = layer if st[b] else n
    assert exit_layer.cpu().tolist() == el
    assert int(n_exited.item()) == sum(st)
    assert int(done.item()) == int(all(st)) and int(L.item()) == (layer if all(st) else n)
    # arg max of every row; a mismatch must be a near tie of the oracle's logits
    z = O.head_logits(m, hidden.to(F64))
    am = argmax.cpu()
    for b in range(Bsz):
        if int(am[b]) != int(am_all[b]):
            top = torch.topk(z[b], 2).values
            assert float(top[0] - top[1]) <= tol * float(z[b].abs().max())
    return near


@pytest.mark.parametrize("dtype", ["fp32", "bf16"])
@pytest.mark.parametrize("conf_mode", [0, 1])
def test_exit_check_matches_oracle(dtype, conf_mode):
    cfg = cfg_of(dtype, 64, 4, n_layers=6, vocab=1024 + 64, logit_scale=2.0, conf_mode=conf_mode, batch=37)
    for layer, thr in ((1, 0.05), (3, 0.2), (5, 0.5)):
        run_exit_check(cfg, seed=20 + layer, layer=layer, threshold=thr, hidden_scale=3.0)


def test_exit_check_fp32_hidden_rows_off_a_16_byte_boundary():
    """The float head reads the caller's hidden rows itself, 16 bytes at a time only where they start on a boundary: rows
    one float further on give the same arg max and, to float rounding of another summation order, the same confidence."""
    cfg = cfg_of("fp32", 64, 4, n_layers=6, vocab=514, logit_scale=2.0, batch=7)
    w = W.make_weights(cfg, seed=19, gain_jitter=0.2)
    model = B.DeviceModel(cfg, w)
    ws = B.Workspace(model.desc, cfg.batch, 16)
    hidden = torch.randn(cfg.batch, cfg.d_model, generator=torch.Generator().manual_seed(19)).mul_(3.0).cuda()
    store = torch.empty(cfg.batch * cfg.d_model + 1, device="cuda")
    off = store[1:].view(cfg.batch, cfg.d_model).copy_(hidden)
    got = []
    for h in (hidden, off):
        z = lambda *s: torch.zeros(*s, dtype=torch.int32, device="cuda")  # noqa: E731
        argmax, conf = z(cfg.batch), torch.zeros(cfg.batch, device="cuda")
        B.ee_exit_check(model, 2, h, 2.0, None, z(cfg.batch), z(cfg.batch), z(1), z(1), z(1), argmax, conf, ws)
        torch.cuda.synchronize()
        got.append((argmax.cpu(), conf.cpu()))
    assert got[0][0].equal(got[1][0])
    assert torch.allclose(got[0][1], got[1][1], rtol=1e-5, atol=0)   # logits of magnitude 10 to 1e-6, scale 4


@pytest.mark.parametrize("dtype", ["fp32", "bf16"])
def test_exit_check_sticky_forced_and_done_flag(dtype):
    cfg = cfg_of(dtype, 64, 4, n_layers=6, vocab=512, logit_scale=2.0, batch=5)
    pre = torch.tensor([1, 0, 1, 0, 0], dtype=torch.int32)
    # threshold above 1: nobody new exits, accepted ones stay accepted
    run_exit_check(cfg, 31, layer=2, threshold=1.5, pre_status=pre)
    # threshold below 1/V: everybody exits -> done flag and batch exit layer
    run_exit_check(cfg, 32, layer=4, threshold=0.0, pre_status=pre)
    # forced injection overrides the confidence
    forced = torch.tensor([6, 3, 2, 4, 6], dtype=torch.int32)
    run_exit_check(cfg, 33, layer=3, threshold=0.5, forced=forced)
    run_exit_check(cfg, 34, layer=6 - 1, threshold=0.5, forced=torch.full((5,), 2, dtype=torch.int32), pre_status=pre)


@pytest.mark.parametrize("batch,heads", [(385, 4), (481, 16), (512, 16)])
def test_exit_check_385_to_512_rows(batch, heads):
    """The row counts at which the LM head runs in the 256 x 256 ring kernel: contraction of one and of four groups
    of sixteen steps (d_model 256 and 1024), a second row block of one row, of three tiles and a row, and full."""
    cfg = cfg_of("bf16", 64, heads, n_layers=4, vocab=1280, logit_scale=2.0, batch=batch)
    run_exit_check(cfg, seed=50 + heads, layer=2, threshold=0.3, hidden_scale=3.0)


@pytest.mark.parametrize("batch,heads,vocab", [(1, 16, 32000), (2, 64, 16416), (3, 8, 24608), (4, 16, 32000), (8, 16, 16416)])
def test_exit_check_of_up_to_eight_rows(batch, heads, vocab):
    """The LM head that normalises its own rows: 513 to 1000 tiles on 256 workgroups, rows of up to 8192 channels."""
    cfg = W.reduced(TINY, dtype="bf16", d_model=heads * 128, n_heads=heads, head_dim=128, n_layers=2, vocab=vocab, batch=batch, logit_scale=0.5,
                    weight_std=0.02)
    run_exit_check(cfg, seed=batch + heads, layer=1, threshold=0.02)


@pytest.mark.parametrize("batch,heads,vocab", [(2, 6, 8224), (4, 5, 8224), (5, 16, 8224), (6, 15, 8224), (8, 15, 8192), (5, 1, 8192)])
def test_exit_check_of_up_to_eight_rows_on_both_sides_of_its_rule(batch, heads, vocab):
    """From more than 256 tiles on, up to four rows take that head from 384 channels on, more from 1024."""
    run_exit_check(cfg_of("bf16", 64, heads, vocab=vocab, logit_scale=2.0, batch=batch), seed=batch * heads, layer=1, threshold=0.3, hidden_scale=3.0)


@pytest.mark.parametrize("batch,heads,vocab", [(129, 2, 32), (150, 6, 1312), (161, 48, 8544), (300, 48, 16416), (600, 2, 1280)])
def test_exit_check_in_blocks(batch, heads, vocab):
    """LM head in 128 x 128 and 128 x 256 blocks: one tile, tiles that leave a wavefront one, or none, of its own (statistics of
    tiles that do not exist would land in the next row's records), more than 512 rows."""
    cfg = cfg_of("bf16", 64, heads, n_layers=4, vocab=vocab, logit_scale=2.0, batch=batch)
    run_exit_check(cfg, seed=70 + heads, layer=2, threshold=0.3, hidden_scale=3.0)


@pytest.mark.parametrize("batch,heads,vocab", [(65, 16, 32 * 18), (96, 13, 32 * 127), (97, 16, 32 * 50), (128, 14, 32 * 255)])
def test_exit_check_of_tiles_that_do_not_come_in_fours(batch, heads, vocab):
    """LM head of 65 to 128 rows in the streaming kernel: three batch tiles one after the other, four at once, the last one of one
    row or full."""
    cfg = cfg_of("bf16", 64, heads, n_layers=4, vocab=vocab, logit_scale=2.0, batch=batch)
    run_exit_check(cfg, seed=74 + heads, layer=2, threshold=0.3, hidden_scale=3.0)


@pytest.mark.parametrize("batch", [3, 40, 100, 200, 450])
def test_exit_check_ties_go_to_the_lowest_index(batch):
    """Every LM-head row four times (16 rows on, in the next tile pair and half a vocabulary on): equal sums bit for bit, so the
    arg max is the lowest of them and top-1 minus top-2 is exactly zero, in each form of the projection and its epilogue."""
    cfg = cfg_of("bf16", 64, 4, n_layers=4, vocab=1280, logit_scale=2.0, batch=batch, conf_mode=1, tied_head=False)
    w = W.make_weights(cfg, seed=23, gain_jitter=0.2)
    lm = w["w_lm"].view(2, 10, 2, 2, 16, -1)
    lm.copy_(lm[:1, :, :1, :1].clone().expand_as(lm))
    w["w_lm"] = lm.view(1280, -1)
    model = B.DeviceModel(cfg, w)
    ws = B.Workspace(model.desc, batch, 16)
    hidden = torch.randn(batch, cfg.d_model, generator=torch.Generator().manual_seed(23)).mul_(3.0).cuda()
    z = lambda *s: torch.zeros(*s, dtype=torch.int32, device="cuda")  # noqa: E731
    argmax, conf = z(batch), torch.full((batch,), 7.0, device="cuda")
    B.ee_exit_check(model, 2, hidden, 2.0, None, z(batch), z(batch), z(1), z(1), z(1), argmax, conf, ws)
    torch.cuda.synchronize()
    assert (argmax < 640).all() and (argmax % 64 < 16).all() and (conf == 0).all()


@pytest.mark.parametrize("dtype,batch,vocab", [
    ("bf16", 5, 1280), ("bf16", 40, 1280), ("bf16", 40, 1312), ("bf16", 100, 1280), ("bf16", 100, 8448),   # one tile a record
    ("bf16", 200, 1280), ("bf16", 450, 1280), ("bf16", 450, 8448),                                         # two
    ("fp32", 5, 130), ("fp32", 5, 514)])
def test_exit_check_of_a_row_of_nan(dtype, batch, vocab):
    """A hidden state of NaN (what attention leaves for a sequence of garbage) has no largest logit, but its arg max stays
    inside the vocabulary, in each form of the projection and its epilogue, and the rows beside it do not change a bit."""
    cfg = cfg_of(dtype, 64, 4, n_layers=4, vocab=vocab, logit_scale=2.0, batch=batch, tied_head=False)
    model = B.DeviceModel(cfg, W.make_weights(cfg, seed=24, gain_jitter=0.2))
    ws = B.Workspace(model.desc, batch, 16)
    hidden = torch.randn(batch, cfg.d_model, generator=torch.Generator().manual_seed(24)).mul_(3.0).cuda()
    bad = torch.tensor([1, batch - 1], device="cuda")
    z = lambda *s: torch.zeros(*s, dtype=torch.int32, device="cuda")  # noqa: E731
    got = []
    for nan in (False, True):
        if nan:
            hidden[bad] = float("nan")
        argmax, conf = z(batch) - 1, torch.zeros(batch, device="cuda")
        B.ee_exit_check(model, 2, hidden, 2.0, None, z(batch), z(batch), z(1), z(1), z(1), argmax, conf, ws)
        torch.cuda.synchronize()
        got.append((argmax, conf))
    assert (got[1][0] >= 0).all() and (got[1][0] < vocab).all(), got[1][0][bad]
    good = torch.ones(batch, dtype=torch.bool, device="cuda")
    good[bad] = False
    assert got[0][0][good].equal(got[1][0][good]) and got[0][1][good].equal(got[1][1][good])


@pytest.mark.parametrize("batch,vocab", [(33, 64), (37, 66), (70, 1030)])
def test_exit_check_fp32_several_row_blocks(batch, vocab):
    """The float projections deal (four batch rows, eight weight rows) out to the workgroups in one list: fewer groups of weight
    rows than XCDs, one more than a multiple, and a last block of few rows."""
    cfg = cfg_of("fp32", 64, 4, n_layers=6, vocab=vocab, logit_scale=2.0, batch=batch)
    run_exit_check(cfg, seed=60 + batch, layer=3, threshold=0.2, hidden_scale=3.0)


def test_exit_check_llama7b_width():
    """LM head of the 7B-shaped workload (vocab 32000 x d 4096, batch 32): every row's confidence and arg max."""
    cfg = W.reduced(L7B, n_layers=2, d_ffn=256)
    run_exit_check(cfg, seed=40, layer=1, threshold=0.9, hidden_scale=1.0)


# ------------------------------------------------------------------------------------------------------
# KV filling
# ------------------------------------------------------------------------------------------------------
def run_kv_fill(cfg, seed, lens, fill_from):
    lens = torch.tensor(lens, dtype=torch.int32)
    cfg = cfg.with_(batch=len(lens), shuffled_blocks=True)
    fill_from = torch.tensor(fill_from, dtype=torch.int32)
    w = W.make_weights(cfg, seed=seed, gain_jitter=0.2)
    m = O.model_from_config(cfg, w)
    run = HipRun(cfg, w, lens, 1, seed=seed, pool_fill=7.0)
    g = torch.Generator().manual_seed(seed)
    hidden = torch.randn(cfg.batch, cfg.d_model, generator=g) * 2.0
    batch = B.make_batch(None, lens.cuda(), run.bt_dev, int(lens.max()) + 1)
    B.ee_kv_fill(run.model, run.cache, batch, hidden.cuda(), fill_from.cuda(), run.ws)
    torch.cuda.synchronize()
    n = cfg.n_layers
    tol = tol_of(cfg)
    # oracle: one sequence at a time with its own first layer
    oc = O.DenseKV(n, cfg.batch, int(lens.max()) + 1, cfg.n_heads, cfg.head_dim, cfg.dtype)
    for b in range(cfg.batch):
        view = O._RowView(oc, [b])
        O.kv_fill(m, view, hidden[b:b + 1].to(F64), lens[b:b + 1].long(), int(fill_from[b]) + 1)
    written = torch.zeros(n, run.num_blocks, 16, dtype=torch.bool)
    for b in range(cfg.batch):
        p = int(lens[b])
        for i in range(1, n + 1):
            k, v = run.kv_at(i, b, p)
            if i > int(fill_from[b]):
                assert_close_scaled(k, oc.K[i - 1][b, p], tol, f"filled K layer {i} sequence {b}")
                assert_close_scaled(v, oc.V[i - 1][b, p], tol, f"filled V layer {i} sequence {b}")
                blk, off = W.slot_of(run.block_tables, b, p, 16)
                written[i - 1, blk, off] = True
    for pool in (run.cache.k, run.cache.v):
        x = pool.cpu().float().permute(0, 1, 3, 2, 4)
        assert bool((x[~written] == 7.0).all()), "KV filling wrote outside the slots it owns"
        assert not bool(written.any()) or bool((x[written] != 7.0).any())


@pytest.mark.parametrize("dtype,dh", [("fp32", 64), ("bf16", 64), ("bf16", 128)])
def test_kv_fill_per_sequence_layers(dtype, dh):
    cfg = cfg_of(dtype, dh, 2, n_layers=5)
    run_kv_fill(cfg, 50, lens=[0, 3, 15, 16, 40, 77, 5], fill_from=[1, 5, 2, 4, 3, 0, 5])


def test_kv_fill_uniform_layer_and_many_rows():
    cfg = cfg_of("bf16", 128, 2, n_layers=4)
    run_kv_fill(cfg, 51, lens=list(range(3, 3 + 45)), fill_from=[2] * 45)        # the paper's rule: one L for all
    run_kv_fill(cfg, 52, lens=[9, 10], fill_from=[4, 4])                           # nothing to fill


def test_kv_fill_width_1280_partly_rearranged_tile_order():
    """80 K/V tiles per layer: 64 take the XCD-aware order, 16 stay in place."""
    cfg = cfg_of("bf16", 128, 10, n_layers=4)
    run_kv_fill(cfg, 54, lens=[0, 17, 31, 64, 5], fill_from=[1, 0, 3, 2, 4])
    run_kv_fill(cfg, 55, lens=list(range(20, 52)), fill_from=[1] * 32)


def test_kv_fill_llama7b_width():
    cfg = W.reduced(L7B, n_layers=3, d_ffn=256, vocab=512)
    run_kv_fill(cfg, 53, lens=[512 + 3 * b for b in range(32)], fill_from=[1] * 32)
