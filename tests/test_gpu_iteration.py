"""Whole-iteration parity on the GPU: ee_decode_iteration against the CPU oracle in lock step (prefill + decode),
the oracle's invariants replayed on the HIP path, and the stored tiny-config trajectory."""
import json
import os

import pytest
import torch

from paper_2407_20272_amd import binding as B
from paper_2407_20272_amd import workloads as W
from gpu_harness import HipRun, lockstep

pytestmark = pytest.mark.gpu
TINY, L7B = W.CONFIGS[0], W.CONFIGS[1]
HERE = os.path.dirname(os.path.abspath(__file__))


def small_bf16(**kw):
    base = dict(n_layers=4, d_model=256, n_heads=2, head_dim=128, d_ffn=352, vocab=1024, batch=5, prompt_len=9,
                min_prompt_len=9, decode_steps=6, weight_std=0.05, logit_scale=1.0, threshold=0.5)
    base.update(kw)
    return W.reduced(L7B, **base)


def test_tiny_fp32_full_trajectory_matches_oracle_and_stored_values():
    """Benchmark config 0 exactly as defined (seed 0, gains 1): all 16 decode steps, zero tolerated divergences."""
    stats = lockstep(TINY, seed=0, steps=TINY.decode_steps, gain_jitter=0.0)
    assert stats["near_threshold"] == 0 and stats["near_tie"] == 0
    with open(os.path.join(HERE, "golden", "tiny_fp32_seed0.json")) as f:
        want = json.load(f)
    assert stats["L"] == want["batch_exit_layer"]


def test_tiny_fp32_untied_head_trajectory_with_varying_tokens():
    """The tiny shape with an untied head and wider weights (the stored second trajectory): every step emits a
    different token per sequence, the batch leaves at layers 2, 3 and 4; all 16 steps, zero tolerated divergences."""
    import importlib.util
    spec = importlib.util.spec_from_file_location("make_golden", os.path.join(HERE, "golden", "make_golden.py"))
    gen = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(gen)
    cfg, seed = gen.case("tiny_fp32_untied_seed4")
    stats = lockstep(cfg, seed=seed, steps=cfg.decode_steps, gain_jitter=0.0)
    assert stats["near_threshold"] == 0 and stats["near_tie"] == 0
    with open(os.path.join(HERE, "golden", "tiny_fp32_untied_seed4.json")) as f:
        want = json.load(f)
    assert stats["L"] == want["batch_exit_layer"]


@pytest.mark.parametrize("seed", [1, 2])
def test_tiny_fp32_other_seeds_with_gain_jitter(seed):
    stats = lockstep(TINY.with_(decode_steps=6, weight_std=0.05, logit_scale=1.0, threshold=0.3), seed=seed, steps=6)
    assert stats["near_threshold"] == 0 and stats["near_tie"] == 0


@pytest.mark.parametrize("dtype", ["fp32", "bf16"])
def test_two_sequences_long_prompts_attention_split_among_workgroups(dtype):
    """Two sequences with prompts of 140 to 300 tokens and two heads: the iteration's attention gives every
    (sequence, head) pair to two workgroups (a part of the context each) and merges them in a second launch."""
    if dtype == "fp32":
        cfg = TINY.with_(batch=2, n_heads=2, head_dim=128, prompt_len=300, min_prompt_len=140, decode_steps=3, weight_std=0.05,
                         logit_scale=1.0, threshold=0.3, shuffled_blocks=True)
    else:
        cfg = small_bf16(batch=2, prompt_len=300, min_prompt_len=140, shuffled_blocks=True)
    stats = lockstep(cfg, seed=47, steps=3)
    total = stats["decisions"] + stats["tokens"]
    assert stats["near_threshold"] + stats["near_tie"] <= max(2, total // 20), stats


@pytest.mark.parametrize("batch,d_ffn,vocab,conf_mode", [(1, 257, 130, 0), (5, 258, 514, 1), (9, 1028, 64, 2), (4, 62, 2, 3)])
def test_fp32_odd_widths(batch, d_ffn, vocab, conf_mode):
    """The float projections take four batch rows a wavefront and 16 bytes a load where a contraction divides by four: rows
    that do not divide by four, widths that do not, a contraction and a vocabulary narrower than a workgroup, every
    confidence measure (the sums of a measure and its decision share a launch)."""
    cfg = TINY.with_(batch=batch, d_ffn=d_ffn, vocab=vocab, conf_mode=conf_mode, prompt_len=12, min_prompt_len=5, weight_std=0.05,
                     logit_scale=1.0, threshold=0.99 if conf_mode == 2 else 0.5, shuffled_blocks=True, tied_head=False)
    stats = lockstep(cfg, seed=7, steps=4)
    assert stats["near_threshold"] + stats["near_tie"] <= 1


@pytest.mark.parametrize("batch,heads,dh,d_ffn,layers,head_mode", [
    (1, 1, 64, 62, 1, True),       # no layer behind the first: the only LM head runs beside KV filling
    (32, 2, 64, 130, 3, 2),        # 64 (sequence, head) pairs: attention multiplies by the output projection; contraction of 130, no 16-byte loads
    (33, 2, 64, 256, 3, True),     # 66: a launch of its own again
    (16, 4, 64, 1028, 3, 2),       # the widest, 64 pairs: four parts; the down projection past 1024 in a loop
    (17, 4, 64, 1024, 3, True),    # 68 pairs; 1024 of a contraction at once, in 160 workgroups
    (32, 2, 128, 1024, 3, 2),      # .. in 256
    (36, 2, 128, 1024, 3, True),   # .. in 288: a loop
    (3, 3, 64, 640, 3, 2),         # three parts, three pieces
    (64, 2, 128, 320, 2, 2),       # the last row count of the four-launch form ..
    (65, 2, 128, 320, 2, True),    # .. past it
    (12, 5, 64, 1028, 3, 2),       # .. and past its width: 320 channels ..
    (16, 4, 128, 1024, 3, True),   # .. 512, the last width of the decision inside QKV ..
    (5, 9, 64, 576, 2, True),      # .. and past that
])
def test_fp32_layers_in_four_launches(batch, heads, dh, d_ffn, layers, head_mode):
    """Float layers of up to 64 rows and 256 channels, at the edges of the forms: the LM head beside the next QKV projection or KV filling,
    the decision in front of attention, the output projection inside it; sequences leave together or one by one."""
    cfg = TINY.with_(batch=batch, n_heads=heads, head_dim=dh, d_model=heads * dh, d_ffn=d_ffn, vocab=130, n_layers=layers, prompt_len=20,
                     min_prompt_len=3, weight_std=0.05, logit_scale=1.0, threshold=0.3, shuffled_blocks=True, tied_head=False)
    forced = torch.randint(1, layers + 1, (3, batch), generator=torch.Generator().manual_seed(batch), dtype=torch.int32)
    if head_mode is True:
        forced = None
    lockstep(cfg, seed=13, steps=3, heads=head_mode, forced_seq=forced)


def test_fp32_ragged_prompts_shuffled_blocks_conf_mode1():
    cfg = TINY.with_(batch=6, prompt_len=21, min_prompt_len=3, shuffled_blocks=True, conf_mode=1, weight_std=0.05,
                     logit_scale=2.0, threshold=0.2, n_layers=5, exit_every=2)
    stats = lockstep(cfg, seed=3, steps=5)
    assert stats["near_threshold"] == 0 and stats["near_tie"] == 0


@pytest.mark.parametrize("batch", [5, 32, 40, 70])
def test_small_bf16_lockstep(batch):
    """bf16 path (MFMA projections, tiled layouts): batch sizes below, at and above one and two 32-row tiles."""
    cfg = small_bf16(batch=batch, shuffled_blocks=True, prompt_len=12, min_prompt_len=4)
    stats = lockstep(cfg, seed=10 + batch, steps=5)
    total = stats["decisions"] + stats["tokens"]
    assert stats["near_threshold"] + stats["near_tie"] <= max(2, total // 20), stats
    assert len(set(stats["L"])) >= 1


@pytest.mark.parametrize("batch,heads,dh,d_ffn,vocab,layers,head_mode", [
    (1, 1, 64, 16, 32, 2, True),       # one tile everywhere, a contraction of one step, wavefronts without a load
    (2, 3, 64, 48, 96, 3, 2),          # three steps: a last load that is not full
    (3, 5, 64, 496, 1344, 3, 2),       # three rows of four, 31 steps
    (4, 2, 128, 80, 64, 2, True),
    (5, 10, 64, 1040, 160, 3, 2),      # the narrowest of five to eight rows ..
    (8, 10, 64, 336, 160, 3, True),
    (5, 6, 64, 1040, 160, 3, 2),       # .. and narrower, in the other kernels (but for the prompt, which has no checks)
    (8, 9, 64, 336, 160, 3, True),
    (8, 5, 64, 336, 160, 3, 2),        # .. the prompt as well
    (4, 4, 64, 336, 8224, 2, True),    # more than 256 tiles of the head: the narrowest of three and four rows ..
    (4, 3, 64, 336, 8224, 2, True),    # .. and narrower
    (8, 24, 128, 32, 64, 1, True),     # the widest of eight rows: 24576 channels; residual updates in 16-row units (8-row ones up to 2048)
    (7, 25, 128, 32, 64, 1, True),     # .. and wider
    (1, 32, 128, 80, 64, 2, True),     # 16-row units, one a workgroup
    (3, 33, 128, 32, 64, 1, True),     # past 4096 channels: operand rows in three groups, 8-row units, three a workgroup
    (2, 52, 128, 32, 64, 1, True),     # past 6144: in four; 16-row units, two a workgroup
    (1, 8, 128, 8240, 16480, 2, True), # 515 tiles of gate/up and of the LM head: two or three a workgroup
    (3, 10, 64, 8240, 24608, 2, 2),    # .. 769: three or four
    (8, 10, 64, 12304, 16480, 2, 2),   # .. of eight rows
])
def test_bf16_up_to_eight_sequences(batch, heads, dh, d_ffn, vocab, layers, head_mode):
    """Projections that build their own operand and add to the residual rows, at the edges of their units, loads and rule; sequences leave
    together or one by one."""
    cfg = small_bf16(batch=batch, n_heads=heads, head_dim=dh, d_model=heads * dh, d_ffn=d_ffn, vocab=vocab, n_layers=layers, prompt_len=19,
                     min_prompt_len=5, shuffled_blocks=True, weight_std=0.05 if heads * dh < 1024 else 0.02)
    forced = torch.randint(1, layers + 1, (3, batch), generator=torch.Generator().manual_seed(batch), dtype=torch.int32)
    stats = lockstep(cfg, seed=17, steps=3, heads=head_mode, forced_seq=forced if head_mode == 2 else None)
    assert stats["near_threshold"] + stats["near_tie"] <= max(2, (stats["decisions"] + stats["tokens"]) // 20), stats


def test_bf16_width_1280_partly_rearranged_tile_order():
    """d_model 1280 (10 heads x 128): the QKV projection has 80 whole and 40 halved tiles, so the XCD-aware tile
    order of the streaming kernel rearranges 64 of each and leaves the rest in place; KV filling runs too."""
    cfg = small_bf16(d_model=1280, n_heads=10, head_dim=128, n_layers=3, batch=7, threshold=0.35, shuffled_blocks=True)
    stats = lockstep(cfg, seed=61, steps=4)
    total = stats["decisions"] + stats["tokens"]
    assert stats["near_threshold"] + stats["near_tie"] <= max(2, total // 20), stats


@pytest.mark.parametrize("batch,n_layers,exit_every,conf_mode,threshold", [
    (1, 3, 1, 0, 0.4), (7, 6, 3, 0, 0.3), (33, 5, 2, 1, 0.2), (64, 4, 1, 0, 0.45), (12, 7, 1, 0, 0.9), (20, 5, 1, 0, 0.05)])
def test_bf16_exit_decision_carried_by_the_next_projection(batch, n_layers, exit_every, conf_mode, threshold):
    """Batches the streaming projection kernel serves (the exit decision of a layer is taken inside the next layer's
    QKV launch): one and two batch tiles, heads after every / every 2nd / 3rd layer, thresholds from "everybody
    leaves at the first head" (the projection after it runs speculatively) to "nobody ever leaves"."""
    cfg = small_bf16(batch=batch, n_layers=n_layers, exit_every=exit_every, conf_mode=conf_mode, threshold=threshold,
                     shuffled_blocks=True, prompt_len=10, min_prompt_len=3)
    stats = lockstep(cfg, seed=70 + batch, steps=4)
    total = stats["decisions"] + stats["tokens"]
    assert stats["near_threshold"] + stats["near_tie"] <= max(2, total // 20), stats


def test_small_bf16_head_dim_64_exit_every_2_mode1():
    cfg = small_bf16(n_heads=4, head_dim=64, n_layers=6, exit_every=2, conf_mode=1, batch=9, threshold=0.3)
    lockstep(cfg, seed=21, steps=4)


def test_threshold_above_one_equals_full_layer_path():
    """Invariant: a threshold no confidence can pass reproduces the head-less full-layer path bit for bit."""
    for cfg in (TINY.with_(decode_steps=4), small_bf16()):
        w = W.make_weights(cfg, seed=4, gain_jitter=0.1)
        prompts, lens = W.make_prompts(cfg, seed=4), W.make_context_lens(cfg, seed=4)
        outs = []
        for heads in (True, False):
            run = HipRun(cfg, w, lens, 4, seed=4)
            tok = run.prefill(prompts, lens)
            pos = lens.clone().long()
            toks = [tok]
            for s in range(4):
                tok, e, L, conf, hid = run.step(tok, pos, 1.0 + 1e-6, heads=heads)
                assert L == cfg.n_layers and bool((e == cfg.n_layers).all())
                toks.append(tok)
                pos += 1
            outs.append((torch.stack(toks), run.cache.k.clone(), run.cache.v.clone()))
        assert torch.equal(outs[0][0], outs[1][0])
        assert torch.equal(outs[0][1], outs[1][1]) and torch.equal(outs[0][2], outs[1][2])     # fp32 and bf16 alike


@pytest.mark.parametrize("cfg", [TINY.with_(n_layers=6, decode_steps=3), small_bf16(n_layers=6)], ids=["fp32", "bf16"])
def test_forced_exit_lockstep(cfg):
    """Synthetic confidence injection: per-sequence forced exit layers, the batch leaves at their maximum."""
    g = torch.Generator().manual_seed(9)
    forced = torch.randint(1, cfg.n_layers + 1, (4, cfg.batch), generator=g, dtype=torch.int32)
    forced[1] = 2                                  # static mode: everybody leaves at layer 2
    forced[2] = cfg.n_layers                       # nobody leaves early
    stats = lockstep(cfg, seed=5, steps=4, forced_seq=forced)
    assert stats["L"] == [int(forced[s].max()) for s in range(4)]


@pytest.mark.parametrize("dtype", ["fp32", "bf16"])
def test_saturated_model_forced_exit_cache_equals_full_pass(dtype):
    """Invariant: when the layers above L0 add nothing to the residual stream, a forced exit at L0 leaves the
    whole cache and the tokens identical to a full pass."""
    cfg = (TINY if dtype == "fp32" else small_bf16()).with_(n_layers=5)
    L0 = 3
    w = W.make_weights(cfg, seed=6, gain_jitter=0.1)
    for i in range(L0, cfg.n_layers):
        w["layers"][i]["w_o"].zero_()
        w["layers"][i]["w_down"].zero_()
    prompts, lens = W.make_prompts(cfg, seed=6), W.make_context_lens(cfg, seed=6)
    res = []
    for forced_mode in (True, False):
        run = HipRun(cfg, w, lens, 3, seed=6)
        tok = run.prefill(prompts, lens)
        pos = lens.clone().long()
        toks = []
        for s in range(3):
            f = torch.full((cfg.batch,), L0, dtype=torch.int32) if forced_mode else None
            tok, e, L, _, _ = run.step(tok, pos, 0.5, forced=f, heads=forced_mode)
            assert L == (L0 if forced_mode else cfg.n_layers)
            toks.append(tok)
            pos += 1
        res.append((torch.stack(toks), run.cache.k.clone(), run.cache.v.clone()))
    assert torch.equal(res[0][0], res[1][0])
    if dtype == "fp32":
        assert torch.equal(res[0][1], res[1][1]) and torch.equal(res[0][2], res[1][2])
    else:
        # Layers up to L0 ran the same kernels on the same values in both runs: identical bits.  Above L0 the filling
        # launch and the full pass's own QKV launch project the same normalised operand but sum the contraction in
        # different orders (different kernels; the V tiles of the forward launch are split between two workgroups), so
        # a value may land on the neighbouring bf16 number (or, where the terms cancel, within float noise of zero).
        for pool in (1, 2):
            assert torch.equal(res[0][pool][:L0], res[1][pool][:L0])
            a, b = res[0][pool][L0:].float(), res[1][pool][L0:].float()
            step = torch.exp2(torch.floor(torch.log2(torch.clamp(b.abs(), min=1e-30))) - 7)        # one bf16 step at b
            assert bool(((a - b).abs() <= torch.clamp(step * 1.001, min=1e-5 * float(b.abs().max()))).all()), \
                "a filled value is more than one bf16 step from the full pass's"
            assert float((a != b).float().mean()) < 0.02, "more than 2 % of the filled values differ in the last bit"


@pytest.mark.parametrize("dtype,batch,conf_mode", [("bf16", 3, 0), ("bf16", 33, 1), ("bf16", 64, 2), ("bf16", 65, 0), ("bf16", 40, 3),
                                                   ("fp32", 5, 0), ("fp32", 5, 2), ("fp32", 65, 1)])
def test_kv_filling_behind_the_last_layer_that_ran_or_was_cached(dtype, batch, conf_mode):
    """The batch leaves at the first, a middle and the last checked layer: every layer above it is cached once, by the projection that shares a
    launch with the decision or by KV filling, whichever the batch and the measure take."""
    base = dict(batch=batch, n_layers=4, conf_mode=conf_mode, prompt_len=12, min_prompt_len=4, shuffled_blocks=True)
    cfg = TINY.with_(**base) if dtype == "fp32" else small_bf16(**base)
    forced = torch.tensor([1, 2, 3], dtype=torch.int32)[:, None].expand(3, batch).contiguous()
    stats = lockstep(cfg, seed=23, steps=3, forced_seq=forced)
    assert stats["L"] == [1, 2, 3]


def test_empty_batch_is_a_noop():
    cfg = TINY
    w = W.make_weights(cfg, seed=0)
    run = HipRun(cfg, w, torch.tensor([3], dtype=torch.int32), 1)
    tok, e, L, conf, hid = run.step(torch.zeros(0, dtype=torch.int32), torch.zeros(0, dtype=torch.long), 0.5,
                                    rows=[])
    assert tok.numel() == 0 and e.numel() == 0


# ------------------------------------------------------------------------------------------------
# confidence measures without an exit head (Section 2.1): hidden states similarity (2), dedicated classifier (3)
# ------------------------------------------------------------------------------------------------
@pytest.mark.parametrize("conf_mode,threshold", [(2, 0.65), (3, 0.62)])
def test_fp32_headless_measures_lockstep(conf_mode, threshold):
    cfg = TINY.with_(decode_steps=4, n_layers=6, conf_mode=conf_mode, threshold=threshold)
    stats = lockstep(cfg, seed=31, steps=4)
    assert stats["near_threshold"] == 0 and stats["near_tie"] == 0
    assert min(stats["L"]) < cfg.n_layers, stats["L"]          # the batch did leave early at least once


@pytest.mark.parametrize("batch", [7, 40])
@pytest.mark.parametrize("conf_mode,threshold", [(2, 0.78), (3, 0.55)])
def test_bf16_headless_measures_lockstep(conf_mode, threshold, batch):
    cfg = small_bf16(n_layers=6, batch=batch, prompt_len=12, min_prompt_len=4, shuffled_blocks=True,
                     conf_mode=conf_mode, threshold=threshold)
    stats = lockstep(cfg, seed=32, steps=5)
    total = stats["decisions"] + stats["tokens"]
    assert stats["near_threshold"] + stats["near_tie"] <= max(2, total // 20), stats
    assert stats["max_conf_err"] < 2e-2


@pytest.mark.parametrize("dtype", ["fp32", "bf16"])
def test_similarity_with_checks_every_second_layer(dtype):
    """The previous hidden state is the one before layer i also where layer i-1 had no check."""
    base = TINY.with_(decode_steps=3) if dtype == "fp32" else small_bf16(batch=9)
    cfg = base.with_(n_layers=7, exit_every=2, conf_mode=2, threshold=0.7)
    lockstep(cfg, seed=33, steps=3)


@pytest.mark.parametrize("conf_mode", [2, 3])
def test_headless_measures_forced_exits(conf_mode):
    cfg = small_bf16(n_layers=6, conf_mode=conf_mode)
    g = torch.Generator().manual_seed(11)
    forced = torch.randint(1, cfg.n_layers + 1, (3, cfg.batch), generator=g, dtype=torch.int32)
    forced[1] = 1
    stats = lockstep(cfg, seed=34, steps=3, forced_seq=forced)
    assert stats["L"] == [int(forced[s].max()) for s in range(3)]


# ------------------------------------------------------------------------------------------------
# per-sequence exit (extension of Algorithm 1): every sequence leaves at its own layer
# ------------------------------------------------------------------------------------------------
@pytest.mark.parametrize("conf_mode,threshold", [(0, 0.8), (2, 0.65), (3, 0.62)])
def test_fp32_per_sequence_exit_lockstep(conf_mode, threshold):
    cfg = TINY.with_(decode_steps=4, n_layers=6, conf_mode=conf_mode, threshold=threshold)
    stats = lockstep(cfg, seed=31, steps=4, heads=2)
    assert stats["near_threshold"] == 0 and stats["near_tie"] == 0


@pytest.mark.parametrize("batch", [7, 40, 70])
@pytest.mark.parametrize("conf_mode,threshold", [(0, 0.5), (2, 0.78)])
def test_bf16_per_sequence_exit_lockstep(conf_mode, threshold, batch):
    cfg = small_bf16(n_layers=6, batch=batch, prompt_len=12, min_prompt_len=4, shuffled_blocks=True,
                     conf_mode=conf_mode, threshold=threshold)
    stats = lockstep(cfg, seed=41, steps=5, heads=2)
    total = stats["decisions"] + stats["tokens"]
    assert stats["near_threshold"] + stats["near_tie"] <= max(2, total // 20), stats


@pytest.mark.parametrize("cfg", [TINY.with_(n_layers=6, decode_steps=3), small_bf16(n_layers=6, batch=9)], ids=["fp32", "bf16"])
def test_per_sequence_forced_exits(cfg):
    """Mixed forced exit layers: sequences leave one by one; their K/V above their own exit layer is filled from
    their own hidden state (checked slot by slot against the oracle by the lock-step comparison)."""
    g = torch.Generator().manual_seed(19)
    forced = torch.randint(1, cfg.n_layers + 1, (4, cfg.batch), generator=g, dtype=torch.int32)
    forced[1] = 3                                  # everybody at layer 3: coincides with Algorithm 1
    forced[2] = cfg.n_layers                       # nobody leaves early
    forced[3, 0] = 1                               # one sequence leaves at once, the rest later
    stats = lockstep(cfg, seed=42, steps=4, forced_seq=forced, heads=2)
    assert stats["L"] == [int(forced[s].max()) for s in range(4)]


def compactable_bf16(**kw):
    """Widths whose weight tiles come in whole groups of four: from 129 rows on the per-sequence rule compacts the rows that are
    still active."""
    return small_bf16(n_layers=6, d_ffn=384, prompt_len=10, min_prompt_len=3, shuffled_blocks=True, **kw)


@pytest.mark.parametrize("batch", [128, 256, 384])
@pytest.mark.parametrize("conf_mode,threshold", [(0, 0.5), (2, 0.78)])
def test_bf16_per_sequence_exit_compacted_rows_lockstep(conf_mode, threshold, batch):
    cfg = compactable_bf16(batch=batch, conf_mode=conf_mode, threshold=threshold)
    stats = lockstep(cfg, seed=43, steps=3, heads=2)
    total = stats["decisions"] + stats["tokens"]
    assert stats["near_threshold"] + stats["near_tie"] <= max(2, total // 20), stats


@pytest.mark.parametrize("batch", [385, 400, 481, 512])
@pytest.mark.parametrize("heads", [1, 2])
def test_bf16_385_to_512_rows_lockstep(batch, heads):
    """385 to 512 rows: the LM head runs in the 256 x 256 ring kernel under Algorithm 1 (a second row block that ends in one row or
    is full), with compacted rows in blocks under the per-sequence rule; everything else runs in blocks."""
    cfg = compactable_bf16(batch=batch)
    stats = lockstep(cfg, seed=46, steps=2, heads=heads)
    total = stats["decisions"] + stats["tokens"]
    assert stats["near_threshold"] + stats["near_tie"] <= max(2, total // 20), stats


@pytest.mark.parametrize("heads,tiles,batch", [(2, 776, 385), (2, 1024, 512), (4, 1544, 400)])
def test_bf16_gate_up_in_the_ring_kernel(heads, tiles, batch):
    """385 to 512 rows and 776 gate/up tiles or more: 256 x 256 blocks in one round (the second row block ends in one row, or is
    full), or in two; one and two turns of the ring."""
    cfg = small_bf16(n_layers=2, d_model=128 * heads, n_heads=heads, d_ffn=16 * tiles, vocab=512, batch=batch, prompt_len=2, min_prompt_len=1,
                     shuffled_blocks=True)
    stats = lockstep(cfg, seed=47, steps=1)
    total = stats["decisions"] + stats["tokens"]
    assert stats["near_threshold"] + stats["near_tie"] <= max(2, total // 20), stats


@pytest.mark.parametrize("batch", [96, 150, 200])
@pytest.mark.parametrize("heads", [1, 2])
def test_bf16_row_counts_with_a_short_last_chunk(batch, heads):
    """Three, five and seven 32-row tiles: a last block of fewer tiles than the others, in the tiled and in the block kernel (under
    the per-sequence rule above 128 rows with the active rows compacted)."""
    cfg = compactable_bf16(batch=batch)
    stats = lockstep(cfg, seed=45, steps=3, heads=heads)
    total = stats["decisions"] + stats["tokens"]
    assert stats["near_threshold"] + stats["near_tie"] <= max(2, total // 20), stats


@pytest.mark.parametrize("heads,dh,batch", [
    (25, 128, 7),      # QKV as 200 whole tiles with half a V tile each: the last 8 past the groups that are rearranged
    (44, 64, 31),      # 264 tiles, one batch tile: too few for two tiles a workgroup
    (49, 64, 31),      # 294: 196 whole tiles with half a V tile each, the fewest
    (22, 128, 33),     # the same in two batch tiles, the second of one row
    (33, 128, 64),     # 396 tiles as 198 pairs; output projection of 132 tiles: three slices of 88 steps of 64 x 64 blocks
    (33, 128, 2),      # ... in one batch tile: pairs
])
def test_bf16_two_output_tiles_per_workgroup(heads, dh, batch):
    cfg = small_bf16(n_layers=2, d_model=heads * dh, n_heads=heads, head_dim=dh, d_ffn=96, vocab=512, batch=batch, prompt_len=3,
                     min_prompt_len=2, weight_std=0.02, shuffled_blocks=True, threshold=2.0)
    stats = lockstep(cfg, seed=61, steps=2)
    assert stats["near_threshold"] + stats["near_tie"] <= max(2, stats["tokens"] // 20), stats


@pytest.mark.parametrize("d_ffn", [16, 48, 80])
def test_bf16_short_contractions_onto_many_tiles(d_ffn):
    """Two batch tiles, 128 weight tiles and a down projection of one, three or five steps: too short for 64 x 64 blocks, which add a
    slice in four parts, or just long enough."""
    cfg = small_bf16(n_layers=1, d_model=4096, n_heads=32, head_dim=128, d_ffn=d_ffn, vocab=512, batch=34, prompt_len=1, min_prompt_len=1,
                     weight_std=0.02, shuffled_blocks=True, threshold=2.0)
    stats = lockstep(cfg, seed=64, steps=1)
    assert stats["near_threshold"] + stats["near_tie"] <= max(2, stats["tokens"] // 20), stats


@pytest.mark.parametrize("heads,d_ffn,layers", [(33, 1104, 2), (40, 2064, 1), (53, 96, 1)])
def test_bf16_rows_do_not_hang_on_the_other_batch_tile(heads, d_ffn, layers):
    """Output and down projection onto 132, 160 and 212 tiles: one batch tile in pairs of tiles in the streaming kernel, two in 64 x 64
    blocks, which add the same parts in the same order.  64 sequences end with the hidden states that they have 32 at a time, bit for
    bit (slices of odd lengths, parts that end inside a stage)."""
    cfg = small_bf16(n_layers=layers, d_model=heads * 128, n_heads=heads, head_dim=128, d_ffn=d_ffn, vocab=512, batch=64, prompt_len=1,
                     min_prompt_len=1, weight_std=0.02)
    lens = torch.full((64,), 3, dtype=torch.int32)
    run = HipRun(cfg, W.make_weights(cfg, seed=65, gain_jitter=0.1), lens, 1, seed=65)
    tokens = torch.randint(0, cfg.vocab, (64,), generator=torch.Generator().manual_seed(65), dtype=torch.int32)
    run.cache.k.normal_()
    run.cache.v.normal_()
    want = run.step(tokens, lens.long(), 2.0, heads=False)[4]
    for half in (list(range(32)), list(range(32, 64))):
        got = run.step(tokens[half], lens[half].long(), 2.0, heads=False, rows=half)[4]
        assert torch.equal(got, want[half])


@pytest.mark.parametrize("heads,dh,batch", [(107, 64, 33), (54, 128, 64)])   # 214 and 216 tiles, the second batch tile of one row or full
def test_bf16_output_projection_in_pairs_of_two_batch_tiles(heads, dh, batch):
    cfg = small_bf16(n_layers=1, d_model=heads * dh, n_heads=heads, head_dim=dh, d_ffn=96, vocab=512, batch=batch, prompt_len=1,
                     min_prompt_len=1, weight_std=0.02, shuffled_blocks=True, threshold=2.0)
    stats = lockstep(cfg, seed=63, steps=1)
    assert stats["near_threshold"] + stats["near_tie"] <= max(2, stats["tokens"] // 20), stats


@pytest.mark.parametrize("heads,dh,d_ffn,batch", [
    (3, 64, 16, 65),        # QKV: 18 tiles in blocks of 3 (64 x 96), the last batch tile of one row; down: a contraction of one step
    (5, 64, 112, 97),       # QKV: 30 tiles; down of seven steps (one past the last pair); gate/up of seven tiles: streaming kernel
    (18, 64, 48, 497),      # QKV: 108 tiles as 128 x 64
    (12, 128, 48, 481),     # 144 as 128 x 96; output projection: 48 tiles
    (17, 128, 48, 512),     # 204 as 128 x 128; output projection: 68 tiles, two slices
    (22, 128, 48, 385),     # 264 as 128 x 192
    (2, 128, 16 * 385, 129),    # gate/up: 385 tiles as 128 x 128, a second row block of one row; down: four slices of 96 or 97 steps
    (2, 128, 16 * 551, 160),    # 551 as 128 x 192, the last block one of five tiles
    (2, 128, 16 * 802, 170),    # 802 as 256 x 128, the last of two tiles
    (1, 128, 16 * 700, 290),    # 700 as 256 x 192, the last of four tiles, a second row block of two
    (43, 64, 4096, 385),        # down: 86 tiles as 256 x 128 in four slices, the last block of two tiles, a second row block that ends in one row
])
def test_bf16_projections_in_blocks(heads, dh, d_ffn, batch):
    """The block shapes of QKV, gate/up, output and down projection from 65 rows on, at ragged edges of rows, tiles and contraction.
    (64 x 64 blocks: test_bf16_two_output_tiles_per_workgroup; the LM head's: test_exit_check_in_blocks; compacted rows: below.)"""
    cfg = small_bf16(n_layers=1, d_model=heads * dh, n_heads=heads, head_dim=dh, d_ffn=d_ffn, vocab=512, batch=batch, prompt_len=2,
                     min_prompt_len=1, weight_std=0.02, shuffled_blocks=True, threshold=2.0)
    stats = lockstep(cfg, seed=62, steps=1)
    assert stats["near_threshold"] + stats["near_tie"] <= max(2, stats["tokens"] // 20), stats


@pytest.mark.parametrize("batch", [65, 200, 512])
def test_keys_cached_by_a_projection_in_blocks_are_those_of_kv_filling(batch):
    """From 65 rows on the QKV projection of a layer and the KV filling of that layer sum the same products in the same order and
    turn them alike, so what they cache is the same bit for bit.  (Where only the rounding inside the rotation differs, about
    one element in two million does: twelve passes, 1.6 to 12.6 million keys.)"""
    cfg = small_bf16(n_layers=1, d_model=2048, n_heads=16, head_dim=128, d_ffn=96, vocab=4096, batch=batch, prompt_len=40, min_prompt_len=1,
                     weight_std=0.02)
    w = W.make_weights(cfg, seed=47, gain_jitter=0.1)
    gen = torch.Generator().manual_seed(47)
    lens = torch.randint(1, 40, (batch,), generator=gen, dtype=torch.int32)
    run = HipRun(cfg, w, lens, 1, seed=47)
    fill_from = torch.zeros(batch, dtype=torch.int32, device="cuda")
    for _ in range(12):
        tokens = torch.randint(0, cfg.vocab, (batch,), generator=gen, dtype=torch.int32)
        run.step(tokens, lens.long(), 2.0, heads=False)
        want = run.cache.k.clone(), run.cache.v.clone()
        run.cache.k.zero_()
        run.cache.v.zero_()
        hidden = w["embed"][tokens.long()].float().cuda()
        B.ee_kv_fill(run.model, run.cache, B.make_batch(None, lens.cuda(), run.bt_dev, 41), hidden, fill_from, run.ws)
        torch.cuda.synchronize()
        assert bool(run.cache.k.any()) and bool(run.cache.v.any())
        assert torch.equal(run.cache.v, want[1]) and torch.equal(run.cache.k, want[0])


@pytest.mark.parametrize("exit_every", [1, 2])
def test_per_sequence_compaction_across_chunk_boundaries(exit_every):
    """Forced exits that take the number of active rows through 129, 128, 127, 1 and 0 (the projections work on
    128-row chunks), with the last sequence staying to the end or leaving one layer before it (KV filling of the
    last layer), and with checks after every second layer only (the row sums of sequences that have left move on
    through layers without a check)."""
    cfg = compactable_bf16(batch=256, exit_every=exit_every)
    n, Bsz = cfg.n_layers, cfg.batch
    forced = torch.full((3, Bsz), 4, dtype=torch.int32)
    forced[:, :127] = 1
    forced[:, 127] = 2
    forced[:, 128] = 3
    forced[0, 255] = n           # one sequence runs every layer
    forced[1, 255] = n - 1       # ... or leaves before the last layer, which is then filled
    forced[2] = torch.randint(1, n + 1, (Bsz,), generator=torch.Generator().manual_seed(5), dtype=torch.int32)
    stats = lockstep(cfg, seed=44, steps=3, forced_seq=forced, heads=2)
    want = [n, n - 1 if exit_every == 1 else n, int(forced[2].max())]
    if exit_every == 1:
        assert stats["L"] == want


@pytest.mark.parametrize("batch", [256, 300])
def test_compacted_rows_in_halves_of_blocks(batch):
    """At most half of the row blocks active: two workgroups share a column block of gate/up (524 tiles in blocks of six, the last one
    of two: its second half has none) and of the LM head (516 in blocks of eight, the last one of four)."""
    cfg = small_bf16(n_layers=5, d_model=128, n_heads=1, d_ffn=16 * 524, vocab=32 * 516, prompt_len=2, min_prompt_len=1, shuffled_blocks=True,
                     batch=batch)
    forced = torch.ones(1, batch, dtype=torch.int32)
    forced[0, torch.randperm(batch, generator=torch.Generator().manual_seed(7))[:128]] = 2   # 128 rows after layer 1
    forced[0, 5] = 3
    forced[0, batch - 1] = 4
    stats = lockstep(cfg, seed=53, steps=1, forced_seq=forced, heads=2)
    assert stats["L"] == [4]


@pytest.mark.parametrize("batch,exit_every", [(129, 1), (256, 1), (257, 1), (200, 6)])   # compacted up to 256 rows; no check ahead of the last layer
def test_last_lm_head_of_the_rows_that_stay(batch, exit_every):
    """Nobody, half of the rows, all but one leave ahead of the last layer: who stays gets a token there, the others keep theirs."""
    cfg = compactable_bf16(batch=batch, exit_every=exit_every)
    forced = torch.full((3, batch), cfg.n_layers, dtype=torch.int32)
    forced[1, ::2] = 2
    forced[2, 1:] = cfg.n_layers - 1
    stats = lockstep(cfg, seed=45, steps=3, forced_seq=forced, heads=2)
    assert stats["L"] == [cfg.n_layers] * 3


@pytest.mark.parametrize("batch,vocab", [(256, 32 * 516), (300, 32 * 64)])
def test_confidences_do_not_hang_on_how_many_rows_are_active(batch, vocab):
    """The sequences that stay have the confidences and hidden states, bit for bit, that they have when the others stay too (whole
    blocks of the projections against halves of them)."""
    cfg = small_bf16(n_layers=3, d_model=256, n_heads=2, d_ffn=16 * 532, vocab=vocab, batch=batch)
    lens = torch.full((batch,), 3, dtype=torch.int32)
    run = HipRun(cfg, W.make_weights(cfg, seed=54, gain_jitter=0.1), lens, 1, seed=54)
    tokens = torch.randint(0, vocab, (batch,), generator=torch.Generator().manual_seed(54), dtype=torch.int32)
    run.cache.k.normal_()
    run.cache.v.normal_()
    forced = torch.full((batch,), cfg.n_layers, dtype=torch.int32)
    _, _, _, want_conf, want = run.step(tokens, lens.long(), 2.0, forced=forced, heads=2)
    stay = torch.zeros(batch, dtype=torch.bool)
    stay[torch.randperm(batch, generator=torch.Generator().manual_seed(55))[:100]] = True
    forced[~stay] = 1
    _, exits, L, conf, hidden = run.step(tokens, lens.long(), 2.0, forced=forced, heads=2)
    assert L == cfg.n_layers and torch.equal(exits, forced)
    assert not want_conf[:2].isnan().any()
    assert torch.equal(conf[0], want_conf[0]) and torch.equal(conf[1, stay], want_conf[1, stay])
    assert torch.equal(hidden[stay], want[stay])


@pytest.mark.parametrize("tiles,batch", [(772, 256), (776, 130), (1036, 200), (1028, 161)])   # 256 x 128 blocks; 256 x 192, the last one of four or two tiles
def test_compacted_gate_up_in_blocks_of_256_rows(tiles, batch):
    """Gate/up of up to 256 rows with exits of their own in one row block: more than 128 rows active, exactly 128 and fewer (the upper
    half is left out), one, none.  (Weights of the usual 0.05: with 0.03 the three largest logits of one prompt lay within 4e-4 of each
    other, where the arithmetic allows 4e-3, and the comparison knows ties of two only.)"""
    cfg = small_bf16(n_layers=6, d_model=128, n_heads=1, d_ffn=16 * tiles, prompt_len=2, min_prompt_len=1, shuffled_blocks=True, batch=batch)
    forced = torch.full((2, batch), 3, dtype=torch.int32)
    forced[:, torch.randperm(batch, generator=torch.Generator().manual_seed(6))[:batch - 128]] = 2
    forced[:, 0] = 1
    forced[0, batch - 1] = 6      # one sequence runs every layer, or leaves before the last
    forced[1, batch - 1] = 5
    stats = lockstep(cfg, seed=51, steps=2, forced_seq=forced, heads=2)
    assert stats["L"] == [6, 5]


@pytest.mark.parametrize("heads", [0, 2])
def test_token_of_a_sequence_of_nan_among_compacted_rows(heads):
    """A sequence whose embedding is NaN among 200 (two row chunks; with exits of their own the rows are compacted): its
    token stays inside the vocabulary and the others' tokens are those of the batch without it."""
    cfg = compactable_bf16(batch=200).with_(n_layers=3)
    w = W.make_weights(cfg, seed=46, gain_jitter=0.1)
    w["embed"][7] = float("nan")
    lens = torch.full((200,), 3, dtype=torch.int32)
    run = HipRun(cfg, w, lens, 2, seed=46)
    tokens = torch.arange(200, dtype=torch.int32) + 8
    forced = torch.arange(200) % 2 + 2 if heads else None
    want = run.step(tokens, lens.long(), 2.0, forced=forced, heads=heads)[0]
    tokens[150] = 7
    got = run.step(tokens, lens.long(), 2.0, forced=forced, heads=heads)[0]
    assert 0 <= int(got[150]) < cfg.vocab
    keep = torch.arange(200) != 150
    assert torch.equal(got[keep], want[keep])


@pytest.mark.parametrize("dtype", ["fp32", "bf16"])
def test_tokens_of_sequences_accepted_before_the_batch_leaves(dtype):
    """Algorithm 1 takes every token from the hidden state at output_layer.  5000 sequences (more than the chip holds in one
    round of the launch that takes a decision), all accepted at layer 1 but the first, whose acceptance at layer 2 ends
    the iteration while later rows' workgroups have not started: their tokens are those of a batch accepted at layer 2."""
    base = TINY if dtype == "fp32" else L7B
    cfg = W.reduced(base, n_layers=3, d_model=128, n_heads=2, head_dim=64, d_ffn=128, vocab=256, batch=5000, prompt_len=1,
                    min_prompt_len=1, weight_std=0.1, tied_head=False)
    lens = torch.ones(5000, dtype=torch.int32)
    run = HipRun(cfg, W.make_weights(cfg, seed=49, gain_jitter=0.1), lens, 1, seed=49)
    tokens = torch.randint(0, 256, (5000,), generator=torch.Generator().manual_seed(49), dtype=torch.int32)
    got = {}
    for name, first, others in (("1", 1, 1), ("2", 2, 2), ("first at 2", 2, 1)):
        forced = torch.full((5000,), others, dtype=torch.int32)
        forced[0] = first
        tok, exits, L, _, _ = run.step(tokens, lens.long(), 2.0, forced=forced)
        assert torch.equal(exits, forced) and L == first
        got[name] = tok
    assert (got["1"] != got["2"]).sum() > 1000, "the two layers have to disagree for the comparison to say anything"
    assert torch.equal(got["first at 2"], got["2"])


def test_prompt_chunk_beside_a_sequence_of_nan():
    """A chunk of three prompts, the tokens of one embedded as NaN: the rows of the others, in the same groups of rows, end
    with the hidden states they have without it, to the rounding of a bf16 layer."""
    cfg = small_bf16(n_layers=2, batch=3, prompt_len=20, min_prompt_len=20)
    w = W.make_weights(cfg, seed=48, gain_jitter=0.1)
    w["embed"][7] = float("nan")
    run = HipRun(cfg, w, torch.full((3,), 20, dtype=torch.int32), 1, seed=48)
    ws = B.Workspace(run.model.desc, 60, 21)
    seq = torch.arange(3, dtype=torch.int32).repeat_interleave(20).cuda()
    pos = torch.arange(20, dtype=torch.int32).repeat(3).cuda()
    tokens = torch.randint(8, cfg.vocab, (60,), generator=torch.Generator().manual_seed(48), dtype=torch.int32).cuda()
    z = lambda *n: torch.zeros(*n, dtype=torch.int32, device="cuda")  # noqa: E731
    got = []
    for nan in (False, True):
        if nan:
            tokens[20:40] = 7
        hidden = torch.zeros(60, cfg.d_model, device="cuda")
        batch = B.make_batch(tokens, pos, run.bt_dev, 21, row_table=seq)
        B.ee_decode_iteration(run.model, run.cache, batch, 2.0, None, B.EE_EXIT_NONE, z(60), z(60), z(1), None, hidden, ws)
        torch.cuda.synchronize()
        got.append(torch.cat([hidden[:20], hidden[40:]]).cpu())
    assert torch.isfinite(got[1]).all()
    assert ((got[1] - got[0]).norm(dim=1) <= 2e-2 * got[0].norm(dim=1)).all()


@pytest.mark.parametrize("batch,d_model", [(1, 256), (64, 256), (65, 256), (9, 512), (9, 576)])
@pytest.mark.parametrize("heads,exit_every", [(1, 1), (2, 2)])
def test_float_exit_decision_inside_the_next_projection(batch, d_model, heads, exit_every):
    """Float models: up to 64 rows of a width up to 512 the decision of a layer is taken by leading workgroups of the next layer's
    QKV launch, beyond in a launch of its own; checks after every layer and after every other one, decided by the confidences (the
    batch as a whole stays to the last layer)."""
    cfg = TINY.with_(batch=batch, d_model=d_model, n_heads=d_model // 64, d_ffn=320, vocab=514, prompt_len=7, min_prompt_len=5, decode_steps=2,
                     weight_std=0.05, logit_scale=1.0, threshold=0.3, exit_every=exit_every)
    lockstep(cfg, seed=81 + batch, steps=2, heads=heads)


@pytest.mark.parametrize("batch,d_model", [(1, 256), (64, 256), (65, 256), (17, 512), (9, 576)])
@pytest.mark.parametrize("heads", [1, 2])
def test_float_batch_that_leaves_inside_the_next_projection(batch, d_model, heads):
    """The same launch when the decision in it ends the iteration: the whole batch leaves at layer 1, in the middle, before the last
    layer, or one by one, the last row early.  The projection behind the decision still runs and caches what KV filling then finds
    cached; everything after it is empty."""
    cfg = TINY.with_(batch=batch, n_layers=5, d_model=d_model, n_heads=d_model // 64, d_ffn=320, vocab=514, prompt_len=7, min_prompt_len=5,
                     decode_steps=4, weight_std=0.05, logit_scale=1.0)
    forced = torch.empty(4, batch, dtype=torch.int32)
    forced[0], forced[1], forced[2] = 1, 3, cfg.n_layers - 1
    forced[3] = torch.arange(batch, 0, -1) % (cfg.n_layers - 1) + 1
    forced[3, 0] = 4
    forced[3, batch - 1] = 2 if batch > 1 else 4
    stats = lockstep(cfg, seed=84 + batch, steps=4, forced_seq=forced, heads=heads)
    assert stats["L"] == [1, 3, 4, 4]


@pytest.mark.parametrize("batch", [2, 31, 32, 33, 63, 64, 65, 97])
def test_rows_that_no_sequence_has(batch):
    """Batches that leave a 32-row tile nearly empty or nearly full, one to four tiles: lanes of missing rows fetch another row's
    operand, and what they compute reaches nothing."""
    cfg = small_bf16(batch=batch, d_model=512, n_heads=4, d_ffn=1056, prompt_len=4, min_prompt_len=3, threshold=0.4)
    lockstep(cfg, seed=90, steps=2, heads=2)


@pytest.mark.parametrize("heads", [1, 2])
def test_batch_of_one_and_prompts_ending_on_block_boundaries(heads):
    """Degenerate sizes: a single sequence, and prompts whose next position opens a new 16-token block."""
    lockstep(small_bf16(batch=1, prompt_len=16, min_prompt_len=16, threshold=0.4), seed=61, steps=3, heads=heads)
    lockstep(small_bf16(batch=3, prompt_len=15, min_prompt_len=15, threshold=0.4), seed=62, steps=3, heads=heads)
    lockstep(TINY.with_(batch=1, prompt_len=31, min_prompt_len=31, decode_steps=3), seed=63, steps=3, heads=heads)


def test_sixty_four_layers_the_most_the_library_takes():
    """EE_MAX_LAYERS layers: the per-layer tables of the KV-filling launch are full; exits spread over the depth."""
    cfg = small_bf16(n_layers=64, d_model=128, n_heads=1, head_dim=128, d_ffn=128, vocab=256, batch=3, prompt_len=6,
                     min_prompt_len=6, weight_std=0.03, logit_scale=0.05, threshold=0.5)
    stats = lockstep(cfg, seed=71, steps=2, check_untouched=False)
    assert all(1 <= L <= 64 for L in stats["L"])
