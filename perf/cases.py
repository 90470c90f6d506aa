"""Performance cases: the calls a program built on this library makes, over the sizes it makes them at.

    listed()             the named cases
    draw(rng)            one more case of the same ranges
    prepare(case, seed)  model, cache, batch and buffers in GPU memory: what a serving program holds before the call
    run(state)           one call of the public entry point and its outputs
    work(case)           bytes and operations no implementation of the call can do without
    tolerance(case)      how far two correct implementations of the same precision may be apart
    exact(case, seed)    the same outputs from plain torch in float64

A case names its entry point in "op":
    iteration   ee_decode_iteration on one token per sequence
    prompt      ee_decode_iteration on a chunk of prompt positions (rows that share block tables, no exit checks)
    check       ee_exit_check
    fill        ee_kv_fill
    attention   ee_paged_attention_decode on one token per sequence
    attention_prompt   ee_paged_attention_decode on a chunk of prompt positions

Models are the repository's own shapes at full width and reduced depth (the layers are alike, so a few of them stand for
all), or narrow ones.  Two things differ from weights drawn independently.  The embedding has unit variance, and the
LM-head row of a token's successor is correlated with the token's embedding: a trained head prefers one token, and an
iteration's tokens then do not hang on the last bit of a near tie.  Exits are forced layer by layer (the library's own
synthetic confidence injection), so that which layers run does not hang on a confidence beside a threshold either.
"""
import math
import random

import torch

from paper_2407_20272_amd import binding as B
from paper_2407_20272_amd import workloads as W

DEVICE = "cuda"
SHAPES = {"tiny_fp32": W.CONFIGS[0], "7b": W.CONFIGS[1], "13b": W.CONFIGS[4]}
ALIGN = 0.5   # correlation of a successor's LM-head row with the token's embedding


# ----------------------------------------------------------------------------------------------------------------
# the cases
# ----------------------------------------------------------------------------------------------------------------
def listed():
    return [
        # The reference-sized float model: four layers, four sequences, an exit check after every layer and one layer left
        # to the KV filling.  The smallest call there is: nothing but launches and their latency.
        dict(name="iteration_tiny_fp32_b4", op="iteration", shape="tiny_fp32", layers=4, batch=4, ctx_min=32, ctx_max=32,
             rule="batch", exits="3", conf_mode=0, shuffled=False),
        # One user's conversation on the 7B shape, full layers: weights streamed for a single row.
        dict(name="iteration_7b_b1", op="iteration", shape="7b", layers=2, batch=1, ctx_min=1000, ctx_max=1000, rule="none",
             exits="", conf_mode=0, shuffled=False),
        # The headline workload: batch 32, contexts of 512 and some decoded tokens, Algorithm 1 with a check after every
        # layer; the batch leaves after layer 3 and the KV of layer 4 is filled.
        dict(name="iteration_7b_b32", op="iteration", shape="7b", layers=4, batch=32, ctx_min=512, ctx_max=640, rule="batch",
             exits="3", conf_mode=0, shuffled=False),
        # A 13B model with the similarity measure, whose checks need no LM head and never fire here.
        dict(name="iteration_13b_b64", op="iteration", shape="13b", layers=2, batch=64, ctx_min=1024, ctx_max=1024,
             rule="batch", exits="", conf_mode=2, shuffled=False),
        # A large ragged batch over a fragmented cache, every sequence leaving at its own layer.
        dict(name="iteration_7b_b256_per_sequence", op="iteration", shape="7b", layers=4, batch=256, ctx_min=128,
             ctx_max=1024, rule="per_sequence", exits="1-4", conf_mode=0, shuffled=True),
        # A prompt chunk as the scheduler cuts it: 512 rows of four prompts that are at different places.
        dict(name="prompt_7b_512_rows", op="prompt", shape="7b", layers=2, rows=512, sequences=4, ctx_min=0, ctx_max=1000,
             shuffled=True),
        # The exit check of a layer in the middle of the model, at the headline batch and at a large odd one.
        dict(name="check_7b_b32", op="check", shape="7b", layer=16, batch=32, conf_mode=0),
        dict(name="check_7b_b500", op="check", shape="7b", layer=16, batch=500, conf_mode=1),
        # KV filling after an early exit: eight of twelve layers.
        dict(name="fill_7b_b32", op="fill", shape="7b", layers=12, batch=32, ctx_min=512, ctx_max=640, fill_from=4,
             shuffled=False),
        # Attention of a single long conversation; of a long-context batch (the most memory traffic); of a prompt chunk.
        dict(name="attention_7b_b1_ctx16k", op="attention", shape="7b", batch=1, ctx_min=16383, ctx_max=16383, shuffled=False),
        dict(name="attention_13b_b64_ctx4k", op="attention", shape="13b", batch=64, ctx_min=4000, ctx_max=4159,
             shuffled=True),
        dict(name="attention_prompt_7b_512_rows", op="attention_prompt", shape="7b", rows=512, sequences=4, ctx_min=0,
             ctx_max=3000, shuffled=True),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi + 0.49)))))))


def draw(rng):
    op = rng.choice(["iteration"] * 6 + ["prompt"] * 3 + ["check"] * 2 + ["fill", "attention", "attention", "attention_prompt"])
    shape = rng.choice(["7b"] * 6 + ["13b"] * 3 + ["narrow"] * 2 + (["tiny_fp32"] if op in ("iteration", "check") else []))
    case = dict(op=op, shape=shape)
    if shape == "narrow":   # a narrow model in bf16, sizes off the powers of two
        dh = rng.choice([64, 128])
        case.update(head_dim=dh, n_heads=rng.randint(3, 2048 // dh), d_ffn=16 * rng.randint(30, 380), vocab=32 * rng.randint(40, 1000))
    cfg = _cfg(case)
    kv_token = 2 * cfg.d_model * (4 if cfg.dtype == "fp32" else 2)
    big = 64 if shape == "tiny_fp32" else 256 if shape == "13b" else 512
    if op in ("iteration", "prompt"):
        case["layers"] = 4 if shape == "tiny_fp32" else rng.randint(1, 2 if shape == "13b" else 3)
    if op in ("prompt", "attention_prompt"):
        case["sequences"] = rng.randint(1, 12)
        case["rows"] = _log_int(rng, max(16, case["sequences"]), 512)
        case["ctx_min"] = 0
        case["ctx_max"] = _log_int(rng, 16, 3000 if op == "attention_prompt" else 1500)
        case["shuffled"] = rng.random() < 0.5
        return case
    case["batch"] = _log_int(rng, 1, big)
    if op == "check":
        case.update(layer=rng.randint(1, cfg.n_layers - 1), conf_mode=rng.choice([0, 0, 1]))
        return case
    if op == "fill":
        case["layers"] = rng.randint(2, 12)
        case["fill_from"] = rng.randint(max(0, case["layers"] - 8), case["layers"] - 1)
    case["shuffled"] = rng.random() < 0.5
    # contexts: ragged or equal, up to what the largest listed case reads
    room = (4e9 if op == "attention" else 1.5e9) / (kv_token * case["batch"])
    top = 200 if shape == "tiny_fp32" else int(max(16, min(room, 16384 if op == "attention" else 2048)))
    case["ctx_max"] = _log_int(rng, min(16, top), top)
    case["ctx_min"] = rng.choice([case["ctx_max"], case["ctx_max"] // 2, case["ctx_max"] // 16])
    if op == "iteration":
        n = case["layers"]
        case["rule"] = rng.choice(["none", "none", "batch", "batch", "per_sequence"])
        case["conf_mode"] = rng.choice([0, 0, 1, 2, 3])
        case["exits"] = "" if case["rule"] == "none" else rng.choice(["", "1-%d" % n, str(rng.randint(1, n))])
    return case


# ----------------------------------------------------------------------------------------------------------------
# what a case says about sizes (the same for every seed)
# ----------------------------------------------------------------------------------------------------------------
def _cfg(case):
    if case["shape"] == "narrow":
        dh, h = case["head_dim"], case["n_heads"]
        cfg = W.reduced(SHAPES["7b"], d_model=h * dh, n_heads=h, head_dim=dh, d_ffn=case["d_ffn"], vocab=case["vocab"])
    else:
        cfg = SHAPES[case["shape"]]
    n = case.get("layers", cfg.n_layers)
    return cfg.with_(n_layers=n, exit_every=1, conf_mode=case.get("conf_mode", 0), tied_head=False)


def _spread(lo, hi, n, key):
    """n whole numbers over [lo, hi], ends included, in a fixed scrambled order."""
    v = [lo + (hi - lo) * i // max(n - 1, 1) for i in range(n)]
    random.Random(key).shuffle(v)
    return v


def _rows(case):
    """(row_table or None, positions): the sequence and position of every batch row."""
    if "rows" not in case:
        return None, _spread(case["ctx_min"], case["ctx_max"], case["batch"], 1)
    S, R = case["sequences"], case["rows"]
    begin = _spread(case["ctx_min"], case["ctx_max"], S, 2)
    table, pos = [], []
    for s in range(S):
        n = R // S + (1 if s < R % S else 0)
        table += [s] * n
        pos += list(range(begin[s], begin[s] + n))
    return table, pos


def _tables(case):
    """(block table rows, number of blocks, number of written blocks).  The blocks that hold a row's own position come
    first in the pool, so that what a call caches is the head of every layer's pool."""
    table, pos = _rows(case)
    seq = table if table is not None else list(range(len(pos)))
    S = max(seq) + 1
    last = [0] * S
    written = [set() for _ in range(S)]
    for s, p in zip(seq, pos):
        last[s] = max(last[s], p)
        written[s].add(p // 16)
    n_written = sum(len(w) for w in written)
    rest = list(range(n_written, sum(l // 16 + 1 for l in last)))
    if case["shuffled"]:
        random.Random(3).shuffle(rest)
    rows, w, r = [], 0, 0
    for s in range(S):
        row = []
        for lb in range(last[s] // 16 + 1):
            if lb in written[s]:
                row.append(w)
                w += 1
            else:
                row.append(rest[r])
                r += 1
        rows.append(row)
    width = max(len(r) for r in rows)
    return [r + [-1] * (width - len(r)) for r in rows], n_written + len(rest), n_written


def _exits(case):
    """Forced exit layers (a layer past the last check never exits), or None: no check fires."""
    spec = case.get("exits", "")
    if not spec:
        return None
    lo, hi = (spec.split("-") + [spec])[:2]
    return _spread(int(lo), int(hi), case["batch"], 4)


def _layers_run(case):
    """(layers that run, [rows that attend in each], checks made)."""
    n, M = case["layers"], len(_rows(case)[1])
    ex = _exits(case) if case.get("rule", "none") != "none" else None
    if ex is None:
        return n, [M] * n, (n - 1 if case.get("rule", "none") != "none" else 0)
    L = max(ex) if max(ex) < n else n
    att = [sum(1 for e in ex if e >= i) if case["rule"] == "per_sequence" else M for i in range(1, L + 1)]
    return L, att, min(L, n - 1)


# ----------------------------------------------------------------------------------------------------------------
# inputs
# ----------------------------------------------------------------------------------------------------------------
def _gen(seed, *key):
    g = torch.Generator(device=DEVICE)
    g.manual_seed(random.Random(repr((seed,) + key)).getrandbits(62))
    return g


def _randn(shape, std, dtype, seed, *key):
    return torch.randn(shape, generator=_gen(seed, *key), device=DEVICE, dtype=torch.float32).mul_(std).to(dtype)


def _weights(case, seed, parts):
    """Plain weights of the parts a call reads ("layers", "qkv", "head"); the others are stubs, never read."""
    cfg = _cfg(case)
    d, f, V, dt, std = cfg.d_model, cfg.d_ffn, cfg.vocab, cfg.torch_dtype, cfg.weight_std
    stub = torch.zeros(32, 16, dtype=dt, device=DEVICE)

    def gain(*key):
        return (1.0 + 0.1 * torch.randn(d, generator=_gen(seed, *key), device=DEVICE)).to(dt)

    w = {"embed": stub, "w_lm": stub, "g_final": gain("g_final"), "layers": []}
    if "head" in parts:
        w["embed"] = _randn((V, d), 1.0, dt, seed, "embed")
        prev = torch.randperm(V, generator=_gen(seed, "successor"), device=DEVICE)
        noise = torch.randn((V, d), generator=_gen(seed, "w_lm"), device=DEVICE)
        w["w_lm"] = (noise.mul_(std * math.sqrt(1 - ALIGN ** 2)).add_(w["embed"].float()[prev], alpha=std * ALIGN)).to(dt)
    for i in range(cfg.n_layers):
        lw = {"g_attn": gain("g_attn", i), "g_ffn": gain("g_ffn", i)}
        for name, shape, part in (("w_q", (d, d), "qkv"), ("w_k", (d, d), "qkv"), ("w_v", (d, d), "qkv"), ("w_o", (d, d), "layers"),
                                  ("w_gate", (f, d), "layers"), ("w_up", (f, d), "layers"), ("w_down", (d, f), "layers")):
            lw[name] = _randn(shape, std, dt, seed, name, i) if part in parts else None
        w["layers"].append(lw)
    w["w_cls"] = _randn((cfg.n_layers, d), 1.5 / d ** 0.5, torch.float32, seed, "w_cls")
    w["b_cls"] = torch.linspace(-2.0, 2.0, cfg.n_layers, device=DEVICE)
    return w


def _stubbed(case, w):
    """The weights with stand-ins of the smallest packable size where a call reads none."""
    cfg = _cfg(case)
    dt = cfg.torch_dtype
    small = {"w_q": (2 * cfg.head_dim, 16), "w_k": (2 * cfg.head_dim, 16), "w_v": (2 * cfg.head_dim, 16), "w_o": (32, 16),
             "w_gate": (cfg.d_ffn, 16), "w_up": (cfg.d_ffn, 16), "w_down": (32, 16)}
    one = {k: torch.zeros(s, dtype=dt, device=DEVICE) for k, s in small.items()}
    return dict(w, layers=[{k: (v if v is not None else one[k]) for k, v in lw.items()} for lw in w["layers"]])


PARTS = {"iteration": ("layers", "qkv", "head"), "prompt": ("layers", "qkv", "head"), "check": ("lm",), "fill": ("qkv",)}


def _inputs(case, seed):
    """Everything random a call reads besides the weights, on the device."""
    cfg, op = _cfg(case), case["op"]
    d, s = cfg.d_model, {}
    if op == "check":
        s["hidden"] = _randn((case["batch"], d), 2.0, torch.float32, seed, "hidden")
        return s
    table, pos = _rows(case)
    rows, blocks, written = _tables(case)
    n_layers = 1 if op.startswith("attention") else cfg.n_layers
    shape = (n_layers, blocks, cfg.n_heads, 16, cfg.head_dim)
    for name in ("k", "v"):
        s[name] = torch.empty(shape, dtype=cfg.torch_dtype, device=DEVICE)
        s[name].normal_(0.0, 1.0, generator=_gen(seed, "pool", name))
    if op == "fill":   # a fill writes the new position of every sequence and reads no cache
        s["hidden"] = _randn((len(pos), d), 2.0, torch.float32, seed, "hidden")
    elif op.startswith("attention"):
        s["q"] = _randn((len(pos), cfg.n_heads, cfg.head_dim), 1.3, torch.float32, seed, "q")
    else:
        s["tokens"] = torch.randint(0, cfg.vocab, (len(pos),), generator=_gen(seed, "tokens"), device=DEVICE, dtype=torch.int32)
    s["pos"] = torch.tensor(pos, dtype=torch.int32, device=DEVICE)
    s["tables"] = torch.tensor(rows, dtype=torch.int32, device=DEVICE)
    s["row_table"] = None if table is None else torch.tensor(table, dtype=torch.int32, device=DEVICE)
    s["written"] = written
    return s


def _check_weights(case, seed):
    """Exit checks read the LM head and the final gain only; independent rows (confidences spread over (0, 1))."""
    cfg = _cfg(case)
    w = _weights(case, seed, ())
    w["w_lm"] = _randn((cfg.vocab, cfg.d_model), cfg.weight_std, cfg.torch_dtype, seed, "w_lm")
    return w


def prepare(case, seed):
    cfg, op = _cfg(case), case["op"]
    s = _inputs(case, seed)
    s["op"] = op
    if op.startswith("attention"):
        s["desc"] = B.make_desc(cfg.with_(n_layers=1))
    else:
        w = _check_weights(case, seed) if op == "check" else _weights(case, seed, PARTS[op])
        s["model"] = B.DeviceModel(cfg, _stubbed(case, w))
        s["desc"] = s["model"].desc
        del w
    M = case["batch"] if op == "check" else len(s["pos"])
    if op != "check":
        cache = B.PagedKV.__new__(B.PagedKV)
        cache.cfg, cache.num_blocks, cache.k, cache.v = cfg, s["k"].shape[1], s["k"], s["v"]
        cache.c = B.ee_kv_cache(s["k"].data_ptr(), s["v"].data_ptr(), cache.num_blocks, 16)
        s["cache"] = cache
        top = int(max(_rows(case)[1])) + 1
        s["batch"] = B.make_batch(s.get("tokens"), s["pos"], s["tables"], top, s["row_table"])
    s["ws"] = B.Workspace(s["desc"], M, 1 if op == "check" else top)
    z = lambda *shape: torch.zeros(*shape, dtype=torch.int32, device=DEVICE)  # noqa: E731
    if op == "check":
        s.update(layer=case["layer"], status=z(M), exit_layer=z(M), n_exited=z(1), done=z(1), L=z(1), argmax=z(M),
                 conf=torch.zeros(M, device=DEVICE))
    elif op in ("iteration", "prompt"):
        rule = case.get("rule", "none")
        ex = _exits(case) if rule != "none" else None
        s.update(rule={"none": 0, "batch": 1, "per_sequence": 2}[rule],
                 forced=None if ex is None else torch.tensor(ex, dtype=torch.int32, device=DEVICE),
                 out_tokens=z(M), out_exit=z(M), out_L=z(1), conf=torch.zeros(cfg.n_layers, M, device=DEVICE),
                 hidden=torch.zeros(M, cfg.d_model, device=DEVICE))
    elif op == "fill":
        s["fill_from"] = torch.full((M,), case["fill_from"], dtype=torch.int32, device=DEVICE)
    else:
        s["out"] = torch.zeros(M, cfg.n_heads, cfg.head_dim, device=DEVICE)
    return s


def run(s):
    op = s["op"]
    if op == "check":   # no confidence exceeds the threshold: nobody has left yet, every row is checked
        B.ee_exit_check(s["model"], s["layer"], s["hidden"], 2.0, None, s["status"], s["exit_layer"], s["n_exited"], s["done"],
                        s["L"], s["argmax"], s["conf"], s["ws"])
        return {"argmax": s["argmax"], "conf": s["conf"], "status": s["status"]}
    if op == "fill":
        B.ee_kv_fill(s["model"], s["cache"], s["batch"], s["hidden"], s["fill_from"], s["ws"])
        return {"k": s["k"][:, :s["written"]], "v": s["v"][:, :s["written"]]}
    if op.startswith("attention"):
        B.ee_paged_attention_decode(s["desc"], s["cache"], 1, s["q"], s["batch"], s["out"], s["ws"])
        return s["out"]
    B.ee_decode_iteration(s["model"], s["cache"], s["batch"], 2.0, s["forced"], s["rule"], s["out_tokens"], s["out_exit"],
                          s["out_L"], s["conf"], s["hidden"], s["ws"])
    return {"tokens": s["out_tokens"], "exit_layer": s["out_exit"], "batch_exit_layer": s["out_L"], "conf": s["conf"],
            "hidden": s["hidden"], "k": s["k"][:, :s["written"]], "v": s["v"][:, :s["written"]]}


# ----------------------------------------------------------------------------------------------------------------
# what a pass cannot do without
# ----------------------------------------------------------------------------------------------------------------
def work(case):
    cfg, op = _cfg(case), case["op"]
    d, f, V, e = cfg.d_model, cfg.d_ffn, cfg.vocab, 4 if cfg.dtype == "fp32" else 2
    if op == "check":
        M = case["batch"]
        return {"bytes": V * d * e + d * e + M * d * 4 + M * 12, "flops": 2 * M * V * d}
    table, pos = _rows(case)
    M = len(pos)
    kv = 2 * d * e                                   # one position's K and V of one layer
    if op == "fill":
        n = case["layers"] - case["fill_from"]
        return {"bytes": n * (2 * d * d * e + M * kv) + M * d * 4, "flops": n * 2 * M * 2 * d * d}
    if table is None:
        cached = sum(p + 1 for p in pos)             # positions read: each sequence's own
    else:
        cached = sum(max(p for t, p in zip(table, pos) if t == s) + 1 for s in set(table))   # each sequence's once
    att_flops = sum(4 * d * (p + 1) for p in pos)
    if op.startswith("attention"):
        return {"bytes": cached * kv + 2 * M * d * 4, "flops": att_flops}
    n = case["layers"]
    L, att, checks = _layers_run(case)
    layer = (4 * d * d + 3 * d * f) * e
    heads = checks if case.get("conf_mode", 0) < 2 else 0
    # one more pass of the head picks the tokens unless the batch left at a check that has one
    heads += 0 if L < n and case.get("conf_mode", 0) < 2 else 1
    share = [a / M for a in att]
    nbytes = L * (layer + M * kv) + sum(share) * cached * kv + heads * V * d * e + (n - L) * (2 * d * d * e + M * kv) + 2 * M * d * 4
    flops = sum(2 * a * (4 * d * d + 3 * d * f) for a in att) + sum(share) * att_flops + heads * 2 * M * V * d + (n - L) * 4 * M * d * d
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    """About four times the distance to float64 measured on the library's first form of each path."""
    if case["shape"] == "tiny_fp32":
        return {"rel": 1e-5}          # float throughout: 1e-7 measured
    if case["op"].startswith("attention"):
        return {"rel": 2e-5}          # float scores, softmax and sums over a bf16 cache: 3e-7 (prompt rows: 3e-6)
    if case["op"] == "fill":
        return {"rel": 2.5e-3}        # one bf16 operand and the bf16 store: 6e-4
    # bf16 operands through whole layers: hidden states 4e-3 to 5e-3, confidences up to 1e-2 (the softmax of logits scaled
    # by up to 15); whole numbers (tokens, arg max) keep a margin, a tie among a few hundred rows may fall the other way
    return {"rel": 0.02, "differ": 0.005}


# ----------------------------------------------------------------------------------------------------------------
# float64 reference
# ----------------------------------------------------------------------------------------------------------------
def _norm(x, g, eps):
    return x * torch.rsqrt(x.square().mean(-1, keepdim=True) + eps) * g.double()


def _rope(x, pos, theta):
    """x [M][H][dh]: channels (j, j + dh/2) turned by pos * theta^(-2j/dh)."""
    half = x.shape[-1] // 2
    ang = pos.double()[:, None] * theta ** (-torch.arange(half, device=x.device, dtype=torch.float64) / half)
    c, s = ang.cos()[:, None], ang.sin()[:, None]
    lo, hi = x[..., :half], x[..., half:]
    return torch.cat([lo * c - hi * s, hi * c + lo * s], -1)


def _attend(q, k_pool, v_pool, pos, tables, row_table):
    """q [M][H][dh] double; every row attends positions 0..its own of its sequence."""
    M, H, dh = q.shape
    out = torch.empty_like(q)
    seq = torch.arange(M, device=q.device) if row_table is None else row_table.long()
    where, at = seq.tolist(), pos.tolist()
    for s in sorted(set(where)):
        rows = torch.tensor([m for m in range(M) if where[m] == s], device=q.device)
        top = max(at[m] for m in rows.tolist()) + 1
        blocks = tables[s, :(top + 15) // 16].long()
        K = k_pool[blocks].double().permute(1, 0, 2, 3).reshape(H, -1, dh)[:, :top]
        V = v_pool[blocks].double().permute(1, 0, 2, 3).reshape(H, -1, dh)[:, :top]
        z = torch.matmul(q[rows].permute(1, 0, 2), K.transpose(1, 2).contiguous()) / math.sqrt(dh)
        z.masked_fill_((torch.arange(top, device=q.device)[None, :] > pos[rows].long()[:, None])[None], -math.inf)
        out[rows] = torch.matmul(z.softmax(-1), V).permute(1, 0, 2)
    return out


def _put(pool, x, pos, tables, row_table):
    """pool [blocks][H][16][dh] takes x [M][H][dh] at every row's position."""
    seq = torch.arange(len(pos), device=x.device) if row_table is None else row_table.long()
    p = pos.long()
    pool[tables[seq, p // 16].long(), :, p % 16] = x


def _head(x, w, cfg):
    return _norm(x, w["g_final"], cfg.rms_eps) @ w["w_lm"].double().T


def _confidence(z, mode):
    p = z.softmax(-1).topk(2, -1).values
    return p[:, 0] if mode == 0 else p[:, 0] - p[:, 1]


def exact(case, seed):
    cfg, op = _cfg(case), case["op"]
    s = _inputs(case, seed)
    if op.startswith("attention"):
        return _attend(s["q"].double(), s["k"][0], s["v"][0], s["pos"], s["tables"], s["row_table"])
    if op == "check":
        z = _head(s["hidden"].double(), _check_weights(case, seed), cfg)
        return {"argmax": None, "conf": _confidence(z * (cfg.logit_scale * case["layer"]), case["conf_mode"]), "status": None}
    w = _weights(case, seed, PARTS[op])
    H, dh, d, eps = cfg.n_heads, cfg.head_dim, cfg.d_model, cfg.rms_eps
    pos, tables, rt, W_ = s["pos"], s["tables"], s["row_table"], s["written"]
    M = len(pos)
    k, v = s["k"][:, :W_].double(), s["v"][:, :W_].double()   # what the call writes, in float64

    def cache_kv(i, x):
        lw = w["layers"][i]
        K = _rope((x @ lw["w_k"].double().T).view(M, H, dh), pos, cfg.rope_theta)
        V = (x @ lw["w_v"].double().T).view(M, H, dh)
        _put(k[i], K, pos, tables, rt)
        _put(v[i], V, pos, tables, rt)

    if op == "fill":
        h = s["hidden"].double()
        for i in range(case["fill_from"], cfg.n_layers):
            cache_kv(i, _norm(h, w["layers"][i]["g_attn"], eps))
        return {"k": k, "v": v}

    n, rule, mode = cfg.n_layers, case.get("rule", "none"), case.get("conf_mode", 0)
    ex = _exits(case) if rule != "none" else None
    status = torch.zeros(M, dtype=torch.bool, device=DEVICE)
    conf = torch.full((n, M), math.nan, dtype=torch.float64, device=DEVICE)
    h = w["embed"][s["tokens"].long()].double()
    L = n
    for i in range(n):
        lw = w["layers"][i]
        frozen = status.clone() if rule == "per_sequence" else torch.zeros_like(status)
        x = _norm(h, lw["g_attn"], eps)
        cache_kv(i, x)
        q = _rope((x @ lw["w_q"].double().T).view(M, H, dh), pos, cfg.rope_theta)
        kp, vp = s["k"][i].double(), s["v"][i].double()
        kp[:W_], vp[:W_] = k[i], v[i]
        a = _attend(q, kp, vp, pos, tables, rt).view(M, d)
        del kp, vp
        h1 = h + a @ lw["w_o"].double().T
        x = _norm(h1, lw["g_ffn"], eps)
        h1 = h1 + (torch.nn.functional.silu(x @ lw["w_gate"].double().T) * (x @ lw["w_up"].double().T)) @ lw["w_down"].double().T
        prev, h = h, torch.where(frozen[:, None], h, h1)
        if rule != "none" and i + 1 < n:
            if mode < 2:
                c = _confidence(_head(h, w, cfg) * (cfg.logit_scale * (i + 1)), mode)
            elif mode == 2:
                c = torch.nn.functional.cosine_similarity(prev, h, dim=-1)
            else:
                c = torch.sigmoid(_norm(h, torch.ones(d, device=DEVICE), eps) @ w["w_cls"][i].double() + w["b_cls"][i].double())
            conf[i] = torch.where(status, conf[i], c)
            if ex is not None:
                status |= torch.tensor([e <= i + 1 for e in ex], device=DEVICE)
            if bool(status.all()):
                L = i + 1
                break
    for i in range(L, n):
        cache_kv(i, _norm(h, w["layers"][i]["g_attn"], eps))
    return {"tokens": None, "exit_layer": None, "batch_exit_layer": None, "conf": conf, "hidden": h, "k": k, "v": v}
