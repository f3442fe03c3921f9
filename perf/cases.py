"""The workloads by which this framework's speed is judged.

One case is one call that a serving loop makes on one layer: decode over a
paged batch, a chunked-prefill step, writing a step's new K/V rows, or moving
blocks out of the elastic id range in every layer. Shapes are those of the
framework's own workloads and tests (32 query heads over 8 kv heads with
head_dim 128; 64 over 8; head_dim 64; the tiny fp32 batch). The pool's commit
and decommit are driver calls with no kernel of this framework in them; the
benchmark times those.
"""
import math
import random

import torch

import paper_2608_23658_amd.kvattn as K

BS = 16                                  # tokens per block, the only size built
ESZ = {"bf16": 2, "f32": 4}
TORCH = {"bf16": torch.bfloat16, "f32": torch.float32}


def listed():
    return [
        # One user's decode step: the smallest call of an interactive session,
        # where latency and idle CUs count. Odd length.
        dict(name="decode_single", op="decode", dtype="bf16", hq=32, hkv=8, d=128,
             batch=1, lo=3971, hi=3971, len_seed=1),
        # A few users with ragged contexts, head_dim 64 and 8 query heads per
        # kv head, through the entry point for captured graphs.
        dict(name="decode_few_d64", op="decode_noalloc", dtype="bf16", hq=64, hkv=8, d=64,
             batch=12, lo=1, hi=4096, len_seed=2),
        # The benchmark's decode step: a full batch of ordinary contexts.
        dict(name="decode_batch", op="decode", dtype="bf16", hq=32, hkv=8, d=128,
             batch=256, lo=512, hi=4096, len_seed=3),
        # Two long documents next to short sessions: most of the grid belongs
        # to two sequences and the merge runs over many splits.
        dict(name="decode_long", op="decode", dtype="bf16", hq=32, hkv=8, d=128,
             batch=6, lo=700, hi=131071, len_seed=12),
        # The tiny fp32 batch of the framework's first workload: launch and
        # latency only.
        dict(name="decode_tiny_f32", op="decode", dtype="f32", hq=4, hkv=2, d=64,
             batch=4, lo=37, hi=130, len_seed=5),
        # The benchmark's chunk: the last 8192 tokens of a 32768-token prompt.
        dict(name="prefill_chunk", op="prefill", hq=32, hkv=8, d=128, prompts=1,
             new_lo=8192, new_hi=8192, ctx_lo=24576, ctx_hi=24576, rows=0, lo=1, hi=1,
             len_seed=6),
        # A step that admits several fresh ragged prompts at once, 8 query
        # heads per kv head.
        dict(name="prefill_prompts", op="prefill", hq=64, hkv=8, d=128, prompts=7,
             new_lo=90, new_hi=2049, ctx_lo=0, ctx_hi=0, rows=0, lo=1, hi=1, len_seed=7),
        # A follow-up question: a short chunk over an earlier conversation.
        # Few row tiles, each with a long walk over the cache.
        dict(name="prefill_short", op="prefill", hq=32, hkv=8, d=128, prompts=1,
             new_lo=201, new_hi=201, ctx_lo=6150, ctx_hi=6150, rows=0, lo=1, hi=1,
             len_seed=8),
        # A unified step of chunked prefill: a chunk of a prompt and a batch
        # of decode sequences, one row each, in one call.
        dict(name="mixed_step", op="prefill", hq=32, hkv=8, d=128, prompts=1,
             new_lo=2048, new_hi=2048, ctx_lo=6144, ctx_hi=6144, rows=128, lo=1024, hi=8192,
             len_seed=9),
        # The new K/V rows of an 8192-token chunk, in block order.
        dict(name="append_chunk", op="append", dtype="bf16", hkv=8, d=128, tokens=8192,
             start=0, blocks=640, scattered=False),
        # The new K/V rows of a decode step: one slot per sequence.
        dict(name="append_step", op="append", dtype="bf16", hkv=8, d=128, tokens=256,
             start=0, blocks=4096, scattered=True),
        # Draining the elastic range before a prefill: live elastic blocks
        # move to free base blocks in all 32 layers.
        dict(name="drain_copy", op="copy", hkv=8, d=128, layers=32, blocks=512, pairs=190),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    op = rng.choice(["decode", "decode", "decode", "prefill", "prefill", "prefill", "append",
                     "append", "copy"])
    seed = rng.randrange(1 << 30)
    if op == "decode":
        dtype, hq, hkv, d = rng.choice([("bf16", 32, 8, 128), ("bf16", 64, 8, 128),
                                        ("bf16", 16, 8, 128), ("bf16", 8, 8, 128),
                                        ("bf16", 12, 3, 128), ("bf16", 64, 8, 64),
                                        ("bf16", 8, 2, 64), ("f32", 4, 2, 64),
                                        ("f32", 16, 4, 64)])
        batch = _log(rng, 1, 256)
        hi = _log(rng, 64, min(131071, max(4096, 1000000 // batch)))
        lo = rng.choice([1, max(1, hi // 8), hi])
        entry = "decode_noalloc" if batch * hq * d * hi <= 256 * 32 * 128 * 3500 and \
            rng.random() < 0.25 else "decode"
        return dict(op=entry, dtype=dtype, hq=hq, hkv=hkv, d=d, batch=batch, lo=lo, hi=hi,
                    len_seed=seed)
    if op == "prefill":
        hq, hkv = rng.choice([(32, 8), (32, 8), (64, 8), (16, 8), (8, 8), (12, 3)])
        prompts = rng.choice([1, 1, 1, 2, 4, 9])
        new_hi = _log(rng, 16, 8192 // prompts)
        new_lo = rng.choice([new_hi, max(1, new_hi // 6)])
        ctx_hi = rng.choice([0, _log(rng, 16, 16384)])
        ctx_lo = ctx_hi // 2
        rows = rng.choice([0, 0, _log(rng, 1, 128)])
        hi = _log(rng, 64, 8192)
        return dict(op="prefill", hq=hq, hkv=hkv, d=128, prompts=prompts, new_lo=new_lo,
                    new_hi=new_hi, ctx_lo=ctx_lo, ctx_hi=ctx_hi, rows=rows, lo=max(1, hi // 8),
                    hi=hi, len_seed=seed)
    if op == "append":
        dtype, hkv, d = rng.choice([("bf16", 8, 128), ("bf16", 8, 128), ("bf16", 3, 128),
                                    ("bf16", 2, 64), ("f32", 4, 64)])
        scattered = rng.random() < 0.5
        tokens = _log(rng, 1, 1024 if scattered else 8192)
        start = 0 if scattered else rng.choice([0, rng.randrange(BS)])
        blocks = (tokens + start) // BS + 1
        return dict(op="append", dtype=dtype, hkv=hkv, d=d, tokens=tokens, start=start,
                    blocks=blocks * 2 + (4 * tokens if scattered else 64), scattered=scattered)
    pairs = _log(rng, 1, 190)
    return dict(op="copy", hkv=rng.choice([8, 4]), d=128, layers=rng.choice([32, 28]),
                blocks=512, pairs=pairs)


# ---------------------------------------------------------------------------
# Sequence lengths: fixed by the case, so that every seed does the same work.

def _decode_lens(c):
    r = random.Random(c["len_seed"])
    lens = [r.randint(c["lo"], c["hi"]) for _ in range(c["batch"])]
    if c["lo"] < c["hi"] and c["hi"] > 65536:      # two long ones, the rest short sessions
        lens = [c["hi"], c["hi"] // 2] + [r.randint(c["lo"], 4096 + c["lo"])
                                         for _ in range(c["batch"] - 2)]
        lens = lens[:c["batch"]]
    return lens


def _prefill_lens(c):
    """(context lengths including the new tokens, new tokens), prompts first."""
    r = random.Random(c["len_seed"])
    new = [r.randint(c["new_lo"], c["new_hi"]) for _ in range(c["prompts"])]
    lens = [n + r.randint(c["ctx_lo"], c["ctx_hi"]) for n in new]
    lens += [r.randint(c["lo"], c["hi"]) for _ in range(c["rows"])]
    return lens, new + [1] * c["rows"]


# ---------------------------------------------------------------------------
# Inputs

def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(seed)


def _randn(shape, dtype, g):
    """N(0, 1) rounded to dtype, drawn in slices so that the fp32 draw of a
    large pool need not exist at once."""
    out = torch.empty(shape, dtype=dtype, device="cuda")
    flat = out.view(-1)
    step = 1 << 28
    for i in range(0, flat.numel(), step):
        n = min(step, flat.numel() - i)
        flat[i:i + n] = torch.randn(n, generator=g, device="cuda")
    return out


def _paged(lens, hkv, d, dtype, g):
    """A layer with 10% free blocks, and the block table of a pool that hands
    blocks out in random order. Slots past a sequence's end and free blocks
    hold other numbers, as a reused pool does."""
    need = [-(-n // BS) for n in lens]
    num_blocks = -(-(sum(need) * 11) // 10 // 32) * 32 + 32
    layer = _randn((num_blocks, 2, hkv, BS * d), dtype, g)
    perm = torch.randperm(num_blocks, generator=g, device="cuda").to(torch.int32)
    table = torch.full((len(lens), max(need)), -1, dtype=torch.int32, device="cuda")
    at = 0
    for s, n in enumerate(need):
        table[s, :n] = perm[at:at + n]
        at += n
    return layer, table, num_blocks


def prepare(case, seed):
    g = _gen(seed)
    op = case["op"]
    if op in ("decode", "decode_noalloc"):
        lens = _decode_lens(case)
        dt = TORCH[case["dtype"]]
        layer, table, nb = _paged(lens, case["hkv"], case["d"], dt, g)
        q = _randn((len(lens), case["hq"], case["d"]), dt, g)
        s = dict(op=op, q=q, layer=layer, table=table, num_blocks=nb, hkv=case["hkv"],
                 lens=torch.tensor(lens, dtype=torch.int32, device="cuda"),
                 max_len=max(lens))
        if op == "decode":
            s["ws"] = K.workspace(K.decode_workspace_bytes(len(lens), case["hq"], case["d"],
                                                           max(lens)))
        else:
            s["out"] = torch.empty_like(q)
        return s
    if op == "prefill":
        lens, new = _prefill_lens(case)
        layer, table, nb = _paged(lens, case["hkv"], case["d"], torch.bfloat16, g)
        total = sum(new)
        cu = [0]
        for n in new:
            cu.append(cu[-1] + n)
        return dict(op=op, q=_randn((total, case["hq"], case["d"]), torch.bfloat16, g),
                    layer=layer, table=table, num_blocks=nb, hkv=case["hkv"],
                    lens=torch.tensor(lens, dtype=torch.int32, device="cuda"),
                    cu=torch.tensor(cu, dtype=torch.int32, device="cuda"), max_len=max(lens),
                    ws=K.workspace(K.prefill_workspace_bytes(len(lens), total, case["hq"],
                                                             case["d"])))
    if op == "append":
        dt = TORCH[case["dtype"]]
        T, nb = case["tokens"], case["blocks"]
        layer = _randn((nb, 2, case["hkv"], BS * case["d"]), dt, g)
        if case["scattered"]:
            slots = torch.randperm(nb * BS, generator=g, device="cuda")[:T]
        else:
            t = torch.arange(case["start"], case["start"] + T, device="cuda")
            perm = torch.randperm(nb, generator=g, device="cuda")
            slots = perm[t // BS] * BS + t % BS
        return dict(op=op, layer=layer, num_blocks=nb, slots=slots.to(torch.int32),
                    k=_randn((T, case["hkv"], case["d"]), dt, g),
                    v=_randn((T, case["hkv"], case["d"]), dt, g))
    block = 2 * case["hkv"] * BS * case["d"]
    layers = [_randn((case["blocks"], block), torch.bfloat16, g) for _ in range(case["layers"])]
    ids = torch.randperm(case["blocks"], generator=g, device="cuda").to(torch.int32)
    n = case["pairs"]
    return dict(op=op, layers=layers, num_blocks=case["blocks"], block_bytes=block * 2,
                src=ids[:n].contiguous(), dst=ids[n:2 * n].contiguous())


def run(s):
    if s["op"] == "decode":
        return K.decode(s["q"], s["layer"], s["num_blocks"], s["table"], s["lens"],
                        num_kv_heads=s["hkv"], max_seq_len=s["max_len"], ws=s["ws"])
    if s["op"] == "decode_noalloc":
        return K.decode_noalloc(s["q"], s["layer"], s["num_blocks"], s["table"], s["lens"],
                                s["out"], num_kv_heads=s["hkv"], max_seq_len=s["max_len"])
    if s["op"] == "prefill":
        return K.prefill_chunk(s["q"], s["layer"], s["num_blocks"], s["table"], s["lens"],
                               s["cu"], num_kv_heads=s["hkv"], max_seq_len=s["max_len"],
                               ws=s["ws"])
    if s["op"] == "append":
        K.kv_append(s["k"], s["v"], s["slots"], s["layer"], s["num_blocks"])
        return s["layer"]
    K.copy_blocks(s["layers"], s["num_blocks"], s["block_bytes"], s["src"], s["dst"])
    return s["layers"]


# ---------------------------------------------------------------------------
# What a pass cannot do without, and how close results have to be

def work(case):
    op = case["op"]
    if op in ("decode", "decode_noalloc"):
        lens = _decode_lens(case)
        e = ESZ[case["dtype"]]
        kv = sum(lens) * case["hkv"] * case["d"] * 2 * e
        qo = 2 * len(lens) * case["hq"] * case["d"] * e
        tab = 4 * sum(-(-n // BS) for n in lens) + 4 * len(lens)
        return {"bytes": kv + qo + tab, "flops": 4 * case["d"] * case["hq"] * sum(lens)}
    if op == "prefill":
        lens, new = _prefill_lens(case)
        pairs = sum(n * (L - n) + n * (n + 1) // 2 for L, n in zip(lens, new))
        kv = sum(lens) * case["hkv"] * case["d"] * 2 * 2
        qo = 2 * sum(new) * case["hq"] * case["d"] * 2
        tab = 4 * sum(-(-n // BS) for n in lens) + 8 * len(lens) + 4
        return {"bytes": kv + qo + tab, "flops": 4 * case["d"] * case["hq"] * pairs}
    if op == "append":
        row = case["hkv"] * case["d"] * ESZ[case["dtype"]]
        return {"bytes": 4 * case["tokens"] * row + 4 * case["tokens"], "flops": 0}
    block = 2 * case["hkv"] * BS * case["d"] * 2
    return {"bytes": 2 * case["pairs"] * case["layers"] * block + 8 * case["pairs"], "flops": 0}


def tolerance(case):
    if case["op"] in ("append", "copy"):
        return "exact"
    if case.get("dtype") == "f32":
        return {"rel": 1e-6, "max": 1e-5}
    # P is rounded to bf16 before the p.v product and the output to bf16:
    # about 2.5e-3 against 64 bits, so another correct order of sums differs
    # by as much again.
    return {"rel": 1e-2, "max": 5e-2}


# ---------------------------------------------------------------------------
# The same results in 64 bits, with plain torch

def _context(s, seq, L, hkv, d):
    """K and V [hkv, L, d] of one sequence in 64 bits, from the layer's bytes:
    K tiles hold 16-byte chunks of 16 slots, V tiles are dim-major."""
    ids = s["table"][seq, :-(-L // BS)].long()
    tiles = s["layer"][ids]                                   # [n, 2, hkv, BS * d]
    vec = 16 // tiles.element_size()
    k = tiles[:, 0].view(-1, hkv, d // vec, BS, vec).permute(1, 0, 3, 2, 4)
    v = tiles[:, 1].view(-1, hkv, d, BS).permute(1, 0, 3, 2)
    return (k.reshape(hkv, -1, d)[:, :L].double(), v.reshape(hkv, -1, d)[:, :L].double())


def _attend(q, k, v, first):
    """Rows q [n, hq, d] at positions first .. first + n - 1, causally."""
    n, hq, d = q.shape
    hkv, L, _ = k.shape
    out = torch.empty(n, hq, d, dtype=torch.float64, device=q.device)
    keys = torch.arange(L, device=q.device)
    step = max(1, (1 << 26) // L)
    for g in range(hkv):
        kt, vg = k[g].t().contiguous(), v[g].contiguous()
        for h in range(g * (hq // hkv), (g + 1) * (hq // hkv)):
            for r in range(0, n, step):
                rows = q[r:r + step, h].double()
                sc = rows @ kt / math.sqrt(d)
                pos = first + r + torch.arange(rows.shape[0], device=q.device)
                sc.masked_fill_(keys[None, :] > pos[:, None], -math.inf)
                out[r:r + step, h] = torch.softmax(sc, dim=-1) @ vg
    return out


def exact(case, seed):
    if case["op"] in ("append", "copy"):
        return None
    s = prepare(case, seed)
    if case["op"] == "prefill":
        lens, new = _prefill_lens(case)
    else:
        lens = _decode_lens(case)
        new = [1] * len(lens)
    out, at = [], 0
    for i, (L, n) in enumerate(zip(lens, new)):
        k, v = _context(s, i, L, case["hkv"], case["d"])
        out.append(_attend(s["q"][at:at + n], k, v, L - n))
        at += n
    return torch.cat(out)
