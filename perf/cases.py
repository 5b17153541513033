"""Cases of the split paged decode-attention library, timed through its public entry points.

One case is one call sequence that a serving program issues per layer and token:

* ``step``    every partition's partial attention, then the merge (the two-call form of attention-level
              migration), through the checked binding or the prepared-argument runner;
* ``fused``   all partitions and their merge in one call;
* ``noalloc`` one partition for a caller that cannot allocate, without any hint;
* ``heads``   the kv heads of one device of a head split;
* ``layer``   the fused call carrying the layer pipeline's fetch and store (pinned host memory);
* ``migrate`` the KV-block copy into another pool.

A case's sequence lengths and ranges come from the case itself (``lens_seed``), so its work is known
without its inputs; queries, keys, values and the block placement come from the seed of ``prepare``.
Keys and values are bf16 N(0, 1) in a pool a fifth larger than needed under a random block table;
unused blocks and slots hold NaN.
"""

import math
import random

import numpy as np
import torch

from paper_2510_13223_amd import bana, workloads
from paper_2510_13223_amd.runner import DeviceWorkload

D, BS = bana.HEAD_DIM, bana.BLOCK_SIZE
TILE_BYTES = 2 * D * BS * 2  # K and V of one (block, kv head)

# Query / kv heads: GQA groups of 4, 8, 7 and 16 and multi-head, as current decoder layers have them.
HEADS = [(8, 2), (32, 8), (64, 8), (40, 40), (28, 4), (32, 2)]


def _case(name, path, batch, hq, hkv, lens, length, parts, cut, **more):
    """``lens``: fixed / uniform / lognormal around ``length``; ``cut``: how a sequence's blocks are split
    into ``parts`` (tail30, random, equal, longonly: only sequences over 2048 tokens, token: at any token)."""
    c = {"path": path, "batch": batch, "hq": hq, "hkv": hkv, "lens": lens, "length": length, "parts": parts,
         "cut": cut, "lens_seed": 0, "scaled": True, "bias": 0.0, "hints": True}
    c.update(more)
    if name is not None:
        c["name"] = name
    return c


def listed():
    return [
        # The smallest call in use: a few short sequences on a small model, latency only.
        _case("tiny_step", "step_runner", 4, 8, 2, "uniform", 640, 2, "random"),
        # One user with a prompt of a few pages: a single sequence, odd length.
        _case("single_fused", "fused", 1, 32, 8, "fixed", 3001, 2, "random"),
        # A lightly loaded server: eight requests, each split between the local and a migrated partition.
        _case("small_step", "step_runner", 8, 32, 8, "uniform", 2300, 2, "random"),
        # A caller that cannot allocate and passes no hints, group of 16, ranges cut at any token.
        _case("ragged_noalloc", "noalloc", 24, 32, 2, "lognormal", 700, 1, "token", hints=False),
        # A chat server's ordinary batch: short prompts with a tail of long ones.
        _case("chat_fused", "fused", 48, 32, 8, "lognormal", 1024, 2, "longonly"),
        # A migration of the last 30 % of every sequence's blocks.
        _case("llama3_8b_migrate", "migrate", 64, 32, 8, "fixed", 4096, 2, "tail30"),
        # Half of the heads of a multi-head layer (the other half lives on another device).
        _case("mha13b_heads", "heads", 32, 40, 40, "fixed", 2048, 1, "tail30", scaled=False),
        # A layer of the pipeline: attention with 500 fetched and 500 stored tokens of KV beside it.
        _case("llama3_8b_layer", "layer", 64, 32, 8, "fixed", 2048, 2, "tail30", scaled=False),
        # The benchmark's layer: 64 sequences of 4096 tokens, the last 30 % migrated.
        _case("llama3_8b_step", "step", 64, 32, 8, "fixed", 4096, 2, "tail30", scaled=False),
        # A full server with mixed lengths; only the long sequences are split.
        _case("mixed_step", "step", 256, 32, 8, "lognormal", 1024, 2, "longonly", scaled=False),
        # Long contexts split four ways into pieces of random sizes.
        _case("long_step", "step", 8, 32, 8, "uniform", 81920, 4, "random", scaled=False),
        # Fine-grained migration of a large model's layer: 16 equal partitions, biased keys.
        _case("fine_step", "step", 512, 64, 8, "fixed", 2048, 16, "equal", scaled=False, bias=2.0),
    ]


def draw(rng):
    path = rng.choice(["step", "step_runner", "fused", "fused", "noalloc", "heads", "layer", "migrate"])
    hq, hkv = rng.choice(HEADS)
    lens = rng.choice(["fixed", "uniform", "lognormal"])
    length = int(round(math.exp(rng.uniform(math.log(200), math.log(65536)))))
    batch = int(round(math.exp(rng.uniform(0, math.log(512)))))
    # At most about 1 GiB of keys and values in a case, 64 MiB where they are made on the host.
    most = (64 << 20) if path == "step_runner" else (1 << 30)
    length = min(length, most // (hkv * 4 * D) // 2)
    batch = max(1, min(batch, most // (length * hkv * 4 * D)))
    parts = 1 if path in ("noalloc", "heads") else 2 if path == "migrate" else rng.choice([1, 2, 2, 3, 4, 16])
    cut = rng.choice(["tail30", "random"]) if path == "migrate" else (
        rng.choice(["random", "token", "longonly", "tail30"]) if parts == 2 else rng.choice(["random", "token", "equal"]))
    return _case(None, path, batch, hq, hkv, lens, length, parts, cut, lens_seed=rng.randrange(1 << 30),
                 scaled=rng.random() < 0.5, hints=path != "noalloc" and rng.random() < 0.8)


# ---- lengths and ranges (host only) ---------------------------------------------------------------

def _lens(case):
    r = np.random.default_rng([case["lens_seed"], case["batch"], case["length"]])
    n, mid = case["batch"], case["length"]
    if case["lens"] == "fixed":
        return np.full(n, mid, dtype=np.int64)
    if case["lens"] == "uniform":
        return r.integers(max(1, int(0.4 * mid)), int(1.6 * mid), size=n, endpoint=True)
    return np.clip(np.rint(mid * np.exp(r.standard_normal(n))), 16, 16 * mid).astype(np.int64)


def _ranges(case):
    """(lens [B], begin [P, B], end [P, B])."""
    lens, P, cut = _lens(case), case["parts"], case["cut"]
    r = random.Random(case["lens_seed"] * 7919 + case["batch"])
    edges = np.zeros((P + 1, len(lens)), dtype=np.int64)
    for b, L in enumerate(int(x) for x in lens):
        nb = -(-L // BS)
        if cut == "token":
            e = [0] + sorted(r.randrange(L + 1) for _ in range(P - 1)) + [L]
            if P == 1:  # a range that starts and ends inside blocks
                e = [r.randrange(min(L, 40)), L]
        else:
            if cut == "tail30":
                js = [nb - int(round(0.3 * nb))] + [nb] * (P - 2)
            elif cut == "equal":
                js = [nb * (p + 1) // P for p in range(P - 1)]
            elif cut == "longonly" and L <= 2048:
                js = [nb] * (P - 1)
            else:
                js = sorted(r.randint(min(1, nb - 1), max(1, nb - 1)) for _ in range(P - 1))
            e = [0] + [min(j * BS, L) for j in js[:P - 1]] + [L]
        edges[:, b] = e
    return lens, edges[:-1].copy(), edges[1:].copy()


def _blocks(begin, end):
    """Blocks that overlap each range."""
    return np.where(end > begin, (end + BS - 1) // BS - begin // BS, 0)


# ---- inputs ---------------------------------------------------------------------------------------

def _pools(case, lens, g, dev):
    """(k, v, table): pools under a random placement, NaN where no token is."""
    hkv = case["hkv"]
    nbs = -(-lens // BS)
    used, mb = int(nbs.sum()), int(nbs.max())
    n = max(1, math.ceil(1.2 * used))
    k = torch.randn((n, hkv, D // 8, BS, 8), generator=g, device=dev, dtype=torch.bfloat16)
    v = torch.randn((n, hkv, D, BS), generator=g, device=dev, dtype=torch.bfloat16)
    if case["bias"]:
        bias = case["bias"] * torch.randn((hkv, D // 8, 1, 8), generator=g, device=dev)
        k += bias.to(torch.bfloat16)
    perm = torch.randperm(n, generator=g, device=dev).to(torch.int32)
    table = torch.full((len(lens), mb), -1, dtype=torch.int32, device=dev)
    live = torch.from_numpy(np.arange(mb)[None, :] < nbs[:, None]).to(dev)
    table[live] = perm[:used]
    rest = perm[used:].long()
    k[rest] = float("nan")
    v[rest] = float("nan")
    tail = lens % BS
    at = np.nonzero(tail)[0]
    if len(at):
        last = table[torch.from_numpy(at).to(dev), torch.from_numpy(nbs[at] - 1).to(dev)].long()
        free = torch.from_numpy(np.arange(BS)[None, :] >= tail[at][:, None]).to(dev)
        k[last] = k[last].masked_fill(free[:, None, None, :, None], float("nan"))
        v[last] = v[last].masked_fill(free[:, None, None, :], float("nan"))
    return k, v, table


def _i32(a, dev):
    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.int32)).to(dev)


def _order(lens, dev):
    """Longest range first: the dispatch order a program passes with uneven ranges."""
    return _i32(np.argsort(-lens, kind="stable"), dev)


def prepare(case, seed):
    dev = torch.device("cuda", torch.cuda.current_device())
    g = torch.Generator(device=dev)
    g.manual_seed(seed)
    lens, begin, end = _ranges(case)
    B, hq, hkv, P = case["batch"], case["hq"], case["hkv"], case["parts"]
    k, v, table = _pools(case, lens, g, dev)
    q = torch.randn((B, hq, D), generator=g, device=dev)
    q = (q / math.sqrt(D) if case["scaled"] else q).to(torch.bfloat16)
    s = {"case": case, "q": q, "k": k, "v": v, "table": table}
    s["lens"], s["begin"], s["end"] = _i32(lens, dev), _i32(begin, dev), _i32(end, dev)
    f32 = dict(dtype=torch.float32, device=dev)

    if case["path"] == "step_runner":
        bits = lambda t: t.view(torch.int16).cpu().numpy().view(np.uint16)
        w = workloads.Workload("case", seed, hq, hkv, bits(q), bits(k), bits(v), table.cpu().numpy(),
                               lens.astype(np.int32), begin.astype(np.int32), end.astype(np.int32),
                               int((end - begin).max()))
        return {"case": case, "runner": DeviceWorkload(w, device=dev, range_hints=case["hints"])}

    if case["path"] == "migrate":
        jb, je = np.where(end[1] > begin[1], begin[1] // BS, 0), np.where(end[1] > begin[1], -(-end[1] // BS), 0)
        n = int((je - jb).sum())
        nd = max(1, math.ceil(1.2 * n))
        at = torch.from_numpy((np.arange(table.shape[1])[None, :] >= jb[:, None])
                              & (np.arange(table.shape[1])[None, :] < je[:, None])).to(dev)
        dst_table = torch.full_like(table, -1)
        dst_table[at] = torch.randperm(nd, generator=g, device=dev)[:n].to(torch.int32)
        s["dst_k"] = torch.zeros((nd,) + tuple(k.shape[1:]), dtype=torch.bfloat16, device=dev)
        s["dst_v"] = torch.zeros((nd,) + tuple(v.shape[1:]), dtype=torch.bfloat16, device=dev)
        s["dst_table"], s["jb"], s["je"] = dst_table, _i32(jb, dev), _i32(je, dev)
        s["longest"] = int((je - jb).max()) * BS if case["hints"] else 0
        return s

    def dims(spans, heads=(hq, hkv)):
        if not case["hints"]:
            return bana.make_dims(B, hq, hkv, table.shape[1], k.shape[0])
        s.setdefault("orders", []).append(_order(spans, dev))
        return bana.make_dims(B, hq, hkv, table.shape[1], k.shape[0], max_range_tokens=int(spans.max()),
                              total_range_tokens=int(spans.sum()), seq_order=s["orders"][-1],
                              nonempty_ranges=int(np.count_nonzero(spans)),
                              waves_hint=4 if case["path"] == "layer" else 0,
                              plan_hint=1 if case["path"] == "layer" else 0)

    spans = end - begin
    s["out"] = torch.zeros((B, hq, D), **f32)
    s["lse"] = torch.zeros((B, hq), **f32)
    if case["path"] == "step":
        s["dims"] = [dims(spans[p]) for p in range(P)]
        s["out_partials"] = torch.zeros((P, B, hq, D), **f32)
        s["lses"] = torch.zeros((P, B, hq), **f32)
        s["rows"] = [(s["begin"][p], s["end"][p], s["out_partials"][p], s["lses"][p]) for p in range(P)]
    elif case["path"] == "heads":
        s["dims"] = [dims(spans[0])]
        s["heads"] = (0, (hkv + 1) // 2)
    else:
        s["dims"] = [dims(spans.sum(axis=0))]
    need = [bana.head_range_dims(d, *s["heads"]) if case["path"] == "heads" else d for d in s["dims"]]
    ws = max(bana.bana_decode_attn_workspace_bytes(d) for d in need)
    s["workspace"] = torch.empty(max(ws, 256), dtype=torch.uint8, device=dev)
    if case["path"] == "layer":
        blocks = -(-500 // BS)  # a request's cached prefix in, its new tokens out
        pin = lambda t: torch.empty(t.shape, dtype=t.dtype).pin_memory()
        some = lambda t: torch.randn((blocks,) + tuple(t.shape[1:]), generator=g, device=dev, dtype=torch.bfloat16)
        s["side"] = []
        for t in (k, v):
            fetch_from = pin(some(t))
            fetch_from.copy_(some(t))
            s["side"].append((torch.zeros_like(some(t)), fetch_from))
            store_from = some(t)
            s["side"].append((pin(store_from), store_from))
    return s


def run(s):
    path = s["case"]["path"]
    if path == "step_runner":
        r = s["runner"]
        r.step()
        return {"out_partials": r.out_partials, "lses": r.lses, "out": r.out, "lse": r.lse_out}
    if path == "migrate":
        bana.bana_migrate_kv_blocks(s["k"], s["v"], s["table"], s["dst_k"], s["dst_v"], s["dst_table"], s["jb"], s["je"],
                                    max_range_tokens=s["longest"])
        return {"dst_k": s["dst_k"].view(torch.int16), "dst_v": s["dst_v"].view(torch.int16)}
    args = (s["q"], s["k"], s["v"], s["table"], s["lens"])
    if path == "step":
        for (begin, end, out, lse), dims in zip(s["rows"], s["dims"]):
            bana.bana_decode_attn_partial(*args, begin, end, out, lse, workspace=s["workspace"], dims=dims)
        bana.bana_merge_partials(s["out_partials"], s["lses"], s["out"], s["lse"])
        return {"out_partials": s["out_partials"], "lses": s["lses"], "out": s["out"], "lse": s["lse"]}
    if path == "noalloc":
        bana.bana_decode_attn_partial_noalloc(*args, s["begin"][0], s["end"][0], s["out"], s["lse"], dims=s["dims"][0])
    elif path == "heads":
        bana.bana_decode_attn_heads(*args, s["begin"][0], s["end"][0], *s["heads"], s["out"], s["lse"],
                                    workspace=s["workspace"], dims=s["dims"][0])
    elif path == "layer":
        bana.bana_decode_attn_fused_copies(*args, s["begin"], s["end"], s["out"], s["lse"], copies=s["side"],
                                           workspace=s["workspace"], dims=s["dims"][0])
        return {"out": s["out"], "lse": s["lse"], "side": [dst.view(torch.int16) for dst, _ in s["side"]]}
    else:
        bana.bana_decode_attn_fused(*args, s["begin"], s["end"], s["out"], s["lse"], workspace=s["workspace"],
                                    dims=s["dims"][0])
    return {"out": s["out"], "lse": s["lse"]}


# ---- what a pass cannot do without, and its result in 64 bits ---------------------------------------

def work(case):
    lens, begin, end = _ranges(case)
    B, hq, hkv, P = case["batch"], case["hq"], case["hkv"], case["parts"]
    blocks = _blocks(begin, end)
    if case["path"] == "migrate":
        n = int(blocks[1].sum())
        return {"bytes": 2 * n * hkv * TILE_BYTES + 8 * n + 8 * B, "flops": 0}
    if case["path"] == "heads":
        hq, hkv = hq // hkv * ((hkv + 1) // 2), (hkv + 1) // 2
    tokens = int((end - begin).sum())
    row = 4 * (D + 1) * B * hq  # an output row and its lse
    moved = tokens * hkv * 4 * D + 4 * int(blocks.sum()) + 8 * P * B + 2 * D * B * hq + row
    if case["path"] in ("step", "step_runner"):
        moved += P * row
    if case["path"] == "layer":
        moved += 2 * 2 * -(-500 // BS) * hkv * TILE_BYTES
    return {"bytes": moved, "flops": 4 * D * tokens * hq}


def tolerance(case):
    # Copies are exact.  Scores are exact bf16 products summed in fp32 and the weights carry 16 bits into
    # the value product.  Measured against 64 bits: outputs off by 3.4e-6 to 4.1e-6 with queries scaled by
    # 1/sqrt(128) (long averages of values), 7e-7 to 1e-6 unscaled, lse by 6e-8; four times the largest.
    return "exact" if case["path"] == "migrate" else {"rel": 1.6e-5, "max": 4e-4}


def exact(case, seed):
    if case["path"] == "migrate":
        return None
    s = prepare(dict(case, path="step" if case["path"] == "step_runner" else case["path"]), seed)
    B, hq, hkv, P = case["batch"], case["hq"], case["hkv"], case["parts"]
    lens, begin, end = _ranges(case)
    group = hq // hkv
    f64 = dict(dtype=torch.float64, device=s["q"].device)
    parts = torch.zeros((P, B, hq, D), **f64)
    lses = torch.full((P, B, hq), -math.inf, **f64)
    for b in range(B):
        for p in range(P):
            t0, t1 = int(begin[p, b]), int(end[p, b])
            if t1 <= t0:
                continue
            j0, j1 = t0 // BS, -(-t1 // BS)
            at = s["table"][b, j0:j1].long()
            cut = slice(t0 - j0 * BS, t1 - j0 * BS)
            for h0 in range(0, hkv, 8):  # eight kv heads at a time bound the 64-bit copies
                h1 = min(hkv, h0 + 8)
                k = s["k"][at, h0:h1].permute(1, 0, 3, 2, 4).reshape(h1 - h0, -1, D)[:, cut].double()
                v = s["v"][at, h0:h1].permute(1, 0, 3, 2).reshape(h1 - h0, -1, D)[:, cut].double()
                rows = slice(h0 * group, h1 * group)
                q = s["q"][b, rows].double().reshape(h1 - h0, group, D)
                x = torch.matmul(q, k.transpose(1, 2).contiguous())
                lses[p, b, rows] = torch.logsumexp(x, -1).reshape(-1)
                parts[p, b, rows] = torch.matmul(torch.softmax(x, -1), v).reshape(-1, D)
    total = torch.logsumexp(lses, 0)
    weight = torch.nan_to_num(torch.exp(lses - total), nan=0.0)
    out = (weight[..., None] * parts).sum(0)
    if case["path"] in ("step", "step_runner"):
        return {"out_partials": parts, "lses": lses, "out": out, "lse": total}
    if case["path"] == "heads":
        first = group * s["heads"][1]  # rows of the other device's heads stay as they were
        out[:, first:] = 0
        total[:, first:] = 0
    if case["path"] == "layer":
        return {"out": out, "lse": total, "side": [None] * len(s["side"])}
    return {"out": out, "lse": total}
