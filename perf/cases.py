"""Timing cases of the token-sparsification operator, through its public entry points.

A case is one packed batch and the call a serving engine makes on it at a drop layer:

  fused    uniprefill_fused                score, block-local top-k, compaction
  top_p    uniprefill_fused_top_p          the same with the block-level top-p rule
  paged    uniprefill_fused_paged          chunks of prompts whose earlier keys sit in a paged KV cache
  lse      uniprefill_fused_lse            the attention layer hands its rows' log-sum-exp over
  scatter  uniprefill_scatter              the way back: compacted rows into the full hidden state

Shapes are those of the repository's workloads, tests and sweeps: 8/8, 32/8 and 40/8 heads, head
dimension 128 (64 and 256 are offered as well), hidden size 1024 to 5120, block sizes 32, 64 and 128,
a query window of 128 rows (32 and 512 in the window study), prompts from about a thousand tokens to
131072, alone, in ragged batches, and mixed with decode rows.

Values: queries, keys and hidden rows are normal in bf16.  Attention over text is concentrated on few
tokens: `key_spread` s scales every key row by exp(s * z), z ~ N(0,1) (0 = plain normal keys, 1 = the
heavy-tailed workload).
"""
import math

import numpy as np
import torch

import paper_2605_06221_amd as up

N_SINK = 128
KV_BLOCK = 16          # tokens per block of the paged cache

_DEFAULTS = {"entry": "fused", "lengths": "4096", "earlier": "", "hidden": 4096, "q_heads": 32, "kv_heads": 8,
             "head_dim": 128, "block": 128, "window": 128, "keep": 0.3, "keep_to": 0.3, "key_spread": 0.5, "scores": False}


def _case(name, **kw):
    return {"name": name, **_DEFAULTS, **kw}


def listed():
    return [
        # the smallest prompt worth sparsifying: launches and host time, hardly any work
        _case("short_1000", lengths="1000", hidden=1024, q_heads=8, block=64, keep=0.5, keep_to=0.5),
        # one 4096-token prompt of a small model, scores wanted by the caller as well
        _case("prompt_4k", lengths="4096", hidden=1024, q_heads=8, block=64, keep=0.5, keep_to=0.5, key_spread=0.0,
              scores=True),
        # one 32768-token prompt of an 8B-shaped layer
        _case("prompt_32k", lengths="32768"),
        # continuous batch of sixteen ragged prompts, every one with its own keep ratio
        _case("batch_16_ragged",
              lengths="28174,21619,17691,10340,11489,3342,4362,2547,7443,27028,21841,30103,17444,20703,32420,18019",
              keep=0.2, keep_to=0.6),
        # the long-context prompt the operator is there for
        _case("prompt_128k", lengths="131072", hidden=5120, q_heads=40, keep=0.25, keep_to=0.25, key_spread=1.0),
        # mixed step: 64 decode rows that pass through, eight prefill chunks with ragged last blocks
        _case("decode_64_chunks_8", lengths="64*1,8137,8165,8160,8176,8171,8190,8188,8191", block=64, keep=0.4, keep_to=0.4),
        # the paper's own rule on a ragged batch of five prompts
        _case("top_p_batch_5", entry="top_p", lengths="20011,2050,9999,4097,14336", block=64, keep=0.95, keep_to=0.99,
              key_spread=1.0, scores=True),
        # chunked prefill: 8192 new tokens after 57344 cached ones, and a short chunk after 5000
        _case("paged_chunks_2", entry="paged", lengths="8192,3001", earlier="57344,5000", block=64),
        # a 64k prompt whose attention kernel returned its log-sum-exp
        _case("lse_64k", entry="lse", lengths="65537", block=128),
        # reconstitution of a 32768-token hidden state from a third of its rows
        _case("scatter_32k", entry="scatter", lengths="32768"),
        # narrow heads, three ragged prompts
        _case("head_64_batch_3", lengths="12289,24576,7011", hidden=2048, head_dim=64, block=64),
        # wide heads, a longer query window
        _case("head_256_window_256", lengths="16384", head_dim=256, q_heads=16, window=256, key_spread=1.0),
    ]


def draw(rng):
    most = work(listed()[3])
    for _ in range(1000):
        entry = rng.choice(["fused", "fused", "fused", "top_p", "paged", "lse", "scatter"])
        total = int(round(math.exp(rng.uniform(math.log(900), math.log(150000)))))
        n_seqs = 1 if rng.random() < 0.4 else rng.randint(2, 20)
        cuts = sorted(rng.randint(1, max(1, total - 1)) for _ in range(n_seqs - 1))
        lengths = [b - a for a, b in zip([0] + cuts, cuts + [total]) if b > a]
        if rng.random() < 0.25:
            lengths = [1] * rng.randint(1, 96) + lengths
        q_heads, kv_heads = rng.choice([(8, 8), (32, 8), (32, 8), (40, 8), (16, 4)])
        keep = round(rng.uniform(0.9, 0.99) if entry == "top_p" else rng.uniform(0.1, 0.7), 3)
        c = {**_DEFAULTS, "entry": entry, "lengths": ",".join(str(n) for n in lengths),
             "hidden": rng.choice([1024, 2048, 4096, 4096, 5120]), "q_heads": q_heads, "kv_heads": kv_heads,
             "head_dim": rng.choice([64, 128, 128, 128, 128, 256]), "block": rng.choice([32, 64, 128]),
             "window": rng.choice([32, 64, 128, 128, 128, 128, 512]), "keep": keep, "keep_to": keep,
             "key_spread": rng.choice([0.5, 1.0]), "scores": entry == "top_p" or (entry != "scatter" and rng.random() < 0.3)}
        if entry == "paged":
            c["earlier"] = ",".join(str(int(math.exp(rng.uniform(math.log(64), math.log(60000))))) for _ in lengths)
        w = work(c)
        # no more than the largest listed case, in work and in memory
        if w["flops"] <= most["flops"] and w["bytes"] <= most["bytes"] and sum(_keys(c)) <= 300000:
            return c
    raise RuntimeError("no case of the range fits")


def _numbers(text):
    out = []
    for part in filter(None, text.split(",")):
        count, _, value = part.rpartition("*")
        out += [int(value)] * (int(count) if count else 1)
    return out


def _keys(case):
    """Keys of every sequence: its own tokens' and, in chunked prefill, those before them."""
    lengths = _numbers(case["lengths"])
    earlier = _numbers(case["earlier"]) or [0] * len(lengths)
    return [n + e for n, e in zip(lengths, earlier)]


def _offsets(lengths):
    return np.concatenate([[0], np.cumsum(lengths)]).astype(np.int32)


def _ratios(case):
    n = len(_numbers(case["lengths"]))
    return np.linspace(case["keep"], case["keep_to"], n).astype(np.float32)


def _params(case):
    lengths = _numbers(case["lengths"])
    return up.make_params(num_seqs=len(lengths), total_tokens=sum(lengths), block_size=case["block"], n_obs=case["window"],
                          n_sink=N_SINK, num_q_heads=case["q_heads"], num_kv_heads=case["kv_heads"],
                          head_dim=case["head_dim"], hidden_dim=case["hidden"])


def _plan(case):
    """(total_kept, workspace bytes) as the library plans them."""
    p, cu, ratios = _params(case), _offsets(_numbers(case["lengths"])), _ratios(case)
    if case["entry"] == "paged":
        _, _, total, ws = up.uniprefill_plan_chunked(p, cu, _offsets(_keys(case)), ratios)
    else:
        _, _, total, ws = up.uniprefill_plan(p, cu, ratios)
    return total, ws


def work(case):
    lengths, keys, entry = _numbers(case["lengths"]), _keys(case), case["entry"]
    row, head = 2 * case["hidden"], 2 * case["head_dim"]
    kept = sum(lengths)
    if entry != "top_p":
        kept, _ = _plan(case)
    else:
        # decided by the data: a little more than the sinks and the window at the least
        kept = sum(min(n, N_SINK + case["window"]) for n in lengths)
    if entry == "scatter":
        return {"bytes": kept * (2 * row + 4), "flops": 0}
    bytes_, flops = kept * (2 * row + 12) + 4 * sum(lengths) * (1 if case["scores"] else 0), 0
    for n, k in zip(lengths, keys):
        if not case["scores"] and entry in ("fused", "lse") and n <= N_SINK + case["window"]:
            continue               # kept whole whatever the scores
        rows = min(n, case["window"])
        bytes_ += k * case["kv_heads"] * head + rows * case["q_heads"] * head
        # a weight is final only when its row has met every key, and the logits fit no memory near the
        # chip: the product is formed once for the rows' sums, once more for the tokens' own keys
        bytes_ -= (k - n) * case["kv_heads"] * head if entry == "lse" else 0
        flops += 2 * rows * case["q_heads"] * case["head_dim"] * ((0 if entry == "lse" else k) + n)
    return {"bytes": bytes_, "flops": flops}


def tolerance(case):
    # rows, positions, indices and offsets are copied or counted: the same bits.  Scores: float32 means
    # of exponentials of float32 sums over the head dimension; logits reach some hundred with heavy tails
    if case["entry"] == "scatter" or not case["scores"]:
        return "exact"
    return {"rel": 1e-5}


def _normal(gen, *shape):
    return torch.randn(shape, generator=gen, device="cuda", dtype=torch.bfloat16)


def _spread_keys(gen, k, spread):
    if spread:
        z = torch.randn(k.shape[0], generator=gen, device="cuda")
        for lo in range(0, k.shape[0], 1 << 15):
            part = k[lo:lo + (1 << 15)]
            part.copy_(part.float() * torch.exp(spread * z[lo:lo + (1 << 15), None, None]))
    return k


def _window_lse(case, q, k, cu):
    """Log-sum-exp of the query window's rows, [heads, tokens], as an attention kernel returns it."""
    hq, group, d = case["q_heads"], case["q_heads"] // case["kv_heads"], case["head_dim"]
    lse = torch.zeros(hq, q.shape[0], device="cuda")
    for r in range(len(cu) - 1):
        lo, hi = int(cu[r]), int(cu[r + 1])
        rows = min(case["window"], hi - lo)
        hidden = torch.arange(hi - lo, device="cuda")[None, :] > torch.arange(hi - lo - rows, hi - lo, device="cuda")[:, None]
        for h in range(hq):
            s = q[hi - rows:hi, h].float() @ k[lo:hi, h // group].float().t().contiguous()
            lse[h, hi - rows:hi] = torch.logsumexp((s / math.sqrt(d)).masked_fill_(hidden, -math.inf), dim=1)
    return lse


def prepare(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    lengths, keys = _numbers(case["lengths"]), _keys(case)
    total, total_keys = sum(lengths), sum(keys)
    kept, ws_bytes = _plan(case)
    s = {"entry": case["entry"], "p": _params(case), "kept": kept, "ws_bytes": ws_bytes,
         "cu_host": _offsets(lengths), "ratio_host": _ratios(case)}
    s["cu"] = torch.from_numpy(s["cu_host"]).cuda()
    s["ratio"] = torch.from_numpy(s["ratio_host"]).cuda()
    room = total if case["entry"] == "top_p" else kept
    if case["entry"] == "scatter":
        # the rows a selection would have kept: a share of every block, ascending
        order = torch.rand(total, generator=gen, device="cuda").argsort()[:kept]
        s["kept_idx"] = order.sort().values.to(torch.int32)
        s["compact"] = _normal(gen, kept, case["hidden"])
        s["full"] = _normal(gen, total, case["hidden"])
        return s
    s["hidden"] = _normal(gen, total, case["hidden"])
    s["q"] = _normal(gen, total, case["q_heads"], case["head_dim"])
    k = _spread_keys(gen, _normal(gen, total_keys, case["kv_heads"], case["head_dim"]), case["key_spread"])
    s["pos"] = torch.cat([torch.arange(kk - n, kk, device="cuda", dtype=torch.int32) for n, kk in zip(lengths, keys)])
    if case["entry"] == "paged":
        s["cu_k_host"] = _offsets(keys)
        s["cu_k"] = torch.from_numpy(s["cu_k_host"]).cuda()
        need = [-(-n // KV_BLOCK) for n in keys]
        order = torch.randperm(sum(need), generator=gen, device="cuda")
        table = torch.zeros(len(keys), max(need), dtype=torch.int32, device="cuda")
        cache = torch.zeros(sum(need) * KV_BLOCK, case["kv_heads"], case["head_dim"], dtype=torch.bfloat16, device="cuda")
        at = 0
        for r, n in enumerate(need):
            table[r, :n] = order[at:at + n].to(torch.int32)
            i = torch.arange(keys[r], device="cuda")
            cache[table[r][i // KV_BLOCK].long() * KV_BLOCK + i % KV_BLOCK] = k[int(s["cu_k_host"][r]):int(s["cu_k_host"][r + 1])]
            at += n
        s["table"], s["k"] = table, cache
    else:
        s["k"] = k
    if case["entry"] == "lse":
        s["lse"] = _window_lse(case, s["q"], k, s["cu_host"])
    # outputs and workspace of the program, allocated once and used by every call
    s["hidden_out"] = torch.zeros(room, case["hidden"], dtype=torch.bfloat16, device="cuda")
    s["pos_out"] = torch.zeros(room, dtype=torch.int32, device="cuda")
    s["kept_idx"] = torch.zeros(room, dtype=torch.int32, device="cuda")
    s["new_cu"] = torch.zeros(len(lengths) + 1, dtype=torch.int32, device="cuda")
    s["scores"] = torch.zeros(total, device="cuda") if case["scores"] else None
    s["workspace"] = torch.empty(ws_bytes + 256, dtype=torch.uint8, device="cuda")
    return s


def run(s):
    if s["entry"] == "scatter":
        up.uniprefill_scatter(s["p"], s["compact"], s["kept_idx"], s["kept"], s["full"])
        return {"hidden": s["full"]}
    outs = (s["hidden_out"], s["pos_out"], s["kept_idx"], s["new_cu"], s["scores"], s["workspace"], s["ws_bytes"])
    ratio = (s["ratio"], s["ratio_host"])
    if s["entry"] == "fused":
        up.uniprefill_fused(s["p"], s["q"], s["k"], s["hidden"], s["pos"], s["cu"], s["cu_host"], *ratio, *outs)
    elif s["entry"] == "top_p":
        up.uniprefill_fused_top_p(s["p"], s["q"], s["k"], s["hidden"], s["pos"], s["cu"], s["cu_host"], *ratio, *outs)
    elif s["entry"] == "paged":
        up.uniprefill_fused_paged(s["p"], s["q"], s["k"], s["hidden"], s["pos"], s["cu"], s["cu_host"], s["cu_k"],
                                  s["cu_k_host"], s["table"], s["table"].shape[1], KV_BLOCK, *ratio, *outs)
    else:
        up.uniprefill_fused_lse(s["p"], s["q"], s["k"], s["lse"], s["lse"].shape[1], s["hidden"], s["pos"], s["cu"],
                                s["cu_host"], None, None, None, 0, KV_BLOCK, *ratio, *outs)
    result = {"hidden": s["hidden_out"], "pos": s["pos_out"], "kept_idx": s["kept_idx"], "new_cu": s["new_cu"]}
    if s["scores"] is not None:
        result["scores"] = s["scores"]
    return result
