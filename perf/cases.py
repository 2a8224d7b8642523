"""The work this library is called for, as cases that a timing program can run.

A case is one pass through the public entry points of `paper_2508_01989_amd`, on tensors that are
already on the GPU:

  "step"       KV append and mixed attention of one batch, one layer, the plan at hand (a serving loop makes
               it once per iteration and uses it for every layer); `fused` says whether the program calls
               tc_mixed_attention_append or tc_kv_append and tc_mixed_attention
  "iteration"  what a serving loop does per iteration: Plan.update, then a step for each of `layers` layers
  "export"     tc_kv_export of whole requests, all layers
  "import"     tc_kv_import of whole requests, all layers

A batch is given by `chunks` (prompt chunks as "tokens@offset", blank-separated) and by `decodes` running
requests whose context lengths follow from `context` ("lognormal mean sigma low high" or "uniform low high")
and `lengths` (the seed of the draw), so that a case says the lengths by itself; the seed given to
prepare() makes tensors and block tables.  Element types are bf16 and IEEE half, head_dim 64 and 128.
"""
import math

import numpy as np
import torch

import paper_2508_01989_amd as tc

BLOCK = 16  # tokens per KV block
GPU = "cuda:0"


def _step(name, heads, kv_heads, head_dim, dtype, chunks, decodes, context, lengths, fused, gain=1.0):
    return {"name": name, "kind": "step", "heads": heads, "kv_heads": kv_heads, "head_dim": head_dim, "dtype": dtype, "chunks": chunks,
            "decodes": decodes, "context": context, "lengths": lengths, "layers": 1, "fused": fused, "gain": gain}


def listed():
    return [
        # The smallest call: a short first chunk with four decodes of a small model; launches and latency are all there is.
        _step("tiny", 8, 8, 64, "bf16", "64@0", 4, "uniform 37 128", 1, False),
        # An instance at low load: a handful of chat requests, decode only.
        _step("decode_few", 32, 8, 128, "bf16", "", 8, "lognormal 1024 0.8 64 8192", 2, True),
        # Two users with long documents: few sequences, long contexts, more query heads.
        _step("decode_long_context", 64, 8, 128, "bf16", "", 2, "uniform 16384 32768", 3, True),
        # An instance of the decode-heavy kind at moderate load, over a whole iteration of sixteen layers: the batch
        # is planned, then each layer appends and attends; a small chunk of a prompt rides along.  The precision and the
        # group of five query heads per KV head are those of the serving experiments this path comes from.
        {**_step("iteration", 40, 8, 128, "fp16", "128@1000", 32, "uniform 512 4096", 4, False, 2.0), "kind": "iteration", "layers": 16},
        # Decode only, at the number of requests that fills the memory.
        _step("pure_decode", 32, 8, 128, "bf16", "", 512, "lognormal 2048 1.0 16 16384", 5, False),
        # The decode-heavy kind at full load: small chunk, many decodes.
        _step("decode_heavy", 32, 8, 128, "bf16", "256@1234", 256, "uniform 512 4096", 6, False),
        # The prefill-heavy kind: a large chunk in the middle of a prompt, some decodes.
        _step("prefill_heavy", 32, 8, 128, "bf16", "2048@4096", 64, "lognormal 1024 0.8 64 8192", 7, False),
        # The same for a model with the smaller head size.
        _step("prefill_heavy_d64", 32, 8, 64, "bf16", "2048@4096", 64, "lognormal 1024 0.8 64 8192", 7, False),
        # New chat prompts: several first chunks of odd lengths in one batch, short contexts, some decodes.
        _step("new_prompts", 40, 8, 128, "fp16", "701@0 333@0 45@0", 16, "lognormal 1024 0.8 64 8192", 8, False, 2.0),
        # The largest call: the last chunk of a long document, with decodes of other long documents.
        _step("long_prompt", 64, 8, 128, "bf16", "8192@24576", 32, "uniform 1024 32768", 9, False),
        # Requests leave an instance: sixteen at once, thirty-two layers, into a transfer buffer.
        {**_step("export", 32, 8, 128, "bf16", "", 16, "lognormal 2048 1.0 16 16384", 10, False), "kind": "export", "layers": 32},
        # One request arrives after its prefill: from the transfer buffer into this instance's blocks.
        {**_step("import_one", 40, 8, 128, "fp16", "", 1, "uniform 1500 1600", 11, False), "kind": "import", "layers": 48},
    ]


def draw(rng):
    """One more case of the same ranges: any load from one decode to a full instance, any chunk from none to the largest."""
    def log(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    heads, kv_heads = rng.choice([(32, 8), (32, 8), (40, 8), (64, 8), (8, 8), (32, 32), (16, 2)])
    case = _step("", heads, kv_heads, rng.choice([128, 128, 64]), rng.choice(["bf16", "bf16", "fp16"]), "", 0, "", rng.randrange(1 << 20), False,
                 rng.choice([1.0, 2.0, 3.0]))
    del case["name"]
    token_bytes = 4 * kv_heads * case["head_dim"]  # K and V of one token, one layer
    kind = rng.choice(["step", "step", "step", "step", "iteration", "export", "import"])
    case["kind"] = kind
    mean = log(64, 16384)
    case["context"] = rng.choice(["lognormal %d 0.8 16 16384" % mean, "lognormal %d 1.0 16 32768" % mean, "uniform %d %d" % (max(1, mean // 4), 2 * mean)])
    if kind in ("export", "import"):
        case["layers"] = rng.choice([16, 32, 48])
        most = int(2.5e9 / (token_bytes * case["layers"] * 2 * mean))
        case["decodes"] = max(1, min(log(1, 32), most))
        return case
    if kind == "iteration":
        case["layers"] = rng.choice([4, 8, 16])
    budget = 2.0e9 / case["layers"]  # bytes of K and V that the decodes of one layer read
    case["decodes"] = max(1, min(log(1, 512), int(budget / (token_bytes * 2 * mean))))
    if rng.random() < 0.7:  # a chunk, or two or three of them
        n = rng.choice([1, 1, 1, 2, 3])
        chunks = []
        for _ in range(n):
            tokens = log(2, 8192 // n)
            offset = rng.choice([0, log(1, 24576)])
            # no more work than a large chunk in the middle of a long prompt
            while 4 * case["head_dim"] * heads * tokens * (offset + tokens / 2) * case["layers"] * n > 3.0e12:
                tokens, offset = (tokens + 1) // 2, offset // 2
            chunks.append("%d@%d" % (max(2, tokens), offset))
        case["chunks"] = " ".join(chunks)
        if rng.random() < 0.2:
            case["decodes"], case["context"] = 0, "uniform 1 1"
    case["fused"] = rng.random() < 0.4
    return case


def _lengths(case):
    """New tokens and cached tokens of every sequence: the chunks, then the decodes (their context counts the new token)."""
    rs = np.random.RandomState(case["lengths"] % (1 << 31))
    law, *num = case["context"].split()
    num = [float(x) for x in num]
    n = case["decodes"]
    if law == "lognormal":
        mean, sigma, lo, hi = num
        kv = np.clip(np.rint(np.exp(rs.normal(math.log(mean) - 0.5 * sigma * sigma, sigma, n))), lo, hi)
    else:
        kv = rs.randint(int(num[0]), int(num[1]) + 1, n)
    chunks = [tuple(int(x) for x in c.split("@")) for c in case["chunks"].split()]
    q_len = np.array([c[0] for c in chunks] + [1] * n, np.int64)
    ctx = np.array([c[1] for c in chunks] + [int(x) - 1 for x in kv], np.int64)
    return q_len, ctx


def _dtype(case):
    return (torch.bfloat16, tc.TC_BF16) if case["dtype"] == "bf16" else (torch.float16, tc.TC_FP16)


def _tables(kv_len, rs):
    """Block tables over a pool with a quarter of its blocks to spare, the blocks scattered as a running allocator leaves them."""
    pages = -(-kv_len // BLOCK)
    blocks = int(pages.sum()) + max(4, int(pages.sum()) // 4)
    ids = rs.permutation(blocks).astype(np.int32)
    table = np.zeros((len(kv_len), int(pages.max())), np.int32)
    at = 0
    for s, n in enumerate(pages):
        table[s, :n] = ids[at:at + n]
        at += n
    return table, blocks


def prepare(case, seed):
    q_len, ctx = _lengths(case)
    dtype, code = _dtype(case)
    heads, kv_heads, dim, layers = case["heads"], case["kv_heads"], case["head_dim"], case["layers"]
    rs = np.random.RandomState((seed * 2 + 1) % (1 << 31))
    gen = torch.Generator(device=GPU).manual_seed(seed)
    table, blocks = _tables(q_len + ctx, rs)
    q_start = np.concatenate([[0], np.cumsum(q_len)]).astype(np.int32)
    tokens = int(q_start[-1])

    def normal(gain, *shape):
        return torch.empty(shape, dtype=dtype, device=GPU).normal_(0.0, gain, generator=gen)

    state = {"case": case, "q_len": q_len, "ctx": ctx.astype(np.int32), "q_start": q_start, "table": table, "scale": 1.0 / math.sqrt(dim)}
    pool_elems = blocks * kv_heads * BLOCK * dim
    state["k"] = normal(1.0, layers, pool_elems)
    state["v"] = normal(1.0, layers, pool_elems)
    pools = [tc.make_pool(heads, kv_heads, dim, blocks, state["k"][i], state["v"][i], dtype=code) for i in range(layers)]
    state["pools"] = pools
    state["plan"] = tc.Plan(pools[0], q_start, state["ctx"], table)
    if case["kind"] in ("export", "import"):
        n_bytes = tc.tc_kv_transfer_bytes(state["plan"], -1, layers)
        state["buffer"] = normal(1.0, n_bytes // 2)
        state["k_layers"], state["v_layers"] = list(state["k"]), list(state["v"])
        return state
    state["q"] = normal(case["gain"], layers, tokens, heads, dim)
    state["k_new"], state["v_new"] = normal(1.0, layers, tokens, kv_heads, dim), normal(1.0, layers, tokens, kv_heads, dim)
    state["out"] = torch.zeros((layers, tokens, heads, dim), dtype=dtype, device=GPU)
    state["workspace"] = torch.empty(max(16, state["plan"].workspace_bytes), dtype=torch.uint8, device=GPU)
    return state


def run(state):
    case, plan = state["case"], state["plan"]
    if case["kind"] == "export":
        tc.tc_kv_export(plan, state["pools"][0], -1, state["k_layers"], state["v_layers"], state["buffer"])
        return state["buffer"].view(torch.int16)
    if case["kind"] == "import":
        tc.tc_kv_import(plan, state["pools"][0], -1, state["k_layers"], state["v_layers"], state["buffer"])
        return state["k"].view(torch.int16), state["v"].view(torch.int16)
    if case["kind"] == "iteration":
        plan.update(state["pools"][0], state["q_start"], state["ctx"], state["table"])
    workspace = state["workspace"]
    for i in range(case["layers"]):
        pool, q, k_new, v_new, out = state["pools"][i], state["q"][i], state["k_new"][i], state["v_new"][i], state["out"][i]
        if case["fused"]:
            tc.tc_mixed_attention_append(plan, pool, q, k_new, v_new, out, state["scale"], workspace)
        else:
            tc.tc_kv_append(plan, pool, k_new, v_new)
            tc.tc_mixed_attention(plan, pool, q, out, state["scale"], workspace)
    # the pools are bit copies: compared as whole numbers
    return state["out"], state["k"].view(torch.int16), state["v"].view(torch.int16)


def work(case):
    q, c = _lengths(case)
    heads, kv_heads, dim, layers = case["heads"], case["kv_heads"], case["head_dim"], case["layers"]
    kv_token = 4 * kv_heads * dim  # bytes of K and V of one token
    if case["kind"] in ("export", "import"):
        return {"bytes": 2 * layers * int((-(-(q + c) // BLOCK) * BLOCK).sum() if case["kind"] == "export" else (q + c).sum()) * kv_token, "flops": 0}
    pairs = int((q * c + q * (q + 1) // 2).sum())
    # cached tokens read once per KV head, the new rows read and stored, Q in, O out
    n_bytes = int(c.sum()) * kv_token + 2 * int(q.sum()) * kv_token + 2 * int(q.sum()) * heads * dim * 2
    return {"bytes": layers * n_bytes, "flops": layers * 4 * dim * heads * pairs}


def tolerance(case):
    """The probabilities and the outputs are rounded to the element type: two correct programs that cut the sums in
    other places differ by about a rounding of each (measured against 64 bits: about 2.3e-3 in bf16 and 3e-4 in half)."""
    if case["kind"] in ("export", "import"):
        return "exact"
    return {"rel": 8e-3, "max": 0.06} if case["dtype"] == "bf16" else {"rel": 1.2e-3, "max": 0.01}


def _slot(t):
    return (t & 3) | ((t & 4) << 1) | ((t & 8) >> 1)


def exact(case, seed):
    if case["kind"] in ("export", "import"):
        return None
    state = prepare(case, seed)
    heads, kv_heads, dim = case["heads"], case["kv_heads"], case["head_dim"]
    group = heads // kv_heads
    slots = torch.tensor([_slot(t) for t in range(BLOCK)], device=GPU)
    out = torch.zeros(state["out"].shape, dtype=torch.float64, device=GPU)
    for i in range(case["layers"]):
        k_pool = state["k"][i].view(-1, kv_heads, dim // 8, BLOCK, 8)
        v_pool = state["v"][i].view(-1, kv_heads, dim, BLOCK)
        for s, (n, c) in enumerate(zip(state["q_len"].tolist(), state["ctx"].tolist())):
            a = int(state["q_start"][s])
            ids = torch.from_numpy(state["table"][s, :-(-(c + n) // BLOCK)].astype(np.int64)).to(GPU)
            k = k_pool[ids].permute(0, 3, 1, 2, 4).reshape(-1, kv_heads, dim)[:c]
            v = v_pool[ids][..., slots].permute(0, 3, 1, 2).reshape(-1, kv_heads, dim)[:c]
            k = torch.cat([k, state["k_new"][i, a:a + n]]).permute(1, 2, 0).double().contiguous()  # [kv_heads][dim][tokens]
            v = torch.cat([v, state["v_new"][i, a:a + n]]).permute(1, 0, 2).double().contiguous()  # [kv_heads][tokens][dim]
            rows = max(1, (1 << 27) // (heads * (c + n)))  # query rows at a time: a gibibyte of scores
            for r in range(0, n, rows):
                m = min(rows, n - r)
                q = state["q"][i, a + r:a + r + m].double().view(m, kv_heads, group, dim).permute(1, 2, 0, 3).reshape(kv_heads, group * m, dim)
                x = torch.bmm(q.contiguous(), k).mul_(state["scale"]).view(kv_heads, group, m, c + n)
                if n > 1:
                    at = torch.arange(c + n, device=GPU)
                    x.masked_fill_(at[None, :] > c + r + torch.arange(m, device=GPU)[:, None], -math.inf)
                x = torch.softmax(x, -1).view(kv_heads, group * m, c + n)
                o = torch.bmm(x, v).view(kv_heads, group, m, dim).permute(2, 0, 1, 3).reshape(m, heads, dim)
                out[i, a + r:a + r + m] = o
    return out, None, None
