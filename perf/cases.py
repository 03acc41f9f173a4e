"""The calls this library is used for, as cases that can be timed and checked.

A case is one call, or the few calls of one step, through the Python binding of the C entry
points: a decode step over a packed cache, the query-key product alone, a prefill's encoders, or a
serving step that appends a key and then attends.  `listed()` names the shapes the repository is
configured, tested and benchmarked on; `draw()` gives further ones from the same ranges.

The packed cache a decode call reads is made here with plain torch (pair, radius, angle,
group-wise quantization, packing), not with the library's own encoders, so that `exact()` can
evaluate the same cache in float64 without any of the library's code.
"""
import math
import random

import torch

import paper_2502_00527_amd as pq

HEAD_DIM = 128
PAIRS = HEAD_DIM // 2
GROUP = 128
DEVICE = "cuda:0"

# ---- cases -----------------------------------------------------------------------------------


def _case(name, op, seqs, q_heads, kv_heads, context, **more):
    case = dict(name=name, op=op, seqs=seqs, q_heads=q_heads, kv_heads=kv_heads, context=context,
                min_context=context, r_bits=4, t_bits=4, grouped_angles=False, v_bits=16, dtype="f16",
                shuffled_pages=False, rope_base=5.0e5)
    case.update(more)
    return case


def listed():
    return [
        # one user, a short prompt: the smallest call a chat turn makes, launches and latency count
        _case("decode_one_short", "decode", 1, 32, 8, 777),
        # a serving batch at long context, 4 query heads per KV head: the benchmark's workload
        _case("decode_gqa", "decode", 16, 32, 8, 32768),
        # every query head has its KV head, moderate context
        _case("decode_mha", "decode", 8, 32, 32, 8192, rope_base=1.0e4),
        # a single very long document at low bits: few sequences, many pages each
        _case("decode_long_r3t3", "decode", 1, 32, 8, 131072, r_bits=3, t_bits=3),
        # continuous batching: lengths all over the place, pages scattered in the pool
        _case("decode_ragged", "decode", 64, 32, 8, 16384, min_context=1024, shuffled_pages=True),
        # wide query groups: 8 query heads per KV head
        _case("decode_group8", "decode", 16, 64, 8, 32768),
        # values quantized too, to 4 bits, at the benchmark's shape
        _case("decode_v4", "decode", 16, 32, 8, 32768, v_bits=4),
        # the smallest cache: 3+3-bit keys, 2-bit values, ragged medium contexts
        _case("decode_r3t3_v2_ragged", "decode", 32, 32, 8, 8192, min_context=512, r_bits=3, t_bits=3, v_bits=2,
              shuffled_pages=True),
        # the group-wise angle quantizer
        _case("decode_grouped_angles", "decode", 16, 32, 8, 16384, grouped_angles=True),
        # the query-key product alone, raw scores to memory (attention variants that bring their own softmax)
        _case("score_batch8", "score", 8, 32, 8, 32768),
        # a long prompt comes in: its keys are packed and its values quantized
        _case("prefill_v4", "prefill", 1, 32, 8, 32768, v_bits=4),
        # one generation step of a ragged batch: append the new key to the fp16 tail, then attend over
        # packed groups and tail; an odd number of sequences, one of them completing a group
        _case("serve_step", "serve", 31, 32, 8, 3000, min_context=200, shuffled_pages=True),
    ]


def draw(rng):
    op = rng.choice(["decode"] * 6 + ["score"] * 2 + ["prefill"] * 2 + ["serve"] * 2)
    r_bits, t_bits = rng.choice([(4, 4), (4, 4), (3, 3), (3, 3), (5, 3), (3, 5), (4, 2), (2, 4)])
    kv_heads = rng.choice([1, 2, 4, 8, 8, 8, 32])
    group = 1 if kv_heads == 32 else rng.choice([1, 2, 4, 4, 4, 8, 6, 7, 16])
    case = _case(None, op, 1, kv_heads * group, kv_heads, 0, r_bits=r_bits, t_bits=t_bits,
                 grouped_angles=rng.random() < 0.2, dtype=rng.choice(["f16", "f16", "f16", "f32"]),
                 v_bits=rng.choice([16, 16, 16, 4, 2]), shuffled_pages=rng.random() < 0.5,
                 rope_base=rng.choice([1.0e4, 5.0e5]))
    del case["name"]
    if op == "prefill":
        case["context"] = case["min_context"] = round(math.exp(rng.uniform(math.log(100), math.log(32768))))
        return case
    # scores per step between a short prompt's and the largest listed case's
    most = 16 * 64 * 32768
    scores = math.exp(rng.uniform(math.log(32 * 300), math.log(most)))
    tokens = max(64, min(16 * 8 * 32768, scores / group) / kv_heads)      # over all sequences
    case["seqs"] = max(1, min(128, round(math.exp(rng.uniform(0.0, math.log(max(2.0, tokens / 64)))))))
    # the longest sequence; lengths of a ragged batch are spread below it
    case["context"] = max(32, min(131072, round(tokens / case["seqs"]) - rng.randrange(3)))
    case["min_context"] = case["context"]
    if case["seqs"] > 1 and rng.random() < 0.6:
        case["min_context"] = max(1, case["context"] // rng.choice([2, 8, 16]))
    return case


def _lengths(case):
    """Context length of every sequence: a property of the case, the same for every seed."""
    if case["op"] == "serve":
        lens = _spread(case)
        lens[0] = lens[0] // GROUP * GROUP + GROUP - 1        # this one completes a group with the appended key
        return lens
    return _spread(case)


def _spread(case):
    if case["min_context"] == case["context"]:
        return [case["context"]] * case["seqs"]
    rng = random.Random(case["context"] * 1009 + case["seqs"])
    return [rng.randint(case["min_context"], case["context"]) for _ in range(case["seqs"])]


# ---- inputs: keys with outlier channels under RoPE, quantized and packed with plain torch -----


def _generator(seed, stream):
    g = torch.Generator(device=DEVICE)
    g.manual_seed((seed * 1000003 + stream) % (2 ** 63))
    return g


def _float_dtype(case):
    return torch.float16 if case["dtype"] == "f16" else torch.float32


def _keys(case, seed, seq, length):
    """Post-RoPE keys [length, kv_heads, d]: N(0, 1) with 2 outlier channels of 8 times the size per head."""
    g = _generator(seed, 10 * seq + 1)
    heads = case["kv_heads"]
    k = torch.randn((length, heads, HEAD_DIM), generator=g, device=DEVICE)
    channel_rng = random.Random(seed)                                    # outliers are a property of the head
    for h in range(heads):
        for pair in channel_rng.sample(range(PAIRS), 2):
            k[:, h, pair + PAIRS * channel_rng.randrange(2)] *= 8.0
    freq = case["rope_base"] ** (-torch.arange(PAIRS, device=DEVICE, dtype=torch.float64) / PAIRS)
    angle = torch.arange(length, device=DEVICE, dtype=torch.float64)[:, None] * freq
    cos, sin = angle.cos().float()[:, None], angle.sin().float()[:, None]
    x, y = k[..., :PAIRS], k[..., PAIRS:]
    return torch.cat([x * cos - y * sin, y * cos + x * sin], dim=-1).to(_float_dtype(case))


def _values(case, seed, seq, length):
    g = _generator(seed, 10 * seq + 2)
    return torch.randn((length, case["kv_heads"], HEAD_DIM), generator=g, device=DEVICE).half()


def _queries(case, seed):
    g = _generator(seed, 3)
    return torch.randn((case["seqs"], case["q_heads"], HEAD_DIM), generator=g, device=DEVICE).to(_float_dtype(case))


def _pages(t, fill):
    """[length, ...] -> [pages, 128, ...], the last page padded with `fill`."""
    pad = -t.shape[0] % GROUP
    if pad:
        t = torch.cat([t, torch.full((pad, *t.shape[1:]), fill, dtype=t.dtype, device=t.device)])
    return t.view(-1, GROUP, *t.shape[1:])


def _min_scale(v, levels):
    """fp16 (scale, zero) over the tokens of each page; v [length, ...]."""
    low = _pages(v, math.inf).amin(dim=1)
    high = _pages(v, -math.inf).amax(dim=1)
    return ((high - low) / levels).half(), low.half()


def _quantize_keys(case, keys):
    """Codes and parameters of one sequence: angle and radius codes [pages, 128, heads, 64], fp16
    (scale, zero) [pages, heads, 64] of the radius and, with grouped angles, of the angle."""
    length = keys.shape[0]
    x, y = keys[..., :PAIRS].float(), keys[..., PAIRS:].float()
    rho = torch.sqrt(x * x + y * y)
    r_levels, t_levels = 2 ** case["r_bits"], 2 ** case["t_bits"]
    s, z = _min_scale(rho, r_levels)
    c = torch.floor((_pages(rho, 0.0) - z.float()[:, None]) / s.float()[:, None])
    c = c.nan_to_num(0.0).clamp_(0, r_levels - 1)
    theta = torch.atan2(y.double(), x.double())
    params = [s, z]
    if case["grouped_angles"]:
        ts, tz = _min_scale(theta, t_levels)
        a = torch.floor((_pages(theta, 0.0) - tz.double()[:, None]) / ts.double()[:, None]).nan_to_num(0.0)
        params += [ts, tz]
    else:
        # a pair on an axis or a diagonal sits exactly on an edge and belongs to the upper bin
        a = torch.floor((_pages(theta, 0.0) + math.pi) * (t_levels / (2 * math.pi)) + 1e-9)
    a = a.clamp_(0, t_levels - 1)
    valid = (torch.arange(c.shape[0] * GROUP, device=DEVICE) < length).view(-1, GROUP, 1, 1)
    return (a * valid).to(torch.uint8), (c * valid).to(torch.uint8), params


def _pack_keys(case, a, c, params):
    """The pools' layout: codes [pages, heads, 4 blocks, 128 tokens, 16 symbols], params {s, z} per pair."""
    n, _, heads, _ = a.shape
    symbol = (a << case["r_bits"]) | c
    symbol = symbol.view(n, GROUP, heads, 4, 16).permute(0, 2, 3, 1, 4)
    if case["r_bits"] + case["t_bits"] == 6:
        four = symbol.reshape(n, heads, 4, GROUP, 4, 4).to(torch.int32)
        word = four[..., 0] | (four[..., 1] << 6) | (four[..., 2] << 12) | (four[..., 3] << 18)
        symbol = torch.stack([word & 255, (word >> 8) & 255, word >> 16], dim=-1).to(torch.uint8).flatten(-2)
    blocks = [torch.stack(params[i:i + 2], dim=-1) for i in range(0, len(params), 2)]
    return symbol.contiguous(), (torch.stack(blocks, dim=2) if len(blocks) == 2 else blocks[0]).contiguous()


def _quantize_values(case, v):
    """Token-wise codes [pages, 128, heads, d] and fp16 (scale, zero) [pages, 128, heads]."""
    v = _pages(v.float(), 0.0)
    levels = 2 ** case["v_bits"] - 1
    low, high = v.amin(dim=-1), v.amax(dim=-1)
    s, z = ((high - low) / levels).half(), low.half()
    code = torch.round((v - z.float()[..., None]) / s.float()[..., None]).nan_to_num(0.0).clamp_(0, levels)
    return code.to(torch.int32), s, z


def _pack_values(case, code, s, z):
    n, _, heads, _ = code.shape
    b = case["v_bits"]
    tokens = 16 // b                                                     # of a 16-byte unit
    per_half = 16 // b if b == 4 else 8                                  # dims in 16 bits
    field = code.view(n, GROUP // tokens, tokens // 2, 2, heads, 16, 8 // per_half, per_half)
    half = torch.zeros(field.shape[:-1], dtype=torch.int32, device=DEVICE)
    for k in range(per_half):
        half |= field[..., k] << (b * k)
    # [page, block, token pair, parity, head, slice, dim half] -> [page, head, block, slice, pair, dim half, parity]
    half = half.permute(0, 4, 1, 5, 2, 6, 3)
    unit = torch.stack([half & 255, half >> 8], dim=-1).to(torch.uint8)
    params = torch.stack([s, z], dim=-1).permute(0, 2, 1, 3)
    return unit.reshape(n, heads, GROUP // tokens, 16, 16), params.contiguous()


def _page_table(case, seed, lens):
    counts = [(n + GROUP - 1) // GROUP for n in lens]
    total = sum(counts)
    ids = torch.arange(total, dtype=torch.int32)
    if case["shuffled_pages"]:
        ids = torch.randperm(total, generator=torch.Generator().manual_seed(seed)).to(torch.int32)
    table = torch.zeros((case["seqs"], max(counts)), dtype=torch.int32)
    at = 0
    for s, n in enumerate(counts):
        table[s, :n] = ids[at:at + n]
        at += n
    return table, counts, total


def _layout(case):
    return pq.Layout(HEAD_DIM, case["r_bits"], case["t_bits"], GROUP, case["kv_heads"], int(case["grouped_angles"]))


def _pools(case, total):
    """Zeroed pools of `total` pages."""
    heads, unit = case["kv_heads"], 2 * (case["r_bits"] + case["t_bits"])
    sets = (2,) if case["grouped_angles"] else ()
    codes = torch.zeros((total, heads, 4, GROUP, unit), dtype=torch.uint8, device=DEVICE)
    params = torch.zeros((total, heads, *sets, PAIRS, 2), dtype=torch.float16, device=DEVICE)
    if case["v_bits"] == 16:
        return codes, params, torch.zeros((total, heads, GROUP, HEAD_DIM), dtype=torch.float16, device=DEVICE), None
    tokens = 16 // case["v_bits"]
    values = torch.zeros((total, heads, GROUP // tokens, 16, 16), dtype=torch.uint8, device=DEVICE)
    return codes, params, values, torch.zeros((total, heads, GROUP, 2), dtype=torch.float16, device=DEVICE)


def prepare(case, seed):
    layout, lens = _layout(case), _lengths(case)
    if case["op"] == "prefill":
        n_pages = (lens[0] + GROUP - 1) // GROUP
        order = torch.arange(n_pages, dtype=torch.int32)
        if case["shuffled_pages"]:
            order = torch.randperm(n_pages, generator=torch.Generator().manual_seed(seed)).to(torch.int32)
        codes, params, v_pool, v_params = _pools(case, n_pages)
        return dict(case=case, layout=layout, keys=_keys(case, seed, 0, lens[0]),
                    values=_values(case, seed, 0, lens[0]), page_ids=order.to(DEVICE), codes=codes, params=params,
                    v_pool=v_pool, v_params=v_params)

    serve = case["op"] == "serve"
    after = [n + 1 for n in lens] if serve else lens                     # a serving step appends one token first
    table, counts, total = _page_table(case, seed, after)
    codes, params, v_pool, v_params = _pools(case, total)
    residual = torch.zeros((case["seqs"], case["kv_heads"], GROUP, HEAD_DIM), dtype=torch.float16,
                           device=DEVICE) if serve else None
    new_keys = torch.empty((case["seqs"], case["kv_heads"], HEAD_DIM), dtype=_float_dtype(case), device=DEVICE)
    for s, length in enumerate(after):
        ids = table[s, :counts[s]].long().to(DEVICE)
        keys = _keys(case, seed, s, length)
        packed = lens[s] // GROUP * GROUP if serve else length           # tokens whose keys are in the pools
        if packed:
            n = (packed + GROUP - 1) // GROUP
            codes[ids[:n]], params[ids[:n]] = _pack_keys(case, *_quantize_keys(case, keys[:packed]))
        if serve:
            new_keys[s] = keys[length - 1]
            tail = keys[packed:length - 1]
            residual[s, :, :tail.shape[0]] = tail.permute(1, 0, 2).half()
        if case["op"] != "score":
            values = _values(case, seed, s, length)
            if v_params is None:
                v_pool[ids] = _pages(values, 0.0).permute(0, 2, 1, 3)
            else:
                v_pool[ids], v_params[ids] = _pack_values(case, *_quantize_values(case, values))
    state = dict(case=case, layout=layout, q=_queries(case, seed), codes=codes, params=params,
                 block_table=table.to(DEVICE), seq_lens=torch.tensor(after, dtype=torch.int32, device=DEVICE),
                 max_seq_len=max(after), sm_scale=1.0 / math.sqrt(HEAD_DIM))
    if case["op"] == "score":
        state["scores"] = torch.zeros((case["seqs"], case["q_heads"], max(after)), device=DEVICE)
        return state
    state.update(v_pool=v_pool, v_params=v_params, v_bits=case["v_bits"],
                 out=torch.zeros((case["seqs"], case["q_heads"], HEAD_DIM), device=DEVICE),
                 workspace=torch.empty(pq.pq_decode_workspace_bytes(layout, case["seqs"], case["q_heads"], max(after)),
                                       dtype=torch.uint8, device=DEVICE))
    if serve:
        # the lengths before the append are kept beside those after it, so that the step can be repeated
        state.update(new_keys=new_keys, residual=residual,
                     lens_before=torch.tensor(lens, dtype=torch.int32, device=DEVICE))
    return state


# ---- one pass --------------------------------------------------------------------------------


def run(state):
    op = state["case"]["op"]
    layout, codes, params = state["layout"], state["codes"], state["params"]
    if op == "prefill":
        pq.pq_encode_keys(layout, state["keys"], state["page_ids"], codes, params)
        if state["v_params"] is None:
            return codes, params
        pq.pq_encode_values(layout, state["case"]["v_bits"], state["values"], state["page_ids"], state["v_pool"],
                            state["v_params"])
        return codes, params, state["v_pool"], state["v_params"]
    if op == "score":
        pq.pq_score_keys(layout, state["q"], codes, params, state["block_table"], state["seq_lens"],
                         state["max_seq_len"], state["scores"])
        return state["scores"]
    residual = None
    if op == "serve":
        residual = state["residual"]
        pq.pq_append_keys(layout, state["new_keys"], residual, state["lens_before"], state["block_table"], codes, params)
    pq.pq_decode_attention(layout, state["q"], codes, params, state["v_pool"], state["block_table"], state["seq_lens"],
                           state["max_seq_len"], state["sm_scale"], state["out"], state["workspace"], None, residual,
                           state["v_bits"], state["v_params"])
    return (state["out"], residual, codes, params) if op == "serve" else state["out"]


# ---- what a pass cannot do without, and how exact its results are ------------------------------


def work(case):
    """Every input read once, every output written once; multiply-adds of q.k and p.v as two operations."""
    lens, heads = _lengths(case), case["kv_heads"]
    tokens = sum(lens) * heads
    code = PAIRS * (case["r_bits"] + case["t_bits"]) / 8 + (4 if case["grouped_angles"] else 2)
    value = 2 * HEAD_DIM if case["v_bits"] == 16 else HEAD_DIM * case["v_bits"] / 8 + 4
    element = 2 if case["dtype"] == "f16" else 4
    if case["op"] == "prefill":
        data = tokens * (HEAD_DIM * element + code)
        if case["v_bits"] != 16:
            data += tokens * (2 * HEAD_DIM + value)
        # per pair: squares, sum, root, angle, minimum and maximum, scaling; per value: minimum, maximum, scaling
        return dict(bytes=data, flops=tokens * (PAIRS * 12 + (0 if case["v_bits"] == 16 else HEAD_DIM * 5)))
    q_rows = case["seqs"] * case["q_heads"] * HEAD_DIM
    scores = sum(lens) * case["q_heads"]
    if case["op"] == "score":
        return dict(bytes=tokens * code + q_rows * element + scores * 4, flops=scores * 2 * HEAD_DIM)
    data = tokens * (code + value) + q_rows * (element + 4)
    if case["op"] == "serve":
        row = heads * HEAD_DIM
        # tail keys are 256 bytes instead of a packed key's; the new row is read and written
        data += sum((n + 1) % GROUP for n in lens) * heads * (2 * HEAD_DIM - code) + case["seqs"] * row * (element + 2)
    return dict(bytes=data, flops=scores * 4 * HEAD_DIM)


def tolerance(case):
    if case["op"] == "prefill":
        return "exact"                                                   # codes are integer decisions
    if case["op"] != "score" and (case["v_bits"] != 16 or case["q_heads"] // case["kv_heads"] >= 8):
        # probabilities meet quantized values, and those of 8-head passes, rounded to 16 bits
        return dict(rel=1.3e-3)
    # 32-bit sums: four times what the path shows against float64
    return dict(rel=5e-7 if case["op"] == "score" else 3e-6)


def _dequantize_keys(case, a, c, params, length):
    """k~ in float64, [heads, length, d]."""
    s, z = params[0].double()[:, None], params[1].double()[:, None]
    rho = (c.double() + 0.5) * s + z
    if case["grouped_angles"]:
        theta = (a.double() + 0.5) * params[2].double()[:, None] + params[3].double()[:, None]
    else:
        theta = (a.double() + 0.5) * (2 * math.pi / 2 ** case["t_bits"]) - math.pi
    k = torch.cat([rho * theta.cos(), rho * theta.sin()], dim=-1)
    return k.view(-1, case["kv_heads"], HEAD_DIM)[:length].permute(1, 0, 2).contiguous()


def exact(case, seed):
    """Scores and attention in float64 over the same cache.  The encoders' outputs are bytes and have
    no float64 counterpart."""
    if case["op"] == "prefill":
        return None
    lens, heads = _lengths(case), case["kv_heads"]
    group = case["q_heads"] // heads
    serve = case["op"] == "serve"
    q = _queries(case, seed).double().view(case["seqs"], heads, group, HEAD_DIM)
    longest = max(lens) + int(serve)
    if case["op"] == "score":
        result = torch.zeros((case["seqs"], heads, group, longest), dtype=torch.float64, device=DEVICE)
    else:
        result = torch.zeros((case["seqs"], heads, group, HEAD_DIM), dtype=torch.float64, device=DEVICE)
    for s, length in enumerate(lens):
        length += int(serve)
        keys = _keys(case, seed, s, length)
        packed = length
        if serve:
            # complete groups are packed -- one that the appended key completes, from its fp16 rows
            packed = length // GROUP * GROUP
            before = (length - 1) // GROUP * GROUP
            keys = torch.cat([keys[:before], keys[before:].half().to(keys.dtype)])
        parts = []
        if packed:
            parts.append(_dequantize_keys(case, *_quantize_keys(case, keys[:packed]), packed))
        if packed < length:
            parts.append(keys[packed:].double().permute(1, 0, 2))
        k = torch.cat(parts, dim=1)
        scores = torch.matmul(k, q[s].transpose(1, 2).contiguous())       # [heads, length, group]
        if case["op"] == "score":
            result[s, :, :, :length] = scores.transpose(1, 2)
            continue
        v = _values(case, seed, s, length)
        if case["v_bits"] == 16:
            v = v.double()
        else:
            code, vs, vz = _quantize_values(case, v)
            v = (code.double() * vs.double()[..., None] + vz.double()[..., None]).view(-1, heads, HEAD_DIM)[:length]
        p = torch.softmax(scores.transpose(1, 2) / math.sqrt(HEAD_DIM), dim=-1).contiguous()
        result[s] = torch.matmul(p, v.permute(1, 0, 2).contiguous())
    result = result.view(case["seqs"], case["q_heads"], -1)
    return (result, None, None, None) if serve else result
