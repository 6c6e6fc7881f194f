"""Performance cases of libpevlm: what a prefill of a long video prompt calls, through the Python binding.

A case is a dict of plain values.  `kind` names the calls of one pass:

  layer     pevlm_rope_seq, pevlm_block_prefill_attn, pevlm_query_attn: one attention layer of a prompt
  attn      the two attention calls on tensors that the caller has already rotated
  fused     pevlm_block_prefill_attn_mrope, pevlm_query_attn_mrope: the layer with three-axis RoPE folded in
  fp8       pevlm_block_prefill_attn_fp8 (both stages)
  append    a new context block at the end of a streamed video: pevlm_rope_seq on its rows and the
            question's, pevlm_block_prefill_attn_blocks, pevlm_query_attn_window
  question  pevlm_query_attn_rope with lse: a further question about a video whose keys are cached
  dense     pevlm_block_prefill_attn over one block without a sink: ordinary full causal attention

`seqs` is a text "S:B:C:Q,S:B:C:Q,...": sink, block, context and question lengths of each packed sequence.
"""
import math

import torch

import paper_2506_19651_amd as P

DEV = "cuda:0"

# Head shapes (query heads, KV heads, head_dim): the 7B video models' attention layers, the larger GQA
# group, and the small one with 64-wide heads.
HEADS_7B, HEADS_GQA8, HEADS_D64 = (28, 4, 128), (32, 8, 128), (14, 2, 64)


def _case(name, kind, heads, seqs, dtype="bf16", **more):
    c = {"name": name} if name else {}
    c.update(kind=kind, dtype=dtype, hq=heads[0], hkv=heads[1], d=heads[2],
             seqs=",".join(":".join(str(int(x)) for x in s) for s in seqs))
    c.update(more)
    return c


def listed():
    return [
        # One layer of a toy prompt in fp32, all 104 tokens of it: six tiny launches, latency only.
        _case("tiny_f32", "layer", (2, 1, 64), [(32, 16, 64, 8)], dtype="f32", base=1.0e4),
        # The fp32 path as a numerical check of a bf16 deployment: a short clip at the real head shape.
        _case("check_f32", "layer", HEADS_7B, [(256, 1024, 2048, 64)], dtype="f32"),
        # A few images and a question, lengths that fill no tile, 64-wide heads.
        _case("short_odd_d64", "layer", HEADS_D64, [(77, 333, 2900, 21)]),
        # 64 frames of 256 tokens (16K): an ordinary clip.
        _case("layer_16k", "layer", HEADS_7B, [(256, 1024, 16384, 64)]),
        # 256 frames (64K): the long video that the headline benchmark runs.
        _case("layer_64k", "layer", HEADS_7B, [(256, 1024, 65536, 128)], offset=0.3),
        # 512 frames of 196 tokens (100K) in blocks of two frames: the many-short-blocks end.
        _case("attn_100k_short_blocks", "attn", HEADS_GQA8, [(392, 392, 100352, 256)]),
        # The same video in blocks of 16 frames with RoPE folded in: the long-block end, the largest case.
        _case("fused_100k_long_blocks", "fused", HEADS_GQA8, [(392, 3136, 100352, 256)]),
        # Four requests of very different length in one batch, every last block partial.
        _case("batch_ragged", "layer", HEADS_7B, [(256, 1024, 256 * f, 64) for f in (33, 97, 161, 255)]),
        # The 8-bit variant of the 64K prefill.
        _case("fp8_64k", "fp8", HEADS_7B, [(256, 1024, 65536, 128)], offset=0.3),
        # Streaming: one block of four frames arrives, the question looks back over 16 of 64 blocks.
        _case("append_64k", "append", HEADS_7B, [(256, 1024, 65536, 128)], window=16),
        # A short follow-up question over 64K cached tokens.
        _case("question_64k", "question", HEADS_7B, [(256, 1024, 65536, 20)]),
        # Full causal attention at 16K, what the method is compared with.
        _case("dense_16k", "dense", HEADS_7B, [(0, 16448, 16448, 0)]),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _prompt(rng, max_ctx, max_block=3200, max_q=256):
    """(S, B, C, Q) of a prompt: video lengths over their logarithm; half of them whole frames, half odd."""
    sink, block = _log_int(rng, 16, 600), _log_int(rng, 128, max_block)
    ctx, q = _log_int(rng, 1024, max_ctx), _log_int(rng, 1, max_q)
    if rng.random() < 0.5:
        frame = rng.choice([196, 256])
        sink, block = frame * rng.choice([1, 2]), frame * max(1, block // frame)
        ctx = frame * max(1, ctx // frame)
    return sink, min(block, ctx), ctx, q


def draw(rng):
    top = listed()
    most = {"bf16": max(work(c)["flops"] for c in top if c["dtype"] == "bf16"),
            "f32": max(work(c)["flops"] for c in top if c["dtype"] == "f32")}
    while True:
        kind = rng.choice(["layer", "layer", "layer", "attn", "fused", "fp8", "append", "question", "dense", "f32"])
        heads = rng.choice([HEADS_7B, HEADS_7B, HEADS_GQA8, HEADS_D64])
        if kind == "f32":
            c = _case("", "layer", heads, [_prompt(rng, 4096, 1100, 64)], dtype="f32")
        elif kind == "dense":
            n = _log_int(rng, 1024, 17000)
            c = _case("", "dense", heads, [(0, n, n, 0)])
        elif kind == "append":
            s, b, n, q = _prompt(rng, 100000)
            c = _case("", "append", heads, [(s, b, n, q)], window=max(1, -(-n // b) // rng.choice([2, 4, 8])))
        else:
            count = rng.choice([1, 1, 1, 2, 4])
            c = _case("", kind, heads, [_prompt(rng, 100000 // count) for _ in range(count)])
            if kind != "question" and rng.random() < 0.25:
                c["offset"] = 0.3
        if work(c)["flops"] <= most[c["dtype"]]:
            return c


# ------------------------------------------------------------------------------------------ sizes
def _seqs(case):
    return [tuple(int(x) for x in s.split(":")) for s in case["seqs"].split(",")]


def _append_span(case):
    """(first row of the newest block, first row of the question, all rows, first visible row of the window)."""
    s, b, c, q = _seqs(case)[0]
    n = -(-c // b)
    return s + (n - 1) * b, s + c, s + c + q, s + max(0, n - case["window"]) * b


def work(case):
    hq, hkv, d = case["hq"], case["hkv"], case["d"]
    e = 4 if case["dtype"] == "f32" else 2
    q_row, kv_row = hq * d * e, hkv * d * e  # bytes of one token's row of Q (or the output) and of K (or V)
    seqs, kind = _seqs(case), case["kind"]
    tri = lambda n: n * (n + 1) // 2
    if kind == "append":
        s = seqs[0][0]
        b0, q0, end, w0 = _append_span(case)
        rows, q, seen = end - b0, end - q0, s + end - w0
        pairs = (q0 - b0) * s + tri(q0 - b0) + q * (s + q0 - w0) + tri(q)
        # new rows: Q read and rotated in place, K rotated, outputs; K and V of what the question sees
        return {"bytes": rows * (3 * q_row + kv_row) + 2 * seen * kv_row, "flops": 4 * d * hq * pairs}
    prefill = sum(tri(s) + (c // b) * (b * s + tri(b)) + (c % b) * s + tri(c % b) for s, b, c, _ in seqs)
    question = sum(q * (s + c) + tri(q) for s, _, c, q in seqs)
    tokens, asked = sum(s + c + q for s, _, c, q in seqs), sum(q for _, _, _, q in seqs)
    if kind == "question":
        return {"bytes": 2 * asked * q_row + 2 * tokens * kv_row + 4 * asked * hq, "flops": 4 * d * hq * question}
    if kind in ("fp8", "dense"):
        rows = tokens - asked
        return {"bytes": rows * (2 * q_row + 2 * kv_row), "flops": 4 * d * hq * prefill}
    bytes_ = tokens * (2 * q_row + 2 * kv_row)  # Q, K, V in, outputs out
    if kind == "layer":
        bytes_ += tokens * (q_row + kv_row)  # Q and K are rotated in place
    elif kind == "fused":
        bytes_ += tokens * (kv_row + 12)  # K in place, three ids a token
    return {"bytes": bytes_, "flops": 4 * d * hq * (prefill + question)}


def tolerance(case):
    # Measured against the same inputs in 64 bits (fp32 path: 4e-7, largest 5e-6) and in fp32 (bf16 path: 2.4e-3, largest
    # 6e-2, one rounding each of the rotated operands, the weights and the result; 8-bit variant: 3.7e-2, codes of
    # three bits), four times that where the limit on a tolerance leaves it.
    if case["kind"] == "fp8":
        return {"rel": 0.03, "max": 0.9}
    return {"rel": 3e-6, "max": 3e-5} if case["dtype"] == "f32" else {"rel": 1e-2, "max": 0.25}


# ------------------------------------------------------------------------------------------ state and pass
def _three_axis_ids(seqs, frame=196, wide=14):
    """Position ids [3][T] of a video prompt: frames of `frame` tokens on a grid, then the question as text."""
    parts = []
    for s, _, c, q in seqs:
        j = torch.arange(s + c, dtype=torch.int32)
        f, r, w = j // frame, j % frame // wide, j % wide
        after = int(max(f.max(), r.max(), w.max())) + 1
        text = after + torch.arange(q, dtype=torch.int32)
        parts.append(torch.cat([torch.stack([f, r, w]), text.expand(3, q)], dim=1))
    return torch.cat(parts, dim=1).contiguous()


def prepare(case, seed):
    seqs, kind = _seqs(case), case["kind"]
    hq, hkv, d = case["hq"], case["hkv"], case["d"]
    dtype = torch.float32 if case["dtype"] == "f32" else torch.bfloat16
    lay, heads = P.Layout.from_seqs(seqs), P.Heads(hq, hkv, d, case["dtype"])
    tokens = lay.total_tokens
    gen = torch.Generator(device=DEV).manual_seed(int(seed))

    def normal(h, scale):
        return torch.randn(tokens, h, d, device=DEV, dtype=dtype, generator=gen).mul_(scale)

    scale = 1.0 if dtype is torch.float32 else 0.5
    q, k, v = normal(hq, scale), normal(hkv, scale), normal(hkv, scale)
    if case.get("offset"):  # keys around a mean of their head, as trained models have them
        k += (torch.randn(1, hkv, d, device=DEV, generator=gen) * case["offset"]).to(dtype)
    base = case.get("base", 1.0e6)
    st = {"kind": kind, "lay": lay, "heads": heads, "base": base, "q": q, "k": k, "v": v, "out": torch.zeros_like(q)}
    space = lambda n: torch.empty(max(int(n), 256), dtype=torch.uint8, device=DEV)
    if kind in ("attn", "fp8", "dense"):  # these callers hold rotated tensors
        P.pevlm_rope_seq(q, k, lay, heads, base)
    elif kind == "question":
        P.pevlm_rope_seq(None, k, lay, heads, base)
    if kind in ("layer", "attn"):
        st["ws_p"] = space(P.pevlm_block_prefill_workspace_bytes(lay, heads))
        st["ws_q"] = space(P.pevlm_query_workspace_bytes(lay, heads))
    elif kind == "dense":
        st["ws_p"] = space(P.pevlm_block_prefill_workspace_bytes(lay, heads))
    elif kind == "fused":
        half = d // 2
        st["section"] = (half // 4, half * 3 // 8, half - half // 4 - half * 3 // 8)
        st["ids"] = _three_axis_ids(seqs).to(DEV)
        st["ws_p"] = space(P.pevlm_block_prefill_rope_workspace_bytes(lay, heads))
        st["ws_q"] = space(P.pevlm_query_rope_workspace_bytes(lay, heads))
    elif kind == "fp8":
        st["ws_p"] = space(P.pevlm_block_prefill_fp8_workspace_bytes(lay, heads))
    elif kind == "question":
        st["lse"] = torch.zeros(tokens, hq, dtype=torch.float32, device=DEV)
        st["ws_q"] = space(P.pevlm_query_rope_workspace_bytes(lay, heads))
        cu = [int(x) for x in lay.cu]
        st["asked"] = [(cu[i + 1] - s[3], cu[i + 1]) for i, s in enumerate(seqs)]
    elif kind == "append":
        b0, q0, end, _ = _append_span(case)
        P.pevlm_rope_seq(None, k, P.Layout.from_seqs([(0, 1, 0, b0)]), heads, base)  # the keys that are cached
        st["b0"], st["new"] = b0, P.Layout.from_seqs([(0, 1, 0, end - b0)])  # the rows that are new
        st["block"], st["window"] = -(-seqs[0][2] // seqs[0][1]) - 1, case["window"]
        st["ws_p"] = space(P.pevlm_block_prefill_workspace_bytes(lay, heads))
        st["ws_q"] = space(P.pevlm_query_window_workspace_bytes(lay, heads))
    return st


def run(st):
    kind, lay, heads, base = st["kind"], st["lay"], st["heads"], st["base"]
    q, k, v, out = st["q"], st["k"], st["v"], st["out"]
    if kind in ("layer", "attn"):
        if kind == "layer":
            P.pevlm_rope_seq(q, k, lay, heads, base)
        P.pevlm_block_prefill_attn(q, k, v, out, lay, heads, workspace=st["ws_p"])
        P.pevlm_query_attn(q, k, v, out, lay, heads, workspace=st["ws_q"])
        return {"out": out, "q": q, "k": k} if kind == "layer" else out
    if kind == "dense":
        P.pevlm_block_prefill_attn(q, k, v, out, lay, heads, workspace=st["ws_p"])
        return out
    if kind == "fp8":
        P.pevlm_block_prefill_attn_fp8(q, k, v, out, lay, heads, workspace=st["ws_p"])
        return out
    if kind == "fused":
        P.pevlm_block_prefill_attn_mrope(q, k, v, out, lay, heads, base, st["ids"], st["section"], workspace=st["ws_p"])
        P.pevlm_query_attn_mrope(q, k, v, out, lay, heads, base, st["ids"], st["section"], workspace=st["ws_q"])
        return {"out": out, "k": k}
    if kind == "question":
        P.pevlm_query_attn_rope(q, k, v, out, lay, heads, base, lse=st["lse"], workspace=st["ws_q"])
        return [(out[a:b], st["lse"][a:b]) for a, b in st["asked"]]
    b0 = st["b0"]
    P.pevlm_rope_seq(q[b0:], k[b0:], st["new"], heads, base, pos_offset=[b0])
    P.pevlm_block_prefill_attn_blocks(q, k, v, out, lay, heads, [st["block"]], [1], False, workspace=st["ws_p"])
    P.pevlm_query_attn_window(q, k, v, out, lay, heads, [st["window"]], workspace=st["ws_q"])
    return {"out": out[b0:], "q": q[b0:], "k": k[b0:]}
