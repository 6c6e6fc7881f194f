"""Kernels at the sizes where their tiling changes: remainders of row groups and key tiles, the borders of
the dispatch rules, the smallest and largest of each range; against the CPU oracle."""
import numpy as np
import pytest
import torch

import paper_2506_19651_amd as P
from paper_2506_19651_amd import cost_model
import workloads as W
from gpu_util import DEV, error_stats, layout_heads, oracle_layout, run_path, to_device, to_host_f32

pytestmark = pytest.mark.gpu

# fp32: sums of n products of N(0,1) values carry about sqrt(n) * 2^-24 relative; every bound of the fp32 path is 1e-5
F32_TOL = 1e-5


@pytest.mark.parametrize("name,Hq,Hkv,D,seqs,splits", [
    # key counts around the 16/32/64-key tiles and the 4 wavefronts that take them in turn
    ("few_keys", 3, 1, 64, [(0, n, n, 0) for n in (1, 15, 16, 17, 32, 33, 63, 64, 65, 127, 128, 129, 257)], 0),
    ("few_keys_d128", 2, 1, 128, [(n, 1, 0, 1) for n in (1, 16, 31, 48, 64, 96, 128, 192, 256)], 0),
    # enough items that a workgroup takes two heads: odd, even and single-head groups, rows that fill no item
    ("pairs_odd_group", 7, 1, 128, [(17, 129, 1290, 33)], 0),
    ("pairs_even_group", 8, 2, 64, [(33, 100, 1111, 17), (0, 16, 47, 1)], 3),
    ("one_head_groups", 8, 8, 64, [(16, 250, 1100, 16)], 2),
    ("empty_splits", 2, 1, 64, [(20, 30, 60, 40)], 64),
], ids=lambda v: v if isinstance(v, str) else None)
def test_fp32_kernel_edges(oracle, name, Hq, Hkv, D, seqs, splits):
    w = W.Workload("f32e_" + name, 31, "f32", Hq, Hkv, D, 1.0e4, seqs, 1.0)
    data = W.generate(w)
    r = run_path(w, data, num_splits=splits, want_lse=True)
    want, want_lse = oracle.forward(data["q"], data["k"], data["v"], oracle_layout(oracle, w), w.rope_base)
    got = to_host_f32(r["out"])
    assert np.isfinite(got).all()
    print(name, error_stats(got, want))
    assert np.max(np.abs(got - want)) <= F32_TOL
    assert np.max(np.abs(to_host_f32(r["lse"]) - want_lse)) <= 1e-4


@pytest.mark.parametrize("splits", [2, 3, 7, 8, 9, 16, 33, 63, 64])
@pytest.mark.parametrize("dtype,Hq,Hkv,D", [("f32", 3, 1, 64), ("f32", 3, 1, 128), ("bf16", 6, 2, 64), ("bf16", 5, 5, 128)])
def test_merge_of_any_number_of_splits(oracle, dtype, Hq, Hkv, D, splits):
    """1-64 splits of question rows, more of them than key tiles included (splits without a key)."""
    w = W.Workload(f"merge{splits}", 32, dtype, Hq, Hkv, D, 1.0e4, [(30, 70, 200, 9), (0, 1, 0, 3), (5, 600, 1200, 33)], 0.5)
    data = W.generate(w)
    r = run_path(w, data, num_splits=splits, want_lse=True)
    want, want_lse = oracle.forward(data["q"], data["k"], data["v"], oracle_layout(oracle, w), w.rope_base)
    st = error_stats(to_host_f32(r["out"]), want)
    lse_err = np.max(np.abs(to_host_f32(r["lse"]) - want_lse))
    if dtype == "f32":
        assert st["max_abs"] <= F32_TOL and lse_err <= 1e-4, st
    else:
        assert st["max_abs"] <= 2e-2 and st["mean_abs"] <= 2e-3 and lse_err <= 2e-2, st


@pytest.mark.parametrize("n_seqs", [1, 4, 5])
@pytest.mark.parametrize("dtype,D", [("f32", 64), ("bf16", 128)])
@pytest.mark.parametrize("splits", [1, 4])
def test_items_formed_in_the_kernel_or_read_from_the_list(oracle, dtype, D, n_seqs, splits):
    """Up to four sequences the attention kernel forms its work items itself, beyond that it reads a built list; the
    workspace holds the enumeration either way.  One split writes the rows directly, several are merged."""
    seqs = [(20, 50, 130, 7), (0, 33, 90, 0), (3, 1, 0, 40), (70, 64, 64, 1), (9, 200, 150, 12)][:n_seqs]
    w = W.Workload(f"inline{n_seqs}", 33, dtype, 4, 2, D, 1.0e4, seqs, 0.5)
    data = W.generate(w)
    lay, heads = layout_heads(w)
    q, k, v = to_device(data["q"]), to_device(data["k"]), to_device(data["v"])
    out = torch.full_like(q, float("nan"))
    lse = torch.full((w.total_tokens, 4), float("nan"), device=DEV)
    offs = [11 * i for i in range(n_seqs)]
    P.pevlm_rope_seq(q, k, lay, heads, w.rope_base, offs)
    ws_p = P.pevlm_block_prefill_attn(q, k, v, out, lay, heads, lse=lse)
    ws_q = P.pevlm_query_attn(q, k, v, out, lay, heads, num_splits=splits, lse=lse)
    torch.cuda.synchronize()
    for ws, host in ((ws_p, P.pevlm_prefill_worklist_host(lay, P.pevlm_prefill_tile_rows(heads))),
                     (ws_q, P.pevlm_query_worklist_host(lay, P.pevlm_query_tile_rows(heads), splits))):
        want_list = b"".join(bytes(it) for it in host)
        assert ws.cpu().numpy()[:len(want_list)].tobytes() == want_list
    want, want_lse = oracle.forward(data["q"], data["k"], data["v"], oracle_layout(oracle, w), w.rope_base, pos_offset=offs)
    st = error_stats(to_host_f32(out), want)
    lse_err = np.max(np.abs(to_host_f32(lse) - want_lse))
    assert st["max_abs"] <= (F32_TOL if dtype == "f32" else 2e-2) and lse_err <= (1e-4 if dtype == "f32" else 2e-2), st
    if dtype == "bf16":  # the question rows with their rotation folded in: the same bits
        q_raw, out2 = to_device(data["q"]), torch.zeros_like(out)
        P.pevlm_query_attn_rope(q_raw, k, v, out2, lay, heads, w.rope_base, offs, num_splits=splits)
        for lo, (S, _B, C, Q) in zip(lay.cu, seqs):
            a = int(lo) + S + C
            assert torch.equal(out2[a:a + Q].view(torch.int16), out[a:a + Q].view(torch.int16))


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("Hq,Hkv,hmap", [(7, 1, None), (6, 2, None), (4, 4, None), (9, 3, [0, 1, 2] * 3), (5, 1, None), (40, 1, None),
                                         (4, 2, [0, 0, 0, 1])], ids=["g7", "g3", "g1", "g3map", "g5", "g40", "unequal"])
@pytest.mark.parametrize("Q", [1, 4, 5, 18, 19, 33, 128, 131])
def test_row_head_pairs_fill_wavefronts(oracle, Hq, Hkv, hmap, Q, D):
    """128 (row, head) pairs per workgroup, 32 per wavefront: row counts on both sides of a full wavefront and a full
    workgroup, groups that do not divide 32, head maps; sink and block rows under the one-item kernel too."""
    w = W.Workload(f"pairs{Q}", 34, "bf16", Hq, Hkv, D, 1.0e4, [(Q, 150, 210, Q), (0, 1, 0, 2)], 0.5)
    data = W.generate(w)
    prev = P.pevlm_set_prefill_kernel("classic")
    try:
        r = run_path(w, data, kv_head_of_q=hmap, want_lse=True)
    finally:
        P.pevlm_set_prefill_kernel(prev)
    want, want_lse = oracle.forward(data["q"], data["k"], data["v"], oracle_layout(oracle, w), w.rope_base, kv_head_of_q=hmap)
    got = to_host_f32(r["out"])
    assert np.isfinite(got).all()
    st = error_stats(got, want)
    assert st["max_abs"] <= 2e-2 and st["mean_abs"] <= 2e-3 and st["max_rel_l2"] <= 3e-2, st
    assert np.max(np.abs(to_host_f32(r["lse"]) - want_lse)) <= 2e-2


@pytest.mark.parametrize("tokens", [1, 33, 700, 5500, 16500])
@pytest.mark.parametrize("dtype,Hq,Hkv,D", [("bf16", 5, 1, 128), ("bf16", 14, 2, 64), ("f32", 3, 3, 64), ("f32", 9, 1, 128)])
def test_rope_heads_shared_between_workgroups(oracle, dtype, Hq, Hkv, D, tokens):
    """Few tokens: the heads of a token are dealt out over several workgroups; from 512 workgroups on one takes all."""
    w = W.Workload(f"rope{tokens}", 35, dtype, Hq, Hkv, D, 1.0e6, [(tokens, 1, 0, 0)], 0.5)
    data = W.generate(w)
    lay, heads = layout_heads(w)
    pos = oracle.positions(oracle_layout(oracle, w)) + 123456
    for which in ("both", "q", "k"):
        q, k = to_device(data["q"]), to_device(data["k"])
        P.pevlm_rope_seq(None if which == "k" else q, None if which == "q" else k, lay, heads, w.rope_base, [123456])
        torch.cuda.synchronize()
        for name, t in (("q", q), ("k", k)):
            got, raw = to_host_f32(t), W.as_float32(data[name])
            if which not in ("both", name):
                assert np.array_equal(got, raw)
                continue
            want = oracle.rope(data[name], pos, w.rope_base)
            # one rounding to the storage type (2^-8 relative in bf16, 2^-23 in fp32) on top of fp32 arithmetic
            assert np.all(np.abs(got - want) <= (2.0 ** -8 if dtype == "bf16" else 2.0 ** -22) * np.abs(want) + 1e-6)


@pytest.mark.parametrize("D,Hq,Hkv", [(128, 28, 4), (64, 6, 3), (128, 5, 1), (64, 14, 7)])
@pytest.mark.parametrize("tokens", [1, 63, 129, 3000])
def test_fp8_both_stages_leave_what_the_stages_leave(D, Hq, Hkv, tokens):
    """Q quantised by the attention kernel (both stages in one call) against the stages called one after the other:
    the same codes, scales and output bits; the maxima are those of the tensors."""
    seqs = [(tokens // 3, max(1, tokens // 4), tokens - tokens // 3, 0)]
    w = W.Workload(f"fp8both{tokens}", 36, "bf16", Hq, Hkv, D, 1.0e6, seqs, 0.5)
    data = W.generate(w)
    rng = np.random.default_rng(7)  # rows of very different magnitude, an all-zero row, zeros of both signs
    x = W.bf16_bits_to_f32(data["q"]) * (2.0 ** rng.integers(-40, 40, (tokens, Hq, 1))).astype(np.float32)
    x[tokens // 2] = 0.0
    x[:, :, 3] = -0.0
    data["q"] = W.f32_to_bf16_bits(x)
    lay, heads = layout_heads(w)
    q, k, v = to_device(data["q"]), to_device(data["k"]), to_device(data["v"])
    plan = P.pevlm_block_prefill_fp8_plan(lay, heads)
    outs, spaces = [], []
    for stages in ((0,), (P.FP8_QUANTISE, P.FP8_ATTEND)):
        ws = torch.full((plan.total,), 0xEE, dtype=torch.uint8, device=DEV)
        out = torch.zeros_like(q)
        for st in stages:
            P.pevlm_block_prefill_attn_fp8(q, k, v, out, lay, heads, workspace=ws, stages=st)
        torch.cuda.synchronize()
        outs.append(out.view(torch.int16).cpu())
        spaces.append(ws.cpu().numpy())
    assert torch.equal(outs[0], outs[1])
    for lo, n in ((plan.q_codes, tokens * Hq * D), (plan.q_scales, tokens * Hq * 4), (plan.kv_amax, 2 * Hkv * 4)):
        assert np.array_equal(spaces[0][lo:lo + n], spaces[1][lo:lo + n])
    amax = spaces[0][plan.kv_amax:plan.kv_amax + 2 * Hkv * 4].view(np.float32).reshape(2, Hkv)
    for i, name in enumerate(("k", "v")):
        assert np.array_equal(amax[i], np.abs(W.bf16_bits_to_f32(data[name])).max(axis=(0, 2)))


@pytest.mark.parametrize("kernel", ["classic", "stream"])
@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("keys", [1, 4, 63, 64, 65, 128, 191, 257])
def test_row_sums_of_equal_weights(D, kernel, keys):
    """Keys of one value: every visible key has the weight 1 and lse - score is the logarithm of their number, for each
    of the lanes and accumulators that the sums are spread over (n weights of 1 add up exactly in fp32: what is
    left is a logarithm and one rounding of the score, 1e-4)."""
    lay, heads = P.Layout.from_seqs([(0, keys, keys, 0)]), P.Heads(4, 2, D, "bf16")
    q = torch.ones(keys, 4, D, device=DEV, dtype=torch.bfloat16)
    k = torch.full((keys, 2, D), 0.25, device=DEV, dtype=torch.bfloat16)
    v = torch.arange(keys, device=DEV, dtype=torch.float32).view(-1, 1, 1).expand(keys, 2, D).to(torch.bfloat16).contiguous()
    out, lse = torch.empty_like(q), torch.empty(keys, 4, device=DEV, dtype=torch.float32)
    prev = P.pevlm_set_prefill_kernel(kernel)
    try:
        P.pevlm_block_prefill_attn(q, k, v, out, lay, heads, lse=lse)
    finally:
        P.pevlm_set_prefill_kernel(prev)
    n = torch.arange(1, keys + 1, dtype=torch.float64)
    want = 0.25 * D / D ** 0.5 + n.log()
    assert (lse.cpu().double() - want.view(-1, 1)).abs().max() <= 1e-4
    mean = torch.cumsum(v[:, 0, 0].cpu().double(), 0) / n
    err = (out.cpu().double() - mean.view(-1, 1, 1)).abs()
    assert (err <= 2.0 ** -8 * mean.view(-1, 1, 1) + 1e-3).all()  # one bf16 rounding of the result


@pytest.mark.parametrize("D,Hq,Hkv", [(128, 7, 1), (64, 6, 3)])
@pytest.mark.parametrize("seqs", [[(3, 50, 70, 129)], [(0, 1, 0, 5), (9, 30, 61, 0), (2, 40, 100, 33), (0, 16, 16, 1)] * 13])
def test_fp8_both_stages_quantise_question_rows(D, Hq, Hkv, seqs):
    """Codes and scales of every row of Q, the question's included, sequences without one and more sequences than a
    table holds: one call of both stages against a QUANTISE stage."""
    w = W.Workload("fp8question", 37, "bf16", Hq, Hkv, D, 1.0e6, seqs, 0.5)
    data = W.generate(w)
    lay, heads = layout_heads(w)
    q, k, v = to_device(data["q"]), to_device(data["k"]), to_device(data["v"])
    plan, out, spaces = P.pevlm_block_prefill_fp8_plan(lay, heads), torch.zeros_like(q), []
    for stages in (0, P.FP8_QUANTISE):
        ws = torch.full((plan.total,), 0xEE, dtype=torch.uint8, device=DEV)
        P.pevlm_block_prefill_attn_fp8(q, k, v, out, lay, heads, workspace=ws, stages=stages)
        spaces.append(ws.cpu().numpy())
    for lo, n in ((plan.q_codes, w.total_tokens * Hq * D), (plan.q_scales, w.total_tokens * Hq * 4)):
        assert np.array_equal(spaces[0][lo:lo + n], spaces[1][lo:lo + n])


@pytest.mark.parametrize("extra", [dict(qk_scale=2.5), dict(qk_scale=1.5, key_ramp=6.0), dict(qk_scale=6.0, key_ramp=3.0)],
                         ids=["peaky", "rising_max", "huge_scores"])
@pytest.mark.parametrize("Hq,Hkv,D", [(8, 2, 128), (7, 1, 128), (6, 2, 64), (4, 4, 64)])
def test_a_row_does_not_depend_on_the_rows_beside_it(Hq, Hkv, D, extra):
    """Reference maxima that have to be raised on the way: the same bits from the one-item kernel (32 (row, head) pairs in a
    wavefront), the streaming kernel (32 rows of one head), the call with RoPE folded in and a prefill block by block."""
    seqs = [(200, 300, 1000, 0), (0, 130, 700, 0), (33, 64, 200, 0)]
    w = W.Workload("beside", 38, "bf16", Hq, Hkv, D, 1.0e6, seqs, 0.5, **extra)
    data = W.generate(w)
    lay, heads = layout_heads(w)
    q, k, v = to_device(data["q"]), to_device(data["k"]), to_device(data["v"])
    raw = q.clone()
    P.pevlm_rope_seq(q, k, lay, heads, w.rope_base)

    def result(call):
        out, lse = torch.zeros_like(q), torch.zeros(w.total_tokens, Hq, device=DEV)
        call(out, lse)
        return out.view(torch.int16).cpu(), lse.view(torch.int32).cpu()

    def in_pieces(out, lse):
        blocks = [-(-c // b) for _s, b, c, _q in seqs]
        for i in range(max(blocks)):
            P.pevlm_block_prefill_attn_blocks(q, k, v, out, lay, heads, [min(i, n - 1) for n in blocks], [int(i < n) for n in blocks], i == 0,
                                              lse=lse)

    results, prev = {}, P.pevlm_set_prefill_kernel("classic")
    try:
        for kernel in ("classic", "stream"):
            P.pevlm_set_prefill_kernel(kernel)
            results[kernel] = result(lambda out, lse: P.pevlm_block_prefill_attn(q, k, v, out, lay, heads, lse=lse))
            results[kernel + " in pieces"] = result(in_pieces)
    finally:
        P.pevlm_set_prefill_kernel(prev)
    results["folded"] = result(lambda out, lse: P.pevlm_block_prefill_attn_rope(raw, k, v, out, lay, heads, w.rope_base, k_is_rotated=True, lse=lse))
    for name, (out, lse) in results.items():
        assert torch.equal(out, results["classic"][0]) and torch.equal(lse, results["classic"][1]), name


@pytest.mark.parametrize("seqs", [[(256, 1024, 256 * f, 64) for f in (33, 97, 161, 255)], [(256, 1024, 65536, 128)] * 2])
def test_static_call_takes_batches_with_the_librarys_split_count(seqs):
    """Batches whose partials nearly fill the built-in array: accepted, and the bits of the call with a workspace."""
    lay, heads = P.Layout.from_seqs(seqs), P.Heads(28, 4, 128, "bf16")
    gen = torch.Generator(device=DEV).manual_seed(3)
    q, k, v = (torch.randn(lay.total_tokens, h, 128, device=DEV, dtype=torch.bfloat16, generator=gen) for h in (28, 4, 4))
    outs = [torch.zeros_like(q), torch.zeros_like(q)]
    P.pevlm_query_attn(q, k, v, outs[0], lay, heads)
    P.pevlm_query_attn_static(q, k, v, outs[1], lay, heads)
    assert torch.equal(outs[0].view(torch.int16), outs[1].view(torch.int16)) and outs[0].any()


@pytest.mark.parametrize("Hq,Hkv", [(128, 2), (132, 2), (9, 3), (12, 4)])
@pytest.mark.parametrize("D", [64, 128])
def test_head_maps_against_the_default_map(Hq, Hkv, D):
    """Query heads dealt out over the KV heads in turn: groups that a wavefront's lanes can hold (up to 64 heads) and a larger
    one; the same bits as the default map on reordered heads, every call."""
    lay = P.Layout.from_seqs([(9, 70, 150, 21), (0, 64, 40, 3)])
    T = lay.total_tokens
    gen = torch.Generator(device=DEV).manual_seed(4)
    q, k, v = (torch.randn(T, h, D, device=DEV, dtype=torch.bfloat16, generator=gen) for h in (Hq, Hkv, Hkv))
    mapped = P.Heads(Hq, Hkv, D, "bf16", [i % Hkv for i in range(Hq)])
    order = sorted(range(Hq), key=lambda i: (i % Hkv, i))  # query heads by KV head
    plain, q2 = P.Heads(Hq, Hkv, D, "bf16"), q[:, order].contiguous()
    prev = P.pevlm_set_prefill_kernel("classic")
    try:
        res = []
        for heads, x in ((mapped, q), (plain, q2)):
            out, lse = torch.zeros_like(x), torch.zeros(T, Hq, device=DEV)
            P.pevlm_block_prefill_attn(x, k, v, out, lay, heads, lse=lse)
            P.pevlm_query_attn(x, k, v, out, lay, heads, num_splits=3, lse=lse)
            res.append((out.view(torch.int16), lse.view(torch.int32)))
    finally:
        P.pevlm_set_prefill_kernel(prev)
    assert torch.equal(res[0][0][:, order], res[1][0]) and torch.equal(res[0][1][:, order], res[1][1])


@pytest.mark.parametrize("Hkv", [1, 2, 4])
@pytest.mark.parametrize("seqs", [[(0, 900, 900, 0)], [(0, 1024, 1024, 3)], [(0, 1100, 1100, 0)], [(130, 1500, 1700, 5)], [(40, 700, 1400, 0)],
                                  [(0, 60, 60, 0), (0, 2000, 2000, 7)], [(0, 200, 5000, 0)],
                                  [(0, 8500, 8500, 0)], [(0, 9100, 9100, 0)]])
def test_items_dealt_over_xcds(Hkv, seqs):
    """One region that fills the runs of the XCDs on a KV head (7 to 72 items over 2, 4 or 8 runs, remainders among them; from
    257 workgroups on they are dealt), and layouts on the other side of the rule: every row once, with the bits of the streaming kernel, folded calls too."""
    lay, heads = P.Layout.from_seqs(seqs), P.Heads(3 * Hkv, Hkv, 128, "bf16")
    gen = torch.Generator(device=DEV).manual_seed(9)
    q, k, v = (torch.randn(lay.total_tokens, h, 128, device=DEV, dtype=torch.bfloat16, generator=gen) for h in (3 * Hkv, Hkv, Hkv))
    rot = q.clone()
    P.pevlm_rope_seq(rot, k, lay, heads, 1.0e6)
    outs, prev = {}, P.pevlm_set_prefill_kernel("auto")
    try:
        for kernel in ("classic", "stream", "folded"):
            outs[kernel] = torch.full_like(q, float("nan"))
            if kernel == "folded":
                P.pevlm_block_prefill_attn_rope(q, k, v, outs[kernel], lay, heads, 1.0e6, k_is_rotated=True)
                continue
            P.pevlm_set_prefill_kernel(kernel)
            P.pevlm_block_prefill_attn(rot, k, v, outs[kernel], lay, heads)
    finally:
        P.pevlm_set_prefill_kernel(prev)
    question = sum(s[3] for s in seqs)
    assert int(torch.isnan(outs["classic"].float()).any(dim=-1).any(dim=-1).sum()) == question  # rows that the call does not compute
    for kernel in ("stream", "folded"):
        assert torch.equal(outs[kernel].view(torch.int16), outs["classic"].view(torch.int16)), kernel


@pytest.mark.parametrize("Hq,Hkv,seqs", [
    (2, 1, [(0, 40, 40, 3)]),                                            # fewer items than XCDs
    (7, 1, [(100, 1024, 20480, 0)]),                                     # fewer rounds than are sorted together
    (14, 2, [(256, 1024, 30000, 1), (0, 64, 0, 9), (33, 700, 5000, 0)]),  # dealt there and back first; an empty context, short last blocks
    (16, 8, [(392, 392, 39592, 0)]),                                     # even as listed, a short last block
    (4, 2, [(16, 500, 900, 2)] * 50),                                    # more sequences than a table holds: as listed
])
def test_shares_of_the_streaming_kernel(Hq, Hkv, seqs):
    """The order that the builder leaves behind the list: every item once, gaps in the last round only, each XCD's share of the
    work within an item of the others', no workgroup far above the mean; and the bits of the one-item kernel."""
    lay, heads = P.Layout.from_seqs(seqs), P.Heads(Hq, Hkv, 128, "bf16")
    gen = torch.Generator(device=DEV).manual_seed(12)
    q, k, v = (torch.randn(lay.total_tokens, h, 128, device=DEV, dtype=torch.bfloat16, generator=gen) for h in (Hq, Hkv, Hkv))
    ws = torch.zeros(P.pevlm_block_prefill_workspace_bytes(lay, heads), dtype=torch.uint8, device=DEV)
    outs, prev = [], P.pevlm_set_prefill_kernel("classic")
    try:
        for kernel in ("classic", "stream"):
            P.pevlm_set_prefill_kernel(kernel)
            outs.append(torch.full_like(q, float("nan")))
            P.pevlm_block_prefill_attn(q, k, v, outs[-1], lay, heads, workspace=ws)
        items = P.pevlm_prefill_stream_items_host(lay, heads)
    finally:
        P.pevlm_set_prefill_kernel(prev)
    assert torch.equal(outs[0].view(torch.int16), outs[1].view(torch.int16))
    n, W = len(items), torch.cuda.get_device_properties(0).multi_processor_count // 8
    cost = np.array([7 + 3 * it.n_tiles for it in items])
    before, dealt = np.cumsum(cost) - cost, len(seqs) <= 48
    # an XCD's run ends with the last item of which it would take the larger part
    first = [int((2 * (cost.sum() * x // 8 - before) >= cost).sum()) if dealt and 0 < x < 8 else n * x // 8 for x in range(9)]
    order = ws.cpu().numpy()[(n * 160 + 255) // 256 * 256:].view(np.int32)
    for x in range(8):
        mine = first[x + 1] - first[x]
        rounds = -(-mine // W)
        seg = order[first[x] + x * W:][:rounds * W].reshape(W, rounds)
        assert np.array_equal(np.sort(seg[seg >= 0]), np.arange(first[x], first[x + 1])) and (seg[:, :-1] >= 0).all()
        if mine and dealt:
            load = np.where(seg >= 0, cost[seg], 0).sum(axis=1)
            assert load.max() <= max(1.04 * load.mean(), load.mean() + cost[first[x]:first[x + 1]].max())


@pytest.mark.parametrize("Hq,Hkv,seqs", [
    (28, 4, [(196, 196, 33712, 0)]),                               # 7 items a head, even as listed
    (32, 8, [(196, 196, 33712, 0)]),                               # 4, four workgroups of 32 always the longest
    (28, 4, [(256, 1024, 32768, 0)]),                              # 28
    (16, 8, [(392, 3136, 50000, 0)]),                              # 25 and a short last block
    (14, 2, [(256, 1024, 256 * f, 0) for f in (33, 97, 41, 63)]),  # runs that end in another sequence
    (6, 2, [(5, 64, 300 + 40 * i, 3) for i in range(48)]),         # as many sequences as a table holds
    (12, 2, [(0, 640, 12800, 0), (700, 64, 0, 5), (0, 33, 1000, 0)]),
])
def test_items_are_dealt_where_listed_ones_come_out_uneven(Hq, Hkv, seqs):
    """The rule looks at one period of a run of equal regions: as the loads of all listed items added up."""
    lay, heads = P.Layout.from_seqs(seqs), P.Heads(Hq, Hkv, 128, "bf16")
    q, k, v = (torch.zeros(lay.total_tokens, h, 128, device=DEV, dtype=torch.bfloat16) for h in (Hq, Hkv, Hkv))
    ws = torch.zeros(P.pevlm_block_prefill_workspace_bytes(lay, heads), dtype=torch.uint8, device=DEV)
    prev = P.pevlm_set_prefill_kernel("stream")
    try:
        P.pevlm_block_prefill_attn(q, k, v, torch.empty_like(q), lay, heads, workspace=ws)
        tiles = np.array([it.n_tiles for it in P.pevlm_prefill_stream_items_host(lay, heads)])
    finally:
        P.pevlm_set_prefill_kernel(prev)
    n, cus = len(tiles), torch.cuda.get_device_properties(0).multi_processor_count
    shares = cost_model.stream_shares(tiles, len(seqs), cus)
    order = ws.cpu().numpy()[(n * 160 + 255) // 256 * 256:].view(np.int32)
    at = 0
    for x in range(8):
        mine = shares[x * (cus // 8):(x + 1) * (cus // 8)]
        count = sum(len(i) for i in mine)
        rounds = -(-count // len(mine))
        for w, want in enumerate(mine):
            got = order[at + x * len(mine) + w * rounds:][:rounds]
            assert np.array_equal(tiles[got[got >= 0]], tiles[want]), (x, w)  # equal ones may stand for each other
        at += count


@pytest.mark.parametrize("Hq,Hkv,D,seqs,splits", [
    (56, 8, 128, [(37, 150, 480, 70)], 13),            # 7 heads: 112 of 128 columns, the last item of 5 rows
    (64, 8, 64, [(0, 533, 533, 16), (5, 64, 30, 1)], 9),  # 8 heads: every column; a block that ends inside a tile of 32 keys
    (72, 8, 64, [(16, 90, 300, 33)], 12),              # 9 heads: two workgroups of an item
    (64, 4, 128, [(20, 130, 300, 40)], 16),            # 16 heads: two full ones
    (64, 16, 64, [(33, 100, 470, 35)], 8),             # 4 heads, items one by one: half of the columns
    (64, 16, 64, [(33, 135, 860, 50)], 13),            # 4 heads, two items together, regions of an odd number of items
    (48, 16, 64, [(33, 100, 870, 50)], 12),            # 3 heads, two items together
    (32, 16, 128, [(0, 70, 1200, 40)], 40),            # 2 heads, two or four items together, short blocks
    (56, 8, 64, [(7, 60, 100, 17)] * 6, 7),            # a list that is read
    (28, 4, 64, [(0, 1100, 1100, 5)], 3),              # 69 items over two XCDs
    (14, 2, 64, [(0, 2080, 2080, 1)], 5),              # 130 over four
])
def test_fp32_groups_of_heads(oracle, Hq, Hkv, D, seqs, splits):
    """The fp32 kernel that takes all heads of a group: column and key remainders, items joined inside a region and not across
    its end, questions; against the oracle, and windowed questions against the kernel that takes one head (a KV head at
    a time does not fill the chip)."""
    w = W.Workload("f32g", 34, "f32", Hq, Hkv, D, 1.0e4, seqs, 1.0)
    data = W.generate(w)
    r = run_path(w, data, num_splits=splits, want_lse=True)
    want, want_lse = oracle.forward(data["q"], data["k"], data["v"], oracle_layout(oracle, w), w.rope_base)
    got = to_host_f32(r["out"])
    assert np.isfinite(got).all()
    print(error_stats(got, want))
    assert np.max(np.abs(got - want)) <= F32_TOL
    assert np.max(np.abs(to_host_f32(r["lse"]) - want_lse)) <= 1e-4
    G, q, k, v = Hq // Hkv, r["q_rot"], r["k_rot"], r["v"]
    outs = [torch.zeros_like(q), torch.zeros_like(q)]
    window = [2 - i % 2 for i in range(len(seqs))]
    P.pevlm_query_attn_window(q, k, v, outs[0], r["lay"], r["heads"], window, num_splits=splits)
    one = P.Heads(G, 1, D, "f32")
    for g in range(Hkv):
        part = torch.zeros_like(q[:, g * G:(g + 1) * G])
        P.pevlm_query_attn_window(q[:, g * G:(g + 1) * G].contiguous(), k[:, g:g + 1].contiguous(), v[:, g:g + 1].contiguous(), part, r["lay"], one, window,
                                  num_splits=splits)
        outs[1][:, g * G:(g + 1) * G] = part
    assert outs[0].any() and (outs[0] - outs[1]).abs().max() <= F32_TOL


def attention_in_64_bits(q, k, v, seq):
    """Rows of one sequence (rotated operands on the CPU), on the device and in 64 bits."""
    S, B, C, _Q = seq
    T, Hq, D = q.shape
    i = torch.arange(T, device=DEV)
    region = torch.where(i < S, -1, torch.where(i < S + C, (i - S) // B, T))
    sees = (i[None, :] <= i[:, None]) & ((region[None, :] == region[:, None]) | (region[None, :] == -1) | (region[:, None] == T))
    q, k, v = (x.to(DEV).double() for x in (q, k, v))
    want = torch.zeros(T, Hq, D, dtype=torch.float64, device=DEV)
    for h in range(Hq):
        g = h * k.shape[1] // Hq
        w = torch.softmax((q[:, h] @ k[:, g].T / D ** 0.5).masked_fill(~sees, float("-inf")), dim=-1)
        want[:, h] = w @ v[:, g]
    return want


def fp32_attention(q, k, v, seq, splits):
    lay, heads = P.Layout.from_seqs([seq]), P.Heads(q.shape[1], k.shape[1], q.shape[2], "f32")
    dev = [x.to(DEV) for x in (q, k, v)]
    out = torch.full_like(dev[0], float("nan"))
    P.pevlm_block_prefill_attn(*dev, out, lay, heads)
    P.pevlm_query_attn(*dev, out, lay, heads, num_splits=splits)
    return out.double()


@pytest.mark.parametrize("Hq,Hkv,D,seq,splits,tol", [
    (28, 4, 128, (100, 333, 500, 40), 4, 4.6e-7),  # the two-head kernel of before had 4.65e-7, one sum a score 6.5e-7
    (14, 2, 64, (77, 333, 900, 21), 4, 3.5e-7),    # 3.53e-7, 4.96e-7
    (2, 1, 64, (32, 16, 64, 8), 1, 2.9e-7),        # (one head then too) 3.1e-7
    (4, 1, 128, (64, 300, 1500, 64), 6, 5.0e-7),   # 6.7e-7
    (28, 4, 128, (256, 1024, 2048, 64), 16, 3.9e-7),  # all heads of a group: 5.6e-7
])
def test_fp32_distance_to_64_bits(Hq, Hkv, D, seq, splits, tol):
    """Relative 2-norm of the error over all rows, scores of standard deviation 2: no more than the fp32 matrix instructions of two heads
    a workgroup had.  The limit lies between what two sums a score measure (10 to 15 % below it) and what one does."""
    gen = torch.Generator().manual_seed(15)
    q, k, v = (torch.randn(sum(seq) - seq[1], h, D, generator=gen) for h in (Hq, Hkv, Hkv))
    q *= 2.0
    want = attention_in_64_bits(q, k, v, seq)
    err = float((fp32_attention(q, k, v, seq, splits) - want).norm() / want.norm())
    print(err)
    assert err <= tol


@pytest.mark.parametrize("Hq,Hkv,D", [(56, 8, 64), (64, 16, 128)])
@pytest.mark.parametrize("q_exp,k_exp,v_exp", [(0, 0, -112), (0, 0, -118), (0, 0, -126), (0, 0, 100), (0, 0, 123), (112, -112, 0), (-112, 112, 0), (-60, 60, -60)])
def test_fp32_groups_of_heads_over_all_magnitudes(Hq, Hkv, D, q_exp, k_exp, v_exp):
    """Operands whose bf16 parts would not all be normal numbers, and ones that leave no room for a power of two: as exact as others.
    The limit is that of the test before for scores of deviation 1, twice it for rows that are done again one by one."""
    seq, gen = (37, 150, 480, 70), torch.Generator().manual_seed(17)
    q, k, v = (torch.randn(sum(seq) - seq[1], h, D, generator=gen) for h in (Hq, Hkv, Hkv))
    tensors = [(x * 2.0 ** e, e) for x, e in ((q, q_exp), (k, k_exp), (v, v_exp))]
    want = attention_in_64_bits(*(x.double() * 2.0 ** -e for x, e in tensors), seq)  # of what the denormals among them hold
    got = fp32_attention(*(x for x, _e in tensors), seq, 13) * 2.0 ** -v_exp
    if v_exp == -126:  # results about 2^-126: a step of the smallest denormal, 2^-23 here, beside the largest error of the others
        assert float((got - want).abs().max()) <= 2.0 ** -23 + 1e-6
    else:
        err = float((got - want).norm() / want.norm())
        print(err)
        assert err <= 6e-7


def test_fp32_groups_of_heads_with_vanishing_weights_of_large_values():
    """A key whose weight is 2^-118 to 2^-125 of the largest and whose value is 2^103, beside values of 2^-17: a good part of the
    result.  The weight's own error is its exponent's, 86 x 2^-24; a weight in fewer bits than fp32 has would be seen."""
    Hq, Hkv, D, seq, gen = 56, 8, 64, (37, 150, 480, 70), torch.Generator().manual_seed(18)
    T = sum(seq) - seq[1]
    q, k, v = (torch.randn(T, h, D, generator=gen) for h in (Hq, Hkv, Hkv))
    q[:, :, 0], k[:, :, 0], k[0, :, 1:], k[0, :, 0] = 8.0, 0.0, 0.0, -82.0
    v[:, :, 5] = 2.0 ** -17 * (1.0 + torch.rand(T, Hkv, generator=gen))
    v[0, :, 5] = 1.999 * 2.0 ** 102
    want = attention_in_64_bits(q, k, v, seq)[1:, :, 5]
    got = fp32_attention(q, k, v, seq, 13)[1:, :, 5]
    assert float(((got - want) / want).abs().max()) <= 2e-5


@pytest.mark.parametrize("Hq,Hkv,D", [(2, 1, 64), (3, 3, 128), (4, 2, 128)])
@pytest.mark.parametrize("before", [3, 16, 37, 100])
def test_fp32_rows_do_not_depend_on_their_place_in_the_batch(Hq, Hkv, D, before):
    """One head at a time: a sequence alone and behind another one of any length, the same bits, question and lse too."""
    seq, gen = (21, 100, 330, 37), torch.Generator(device=DEV).manual_seed(16)
    T = sum(seq) - seq[1]
    q, k, v = (torch.randn(T + before, h, D, device=DEV, generator=gen) for h in (Hq, Hkv, Hkv))
    heads, res = P.Heads(Hq, Hkv, D, "f32"), []
    for seqs in ([seq], [(0, 8, before, 0), seq]):
        lay, x = P.Layout.from_seqs(seqs), [t[before if len(seqs) == 1 else 0:].clone() for t in (q, k, v)]
        out, lse = torch.zeros_like(x[0]), torch.zeros(lay.total_tokens, Hq, device=DEV)
        P.pevlm_block_prefill_attn(*x, out, lay, heads, lse=lse)
        P.pevlm_query_attn(*x, out, lay, heads, num_splits=3, lse=lse)
        res.append((out[-T:].view(torch.int32), lse[-T:].view(torch.int32)))
    assert torch.equal(res[0][0], res[1][0]) and torch.equal(res[0][1], res[1][1])


@pytest.mark.parametrize("Hq,Hkv,D,seqs,splits", [
    (3, 3, 128, [(0, 64, 0, 1), (0, 512, 9000, 1)], 16),                    # one pair; one key and empty splits beside long ones
    (7, 1, 128, [(65, 128, 300, 18), (9, 1000, 8000, 18)], 13),             # 126 of 128 pairs; key ranges of part of a tile
    (8, 2, 64, [(1, 64, 1000, 32), (0, 100, 0, 31), (5, 50, 5000, 1)], 9),  # 128 pairs; sequences of 1 to 80 tiles, in a batch
    (14, 2, 128, [(256, 1024, 36000, 36)], 64),                             # 252 of 256 pairs, half of the compute units: the other kernel
    (28, 4, 128, [(256, 1024, 36000, 36)], 64),                             # ... all of them
    (28, 4, 128, [(256, 1024, 30000, 36)], 64),                             # ... and splits below the line: the other kernel
    (12, 4, 128, [(0, 512, 15000, 64), (0, 0, 0, 0), (7, 64, 900, 65)], 28),  # more rows than angles go without a table
    (4, 2, 64, [(3, 512, 16000, 64), (0, 64, 0, 0), (7, 64, 900, 3)], 30),    # as many
    (16, 8, 64, [(30, 700, 17000, 128)], 32),                               # 256 pairs, 128 rows of the diagonal: two tiles of it
    (64, 1, 128, [(0, 512, 26000, 4)] + [(0, 512, 3000, 4)] * 4, 50),       # 256 pairs of a wide group; more sequences than kernel arguments hold
    (16, 2, 64, [(0, 512, 11000, 16)] + [(5, 64, 700 + i, 16 - i) for i in range(5)], 20),  # more sequences, two KV heads
])
@pytest.mark.parametrize("call", ["plain", "rope", "window", "bad"])
def test_short_questions(Hq, Hkv, D, seqs, splits, call):
    """The kernel that stages the keys once for all pairs of a KV head, with the bits of the one-item kernel: that one
    takes the same question under a map to the KV heads in reverse."""
    lay = P.Layout.from_seqs(seqs)
    back = [Hkv - 1 - h * Hkv // Hq for h in range(Hq)]
    gen = torch.Generator(device=DEV).manual_seed(14)
    q, k, v = (torch.randn(lay.total_tokens, h, D, device=DEV, dtype=torch.bfloat16, generator=gen) for h in (Hq, Hkv, Hkv))
    if call == "bad":  # a question row's own key and a value, both seen by the rows behind them only
        k[-1, 0], v[-1, -1, 0] = float("nan"), float("inf")
    res = []
    for hmap in (None, back):
        heads = P.Heads(Hq, Hkv, D, "bf16", kv_head_of_q=hmap)
        kk, vv = (k, v) if hmap is None else (k.flip(1).contiguous(), v.flip(1).contiguous())
        out, lse = torch.full_like(q, 7.0), torch.full((lay.total_tokens, Hq), 7.0, device=DEV)
        if call == "rope":
            P.pevlm_query_attn_rope(q, kk, vv, out, lay, heads, 1.0e6, pos_offset=[70 * i for i in range(len(seqs))], num_splits=splits, lse=lse)
        elif call == "window":
            P.pevlm_query_attn_window(q, kk, vv, out, lay, heads, [30] * len(seqs), num_splits=splits, lse=lse)
        else:
            P.pevlm_query_attn(q, kk, vv, out, lay, heads, num_splits=splits, lse=lse)
        res.append((out.view(torch.int16), lse.view(torch.int32)))
    assert torch.equal(res[0][0], res[1][0]) and torch.equal(res[0][1], res[1][1])


@pytest.mark.parametrize("Hq,D,seqs,splits", [
    (7, 128, [(65, 128, 300, 18), (9, 1000, 8000, 18)], 13),
    (64, 128, [(0, 900, 26000, 4)] + [(0, 512, 3000, 4)] * 4, 50),
    (16, 64, [(3, 1200, 34000, 8), (0, 64, 0, 0), (7, 64, 900, 3)], 60),
])
@pytest.mark.parametrize("call", ["plain", "rope", "window"])
def test_short_questions_of_one_kv_head(Hq, D, seqs, splits, call):
    """One KV head has no other head map: the one-item kernel takes its heads as the second half of a call with two KV heads
    under a map that swaps them."""
    lay, gen = P.Layout.from_seqs(seqs), torch.Generator(device=DEV).manual_seed(19)
    q, k, v = (torch.randn(lay.total_tokens, h, D, device=DEV, dtype=torch.bfloat16, generator=gen) for h in (2 * Hq, 2, 2))
    res = []
    for heads, x, kk, vv in ((P.Heads(Hq, 1, D, "bf16"), *(t.contiguous() for t in (q[:, Hq:], k[:, :1], v[:, :1]))),
                             (P.Heads(2 * Hq, 2, D, "bf16", kv_head_of_q=[1] * Hq + [0] * Hq), q, k, v)):
        out, lse = torch.full_like(x, 7.0), torch.full((lay.total_tokens, x.shape[1]), 7.0, device=DEV)
        if call == "rope":
            P.pevlm_query_attn_rope(x, kk, vv, out, lay, heads, 1.0e6, pos_offset=[70 * i for i in range(len(seqs))], num_splits=splits, lse=lse)
        elif call == "window":
            P.pevlm_query_attn_window(x, kk, vv, out, lay, heads, [30] * len(seqs), num_splits=splits, lse=lse)
        else:
            P.pevlm_query_attn(x, kk, vv, out, lay, heads, num_splits=splits, lse=lse)
        res.append((out[:, -Hq:].contiguous().view(torch.int16), lse[:, -Hq:].contiguous().view(torch.int32)))
    assert torch.equal(res[0][0], res[1][0]) and torch.equal(res[0][1], res[1][1])
