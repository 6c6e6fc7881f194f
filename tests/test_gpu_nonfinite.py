"""Infinite and invalid values in keys and values: they reach the rows that see them and no others."""
import numpy as np
import pytest
import torch

import paper_2506_19651_amd as P
import workloads as W
from gpu_util import DEV, oracle_layout, run_path, to_host_f32

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("Hq,Hkv,D,splits", [(2, 1, 64, 0), (7, 1, 128, 3), (8, 8, 64, 1), (8, 2, 128, 5)])
@pytest.mark.parametrize("where", ["value", "key"])
def test_fp32_rows_that_do_not_see_a_bad_key_stay_finite(oracle, Hq, Hkv, D, splits, where):
    """fp32 kernel, one and two heads per workgroup: bad keys at both ends of a key tile, of an item of 16 rows, of a block
    and of the sequence, in the sink, the block and the question."""
    seqs = [(21, 100, 330, 37), (5, 40, 0, 0), (0, 64, 1600, 3)]
    w = W.Workload("bad_f32", 41, "f32", Hq, Hkv, D, 1.0e4, seqs, 1.0)
    data = W.generate(w)
    starts = np.concatenate([[0], np.cumsum([s + c + q for s, _b, c, q in seqs])])
    # sequence 0: last sink key, a block's first and middle keys, question keys; 1: a sink key; 2: a block's last key
    bad = [20, 121, 160, 351, 357, 387, starts[1] + 3, starts[2] + 64 * 7 + 63]
    numbers = [np.nan, np.inf, -np.inf]
    for i, t in enumerate(bad):
        x = data["v" if where == "value" else "k"]
        x[t, i % Hkv, (5 * i) % D] = numbers[i % 3] if where == "value" else np.nan
    r = run_path(w, data, num_splits=splits, want_lse=True)
    got, lse = to_host_f32(r["out"]), to_host_f32(r["lse"])
    want, want_lse = oracle.forward(data["q"], data["k"], data["v"], oracle_layout(oracle, w), w.rope_base)
    fine = np.isfinite(want)
    assert 0.2 < fine.mean() < 1.0  # the inputs do what they are meant to
    assert np.array_equal(np.isfinite(got), fine)
    assert np.abs(got[fine] - want[fine]).max() <= 1e-5  # the bound of every fp32 test
    both = np.isfinite(want_lse)
    assert np.array_equal(np.isfinite(lse), both) and np.abs(lse[both] - want_lse[both]).max() <= 1e-4


@pytest.mark.parametrize("Hq,Hkv,D", [(56, 8, 64), (32, 8, 128)])
@pytest.mark.parametrize("where", ["value", "key"])
def test_fp32_groups_of_heads_with_bad_keys(oracle, Hq, Hkv, D, where):
    """The same for the kernel that takes all heads of a group, where a bad key meets the other rows and heads in matrix
    instructions; the largest finite numbers too, which overflow their first bf16 plane."""
    seqs = [(21, 100, 430, 37)]
    w = W.Workload("bad_f32g", 42, "f32", Hq, Hkv, D, 1.0e4, seqs, 1.0)
    data = W.generate(w)
    x = data["v" if where == "value" else "k"]
    for i, t in enumerate([20, 121, 160, 351, 457, 487]):
        x[t, i % Hkv, (5 * i) % D] = [np.nan, np.inf, -np.inf][i % 3] if where == "value" else np.nan
    if where == "value":
        x[300, 7, 3] = 3.4e38
    r = run_path(w, data, num_splits=11)
    got = to_host_f32(r["out"])
    want, _ = oracle.forward(data["q"], data["k"], data["v"], oracle_layout(oracle, w), w.rope_base)
    fine = np.isfinite(want)
    assert 0.2 < fine.mean() < 1.0
    assert np.array_equal(np.isfinite(got), fine)
    assert (np.abs(got[fine] - want[fine]) <= 1e-5 * np.maximum(1.0, np.abs(want[fine]))).all()


@pytest.mark.parametrize("Hq,Hkv,D,seqs,splits", [
    (32, 8, 128, [(100, 500, 1400, 70)], 24),   # 4 heads: two items together, 4 of 5 in the question
    (48, 16, 64, [(33, 100, 870, 50)], 12),     # 3 heads: two
    (16, 8, 64, [(56, 500, 3010, 110)], 40),    # 2 heads: four in the prefill and the question, ends of three, two and one
    (32, 16, 128, [(0, 70, 1200, 40)], 40),     # 2 heads: short blocks
])
@pytest.mark.parametrize("where", ["value", "key", "largest"])
def test_fp32_joined_items_with_bad_keys(oracle, Hq, Hkv, D, seqs, splits, where):
    """The same where a workgroup takes several items of 16 rows at once: a bad key or value in every stretch of 16 rows of
    a sink, a block and the question, so that rows of each of the joined items do and do not see one; the largest finite values, which
    overflow their first bf16 plane, in the rows of all of them."""
    w = W.Workload("bad_f32j", 44, "f32", Hq, Hkv, D, 1.0e4, seqs, 1.0)
    data = W.generate(w)
    S, B, C, Q = seqs[0]
    bad = [(t, t // 16 % Hkv) for t in range(S - 1 if S else 0, S)]  # the sink's last key alone: blocks and question see the sink
    for start, n in [(S + b, min(B, C - b)) for b in range(0, C, B)] + [(S + C, Q)]:
        g = start % Hkv  # one KV head to a region: the others' rows stay as they are
        bad += [(start + r, g) for r in (18, 33, 50, n - 2) if r < n and start != S]
    x = data["k" if where == "key" else "v"]
    for i, (t, g) in enumerate(bad):
        x[t, g, (5 * i) % D] = np.nan if where == "key" else (3.399e38 if where == "largest" else [np.nan, np.inf, -np.inf][i % 3])
    r = run_path(w, data, num_splits=splits, want_lse=True)
    got, lse = to_host_f32(r["out"]), to_host_f32(r["lse"])
    want, want_lse = oracle.forward(data["q"], data["k"], data["v"], oracle_layout(oracle, w), w.rope_base)
    fine = np.isfinite(want)
    assert 0.2 < fine.mean() < 1.0 or where == "largest" and fine.all()
    assert np.array_equal(np.isfinite(got), fine)
    assert (np.abs(got[fine] - want[fine]) <= 1e-5 * np.maximum(1.0, np.abs(want[fine]))).all()
    both = np.isfinite(want_lse)
    assert np.array_equal(np.isfinite(lse), both) and np.abs(lse[both] - want_lse[both]).max() <= 1e-4


@pytest.mark.parametrize("Hq,Hkv,D", [(72, 8, 64), (64, 4, 64), (96, 2, 128)])
def test_fp32_wide_groups_with_bad_keys(oracle, Hq, Hkv, D):
    """Groups of 9, 16 and 48 heads, whose items are dealt out over several workgroups (an item's 16 rows, over the ends of
    them): a row that is done again is stored once, by the workgroup that has it.  Right against the oracle, lse too, and the same
    bits whatever the buffers held before."""
    seqs = [(21, 100, 430, 37)]
    w = W.Workload("bad_f32w", 43, "f32", Hq, Hkv, D, 1.0e4, seqs, 1.0)
    data = W.generate(w)
    for i, t in enumerate([20, 121, 160, 351, 457, 487]):
        data["v"][t, i % Hkv, (5 * i) % D] = [np.nan, np.inf, -np.inf, 3.4e38][i % 4]
    r = run_path(w, data, num_splits=11, want_lse=True)
    got, lse = to_host_f32(r["out"]), to_host_f32(r["lse"])
    want, want_lse = oracle.forward(data["q"], data["k"], data["v"], oracle_layout(oracle, w), w.rope_base)
    fine = np.isfinite(want)
    assert 0.2 < fine.mean() < 1.0
    assert np.array_equal(np.isfinite(got), fine)
    assert (np.abs(got[fine] - want[fine]) <= 1e-5 * np.maximum(1.0, np.abs(want[fine]))).all()
    assert np.abs(lse - want_lse).max() <= 1e-4  # scores are finite
    once = run_path(w, data, num_splits=11, want_lse=True, poison=False)
    for name in ("out", "lse"):
        assert torch.equal(r[name].nan_to_num(9.0), once[name].nan_to_num(9.0))


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("splits", [1, 2, 9, 64])
def test_infinite_value_behind_a_vanishing_weight(dtype, D, splits):
    """One question row: its weight of every early key underflows (scores 512 and more below the largest), the value of one
    of them is infinite.  0 x inf stays visible however the keys are split: in that element and in no other."""
    n = 700
    lay, heads = P.Layout.from_seqs([(0, n - 1, n - 1, 1)]), P.Heads(2, 1, D, dtype)
    kind = torch.float32 if dtype == "f32" else torch.bfloat16
    q = torch.full((n, 2, D), 8.0, device=DEV, dtype=kind)
    k = torch.zeros((n, 1, D), device=DEV, dtype=kind)
    k[650:] = 8.0
    v = torch.ones((n, 1, D), device=DEV, dtype=kind)
    v[100, 0, 7] = float("inf")
    out = torch.zeros_like(q)
    P.pevlm_query_attn(q, k, v, out, lay, heads, num_splits=splits)
    row = out[n - 1].float().cpu()
    assert not torch.isfinite(row[:, 7]).any()
    row[:, 7] = 1.0
    assert torch.equal(row, torch.ones_like(row))  # equal weights of values 1
