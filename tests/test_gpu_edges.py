"""Kernels at the sizes where their tiling changes: remainders of row groups and key tiles, the borders of
the dispatch rules, the smallest and largest of each range; against the CPU oracle."""
import numpy as np
import pytest
import torch

import paper_2506_19651_amd as P
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
