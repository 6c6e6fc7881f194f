"""Useful-FLOP accounting from the paper's operation counts (Sec. "Formulations", Eq. 6-10).

The paper counts 2*H operations per (query, key) pair with H = n_q_heads * head_dim (one GEMM).
Here both GEMMs (Q K^T and P V) are counted at 2 FLOP per multiply-add, i.e. 4 * head_dim per
visible pair per query head, and only pairs the mask keeps are counted (causal inside regions)."""
from __future__ import annotations

from .binding import Heads, Layout, pevlm_visible_pairs


def useful_flops(layout: Layout, heads: Heads):
    """Returns (prefill_flops, question_flops): sink + context-block rows, question rows."""
    sink, blocks, question = pevlm_visible_pairs(layout)
    per_pair = 4 * heads.head_dim * heads.n_q_heads
    return (sink + blocks) * per_pair, question * per_pair


# ---------------------------------------------------------------------------------------------
# Time model of the block-prefill call and the choice of sink and block size under a latency cap.
# The paper observes that both sizes trade accuracy against attention time and leaves their choice to
# tuning (Sec. on sink and block size; cost side: Eq. 7, Eq. 8 and Eq. 10, quadratic in both).
#
# Streaming kernel (one resident workgroup of 8 wavefronts per compute unit, items dealt by length inside each XCD's
# run of the list): a workgroup needs
#     STREAM_US_PER_ITEM * items + STREAM_US_PER_TILE * key tiles of its items,
# and the launch takes as long as its slowest workgroup.  One-item-per-workgroup kernel (two
# workgroups of 4 wavefronts per compute unit, dispatched as slots free up):
#     time * (2 * CUs) = US_PER_WORKGROUP * workgroups + US_PER_WORKGROUP_TILE * sum of key tiles.
# The constants are fitted to measured runs on one MI355X (profiles/block_prefill_sweep.md); the
# predictions stay within 10 % of them.  The one-item kernel's at head_dim 128 come from 68 prompts of 4 K to
# 40 K tokens that fill the chip at least twice (ratio to the measured time 1.02 +- 0.09).  64-wide heads run on the
# one-item kernel only, unless the streaming kernel is forced, which the model does not cover.
STREAM_US_PER_ITEM = 3.9
STREAM_US_PER_TILE = 1.665
US_PER_WORKGROUP = {128: 6.1, 64: 2.7}
US_PER_WORKGROUP_TILE = {128: 1.865, 64: 1.065}
_TILE_ROWS, _KEY_TILE, _PAIRS = 128, 64, 128


def prefill_work(layout: Layout, heads: Heads):
    """(workgroups, workgroup key tiles) of the one-item-per-workgroup kernel, from the same host
    enumeration the library offers: 128 (row, query head) pairs of an item and KV head per workgroup (one
    head at a time where a head map's groups are unequal, or hold more than 64 heads), which stages the tiles up to
    its own last row."""
    from .binding import pevlm_prefill_worklist_host

    G = heads.n_q_heads // heads.n_kv_heads
    if heads.map is not None:
        kv = [int(g) for g in heads.map]
        equal = all(kv.count(g) == G for g in range(heads.n_kv_heads))
        if not equal or (G > 64 and kv != sorted(kv)):
            G = 1
    groups = heads.n_q_heads // G
    n_wg = n_tiles = 0
    for it in pevlm_prefill_worklist_host(layout, _TILE_ROWS):
        pairs, full = it.q_rows * G, -(-it.full_len // _KEY_TILE)
        for first in range(0, pairs, _PAIRS):
            last_row = it.q_start + (min(first + _PAIRS, pairs) - 1) // G
            n_wg += groups
            n_tiles += groups * (full + (last_row - it.diag_start) // _KEY_TILE + 1)
    return n_wg, n_tiles


_XCDS, _DEALT_ROUNDS, _DEALT_ITEMS, _DEALT_WGS, _DEALT_SEQS, _EVEN_SHARE = 8, 4, 4096, 32, 48, 18


def stream_shares(tiles, num_seqs: int, compute_units: int = 256):
    """The library's own assignment of a stream-item list (key tiles of each item) to workgroups: one array of item
    numbers per workgroup, in its order.  Runs of the list per XCD are cut by cost, 7 an item and 3 a tile; inside a run
    the items go round by round to the workgroups, as listed where that is even enough over all of them, else ranked by cost
    there and back, the last rounds' sorted and to the least loads."""
    import numpy as np

    n, wgs = len(tiles), min(max(compute_units // _XCDS, 1), _DEALT_WGS)
    cost = 7 + 3 * np.asarray(tiles, dtype=np.int64)
    before, total = np.cumsum(cost) - cost, int(cost.sum())
    # a run ends with the last item of which it would take the larger part
    first = [0] + [int((2 * (total * x // _XCDS - before) >= cost).sum()) for x in range(1, _XCDS)] + [n]
    dealt = num_seqs <= _DEALT_SEQS and wgs == _DEALT_WGS and max(np.diff(first)) <= _DEALT_ITEMS
    if not dealt:
        first = [n * x // _XCDS for x in range(_XCDS + 1)]
    listed = [np.arange(lo + w, hi, wgs) for lo, hi in zip(first[:-1], first[1:]) for w in range(wgs)]
    most = max((int(cost[i].sum()) for i in listed), default=0)
    if not dealt or most * len(listed) * _EVEN_SHARE <= total * (_EVEN_SHARE + 1):
        return listed
    shares = []
    for lo, hi in zip(first[:-1], first[1:]):
        c, m = cost[lo:hi], hi - lo
        plain = max(0, -(-m // wgs) - _DEALT_ROUNDS) * wgs
        mine, load = [[] for _ in range(wgs)], np.zeros(wgs, np.int64)
        for r0 in range(0, plain, wgs):
            ranked = r0 + np.argsort(-c[r0:r0 + wgs], kind="stable")
            for w, i in enumerate(ranked if r0 // wgs % 2 == 0 else ranked[::-1]):
                mine[w].append(lo + int(i))
                load[w] += c[i]
        rest = plain + np.argsort(-c[plain:], kind="stable")
        for r0 in range(0, m - plain, wgs):
            for w, i in zip(np.argsort(load, kind="stable"), rest[r0:r0 + wgs]):
                mine[w].append(lo + int(i))
                load[w] += c[i]
        shares += [np.asarray(i, dtype=np.int64) for i in mine]
    return shares


def stream_work(layout: Layout, heads: Heads, compute_units: int = 256):
    """Per workgroup of the streaming kernel: (items, key tiles), as two arrays."""
    import ctypes

    import numpy as np

    from .binding import StreamItem, load_library

    lib = load_library()
    n = lib.pevlm_prefill_stream_items_host(layout.ref(), heads.ref(), None, None, 1, None, 0)
    if n <= 0:
        return np.zeros(0), np.zeros(0)
    items = (StreamItem * n)()
    lib.pevlm_prefill_stream_items_host(layout.ref(), heads.ref(), None, None, 1, items, n)
    words = ctypes.sizeof(StreamItem) // 4
    tiles = np.frombuffer(items, dtype=np.int32).reshape(n, words)[:, 6].astype(np.int64)  # n_tiles
    shares = stream_shares(tiles, len(layout.cu) - 1, compute_units)
    return np.asarray([len(i) for i in shares]), np.asarray([int(tiles[i].sum()) for i in shares])


def predict_block_prefill_ms(layout: Layout, heads: Heads, compute_units: int = 256) -> float:
    from .binding import pevlm_prefill_uses_stream_kernel

    if pevlm_prefill_uses_stream_kernel(layout, heads):
        cnt, til = stream_work(layout, heads, compute_units)
        return float((STREAM_US_PER_ITEM * cnt + STREAM_US_PER_TILE * til).max()) * 1e-3
    n_wg, n_tiles = prefill_work(layout, heads)
    d = heads.head_dim
    return (US_PER_WORKGROUP[d] * n_wg + US_PER_WORKGROUP_TILE[d] * n_tiles) / (2 * compute_units) * 1e-3


def choose_block_len(sink_len: int, ctx_len: int, query_len: int, heads: Heads, candidates, max_ms: float,
                     compute_units: int = 256):
    """Largest candidate block length (the paper's accuracy grows with the block size) whose
    predicted block-prefill time stays within max_ms; None if none does.  Returns (B, predicted_ms)."""
    best = None
    for B in sorted(candidates):
        lay = Layout.from_seqs([(sink_len, B, ctx_len, query_len)])
        ms = predict_block_prefill_ms(lay, heads, compute_units)
        if ms <= max_ms:
            best = (B, ms)
    return best


def video_layout(prefix_tokens: int, tokens_per_frame: int, n_frames: int, query_len: int, sink_frames: int,
                 block_frames: int):
    """(S, B, C, Q) of a video prompt partitioned as in Sec. "Partitioning Strategy": the sink is the
    text prefix plus the first sink_frames frames, the remaining frames form context blocks of
    block_frames frames (the last one may be shorter), the question follows."""
    sink_frames = min(sink_frames, n_frames)
    S = prefix_tokens + sink_frames * tokens_per_frame
    C = (n_frames - sink_frames) * tokens_per_frame
    return S, max(block_frames * tokens_per_frame, 1), C, query_len


def choose_sink_and_block(prefix_tokens: int, tokens_per_frame: int, n_frames: int, query_len: int, heads: Heads,
                          sink_frames, block_frames, max_ms: float, compute_units: int = 256):
    """Both knobs at once.  For every (sink frames, block frames) of the two candidate lists the
    block-prefill time is predicted; among the pairs within max_ms the one that keeps the most
    (query, key) pairs visible is returned -- the pair closest to full attention, which is the direction
    in which the paper's accuracy grows for both sizes -- ties going to the larger block.
    Returns (best, table): best = (sink_frames, block_frames, predicted_ms, visible_pairs) or None,
    table = that tuple for every candidate pair."""
    table = []
    for sf in sink_frames:
        for bf in block_frames:
            lay = Layout.from_seqs([video_layout(prefix_tokens, tokens_per_frame, n_frames, query_len, sf, bf)])
            sink, blocks, _question = pevlm_visible_pairs(lay)
            table.append((sf, bf, predict_block_prefill_ms(lay, heads, compute_units), sink + blocks))
    ok = [r for r in table if r[2] <= max_ms]
    best = max(ok, key=lambda r: (r[3], r[1])) if ok else None
    return best, table
