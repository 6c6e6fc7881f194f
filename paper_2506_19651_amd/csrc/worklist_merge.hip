// Work-list builder kernels and the log-sum-exp merge of split-KV partials.
#include "common.h"

namespace pevlm {

// One thread per work item: locate the sequence in the chunk table, then evaluate the closed-form
// item (the same inline function the host enumeration uses).
__global__ __launch_bounds__(256) void build_prefill_items_kernel(SeqTable tab, int32_t tile_rows,
                                                                  pevlm_work_item *items, int32_t item_offset)
{
    int32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    int32_t total = tab.item_base[tab.num_seqs];
    if (i >= total) return;
    int32_t s = 0;
    while (s + 1 < tab.num_seqs && i >= tab.item_base[s + 1]) ++s;
    items[item_offset + i] = prefill_item_sel(tab.start[s], tab.sink[s], tab.block[s], tab.ctx[s], tile_rows, tab.sel_first[s],
                                              tab.sel_sink, i - tab.item_base[s], tab.seq_index0 + s);
}

__global__ __launch_bounds__(256) void build_query_items_kernel(SeqTable tab, int32_t tile_rows, int32_t num_splits,
                                                                int32_t total_q_rows, int32_t align,
                                                                pevlm_work_item *items, int32_t item_offset,
                                                                int32_t *qrow_of_compact)
{
    int32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    int32_t total = tab.item_base[tab.num_seqs];
    if (i < total) {
        int32_t s = 0;
        while (s + 1 < tab.num_seqs && i >= tab.item_base[s + 1]) ++s;
        items[item_offset + i] =
            tab.windowed ? query_item_window(tab.start[s], tab.sink[s], tab.ctx[s], tab.query[s], tile_rows, num_splits,
                                             i - tab.item_base[s], tab.seq_index0 + s, tab.qrow_base[s], total_q_rows, align,
                                             tab.win_start[s])
                         : query_item(tab.start[s], tab.sink[s], tab.ctx[s], tab.query[s], tile_rows, num_splits,
                                      i - tab.item_base[s], tab.seq_index0 + s, tab.qrow_base[s], total_q_rows, align);
    }
    // packed row of every compact question row of this chunk
    int32_t stride = gridDim.x * blockDim.x;
    for (int32_t s = 0; s < tab.num_seqs; ++s)
        for (int32_t r = i; r < tab.query[s]; r += stride)
            qrow_of_compact[tab.qrow_base[s] + r] = tab.start[s] + tab.sink[s] + tab.ctx[s] + r;
}

// What a dealer keeps of a sequence: the items of a head of its sink, of a block and of a short last block, and where the
// blocks and the short block start.  An item's cost depends on its number inside its head alone.
struct DealtRegion {
    int32_t items, R, full_len;
};
struct DealtSeq {
    int32_t base, blocks, last;
    DealtRegion region[3];
};

// The order of one XCD's items (one workgroup), as StreamShares says where they are dealt.  Keys are all different: equal costs go by
// their place.
constexpr int32_t kDealThreads = 512;
// keys v[0 .. N) above mine; a short loop, since what is fetched of a kernel that runs once costs more than its cycles
template <int N>
__device__ __forceinline__ int32_t keys_above(const uint32_t *v, uint32_t mine)
{
    int32_t rank = 0;
#pragma unroll 2
    for (int32_t j = 0; j < N; j += 4) {
        const uint4 x = *reinterpret_cast<const uint4 *>(v + j);
        rank += x.x > mine;
        rank += x.y > mine;
        rank += x.z > mine;
        rank += x.w > mine;
    }
    return rank;
}
__device__ __forceinline__ void deal_stream_items(const SeqTable &tab, int32_t G, int32_t Hkv, const StreamShares &sh, int32_t xcd, int32_t *order, int32_t deal)
{
    constexpr int32_t W = kMaxWgsPerXcd, TAIL = kDealtRounds * W;
    __shared__ __attribute__((aligned(16))) uint32_t key[kDealtItems];  // cost * 2^7 + 127 - place % 128
    __shared__ __attribute__((aligned(16))) uint32_t tail[TAIL], load[W];  // load: sum of costs * 2^5 + workgroup
    __shared__ DealtSeq seqs[kMaxSeqsPerLaunch];
    __shared__ uint2 sorted[TAIL];  // (item, cost)
    const int32_t tid = threadIdx.x, lo = sh.first[xcd], n = sh.first[xcd + 1] - lo;
    const int32_t rounds = ceil_div(n, W), plain = rounds > kDealtRounds ? rounds - kDealtRounds : 0;  // rounds dealt there and back
    int32_t *const seg = order + share_segment(sh, xcd);
    if (!deal) {
        for (int32_t i = tid; i < rounds * W; i += kDealThreads) seg[i % W * rounds + i / W] = i < n ? lo + i : -1;
        return;
    }
    const int32_t num_seqs = tab.num_seqs;
    if (tid < num_seqs) {
        const int32_t S = tab.sink[tid], B = tab.block[tid], C = tab.ctx[tid], first = tab.sel_first[tid], count = C > 0 ? tab.sel_count[tid] : 0;
        const int32_t nb = C > 0 ? ceil_div(C, B) : 0, rest = C > 0 && first + count == nb ? C - (nb - 1) * B : B;
        DealtSeq d;
        d.base = tab.item_base[tid];
        d.region[0] = {stream_items_of_region(S, G), S, 0};
        d.region[1] = {stream_items_of_region(B, G), B, S};
        d.region[2] = {stream_items_of_region(rest, G), rest, S};
        d.blocks = d.base + (tab.sel_sink ? d.region[0].items * Hkv : 0);
        d.last = d.blocks + (count > 0 ? (count - 1) * d.region[1].items * Hkv : 0);
        seqs[tid] = d;
    }
    if (tid < W) load[tid] = (uint32_t)tid;
    __syncthreads();
    for (int32_t i = tid; i < n; i += kDealThreads) {
        const int32_t idx = lo + i;
        int32_t s = 0;
        while (s + 1 < num_seqs && idx >= seqs[s + 1].base) ++s;
        const DealtSeq &d = seqs[s];
        const bool in_sink = idx < d.blocks, in_last = idx >= d.last;
        const DealtRegion r = d.region[in_sink ? 0 : (in_last ? 2 : 1)];
        const uint32_t c = stream_item_cost(r.R, r.full_len, G, (idx - (in_sink ? d.base : (in_last ? d.last : d.blocks))) % r.items);
        key[i] = (c << 7) + (uint32_t)(127 - i % 128);
    }
    __syncthreads();
    const int32_t t0 = plain * W, m = n - t0;  // at most TAIL items are left
    if (tid < TAIL) tail[tid] = tid < m ? key[t0 + tid] : (uint32_t)tid;
    for (int32_t i = tid; i < t0; i += kDealThreads) {
        const int32_t round = i / W, rank = keys_above<W>(key + round * W, key[i]), w = round & 1 ? W - 1 - rank : rank;
        seg[w * rounds + round] = lo + i;
        atomicAdd(&load[w], key[i] >> 7 << 5);
    }
    __syncthreads();
    if (tid < TAIL) sorted[keys_above<TAIL>(tail, tail[tid])] = make_uint2(tid < m ? lo + t0 + tid : -1, tail[tid] >> 7 << 5);
    __syncthreads();
    if (tid >= W) return;
    // lane w for workgroup w: the round's longest item to the least load, and so on
    for (int32_t round = plain; round < rounds; ++round) {
        const uint32_t mine = load[tid];
        const uint2 item = sorted[(round - plain) * W + W - 1 - keys_above<W>(load, mine)];
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
        seg[tid * rounds + round] = (int32_t)item.x;
        load[tid] = mine + item.y;
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
    }
}

// Same for the stream items of the bf16 streaming block-prefill kernel (item_base counts stream items) and their order: the
// first kXcds workgroups list it or deal it out if the chunk is the whole list, otherwise every thread lists its own item (100 K tokens in blocks
// of 392: 7.4 us, by the threads 10.6).
__global__ __launch_bounds__(kDealThreads) void build_stream_items_kernel(SeqTable tab, int32_t G, int32_t Hkv, HeadTable heads,
                                                                          pevlm_stream_item *items, int32_t item_offset, StreamShares shares,
                                                                          int32_t *order, int32_t dealers, int32_t deal)
{
    if ((int32_t)blockIdx.x < dealers) {
        deal_stream_items(tab, G, Hkv, shares, blockIdx.x, order, deal);
        return;
    }
    int32_t i = ((int32_t)blockIdx.x - dealers) * kDealThreads + threadIdx.x;
    int32_t total = tab.item_base[tab.num_seqs];
    if (i >= total) return;
    int32_t s = 0;
    while (s + 1 < tab.num_seqs && i >= tab.item_base[s + 1]) ++s;
    items[item_offset + i] = stream_item(tab.start[s], tab.sink[s], tab.block[s], tab.ctx[s], G, Hkv, tab.sel_first[s], tab.sel_sink,
                                         i - tab.item_base[s], tab.seq_index0 + s, heads.head_order);
    if (dealers) return;
    i += item_offset;
    int32_t x = 0;
    while (i >= shares.first[x + 1]) ++x;
    const int32_t n = shares.first[x + 1] - shares.first[x], W = shares.wgs, rounds = ceil_div(n, W), at = i - shares.first[x];
    int32_t *const seg = order + share_segment(shares, x);
    seg[at % W * rounds + at / W] = i;
    if (at == n - 1)  // no items in the rest of the last round
        for (int32_t left = n; left < rounds * W; ++left) seg[left % W * rounds + rounds - 1] = -1;
}

hipError_t launch_build_stream_items(const SeqTable &tab, int32_t G, int32_t Hkv, const HeadTable &heads, pevlm_stream_item *items,
                                     int32_t item_offset, const StreamShares &shares, int32_t *order, bool whole, bool deal, hipStream_t stream)
{
    const int32_t total = tab.item_base[tab.num_seqs], dealers = whole ? kXcds : 0;
    hipLaunchKernelGGL(build_stream_items_kernel, dim3(dealers + (total + kDealThreads - 1) / kDealThreads), dim3(kDealThreads), 0, stream, tab, G, Hkv,
                       heads, items, item_offset, shares, order, dealers, (int32_t)deal);
    return hipGetLastError();
}

hipError_t launch_build_prefill_items(const SeqTable &tab, int32_t tile_rows, pevlm_work_item *items,
                                      int32_t item_offset, hipStream_t stream)
{
    int32_t total = tab.item_base[tab.num_seqs];
    hipLaunchKernelGGL(build_prefill_items_kernel, dim3((total + 255) / 256), dim3(256), 0, stream, tab, tile_rows, items,
                       item_offset);
    return hipGetLastError();
}

hipError_t launch_build_query_items(const SeqTable &tab, int32_t tile_rows, int32_t num_splits, int32_t total_q_rows,
                                    int32_t align, pevlm_work_item *items, int32_t item_offset, int32_t *qrow_of_compact,
                                    hipStream_t stream)
{
    int32_t total = tab.item_base[tab.num_seqs];
    int32_t blocks = (total + 255) / 256;
    if (blocks < 1) blocks = 1;
    hipLaunchKernelGGL(build_query_items_kernel, dim3(blocks), dim3(256), 0, stream, tab, tile_rows, num_splits,
                       total_q_rows, align, items, item_offset, qrow_of_compact);
    return hipGetLastError();
}

// ------------------------------------------------------------------------------------------
// Merge of split-KV partials.  For one (question row, head) with partial s holding the running
// max m_s of the raw scores, l_s = sum exp(scale (score - m_s)) and acc_s = sum exp(...) v:
//   M = max_s m_s,  w_s = exp(scale (m_s - M)),  out = sum_s w_s acc_s / sum_s w_s l_s,
//   lse = scale M + log(sum_s w_s l_s).           (exact identity of Eq. 1's softmax)
// One wavefront per (row, head): lane s fetches (m, l) of split s, so the weights of all splits are known after
// one memory round trip; then D/4 lanes cover a row of values with 16 bytes each and the wavefront's 64 / (D/4)
// groups of them take the splits in turn, four in flight per lane.  Bound by reading the partials once
// (33 MB for 128 rows x 28 heads x 18 splits: 6.5 us at the copy rate); a thread that walks all splits of its
// four outputs takes one round trip per split: 47 us for 20 rows x 28 heads x 64 splits.
//
// FEW splits leave most of such a wavefront idle: up to 8 of them D/4 lanes take a row, and a wavefront two or four rows.
// us, wavefront per row against D/4 lanes: 1600 rows x 28 heads x 128, 2 splits 18.4 / 12.2, 8 splits 24.9 / 21.6;
// 1600 x 14 x 64, 2 splits 10.8 / 5.0; 8 rows x 28 heads, 8 splits 3.7 / 4.1, 16 splits 4.0 / 4.7.
// ------------------------------------------------------------------------------------------
constexpr int32_t kFewSplits = 8;

__device__ inline uint16_t f32_to_bf16_rne(float f)
{
    uint32_t u = __float_as_uint(f);
    u += 0x7fffu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}

template <int D, bool FEW>
__global__ __launch_bounds__(256) void merge_kernel(MergeParams p)
{
    constexpr int LPR = D / 4, UNIT = FEW ? LPR : 64, NSUB = UNIT / LPR, UNROLL = 4;
    const int32_t lane = threadIdx.x & 63, split = lane % UNIT, first_lane = lane - split;
    const int64_t n_units = (int64_t)p.total_q_rows * p.n_q_heads;
    int64_t unit = ((int64_t)blockIdx.x * 256 + threadIdx.x) / UNIT;  // (compact row, head)
    if (!FEW) unit = (int64_t)blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (unit >= n_units) return;
    float m = -INFINITY, l = 0.f;
    if (split < p.num_splits) {
        const float2 ml = *reinterpret_cast<const float2 *>(p.part_ml + ((int64_t)split * n_units + unit) * 2);
        m = ml.x;
        l = ml.y;
    }
    float M = m;
#pragma unroll
    for (int o = UNIT / 2; o > 0; o >>= 1) M = fmaxf(M, __shfl_xor(M, o));
    const uint64_t seen = __ballot(m != -INFINITY) >> first_lane;  // splits that saw a key of the row
    const float w = m == -INFINITY ? 0.f : expf((m - M) * p.scale);
    float denom = w * l;
#pragma unroll
    for (int o = UNIT / 2; o > 0; o >>= 1) denom += __shfl_xor(denom, o);

    const int32_t sub = split / LPR, d4 = (lane % LPR) * 4;
    const float *acc_row = p.part_acc + unit * D + d4;
    float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
    for (int32_t s0 = 0; s0 < p.num_splits; s0 += NSUB * UNROLL) {
        float4 a[UNROLL];
        float ws[UNROLL];
#pragma unroll
        for (int u = 0; u < UNROLL; ++u) {
            const int32_t s = s0 + u * NSUB + sub;  // below UNIT: the last step of UNIT splits ends there
            ws[u] = __shfl(w, first_lane + s);
            a[u] = make_float4(0.f, 0.f, 0.f, 0.f);
            // a weight too small for fp32 is no reason to leave a split out: its values may be infinite
            if (seen >> s & 1) a[u] = *reinterpret_cast<const float4 *>(acc_row + s * n_units * D);
        }
#pragma unroll
        for (int u = 0; u < UNROLL; ++u) {
            acc.x += ws[u] * a[u].x; acc.y += ws[u] * a[u].y; acc.z += ws[u] * a[u].z; acc.w += ws[u] * a[u].w;
        }
    }
#pragma unroll
    for (int o = LPR; o < UNIT; o <<= 1) {
        acc.x += __shfl_xor(acc.x, o); acc.y += __shfl_xor(acc.y, o);
        acc.z += __shfl_xor(acc.z, o); acc.w += __shfl_xor(acc.w, o);
    }
    if (sub != 0) return;
    const float inv = 1.f / denom;
    const int32_t cr = (int32_t)(unit / p.n_q_heads);
    const int32_t row = p.qrow_of_compact ? p.qrow_of_compact[cr] : inline_question_row(p.seqs, cr);
    const int32_t h = (int32_t)(unit % p.n_q_heads);
    const int64_t o = ((int64_t)row * p.n_q_heads + h) * D + d4;
    if (p.is_bf16) {
        ushort4 r;
        r.x = f32_to_bf16_rne(acc.x * inv); r.y = f32_to_bf16_rne(acc.y * inv);
        r.z = f32_to_bf16_rne(acc.z * inv); r.w = f32_to_bf16_rne(acc.w * inv);
        *reinterpret_cast<ushort4 *>((uint16_t *)p.out + o) = r;
    } else {
        *reinterpret_cast<float4 *>((float *)p.out + o) = make_float4(acc.x * inv, acc.y * inv, acc.z * inv, acc.w * inv);
    }
    if (p.lse && d4 == 0) p.lse[(int64_t)row * p.n_q_heads + h] = M * p.scale + logf(denom);
}

hipError_t launch_merge(const MergeParams &p, hipStream_t stream)
{
    static_assert(PEVLM_MAX_SPLITS == 64, "one lane per split, steps of 8 or 16 splits");
    const int64_t units = (int64_t)p.total_q_rows * p.n_q_heads;
    const bool few = p.num_splits <= kFewSplits;
    const int64_t lanes = units * (few ? p.head_dim / 4 : 64);
    const dim3 grid((uint32_t)((lanes + 255) / 256)), block(256);
    const auto kernel = p.head_dim == 128 ? (few ? merge_kernel<128, true> : merge_kernel<128, false>)
                                          : (few ? merge_kernel<64, true> : merge_kernel<64, false>);
    hipLaunchKernelGGL(kernel, grid, block, 0, stream, p);
    return hipGetLastError();
}

}  // namespace pevlm
