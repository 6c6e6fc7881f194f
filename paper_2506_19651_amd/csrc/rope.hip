// Sequential rotary position embedding (Sec. "Position Encoding"): every token of a sequence is
// rotated at its index in the whole sequence; nothing restarts at a block boundary.
// HBM-bound: each element of q and k is read once and written once.
#include <algorithm>
#include <type_traits>

#include "common.h"
#include "rope_math.h"

namespace pevlm {

// Rows (or table entries) of a chunk of sequences: entry e of sequence s, first[s] <= e < first[s + 1], has the position
// e - first[s] + pos[s] and is packed row e - first[s] + row[s].
struct RopeRows {
    int32_t num_seqs;
    int32_t first[kMaxSeqsPerLaunch], pos[kMaxSeqsPerLaunch], row[kMaxSeqsPerLaunch];
};

// Pair indices of a lane.  Two: 64 lanes take two tokens of 128-wide heads, 4 bytes each in bf16.  With eight (16 bytes) the eight
// sines and cosines in a row are 8 KB of instructions, and a launch too small to run them more than a few times on a compute unit
// waits for them to be fetched (about 0.37 us a KB); large launches are not faster for it.  us, eight / two: 104 tokens x
// 28/4 heads 4.1 / 2.9 (fp32 5.6 / 3.3), 1152 5.7 / 5.0, 16 K 42.0 / 40.5, 66 K 222.5 / 211.6; 66 K x 32/8 heads 290 / 258.  Passes over
// the same 26 to 42 MB, which the L2s then hold, can be slower with two (32/8 heads, 2.5 K tokens 8.3 / 9.3, 3.3 K 11.1 / 11.6, 4.1 K 13.3 /
// 14.9; 3.7 K 12.4 / 12.1): it depends on which XCD had the rows last.  On rows that come from further off two are faster at every size
// (2.5 K 15.2 / 13.5, 3.3 K 18.2 / 17.5, 4.1 K 21.8 / 19.7), so there is no rule for it.
constexpr int kPairsPerLane = 2;
// a lane's values of one half of a row, as they lie in memory
template <bool BF16>
struct RopeWords {
    typedef typename std::conditional<BF16, uint32_t, uint2>::type Word;
    static constexpr int WORDS = BF16 ? kPairsPerLane / 2 : kPairsPerLane;
    union {
        Word all;
        uint32_t w[WORDS];
    };
    static_assert(sizeof(Word) == WORDS * 4, "one access a half row");
    __device__ __forceinline__ void load(const void *src) { all = *reinterpret_cast<const Word *>(src); }
    __device__ __forceinline__ void store(void *dst) const { *reinterpret_cast<Word *>(dst) = all; }
};

// A lane owns PPL consecutive pair indices i of one token: it loads x[i..i+PPL) and x[i+D/2..i+D/2+PPL), forms the PPL
// angles once in fp64, reduces them to [-pi, pi], and then walks over the query heads and key heads of that token.
// blockIdx.y takes heads_per_y of them: with enough tokens to fill the chip all (the angles are formed once),
// with few tokens a share, so that the chip is filled and the walk is short (1152 tokens x 32 heads: 36
// workgroups, 12.4 us, against 288 workgroups, 6 us).
//
// MROPE (three position axes: temporal, height, width; the scheme of the Qwen2.5-VL models of the
// paper's experiments): the token's three ids come from pos3 [3][T] in device memory and pair index
// i takes the id of the axis whose section holds i (sections are consecutive: [0, sec0),
// [sec0, sec01), [sec01, D/2)); `rows` is not used.
template <int D, bool BF16, bool MROPE>
__global__ __launch_bounds__(256) void rope_kernel(void *q, void *k, RopeRows rows, RopeFreq fr, int32_t Hq, int32_t Hkv,
                                                   int32_t row_begin, int32_t row_end, const int32_t *pos3, int64_t T,
                                                   int32_t sec0, int32_t sec01, float2 *table, int32_t heads_per_y)
{
    constexpr int PPL = kPairsPerLane, LANES_PER_TOKEN = D / 2 / PPL, EL = BF16 ? 2 : 4;
    constexpr int TOKENS_PER_BLOCK = 256 / LANES_PER_TOKEN;
    int32_t tok = row_begin + blockIdx.x * TOKENS_PER_BLOCK + threadIdx.x / LANES_PER_TOKEN;
    if (tok >= row_end) return;
    int32_t i0 = (threadIdx.x % LANES_PER_TOKEN) * PPL;
    // The first rows of the token are requested before the angles are formed, and each row is requested PF rows ahead of its use,
    // so that the sine/cosine arithmetic and the rotation run under the memory latency.  Rows of the token: its Hq
    // query heads, then its Hkv key heads.
    constexpr int PF = BF16 ? 4 : 1;
    const int32_t nq = q ? Hq : 0, all = nq + (k ? Hkv : 0);
    const int32_t first = blockIdx.y * heads_per_y, nrows = min(first + heads_per_y, all);
    char *const qrow = (char *)q + (((int64_t)tok * Hq) * D + i0) * EL;
    char *const krow = (char *)k + (((int64_t)tok * Hkv) * D + i0) * EL;
    const auto at = [&](int32_t r) { return r < nq ? qrow + (int64_t)r * (D * EL) : krow + (int64_t)(r - nq) * (D * EL); };
    RopeWords<BF16> plo[PF], phi[PF];
#pragma unroll
    for (int j = 0; j < PF; ++j)
        if (first + j < nrows) {
            plo[j].load(at(first + j));
            phi[j].load(at(first + j) + D / 2 * EL);
        }
    double pos = 0.0, pos_axis[3] = {0.0, 0.0, 0.0};
    if (MROPE) {
#pragma unroll
        for (int a = 0; a < 3; ++a) pos_axis[a] = (double)pos3[(int64_t)a * T + tok];
    } else {
        int32_t s = 0;
        while (s + 1 < rows.num_seqs && tok >= rows.first[s + 1]) ++s;
        pos = (double)(tok - rows.first[s] + rows.pos[s]);
    }
    float cs[PPL], sn[PPL];
#pragma unroll
    for (int j = 0; j < PPL; ++j) {
        if (MROPE) pos = i0 + j < sec0 ? pos_axis[0] : (i0 + j < sec01 ? pos_axis[1] : pos_axis[2]);
        rope_cos_sin<!BF16>(pos, fr.inv_freq[i0 + j], cs[j], sn[j]);
    }
    if (table && first == 0) {  // by-product for the fused query rotation of the attention kernels: entry = packed row
        float2 *dst = table + (int64_t)tok * (D / 2) + i0;
#pragma unroll
        for (int j = 0; j < PPL; j += 2) *reinterpret_cast<float4 *>(dst + j) = make_float4(cs[j], sn[j], cs[j + 1], sn[j + 1]);
    }
    for (int32_t r0 = first; r0 < nrows; r0 += PF) {
#pragma unroll
        for (int j = 0; j < PF; ++j) {
            const int32_t r = r0 + j;
            if (r >= nrows) break;
            char *const x = at(r);
            const RopeWords<BF16> lo = plo[j], hi = phi[j];
            if (r + PF < nrows) {
                plo[j].load(at(r + PF));
                phi[j].load(at(r + PF) + D / 2 * EL);
            }
            RopeWords<BF16> ol, ou;
            if constexpr (BF16) {
#pragma unroll
                for (int w = 0; w < PPL / 2; ++w) {
                    float a0 = __uint_as_float(lo.w[w] << 16), a1 = __uint_as_float(lo.w[w] & 0xffff0000u);
                    float b0 = __uint_as_float(hi.w[w] << 16), b1 = __uint_as_float(hi.w[w] & 0xffff0000u);
                    float r0f, r1f, t0f, t1f;
                    rope_rotate(a0, b0, cs[2 * w], sn[2 * w], r0f, t0f);
                    rope_rotate(a1, b1, cs[2 * w + 1], sn[2 * w + 1], r1f, t1f);
                    ol.w[w] = rope_pack_bf16(r0f, r1f);
                    ou.w[w] = rope_pack_bf16(t0f, t1f);
                }
            } else {
#pragma unroll
                for (int w = 0; w < PPL; ++w) {
                    float rf, tf;
                    rope_rotate(__uint_as_float(lo.w[w]), __uint_as_float(hi.w[w]), cs[w], sn[w], rf, tf);
                    ol.w[w] = __float_as_uint(rf);
                    ou.w[w] = __float_as_uint(tf);
                }
            }
            ol.store(x);
            ou.store(x + D / 2 * EL);
        }
    }
}

// cos/sin table for the query rotation fused into the bf16 attention kernel: entry e holds, for
// every pair index i, (cos, sin) of the angle of packed row e (of the e-th question row of the batch where
// `rows` counts those).  Same arithmetic as rope_kernel, so a query rotated from the table gets the
// bits pevlm_rope_seq would have stored.  One thread per (entry, PPL pair indices).
template <int D>
__global__ __launch_bounds__(256) void rope_table_kernel(float2 *table, RopeRows rows, RopeFreq fr,
                                                         int32_t entry_begin, int32_t entry_end, const int32_t *pos3, int64_t T,
                                                         int32_t sec0, int32_t sec01)
{
    constexpr int PPL = kPairsPerLane, LANES_PER_ENTRY = D / 2 / PPL;
    const int32_t e = entry_begin + (blockIdx.x * 256 + threadIdx.x) / LANES_PER_ENTRY;
    if (e >= entry_end) return;
    const int32_t i0 = (threadIdx.x % LANES_PER_ENTRY) * PPL;
    int32_t s = 0;
    while (s + 1 < rows.num_seqs && e >= rows.first[s + 1]) ++s;
    double pos_axis[3];
    if (pos3) {  // three position axes: pair index i takes the id of the axis whose section holds it
        const int32_t row = e - rows.first[s] + rows.row[s];
#pragma unroll
        for (int a = 0; a < 3; ++a) pos_axis[a] = (double)pos3[(int64_t)a * T + row];
    } else {
        pos_axis[0] = pos_axis[1] = pos_axis[2] = (double)(e - rows.first[s] + rows.pos[s]);
        sec0 = sec01 = D;  // every pair index on axis 0
    }
    float2 *dst = table + (int64_t)e * (D / 2) + i0;
#pragma unroll
    for (int j = 0; j < PPL; j += 2) {
        float c0, s0, c1, s1;
        const int32_t ia = i0 + j, ib = i0 + j + 1;
        rope_cos_sin<false>(ia < sec0 ? pos_axis[0] : (ia < sec01 ? pos_axis[1] : pos_axis[2]), fr.inv_freq[ia], c0, s0);
        rope_cos_sin<false>(ib < sec0 ? pos_axis[0] : (ib < sec01 ? pos_axis[1] : pos_axis[2]), fr.inv_freq[ib], c1, s1);
        *reinterpret_cast<float4 *>(dst + j) = make_float4(c0, s0, c1, s1);
    }
}

// rope_base^(-2i/D): 64 powers cost more than a kernel launch's share of the call, and a program asks for one or
// two (D, base) again and again: each thread keeps the last one it asked for
static const RopeFreq &frequencies(int32_t D, double rope_base)
{
    static thread_local RopeFreq fr;
    static thread_local int32_t have_d = 0;
    static thread_local double have_base = 0.0;
    if (have_d != D || have_base != rope_base) {
        for (int i = 0; i < 64; ++i) fr.inv_freq[i] = i < D / 2 ? pow(rope_base, -2.0 * (double)i / (double)D) : 0.0;
        have_d = D;
        have_base = rope_base;
    }
    return fr;
}

// the rows of a chunk of sequences, or its question rows as they are counted over the batch
static RopeRows rope_rows(const SeqTable &tab, bool question)
{
    RopeRows r;
    r.num_seqs = tab.num_seqs;
    for (int32_t s = 0; s < tab.num_seqs; ++s) {
        const int32_t before = question ? tab.sink[s] + tab.ctx[s] : 0;
        r.first[s] = question ? tab.qrow_base[s] : tab.start[s];
        r.pos[s] = before + tab.pos_offset[s];
        r.row[s] = tab.start[s] + before;
    }
    return r;
}

void question_angles(const SeqTable &tab, int32_t D, double rope_base, RopeAngles *angles)
{
    static_assert(kInlineSeqs <= 4, "RopeAngles holds the sequences of a call without a list");
    const RopeRows rows = rope_rows(tab, true);
    angles->freq = frequencies(D, rope_base);
    angles->num_seqs = rows.num_seqs;
    for (int32_t s = 0; s < rows.num_seqs; ++s) {
        angles->first[s] = rows.first[s];
        angles->pos[s] = rows.pos[s];
    }
}

hipError_t launch_rope_table(float *table, bool question, const SeqTable &tab, int32_t D, double rope_base,
                             int32_t entry_begin, int32_t entry_end, const int32_t *pos3, int64_t T, int32_t sec0, int32_t sec01,
                             hipStream_t stream)
{
    if (entry_end <= entry_begin) return hipSuccess;
    const RopeFreq &fr = frequencies(D, rope_base);
    const RopeRows rows = rope_rows(tab, question);
    const int32_t per_block = 256 / (D / 2 / kPairsPerLane);
    dim3 grid((entry_end - entry_begin + per_block - 1) / per_block);
    const auto kernel = D == 128 ? rope_table_kernel<128> : rope_table_kernel<64>;
    hipLaunchKernelGGL(kernel, grid, dim3(256), 0, stream, (float2 *)table, rows, fr, entry_begin, entry_end, pos3, T, sec0, sec01);
    return hipGetLastError();
}

template <bool MROPE>
static hipError_t launch_rope_any(void *q, void *k, const RopeRows &rows, int32_t Hq, int32_t Hkv, int32_t D, bool bf16,
                                  double rope_base, int32_t row_begin, int32_t row_end, const int32_t *pos3, int64_t T,
                                  int32_t sec0, int32_t sec01, float *table, hipStream_t stream)
{
    const RopeFreq &fr = frequencies(D, rope_base);
    if (row_end <= row_begin) return hipSuccess;
    // heads per workgroup: all of them from 2048 workgroups on (8 to a compute unit), below that as few as it takes to have
    // 2048, at least 4 (512 workgroups: 5 K tokens x 28/4 heads 14.3 us, 12.9 with 2048, 13.2 with 4096)
    const int32_t heads = (q ? Hq : 0) + (k ? Hkv : 0);
    const int32_t tokens_per_block = 256 / (D / 2 / kPairsPerLane), blocks = (row_end - row_begin + tokens_per_block - 1) / tokens_per_block;
    int32_t shares = std::max(1, std::min(2048 / blocks, heads / 4));
    const int32_t per_y = (heads + shares - 1) / shares;
    shares = (heads + per_y - 1) / per_y;
    dim3 grid(blocks, shares);
#define PEVLM_ROPE_LAUNCH(DD, BB) \
    hipLaunchKernelGGL((rope_kernel<DD, BB, MROPE>), grid, dim3(256), 0, stream, q, k, rows, fr, Hq, Hkv, row_begin, row_end, pos3, T, sec0, sec01, (float2 *)table, per_y)
    if (D == 128 && bf16) PEVLM_ROPE_LAUNCH(128, true);
    else if (D == 128) PEVLM_ROPE_LAUNCH(128, false);
    else if (bf16) PEVLM_ROPE_LAUNCH(64, true);
    else PEVLM_ROPE_LAUNCH(64, false);
#undef PEVLM_ROPE_LAUNCH
    return hipGetLastError();
}

hipError_t launch_rope(void *q, void *k, const SeqTable &tab, int32_t Hq, int32_t Hkv, int32_t D, bool bf16,
                       double rope_base, float *table, hipStream_t stream)
{
    int32_t n = tab.num_seqs;
    int32_t row_begin = tab.start[0];
    int32_t row_end = tab.start[n - 1] + tab.sink[n - 1] + tab.ctx[n - 1] + tab.query[n - 1];
    return launch_rope_any<false>(q, k, rope_rows(tab, false), Hq, Hkv, D, bf16, rope_base, row_begin, row_end, nullptr, 0, 0, 0, table, stream);
}

hipError_t launch_rope_mrope(void *q, void *k, int64_t T, int32_t Hq, int32_t Hkv, int32_t D, bool bf16, double rope_base,
                             const int32_t *pos3, int32_t sec0, int32_t sec01, float *table, hipStream_t stream)
{
    RopeRows rows = {};
    return launch_rope_any<true>(q, k, rows, Hq, Hkv, D, bf16, rope_base, 0, (int32_t)T, pos3, T, sec0, sec01, table, stream);
}

}  // namespace pevlm
