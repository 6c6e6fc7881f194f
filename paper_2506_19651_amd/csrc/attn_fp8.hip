// FP8 (OCP E4M3) variant of the block-prefill step for gfx950 (CDNA4): rows of the sink (Eq. 3) and of the
// context blocks (Eq. 4) with Q K^T and P V on v_mfma_f32_32x32x64_f8f6f4 (fp32 accumulation, fp32
// online softmax).  Two stages:
//
//   quantise   bf16 Q, K, V -> E4M3 codes times power-of-two scales (Q: one scale per token and query
//              head; K, V: one scale per KV head over all tokens).  K and V are written as the
//              64-key tiles the attention kernel stages, one run of tiles per region (sink, each
//              context block), zero padded, already in the byte order the tile has in LDS; V tiles
//              are transposed (head_dim major) with the keys in the order in which a lane of the
//              score MFMA holds them, so that the weights go from the score registers to the value
//              MFMA without any exchange between lanes.
//   attend     one workgroup (4 wavefronts x 32 rows) per 128 query rows of a region and query head;
//              a K tile and a V tile per step are copied into LDS (two stages each) by asynchronous
//              global->LDS loads issued one tile ahead.
//
// Scores.  Q is quantised after multiplication by c = softmax factor * log2(e); the power-of-two scales of
// the query row and of the K head enter the score MFMAs as their 8-bit block exponents, and the
// accumulators start from 7 - m (m: the row's reference maximum): the MFMAs deliver the exponents of the
// weights, and the vector ALU is left with exp2, the row sum, the row maximum and the conversion.
//
// Weights.  p = exp2(c s - m + 7) is rounded to E4M3; m is a reference maximum of the row that is
// raised to the running maximum whenever that has outgrown it by more than one octave, so the
// largest weight of a row lies in [2^7, 2^8] (E4M3 reaches 448) and weights down to 2^-16 of the
// largest keep at least one significant bit.  The row sum is taken over the unrounded weights.
#include <algorithm>
#include <type_traits>

#include "attn_bf16_tile.h"

namespace pevlm {

namespace {

typedef __attribute__((ext_vector_type(8))) int32_t i32x8;
typedef __attribute__((ext_vector_type(4))) int32_t i32x4v;

constexpr int32_t kExpLimit = 100;
constexpr float kWeightShift = 7.f;  // log2 of the weight of a key whose score equals the reference maximum
constexpr float kWeightLag = 1.f;    // octaves the running maximum may exceed the reference

// smallest e with amax * 2^-e <= 448 (0 for amax == 0), within [-100, 100]
__device__ __forceinline__ int32_t scale_exponent(float amax)
{
    if (!(amax > 0.f)) return 0;
    int x;
    const float f = frexpf(amax, &x);  // amax = f 2^x, f in [0.5, 1); 448 = 0.875 * 2^9
    int32_t e = (f <= 0.875f) ? x - 9 : x - 8;
    e = e < -kExpLimit ? -kExpLimit : e;
    return e > kExpLimit ? kExpLimit : e;
}
__device__ __forceinline__ float pow2(int32_t e) { return __int_as_float((127 + e) << 23); }  // |e| <= 126

// two fp32 values -> two E4M3 codes in the low or high half of a 32-bit word (round to nearest even)
template <bool HIGH>
__device__ __forceinline__ int32_t pack2(float a, float b, int32_t old)
{
    return __builtin_amdgcn_cvt_pk_fp8_f32(a, b, old, HIGH);
}
// four fp32 values -> four codes; both halves of the word are written, so what it held before does not matter
// (a word started from 0 costs a move per pair of conversions)
__device__ __forceinline__ int32_t pack4(float a, float b, float c, float d)
{
    int32_t v;
    asm("" : "=v"(v));
    return pack2<true>(c, d, pack2<false>(a, b, v));
}
__device__ __forceinline__ i32x4v quantise16(const float (&x)[16], float inv_scale)
{
    i32x4v r;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
        r[w] = pack4(x[4 * w] * inv_scale, x[4 * w + 1] * inv_scale, x[4 * w + 2] * inv_scale, x[4 * w + 3] * inv_scale);
    }
    return r;
}
__device__ __forceinline__ void bf16x8_to_f32(const uint4 &raw, float *dst)
{
    const uint32_t w[4] = {raw.x, raw.y, raw.z, raw.w};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        dst[2 * i] = __uint_as_float(w[i] << 16);
        dst[2 * i + 1] = __uint_as_float(w[i] & 0xffff0000u);
    }
}

// largest magnitude of eight pairs of bf16 values, as the bit pattern of an fp32 value: magnitudes order like the
// 15-bit integers that encode them, so the two halves of a word are compared by one packed maximum
__device__ __forceinline__ uint32_t largest_magnitude(const uint32_t (&w)[8])
{
    typedef __attribute__((ext_vector_type(2))) uint16_t u16x2;
    u16x2 m = {0, 0};
#pragma unroll
    for (int i = 0; i < 8; ++i) m = __builtin_elementwise_max(m, __builtin_bit_cast(u16x2, w[i] & 0x7fff7fffu));
    return (uint32_t)(m[0] > m[1] ? m[0] : m[1]) << 16;
}

// position of the 16-byte chunk c of row r inside a staged tile whose rows hold CPR chunks: rows that
// 16 consecutive lanes read together are spread over all LDS banks
template <int CPR>
__host__ __device__ __forceinline__ int32_t swizzled_chunk(int32_t r, int32_t c)
{
    return c ^ ((r / (16 / CPR)) % CPR);
}

// One k-step of the scores of 64 keys x 32 rows: s[kc] = c + K Q^T with the block exponents of K and Q, c = 0, the
// start values or s[kc].  Written as instructions because both chunks start from the same 16 registers:
// left to the compiler the start values are copied for one of the chunks on every tile.  The compiler sees no matrix
// instruction here, so the waits are part of the block: two states in front, for operands that a vector instruction has
// just written, and after the LAST step the 16 passes and 4 states that a reader of the results needs (row_max_grouped
// reads them in instructions of its own, so that a builtin as the last step would not do).  Between two steps a
// chunk's MFMAs are one MFMA (64 cycles) apart, which the chained accumulator needs no wait for.
enum { kFromZero, kFromStart, kContinue };
template <int FROM, bool LAST>
__device__ __forceinline__ void score_step(const i32x8 &k0, const i32x8 &k1, const i32x8 &q, const f32x16 &start, int32_t k_exp8,
                                           int32_t q_exp8, f32x16 (&s)[2])
{
#define PEVLM_SCORE(dst, kreg, creg) "v_mfma_scale_f32_32x32x64_f8f6f4 " dst ", " kreg ", %4, " creg ", %5, %6 op_sel_hi:[0,0,0]\n\t"
#define PEVLM_SCORES(bind, c0, c1, tail, ...)                                                                   \
    asm volatile("s_nop 1\n\t" PEVLM_SCORE("%0", "%2", c0) PEVLM_SCORE("%1", "%3", c1) tail                     \
                 : bind(s[0]), bind(s[1]) : "v"(k0), "v"(k1), "v"(q), "v"(k_exp8), "v"(q_exp8), ##__VA_ARGS__)
#define PEVLM_WAIT "s_nop 15\n\ts_nop 3"
    if (FROM == kFromZero) {
        if (LAST) PEVLM_SCORES("=&v", "0", "0", PEVLM_WAIT);
        else PEVLM_SCORES("=&v", "0", "0", "");
    } else if (FROM == kFromStart) {
        if (LAST) PEVLM_SCORES("=&v", "%7", "%7", PEVLM_WAIT, "v"(start));
        else PEVLM_SCORES("=&v", "%7", "%7", "", "v"(start));
    } else {
        if (LAST) PEVLM_SCORES("+v", "%0", "%1", PEVLM_WAIT);
        else PEVLM_SCORES("+v", "%0", "%1", "");
    }
#undef PEVLM_WAIT
#undef PEVLM_SCORES
#undef PEVLM_SCORE
}

// maximum of 8 values without the quieting moves that plain fmaxf puts in front of values it cannot prove canonical
__device__ __forceinline__ float max8(float a, float b, float c, float d, float e, float f, float g, float h)
{
    float r;
    asm("v_max3_f32 %0, %1, %2, %3\n\tv_max3_f32 %0, %0, %4, %5\n\tv_max3_f32 %0, %0, %6, %7\n\tv_max_f32 %0, %0, %8"
        : "=&v"(r) : "v"(a), "v"(b), "v"(c), "v"(d), "v"(e), "v"(f), "v"(g), "v"(h));
    return r;
}
// maximum over the 64 keys of the tile for this lane's row (both lanes of a row end up with it)
__device__ __forceinline__ float row_max_grouped(const f32x16 (&s)[2])
{
    const float m0 = max8(s[0][0], s[0][1], s[0][2], s[0][3], s[0][4], s[0][5], s[0][6], s[0][7]);
    const float m1 = max8(s[0][8], s[0][9], s[0][10], s[0][11], s[0][12], s[0][13], s[0][14], s[0][15]);
    const float m2 = max8(s[1][0], s[1][1], s[1][2], s[1][3], s[1][4], s[1][5], s[1][6], s[1][7]);
    const float m3 = max8(s[1][8], s[1][9], s[1][10], s[1][11], s[1][12], s[1][13], s[1][14], s[1][15]);
    const float mx = fmaxf(max3f(m0, m1, m2), m3);
    const auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(mx), __float_as_uint(mx), false, false);
    return fmaxf(__uint_as_float(sw[0]), __uint_as_float(sw[1]));
}

// Q: one scale per (token, head); D/16 consecutive lanes share a row of one head (rh: token x heads + head, c: the lane's
// 16 values).  What is quantised is q * factor (factor = softmax factor * log2(e), one fp32 multiplication per element),
// so that the score MFMAs deliver base-2 exponents.
template <int D>
__device__ __forceinline__ void quantise_q_part(const uint16_t *q, int64_t rh, bool live, int32_t c, float factor, uint8_t *codes, float *scales)
{
    float x[16];
    if (live) {
        const uint4 *src = reinterpret_cast<const uint4 *>(q + rh * D + c * 16);
        bf16x8_to_f32(src[0], x);
        bf16x8_to_f32(src[1], x + 8);
#pragma unroll
        for (int i = 0; i < 16; ++i) x[i] = __fmul_rn(x[i], factor);
    } else {
#pragma unroll
        for (int i = 0; i < 16; ++i) x[i] = 0.f;
    }
    float m = 0.f;
#pragma unroll
    for (int i = 0; i < 16; ++i) m = fmaxf(m, fabsf(x[i]));
#pragma unroll
    for (int off = D / 32; off >= 1; off >>= 1) m = fmaxf(m, __shfl_xor(m, off));
    const int32_t e = scale_exponent(m);
    if (live) {
        *reinterpret_cast<i32x4v *>(codes + rh * D + c * 16) = quantise16(x, pow2(-e));
        if (c == 0) scales[rh] = pow2(e);
    }
}

}  // namespace

// ---------------------------------------------------------------- work lists
// Both lists of a chunk of sequences (tiles.item_base counts 64-row key tiles, items.item_base 128-row items) and,
// with the first chunk, the zeros that the maxima start from: one launch instead of three of 4-5 us each.  Workgroups
// from list_blocks on quantise the chunk's question rows (n_question of them, tab.qrow_base counts them) in a call
// whose attention kernel quantises the other rows.
template <int D>
__global__ __launch_bounds__(256) void fp8_setup_kernel(SeqTable tab, Fp8TileBases bases, Fp8ItemBases items_of, pevlm_work_item *key_tiles,
                                                        int32_t tile_offset, Fp8Item *items, int32_t item_offset, uint32_t *zero, int32_t n_zero,
                                                        int32_t list_blocks, Fp8Question qu)
{
    if ((int32_t)blockIdx.x >= list_blocks) {
        // 32 bits hold a (row, head) number: 2^32 rows of one head would be a tensor of 512 GB and more
        const uint32_t block = (uint32_t)((int32_t)blockIdx.x - list_blocks), unit = block * (256 / (D / 16)) + threadIdx.x / (D / 16);
        const int32_t r = (int32_t)(unit / (uint32_t)qu.n_q_heads), head = (int32_t)(unit - (uint32_t)r * (uint32_t)qu.n_q_heads);
        int32_t s = 0;
        while (s + 1 < tab.num_seqs && r >= tab.qrow_base[s + 1]) ++s;
        const int64_t row = tab.start[s] + tab.sink[s] + tab.ctx[s] + r - tab.qrow_base[s];
        quantise_q_part<D>((const uint16_t *)qu.q, row * qu.n_q_heads + head, r < qu.n_rows, (int32_t)(threadIdx.x % (D / 16)), qu.factor, qu.codes, qu.scales);
        return;
    }
    const int32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n_zero) zero[i] = 0u;
    if (i < tab.item_base[tab.num_seqs]) {
        int32_t s = 0;
        while (s + 1 < tab.num_seqs && i >= tab.item_base[s + 1]) ++s;
        key_tiles[tile_offset + i] = prefill_item(tab.start[s], tab.sink[s], tab.block[s], tab.ctx[s], kKeyTile, i - tab.item_base[s], tab.seq_index0 + s);
    }
    if (i < items_of.base[tab.num_seqs]) {
        int32_t s = 0;
        while (s + 1 < tab.num_seqs && i >= items_of.base[s + 1]) ++s;
        const int32_t S = tab.sink[s], B = tab.block[s];
        const pevlm_work_item w = prefill_item(tab.start[s], S, B, tab.ctx[s], kFp8TileRows, i - items_of.base[s], tab.seq_index0 + s);
        Fp8Item it;
        it.q_start = w.q_start;
        it.q_rows = w.q_rows;
        it.full_start = w.full_start;
        it.full_len = w.full_len;
        it.full_tile0 = bases.base[s];  // the sink is the first region of the sequence
        it.diag_start = w.diag_start;
        it.diag_len = w.diag_len;
        const int32_t local = w.diag_start - tab.start[s];  // first position of the item's own region
        it.diag_tile0 = bases.base[s] + (local < S ? 0 : ceil_div(S, kKeyTile) + ((local - S) / B) * ceil_div(B, kKeyTile));
        items[item_offset + i] = it;
    }
}

// ---------------------------------------------------------------- quantise
// Largest magnitude per KV head of K (amax[g]) and V (amax[Hkv + g]): blockIdx.y = tensor.  The tensor is read
// front to back, 16 bytes a lane, in steps that are a multiple of a token's row, so that a lane stays in one
// head (reading one head's 256 bytes out of every row: 40 us for the 135 MB of 66K tokens x 4 heads; whole rows:
// 33 us, of which 5 us are the launch).  Bit patterns of non-negative floats order like the floats, so the reduction is an integer
// maximum, and a bf16 pair's magnitudes compare as its two halves.
template <int D>
__global__ __launch_bounds__(256) void amax_kv_kernel(const uint16_t *k, const uint16_t *v, int64_t T, int32_t Hkv, uint32_t *amax)
{
    const int32_t chunks = Hkv * (D / 8);  // 16-byte chunks of a token's row
    const int64_t total = T * chunks;
    const int64_t lanes = (int64_t)gridDim.x * 256, step = lanes / chunks * chunks;  // the launch has at least one row of lanes
    const int64_t first = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const uint4 *src = reinterpret_cast<const uint4 *>(blockIdx.y ? v : k);
    __shared__ uint32_t head_max[kMaxHeads];
    for (int32_t i = threadIdx.x; i < Hkv; i += 256) head_max[i] = 0u;
    __syncthreads();
    uint32_t lo = 0u, hi = 0u;  // maxima of the magnitudes in the low and high halves, both as (value << 16)
    auto take = [&](uint32_t w) {
        const uint32_t l = (w << 16) & 0x7fff0000u, h = w & 0x7fff0000u;
        lo = l > lo ? l : lo;
        hi = h > hi ? h : hi;
    };
    if (first < step) {
        int64_t i = first;
        constexpr int U = 8;  // loads in flight per lane
        for (; i + (U - 1) * step < total; i += U * step) {
            uint4 raw[U];
#pragma unroll
            for (int u = 0; u < U; ++u) raw[u] = src[i + u * step];
#pragma unroll
            for (int u = 0; u < U; ++u) { take(raw[u].x); take(raw[u].y); take(raw[u].z); take(raw[u].w); }
        }
        for (; i < total; i += step) {
            const uint4 raw = src[i];
            take(raw.x); take(raw.y); take(raw.z); take(raw.w);
        }
        // lanes of a head first (D/8 neighbours share one), then the workgroup, then one atomic per workgroup and head
        uint32_t m = lo > hi ? lo : hi;
#pragma unroll
        for (int off = D / 16; off >= 1; off >>= 1) {
            const uint32_t x = (uint32_t)__shfl_xor((int32_t)m, off);
            m = x > m ? x : m;
        }
        if (threadIdx.x % (D / 8) == 0) atomicMax(&head_max[(int32_t)((first % chunks) / (D / 8))], m);
    }
    __syncthreads();
    for (int32_t i = threadIdx.x; i < Hkv; i += 256)
        if (head_max[i]) atomicMax(amax + blockIdx.y * Hkv + i, head_max[i]);
}

template <int D>
__global__ __launch_bounds__(256) void quantise_q_kernel(const uint16_t *q, int64_t n_rows_heads, float factor, uint8_t *codes, float *scales)
{
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    quantise_q_part<D>(q, t / (D / 16), t / (D / 16) < n_rows_heads, (int32_t)(t % (D / 16)), factor, codes, scales);
}

// K and V tiles: blockIdx.x = key tile (64 rows of one region), blockIdx.y = KV head.
//   K tile image: 64 rows of D bytes, chunk c of row r at chunk position swizzled_chunk<D/16>(r, c).
//   V tile image: D rows (head_dim) of 64 bytes; byte j of a row is key
//       kappa(j) = ((j % 32) / 16) * 32 + ((j % 16) / 4) * 8 + (j / 32) * 4 + j % 4
//   of the tile (the order in which the two halves of a wavefront hold the keys of a score tile);
//   chunk c of row d at chunk position swizzled_chunk<4>(d, c).
template <int D>
__global__ __launch_bounds__(256) void quantise_kv_tiles_kernel(const uint16_t *k, const uint16_t *v, const pevlm_work_item *key_tiles,
                                                                int32_t Hkv, const uint32_t *amax, uint8_t *k_tiles, uint8_t *v_tiles)
{
    constexpr int CPR = D / 16, TILEB = kKeyTile * D;
    __shared__ uint16_t vt[kKeyTile][D + 2];
    const int32_t tile = blockIdx.x, g = blockIdx.y, tid = threadIdx.x;
    const pevlm_work_item it = key_tiles[tile];
    const float k_inv = pow2(-scale_exponent(__uint_as_float(amax[g])));
    const float v_inv = pow2(-scale_exponent(__uint_as_float(amax[Hkv + g])));
    uint8_t *kdst = k_tiles + ((int64_t)tile * Hkv + g) * TILEB;
    uint8_t *vdst = v_tiles + ((int64_t)tile * Hkv + g) * TILEB;
    // K: 16 values of one row per step; V rows into LDS
    for (int32_t u = tid; u < kKeyTile * CPR; u += 256) {
        const int32_t r = u / CPR, c = u % CPR;
        float x[16];
        uint4 v0 = {0, 0, 0, 0}, v1 = {0, 0, 0, 0};
        if (r < it.q_rows) {
            const int64_t row = ((int64_t)(it.q_start + r) * Hkv + g) * D + c * 16;
            const uint4 *ks = reinterpret_cast<const uint4 *>(k + row);
            bf16x8_to_f32(ks[0], x);
            bf16x8_to_f32(ks[1], x + 8);
            const uint4 *vs = reinterpret_cast<const uint4 *>(v + row);
            v0 = vs[0];
            v1 = vs[1];
        } else {
#pragma unroll
            for (int i = 0; i < 16; ++i) x[i] = 0.f;
        }
        *reinterpret_cast<i32x4v *>(kdst + r * D + swizzled_chunk<CPR>(r, c) * 16) = quantise16(x, k_inv);
        const uint32_t w[8] = {v0.x, v0.y, v0.z, v0.w, v1.x, v1.y, v1.z, v1.w};
#pragma unroll
        for (int i = 0; i < 8; ++i) *reinterpret_cast<uint32_t *>(&vt[r][c * 16 + 2 * i]) = w[i];
    }
    __syncthreads();
    for (int32_t u = tid; u < D * 4; u += 256) {
        const int32_t d = u / 4, c = u % 4;
        float x[16];
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            const int32_t j = c * 16 + i;
            const int32_t key = ((j % 32) / 16) * 32 + ((j % 16) / 4) * 8 + (j / 32) * 4 + j % 4;
            x[i] = __uint_as_float((uint32_t)vt[key][d] << 16);
        }
        *reinterpret_cast<i32x4v *>(vdst + d * kKeyTile + swizzled_chunk<4>(d, c) * 16) = quantise16(x, v_inv);
    }
}

// ---------------------------------------------------------------- attend
// Three wavefronts per SIMD (the second launch bound): it keeps the kernel within 168 registers (head_dim 128 uses
// them all and, where it quantises Q, spills two), all of them ordinary vector registers -- given more, the
// compiler parks the MFMA results in accumulation registers and copies them back and forth around every softmax
// step (measured 24 % slower) -- and lets the vector work of one wavefront run under the MFMAs of the others.
//
// QUANTISE_Q (a call of both stages): every row of Q is used by exactly one wavefront, which quantises it on the
// way in and leaves codes and scales in the workspace for later ATTEND calls.  The separate kernel reads 472 MB
// and writes 236 MB of codes that are then read back (64K tokens x 28 heads: 115 us); here the same rows cost
// 55 us of vector arithmetic inside a kernel that leaves HBM three quarters idle (attention 464 -> 520 us).
template <int D, bool QUANTISE_Q>
__global__ __launch_bounds__(256, 3) void attn_fp8_kernel(Fp8Params p)
{
    constexpr int KT = kKeyTile, CPR = D / 16, TILEB = KT * D;
    constexpr int KQ = D / 64;            // score MFMAs (64 values of head_dim each) per 32-key chunk
    constexpr int DBLK = D / 32;          // 32-wide blocks of head_dim in O^T
    constexpr int NLD = TILEB / (256 * 16);
    constexpr int ROWB = D * 2, CH = D / 8, RPI = 1024 / ROWB, NOL = 32 * ROWB / 1024;  // output rows through LDS
    static_assert(4 * TILEB == 4 * 32 * ROWB, "the output slices reuse the four tile stages");
    __shared__ __attribute__((aligned(1024))) uint8_t lds[4 * TILEB];  // K stage 0, 1, V stage 0, 1

    // consecutive (item, head) pairs on one XCD: workgroup b runs on XCD b % 8
    const int32_t n_work = p.n_items * p.n_q_heads;
    const int32_t per_xcd = (n_work + 7) >> 3;
    const int32_t work = (int32_t)(blockIdx.x & 7) * per_xcd + (int32_t)(blockIdx.x >> 3);
    if ((int32_t)(blockIdx.x >> 3) >= per_xcd || work >= n_work) return;
    const Fp8Item it = p.items[work / p.n_q_heads];
    const int32_t head = __builtin_amdgcn_readfirstlane((int32_t)p.heads.head_order[work % p.n_q_heads]);
    const int32_t g = __builtin_amdgcn_readfirstlane((int32_t)p.heads.kv_of_q[head]);
    const int32_t Hq = p.n_q_heads, Hkv = p.n_kv_heads;

    const int32_t tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int32_t l32 = lane & 31, g32 = lane >> 5;
    const int32_t n_full = ceil_div(it.full_len, KT), n_tiles = n_full + ceil_div(it.diag_len, KT);
    const int32_t w_rows = min(max(it.q_rows - wave * 32, 0), 32);
    const int32_t wr_lo = it.q_start + wave * 32, wr_hi = wr_lo + w_rows - 1;
    int32_t n_w = 0;  // tiles this wavefront computes: all of the sink, its own region up to its last row
    if (w_rows > 0) n_w = n_full + min((wr_hi - it.diag_start) / KT + 1, n_tiles - n_full);
    const int32_t my_row = w_rows > 0 ? wr_lo + (l32 < w_rows ? l32 : w_rows - 1) : it.q_start;  // always a row of the item

    const uint32_t lds_addr = (uint32_t)(size_t)LDS_PTR(void, lds);
    const uint8_t *const k_head = p.k_tiles + (int64_t)g * TILEB, *const v_head = p.v_tiles + (int64_t)g * TILEB;
    const int64_t tile_stride = (int64_t)Hkv * TILEB;
#define PEVLM_FP8_LOAD_TILE(t, stage)                                                                              \
    do {                                                                                                           \
        const int64_t ti_ = (t) < n_full ? it.full_tile0 + (t) : it.diag_tile0 + ((t) - n_full);                   \
        const uint8_t *ks_ = uniform_ptr(k_head + ti_ * tile_stride), *vs_ = uniform_ptr(v_head + ti_ * tile_stride); \
        _Pragma("unroll") for (int j = 0; j < NLD; ++j) {                                                          \
            load_lds_16_base(ks_, (uint32_t)((j * 256 + tid) * 16), lds_addr + (stage) * TILEB + (j * 4 + wave) * 1024); \
            load_lds_16_base(vs_, (uint32_t)((j * 256 + tid) * 16), lds_addr + (2 + (stage)) * TILEB + (j * 4 + wave) * 1024); \
        }                                                                                                          \
    } while (0)

    PEVLM_FP8_LOAD_TILE(0, 0);

    // query fragments: lane (row l32, half g32) holds head_dim [64 kk + 32 g32, +32) of its row
    i32x8 qf[KQ];
    int32_t q_exp8;
    const int64_t q_unit = (int64_t)my_row * Hq + head;
    if (QUANTISE_Q) {
        // D/16 lanes share a row, so that rows are read and codes written as whole lines; the codes reach the lanes
        // that need them through a wavefront-private quarter of tile stage 1, which is free until every wavefront
        // has passed the top of tile 0.
        constexpr int LPR = D / 16, RPS = 64 / LPR, NS = 32 / RPS;  // lanes per row, rows per step, steps
        uint8_t *const slice = lds + ((wave >> 1) * 2 + 1) * TILEB + (wave & 1) * (32 * D);
        const int32_t c = lane % LPR;
        uint4 raw[NS][2];
#pragma unroll
        for (int st = 0; st < NS; ++st) {
            const int32_t r = st * RPS + lane / LPR, row = w_rows > 0 ? wr_lo + (r < w_rows ? r : w_rows - 1) : it.q_start;
            const uint4 *src = reinterpret_cast<const uint4 *>((const uint16_t *)p.q + ((int64_t)row * Hq + head) * D + c * 16);
            raw[st][0] = src[0];
            raw[st][1] = src[1];
        }
        q_exp8 = 0;
#pragma unroll
        for (int st = 0; st < NS; ++st) {
            const uint32_t w[8] = {raw[st][0].x, raw[st][0].y, raw[st][0].z, raw[st][0].w, raw[st][1].x, raw[st][1].y, raw[st][1].z, raw[st][1].w};
            uint32_t m = largest_magnitude(w);
#pragma unroll
            for (int off = LPR / 2; off >= 1; off >>= 1) m = max(m, (uint32_t)__shfl_xor((int32_t)m, off));
            // rounding is monotonic: the largest |q * factor| is the largest |q| times factor.  Multiplying by factor
            // and then by the power of two rounds like multiplying by their product, but where the product of the
            // first multiplication is subnormal, and there the code is 0 either way.
            const int32_t e = scale_exponent(__fmul_rn(__uint_as_float(m), p.q_factor));
            const float mul = p.q_factor * pow2(-e);
            float x[16];
            bf16x8_to_f32(raw[st][0], x);
            bf16x8_to_f32(raw[st][1], x + 8);
            const i32x4v codes = quantise16(x, mul);
            const int32_t r = st * RPS + lane / LPR;
            *reinterpret_cast<i32x4v *>(slice + r * D + swizzled_chunk<CPR>(r, c) * 16) = codes;
            const int32_t mine = __shfl(127 + e, (l32 % RPS) * LPR);
            if (l32 / RPS == st) q_exp8 = mine;
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
        for (int kk = 0; kk < KQ; ++kk) {
            const int32_t c0 = kk * 4 + g32 * 2;
            const i32x4v a = *reinterpret_cast<const i32x4v *>(slice + l32 * D + swizzled_chunk<CPR>(l32, c0) * 16);
            const i32x4v b = *reinterpret_cast<const i32x4v *>(slice + l32 * D + swizzled_chunk<CPR>(l32, c0 + 1) * 16);
            qf[kk] = i32x8{a[0], a[1], a[2], a[3], b[0], b[1], b[2], b[3]};
        }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // the slice has been read before this wavefront passes a barrier
    } else {
        const uint8_t *qrow = p.q_codes + q_unit * D;
#pragma unroll
        for (int kk = 0; kk < KQ; ++kk) {
            const i32x4v a = *reinterpret_cast<const i32x4v *>(qrow + kk * 64 + g32 * 32);
            const i32x4v b = *reinterpret_cast<const i32x4v *>(qrow + kk * 64 + g32 * 32 + 16);
            qf[kk] = i32x8{a[0], a[1], a[2], a[3], b[0], b[1], b[2], b[3]};
        }
        q_exp8 = (__float_as_int(p.q_scales[q_unit]) >> 23) & 0xff;
    }
    // The scales of K (per head) and of the query row (per lane: both halves of the wavefront hold the same
    // rows) go into the score MFMAs as 8-bit exponents; the accumulators start from kWeightShift minus the
    // row's reference maximum, so the MFMAs deliver the exponents of the weights directly.
    const int32_t k_exp8 = 127 + scale_exponent(__uint_as_float(p.kv_amax[g]));
    const float v_scale = pow2(scale_exponent(__uint_as_float(p.kv_amax[Hkv + g])));

    f32x16 o[DBLK], s[2];
    float m_ref = -INFINITY, l_run = 0.f;
    float shift = 0.f;  // kWeightShift - reference maximum, once there is one
    f32x16 start;       // the same in all 16 accumulator registers of the lane

    // Tile t for this wavefront.  The first one has no reference yet: its scores start from the inline constant 0
    // and are moved to their own maximum, its value MFMAs start the accumulators -- no clearing and rescaling of
    // 64 + 16 registers that hold nothing (150 of the 2700 vector instructions of an item of 12 tiles).
    auto tile_top = [&](int32_t t) {
        __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0): this wavefront's share of tile t has landed
        __builtin_amdgcn_s_barrier();        // ... everybody's has, and everybody has left tile t - 1
        asm volatile("" ::: "memory");
        if (t + 1 < n_tiles) PEVLM_FP8_LOAD_TILE(t + 1, (t + 1) & 1);
    };
    auto tile_step = [&](auto first_tag, int32_t t) {
        constexpr bool FIRST = decltype(first_tag)::value;
        const uint8_t *tk = lds + (t & 1) * TILEB, *tv = lds + (2 + (t & 1)) * TILEB;
        // ---- S^T = K Q^T: rows = keys of the chunk, columns = this wavefront's query rows
        auto read_k = [&](int kk, int kc) {
            const int32_t r = kc * 32 + l32, c0 = kk * 4 + g32 * 2;
            const i32x4v a = *reinterpret_cast<const i32x4v *>(tk + r * D + swizzled_chunk<CPR>(r, c0) * 16);
            const i32x4v b = *reinterpret_cast<const i32x4v *>(tk + r * D + swizzled_chunk<CPR>(r, c0 + 1) * 16);
            return i32x8{a[0], a[1], a[2], a[3], b[0], b[1], b[2], b[3]};
        };
        score_step<FIRST ? kFromZero : kFromStart, KQ == 1>(read_k(0, 0), read_k(0, 1), qf[0], start, k_exp8, q_exp8, s);
        if (KQ == 2) score_step<kContinue, true>(read_k(KQ - 1, 0), read_k(KQ - 1, 1), qf[KQ - 1], start, k_exp8, q_exp8, s);
        int32_t k0, kend;
        bool causal;
        if (t < n_full) {
            k0 = it.full_start + t * KT; kend = it.full_start + it.full_len; causal = false;
        } else {
            k0 = it.diag_start + (t - n_full) * KT; kend = it.diag_start + it.diag_len; causal = true;
        }
        if ((k0 + KT > kend) || (causal && (k0 + KT - 1 > wr_lo))) mask_tile(s, k0, kend, causal, my_row, g32);
        // ---- reference maximum: raised to the running maximum once that is more than kWeightLag above it
        const float mx = row_max_grouped(s) - shift;
        const bool raise = mx > m_ref + kWeightLag;
        if (FIRST || __any(raise)) {
            const float m_new = raise ? mx : m_ref;
            if (!FIRST) {
                const float alpha = __builtin_amdgcn_exp2f(m_ref - m_new);  // 1 where nothing changes
                l_run *= alpha;
#pragma unroll
                for (int b = 0; b < DBLK; ++b)
#pragma unroll
                    for (int i = 0; i < 16; ++i) o[b][i] *= alpha;
            }
            m_ref = m_new;
            // the scores of this tile move to the new reference; later tiles start from it
            const float new_shift = kWeightShift - m_ref;
            const float delta = new_shift - shift;
            shift = new_shift;
#pragma unroll
            for (int kc = 0; kc < 2; ++kc)
#pragma unroll
                for (int i = 0; i < 16; ++i) s[kc][i] += delta;
#pragma unroll
            for (int i = 0; i < 16; ++i) start[i] = shift;
        }
        // the V fragments of the first value MFMA are requested before the weights are formed
        auto read_v = [&](int b) {
            const int32_t d = b * 32 + l32;
            const i32x4v a = *reinterpret_cast<const i32x4v *>(tv + d * KT + swizzled_chunk<4>(d, g32 * 2) * 16);
            const i32x4v c = *reinterpret_cast<const i32x4v *>(tv + d * KT + swizzled_chunk<4>(d, g32 * 2 + 1) * 16);
            return i32x8{a[0], a[1], a[2], a[3], c[0], c[1], c[2], c[3]};
        };
        i32x8 vf[2];
        vf[0] = read_v(0);
        __builtin_amdgcn_sched_barrier(0);
        // ---- weights: E4M3 codes in the order the value MFMA wants them (byte 16 kc + i of the lane)
        float psum = 0.f;
        i32x8 pf;
#pragma unroll
        for (int kc = 0; kc < 2; ++kc)
#pragma unroll
            for (int w = 0; w < 4; ++w) {
                const float w0 = __builtin_amdgcn_exp2f(s[kc][4 * w]);
                const float w1 = __builtin_amdgcn_exp2f(s[kc][4 * w + 1]);
                const float w2 = __builtin_amdgcn_exp2f(s[kc][4 * w + 2]);
                const float w3 = __builtin_amdgcn_exp2f(s[kc][4 * w + 3]);
                psum += (w0 + w1) + (w2 + w3);
                pf[kc * 4 + w] = pack4(w0, w1, w2, w3);
            }
        l_run += psum;
        // ---- O^T += V^T P^T
        const f32x16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int b = 0; b < DBLK; ++b) {
            if (b + 1 < DBLK) vf[(b + 1) & 1] = read_v(b + 1);
            o[b] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(vf[b & 1], pf, FIRST ? zero : o[b], 0, 0, 0, 0, 0, 0);
        }
    };
    tile_top(0);
    if (n_w > 0) tile_step(std::true_type(), 0);
    for (int32_t t = 1; t < n_tiles; ++t) {
        tile_top(t);
        if (t < n_w) tile_step(std::false_type(), t);
    }
#undef PEVLM_FP8_LOAD_TILE

    // The codes and scales of Q leave with the output: stored in front of the loop they would be waited for at the top
    // of the first tile (stores and the tile loads share a counter).
    if (QUANTISE_Q && l32 < w_rows) {
        uint8_t *dst = p.q_codes + q_unit * D + g32 * 32;
#pragma unroll
        for (int kk = 0; kk < KQ; ++kk) {
            *reinterpret_cast<i32x4v *>(dst + kk * 64) = i32x4v{qf[kk][0], qf[kk][1], qf[kk][2], qf[kk][3]};
            *reinterpret_cast<i32x4v *>(dst + kk * 64 + 16) = i32x4v{qf[kk][4], qf[kk][5], qf[kk][6], qf[kk][7]};
        }
        if (g32 == 0) p.q_scales[q_unit] = pow2(q_exp8 - 127);
    }
    // ---- output: normalise, undo the V scale, rows out through LDS as whole 2 D-byte rows (non-temporal: nothing here
    // reads them again; 64K call 604 -> 595 us)
    __syncthreads();  // every wavefront has left the tile stages
    uint8_t *slice = lds + wave * 32 * ROWB;
    const float l_tot = l_run + __shfl_xor(l_run, 32);
    const float inv = v_scale / l_tot;
#pragma unroll
    for (int b = 0; b < DBLK; ++b)
#pragma unroll
        for (int i4 = 0; i4 < 4; ++i4) {
            bf16x4 v4;
            v4[0] = (__bf16)(o[b][i4 * 4] * inv);
            v4[1] = (__bf16)(o[b][i4 * 4 + 1] * inv);
            v4[2] = (__bf16)(o[b][i4 * 4 + 2] * inv);
            v4[3] = (__bf16)(o[b][i4 * 4 + 3] * inv);
            *reinterpret_cast<bf16x4 *>(slice + l32 * ROWB + (((b * 4 + i4) ^ (l32 & (CH - 1))) << 4) + g32 * 8) = v4;
        }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    uint8_t *const obase = (uint8_t *)p.out + ((int64_t)wr_lo * Hq + head) * ROWB;  // wavefront-uniform
    const int32_t cp = lane % CH;
    uint32_t off = (uint32_t)(lane / CH * Hq * ROWB + cp * 16);
#pragma unroll
    for (int j = 0; j < NOL; ++j, off += (uint32_t)(RPI * Hq * ROWB)) {
        const int32_t rl = j * RPI + lane / CH;
        const uint4 val = *reinterpret_cast<const uint4 *>(slice + rl * ROWB + ((cp ^ (rl & (CH - 1))) << 4));
        if (rl < w_rows) __builtin_nontemporal_store(__builtin_bit_cast(u32x4, val), reinterpret_cast<u32x4 *>(obase + off));
    }
    if (p.lse && g32 == 0 && l32 < w_rows)
        p.lse[(int64_t)(wr_lo + l32) * Hq + head] = (m_ref - kWeightShift + __log2f(l_tot)) * 0.69314718056f;
}

// ---------------------------------------------------------------- launchers
hipError_t launch_fp8_setup(const SeqTable &tab, const Fp8TileBases &bases, const Fp8ItemBases &items_of, pevlm_work_item *key_tiles,
                            int32_t tile_offset, Fp8Item *items, int32_t item_offset, uint32_t *zero, int32_t n_zero, const Fp8Question &qu,
                            int32_t D, hipStream_t stream)
{
    const int32_t n = std::max(std::max(tab.item_base[tab.num_seqs], items_of.base[tab.num_seqs]), n_zero);
    const int32_t list_blocks = ceil_div(n, 256);
    const int64_t threads = (int64_t)qu.n_rows * qu.n_q_heads * (D / 16), blocks = list_blocks + (threads + 255) / 256;
    if (blocks == 0) return hipSuccess;
    const auto kernel = D == 128 ? fp8_setup_kernel<128> : fp8_setup_kernel<64>;
    hipLaunchKernelGGL(kernel, dim3((uint32_t)blocks), dim3(256), 0, stream, tab, bases, items_of, key_tiles, tile_offset, items,
                       item_offset, zero, n_zero, list_blocks, qu);
    return hipGetLastError();
}

template <int D>
static void quantise_launches(const uint16_t *q, const uint16_t *k, const uint16_t *v, int64_t T, int32_t Hq, int32_t Hkv, float q_factor,
                              const pevlm_work_item *key_tiles, int32_t n_key_tiles, uint32_t *kv_amax, float *q_scales, uint8_t *q_codes,
                              uint8_t *k_tiles, uint8_t *v_tiles, int32_t compute_units, bool with_q, hipStream_t stream)
{
    // K and V twice in a row, so that the second reading finds what the last-level cache kept of the first (64K
    // tokens: tiles 31 us, 43 us with Q's kernel in between).  One workgroup per compute unit and tensor for the maxima:
    // with four, 4096 atomics on 8 words cost 5 us of 38.
    const int64_t chunks = T * Hkv * (D / 8);
    const int32_t row_blocks = (Hkv * (D / 8) + 255) / 256;  // at least one row of lanes
    const int32_t bx = (int32_t)std::max<int64_t>(row_blocks, std::min<int64_t>((chunks + 2047) / 2048, compute_units));
    hipLaunchKernelGGL((amax_kv_kernel<D>), dim3(bx, 2), dim3(256), 0, stream, k, v, T, Hkv, kv_amax);
    hipLaunchKernelGGL((quantise_kv_tiles_kernel<D>), dim3(n_key_tiles, Hkv), dim3(256), 0, stream, k, v, key_tiles, Hkv, kv_amax, k_tiles, v_tiles);
    if (with_q) {
        const int64_t q_threads = T * Hq * (D / 16);
        hipLaunchKernelGGL((quantise_q_kernel<D>), dim3((uint32_t)((q_threads + 255) / 256)), dim3(256), 0, stream, q, T * Hq, q_factor, q_codes, q_scales);
    }
}

hipError_t launch_fp8_quantise(const void *q, const void *k, const void *v, int64_t T, int32_t Hq, int32_t Hkv, int32_t D,
                               float q_factor, const pevlm_work_item *key_tiles, int32_t n_key_tiles, uint32_t *kv_amax, float *q_scales,
                               uint8_t *q_codes, uint8_t *k_tiles, uint8_t *v_tiles, int32_t compute_units, bool with_q, hipStream_t stream)
{
    const auto launches = D == 128 ? quantise_launches<128> : quantise_launches<64>;
    launches((const uint16_t *)q, (const uint16_t *)k, (const uint16_t *)v, T, Hq, Hkv, q_factor, key_tiles, n_key_tiles, kv_amax, q_scales, q_codes,
             k_tiles, v_tiles, compute_units, with_q, stream);
    return hipGetLastError();
}

hipError_t launch_attn_fp8(const Fp8Params &p, int32_t D, hipStream_t stream)
{
    const int32_t n_work = p.n_items * p.n_q_heads;
    const dim3 grid(8 * ((n_work + 7) / 8)), block(256);
    const bool quantise_q = p.q != nullptr;
    if (D == 128) {
        if (quantise_q) hipLaunchKernelGGL((attn_fp8_kernel<128, true>), grid, block, 0, stream, p);
        else hipLaunchKernelGGL((attn_fp8_kernel<128, false>), grid, block, 0, stream, p);
    } else {
        if (quantise_q) hipLaunchKernelGGL((attn_fp8_kernel<64, true>), grid, block, 0, stream, p);
        else hipLaunchKernelGGL((attn_fp8_kernel<64, false>), grid, block, 0, stream, p);
    }
    return hipGetLastError();
}

}  // namespace pevlm
