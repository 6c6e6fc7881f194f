// fp32 attention: the numerical anchor of the library and the path taken for fp32 tensors.  Two kernels over the same work
// items (<= 16 query rows), both with scores formed transposed, S^T = K Q^T (A: keys, B: query rows): what a lane then holds of
// a query row is the B operand of O^T += V^T P^T as it stands.
//
// attn_f32_group, where it gives every compute unit a workgroup: all heads of a KV group together, 128 (row, head) columns to a
// workgroup of 4 wavefronts, on the bf16 matrix instructions: every fp32 value is split into three bf16 ones that add up to it
// exactly, and six of their nine products are taken (the others come to 2^-27 of the product, root mean square).  Six bf16
// instructions take 192 cycles where the fp32 ones take 512, and leave the vector ALU its cycles.  K and V are split once per
// workgroup, on their way into LDS.  Prefill of 2304 rows (sink 256, two blocks of 1024) x 28/4 heads x 128: 261 us on the fp32
// instructions (two heads x 16 rows, 56 % of the time matrix instructions, every wavefront loading its own keys), 170 now; 20.7 K
// rows 2350 -> 1360 us, 1.2 PFLOP/s of bf16 products.  Distance to the same attention in 64 bits 1.8e-7, 2.9e-7 before.  Bound: the
// bf16 matrix instructions, and with few workgroups their unequal lengths.
//
// attn_f32_single elsewhere: one head on 16 columns of v_mfma_f32_16x16x4_f32; the 4 wavefronts take the item's key tiles in turn,
// each with an online softmax of its own, and are joined at the end by the log-sum-exp identity, so that an item of a few
// hundred keys is a chain of one or two tiles, and a short prompt still spreads over the chip.  The order of a
// contraction and of the output rows is free, and is chosen so that a lane feeds 4 MFMA steps from one 16-byte load.
//
// A key that a row must not see enters its value MFMAs with the weight 0, which hides every finite value but not an
// infinite or invalid one (nor one that overflows its first bf16 part, from 2^104 on).  Such a value leaves a NaN in the row, so
// rows that do not come out finite are done again over the keys that they see and no others (attn_f32_row).
#include <algorithm>
#include <type_traits>

#include "attn_bf16_tile.h"

namespace pevlm {

namespace {

constexpr int kRows = 16;  // query rows of an item
constexpr int NW = 4;      // wavefronts of a workgroup

template <int D>
struct F32Row {  // a wavefront's query row and weights of 64 keys
    float q[D], w[64];
};
template <int D>
struct F32Shared {
    float ml[NW][kRows][2];           // per first tile of a wavefront, and row: maximum of the raw scores, sum of the weights
    float o[NW][kRows][D + 4];        // values of each, scaled to the common maximum
    F32Row<D> row[NW];                // attn_f32_row
};

// exp(d * scale) for c = scale * log2(e): two instructions where expf takes twelve.  c and the product are rounded where expf's
// argument was rounded once; the outputs' distance to 64 bits does not show it (28/4 heads x 384 rows 2.894e-7, 2.889e-7 with expf; 2/1 x
// 104 rows 1.900e-7, 1.901e-7; 4/1 x 1.9 K rows 3.446e-7, 3.453e-7).
__device__ __forceinline__ float weight_of(float d, float c) { return __builtin_amdgcn_exp2f(d * c); }
__device__ __forceinline__ float other_half(float x)  // the value of lane ^ 32
{
    const auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return __uint_as_float((threadIdx.x & 32) ? sw[0] : sw[1]);
}
// A row's weights are formed against the reference maximum it has; it is raised (and the row scaled) on its first tile and when
// a lane's sum of weights reaches this bound: they are not negative, so each stays below it, and an overflow is seen.
constexpr float kSumBound = 256.f;
// The wavefronts of a workgroup take its tiles in turn, wavefront 0 not always first: it sits on the same SIMD in every
// workgroup, and where the tiles do not divide by four that one had the most to do.  What a wavefront brings to the join goes by
// its first tile's number, so that a row's result does not depend on who came first, on the row's place in the batch for one.
__device__ __forceinline__ int32_t first_tile(const pevlm_work_item &it, int32_t u, int32_t wave) { return (wave + u + (it.q_start >> 4) + (it.q_start >> 7)) % NW; }

// Rows of one head: the wavefronts' values in sh.o, already scaled to
// the row's common maximum, are added and stored, four rows by a wavefront.  Returns false, with none of the
// wavefront's rows stored, if one of them is not finite.
constexpr int kRowsPerWave = kRows / NW;
template <int D, bool PARTIAL>
__device__ __forceinline__ bool store_rows(const AttnParams &p, const pevlm_work_item &it, int32_t head, const F32Shared<D> &sh)
{
    const int32_t orow = threadIdx.x / 16, c = threadIdx.x % 16, Hq = p.n_q_heads;
    const bool live = orow < it.q_rows;
    f32x4 x[D / 64];
    float zero = 0.f;  // stays 0 while every value is finite
#pragma unroll
    for (int i = 0; i < D / 64; ++i) {
        x[i] = *reinterpret_cast<const f32x4 *>(&sh.o[0][orow][64 * i + 4 * c]);
#pragma unroll
        for (int w = 1; w < NW; ++w) x[i] += *reinterpret_cast<const f32x4 *>(&sh.o[w][orow][64 * i + 4 * c]);
#pragma unroll
        for (int j = 0; j < 4; ++j) zero = fmaf(x[i][j], 0.f, zero);
    }
    if (__any(live && zero != 0.f)) return false;
    if (!live) return true;
    float M = -INFINITY, L = 0.f;
#pragma unroll
    for (int w = 0; w < NW; ++w) M = fmaxf(M, sh.ml[w][orow][0]);
#pragma unroll
    for (int w = 0; w < NW; ++w) {
        const float mw = sh.ml[w][orow][0];
        L += mw == -INFINITY ? 0.f : sh.ml[w][orow][1] * expf((mw - M) * p.scale);
    }
    const float inv = PARTIAL ? 1.f : 1.f / L;
    const int64_t slot = PARTIAL ? it.reserved + orow : it.q_start + orow;
    float *dst = (PARTIAL ? p.part_acc : (float *)p.out) + (slot * Hq + head) * D;
#pragma unroll
    for (int i = 0; i < D / 64; ++i) *reinterpret_cast<f32x4 *>(dst + 64 * i + 4 * c) = x[i] * inv;
    if (c == 0) {
        if (PARTIAL) {
            p.part_ml[(slot * Hq + head) * 2] = M;
            p.part_ml[(slot * Hq + head) * 2 + 1] = L;
        } else if (p.lse) {
            p.lse[slot * Hq + head] = M * p.scale + logf(L);
        }
    }
    return true;
}

// Row rr of an item by one wavefront, with plain multiply-adds over the keys that the row sees and no others: lanes over the keys
// for the scores and over head_dim for the values.  Taken where infinite or invalid numbers are about.
template <int D, bool PARTIAL>
__device__ __forceinline__ void attn_f32_row(const AttnParams &p, const pevlm_work_item &it, int32_t rr, int32_t h, int32_t g, F32Row<D> &own)
{
    constexpr int DV = D / 64;
    int32_t lane = threadIdx.x & 63;
    asm volatile("" : "+v"(lane));  // nothing of this is formed ahead of the tile loop, whose registers are full
    const int32_t Hq = p.n_q_heads, Hkv = p.n_kv_heads;
    const float *Q = (const float *)p.q, *K = (const float *)p.k, *V = (const float *)p.v;
    float *const q_s = own.q, *const w_s = own.w;
    auto exchanged = [] {  // what a lane has written to the wavefront's own LDS is read by its other lanes
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    };
    const int32_t row = it.q_start + rr;
    exchanged();
    for (int c = 0; c < DV; ++c) q_s[lane + 64 * c] = Q[((int64_t)row * Hq + h) * D + lane + 64 * c];
    exchanged();
    float m = -INFINITY, l = 0.f, acc[DV];
    for (int c = 0; c < DV; ++c) acc[c] = 0.f;
    for (int seg = 0; seg < 2; ++seg) {
        const int32_t start = seg == 0 ? it.full_start : it.diag_start;
        const int32_t n = seg == 0 ? it.full_len : (row - start + 1 < it.diag_len ? row - start + 1 : it.diag_len);
        for (int32_t k0 = 0; k0 < n; k0 += 64) {
            const int32_t j = k0 + lane, cnt = n - k0 < 64 ? n - k0 : 64;
            float s = -INFINITY;
            if (j < n) {
                const f32x4 *kp = reinterpret_cast<const f32x4 *>(K + ((int64_t)(start + j) * Hkv + g) * D);
                s = 0.f;
                for (int d = 0; d < D / 4; ++d) {
                    const f32x4 x = kp[d];
                    s += q_s[4 * d] * x[0] + q_s[4 * d + 1] * x[1] + q_s[4 * d + 2] * x[2] + q_s[4 * d + 3] * x[3];
                }
            }
            float mx = s;
            for (int o = 32; o > 0; o >>= 1) mx = fmaxf(mx, __shfl_xor(mx, o));
            const float m_new = fmaxf(m, mx);
            const float w = j < n ? expf((s - m_new) * p.scale) : 0.f;
            const float alpha = expf((m - m_new) * p.scale);  // m = -inf gives 0
            float sum = w;
            for (int o = 32; o > 0; o >>= 1) sum += __shfl_xor(sum, o);
            l = l * alpha + sum;
            for (int c = 0; c < DV; ++c) acc[c] *= alpha;
            m = m_new;
            exchanged();
            w_s[lane] = w;
            exchanged();
            for (int32_t jj = 0; jj < cnt; ++jj) {
                const float *vp = V + ((int64_t)(start + k0 + jj) * Hkv + g) * D;
                for (int c = 0; c < DV; ++c) acc[c] += w_s[jj] * vp[lane + 64 * c];
            }
        }
    }
    const int64_t slot = ((int64_t)(PARTIAL ? it.reserved + rr : row)) * Hq + h;
    float *const dst = (PARTIAL ? p.part_acc : (float *)p.out) + slot * D;
    for (int c = 0; c < DV; ++c) dst[lane + 64 * c] = PARTIAL ? acc[c] : acc[c] * (1.f / l);
    if (lane == 0) {
        if (PARTIAL) {
            p.part_ml[slot * 2] = m;
            p.part_ml[slot * 2 + 1] = l;
        } else if (p.lse) {
            p.lse[slot] = m * p.scale + logf(l);
        }
    }
}

// One head on 16 columns: lane % 16 is the row, lane / 16 the k index; step j of group i of Q K^T contracts
// head_dim 16 i + 4 kq + j, the lane's score v of a block of 16 keys is that of key 4 kq + v, row r of
// block 4 hh + b of O^T is head_dim 64 hh + 4 r + b.  A score is two sums over half of head_dim each: one sum has a third more
// error in the output (28/4 heads x 128, blocks of 333: 2.2e-7 and 3.2e-7; 14/2 x 64 1.9e-7 and 2.6e-7) and takes as long.
template <int D, bool PARTIAL>
__device__ __forceinline__ int32_t attn_f32_single(const AttnParams &p, const pevlm_work_item &it, int32_t h, int32_t g, int32_t u, F32Shared<D> &sh)
{
    constexpr int KI = D / 16;  // 16-wide groups of head_dim in Q K^T
    constexpr int VH = D / 64;  // 64-wide halves of head_dim in O^T
    const int32_t tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int32_t r16 = lane & 15, kq = lane >> 4;
    const int32_t Hq = p.n_q_heads, Hkv = p.n_kv_heads;
    const float *Q = (const float *)p.q, *K = (const float *)p.k, *V = (const float *)p.v;
    const int32_t row = it.q_start + (r16 < it.q_rows ? r16 : it.q_rows - 1);

    f32x4 qf[KI];
#pragma unroll
    for (int i = 0; i < KI; ++i) qf[i] = *reinterpret_cast<const f32x4 *>(Q + ((int64_t)row * Hq + h) * D + 16 * i + 4 * kq);

    // keys per tile: 64, fewer where an item has so few keys that wavefronts would get none
    const int32_t n_keys = it.full_len + it.diag_len;
    const int32_t KT = n_keys <= 4 * 16 ? 16 : (n_keys <= 4 * 32 ? 32 : 64);
    const int32_t n_full = ceil_div(it.full_len, KT), n_tiles = n_full + ceil_div(it.diag_len, KT);

    float m = -INFINITY, l = 0.f;
    f32x4 o[4 * VH];
#pragma unroll
    for (int b = 0; b < 4 * VH; ++b) o[b] = f32x4{0.f, 0.f, 0.f, 0.f};
    const float c_log2 = p.scale * 1.4426950408889634f;
    const int32_t turn = first_tile(it, u, wave);
    for (int32_t t = turn; t < n_tiles; t += NW) {
        const bool causal = t >= n_full;
        const int32_t k0 = causal ? it.diag_start + (t - n_full) * KT : it.full_start + t * KT;
        const int32_t kend = causal ? it.diag_start + it.diag_len : it.full_start + it.full_len;
        const int32_t last = (kend - k0 < KT ? kend - k0 : KT) - 1;  // last key of the tile, relative
        const int32_t nblk = (last >> 4) + 1;
        // ---- scores: 16 keys x 16 rows per block
        f32x4 s[4];
#pragma unroll
        for (int b = 0; b < 4; ++b) {
            s[b] = f32x4{0.f, 0.f, 0.f, 0.f};
            if (b < nblk) {
                const int32_t key = b * 16 + r16 < last ? b * 16 + r16 : last;
                const float *kp = K + ((int64_t)(k0 + key) * Hkv + g) * D + 4 * kq;
                f32x4 a[KI], s2 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int i = 0; i < KI; ++i) a[i] = *reinterpret_cast<const f32x4 *>(kp + 16 * i);
#pragma unroll
                for (int i = 0; i < KI; ++i)
#pragma unroll
                    for (int j = 0; j < 4; j += 2) {
                        s[b] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[i][j], qf[i][j], s[b], 0, 0, 0);
                        s2 = __builtin_amdgcn_mfma_f32_16x16x4f32(a[i][j + 1], qf[i][j + 1], s2, 0, 0, 0);
                    }
                s[b] += s2;
            }
        }
        // ---- weights: this lane holds keys 16 b + 4 kq + v of its row
        const int32_t lim = (causal && row - k0 < last ? row - k0 : last) - 4 * kq;
        float mx = -INFINITY;
#pragma unroll
        for (int b = 0; b < 4; ++b)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                s[b][v] = b * 16 + v <= lim ? s[b][v] : -INFINITY;
                mx = fmaxf(mx, s[b][v]);
            }
        mx = fmaxf(mx, __shfl_xor(mx, 16));
        mx = fmaxf(mx, __shfl_xor(mx, 32));
        const float m_new = fmaxf(m, mx);
        const float m_use = m_new == -INFINITY ? 0.f : m_new;  // no visible key yet: all weights come out 0
        float psum = 0.f;
#pragma unroll
        for (int b = 0; b < 4; ++b)
            if (b < nblk) {
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    s[b][v] = weight_of(s[b][v] - m_use, c_log2);
                    psum += s[b][v];
                }
            }
        if (__any(m_new > m)) {
            const float alpha = weight_of(m - m_use, c_log2);  // m = -inf gives 0
            l *= alpha;
#pragma unroll
            for (int b = 0; b < 4 * VH; ++b) o[b] *= alpha;
            m = m_new;
        }
        l += psum;
        // ---- values: step v of a block takes keys 16 b + 4 kq + v, d-block 4 hh + b' the indices 64 hh + 4 r + b'
#pragma unroll
        for (int b = 0; b < 4; ++b)
            if (b < nblk) {
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const int32_t kl = b * 16 + 4 * kq + v, key = kl < last ? kl : last;
                    const float *vp = V + ((int64_t)(k0 + key) * Hkv + g) * D + 4 * r16;
#pragma unroll
                    for (int hh = 0; hh < VH; ++hh) {
                        const f32x4 a = *reinterpret_cast<const f32x4 *>(vp + 64 * hh);
#pragma unroll
                        for (int bb = 0; bb < 4; ++bb)
                            o[4 * hh + bb] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[bb], s[b][v], o[4 * hh + bb], 0, 0, 0);
                    }
                }
            }
    }

    // ---- join the wavefronts, as above
    l += __shfl_xor(l, 16);
    l += __shfl_xor(l, 32);
    if (kq == 0) {
        sh.ml[turn][r16][0] = m;
        sh.ml[turn][r16][1] = l;
    }
    __syncthreads();
    float M = -INFINITY;
#pragma unroll
    for (int w = 0; w < NW; ++w) M = fmaxf(M, sh.ml[w][r16][0]);
    const float f = m == -INFINITY ? 0.f : expf((m - M) * p.scale);
#pragma unroll
    for (int hh = 0; hh < VH; ++hh)
#pragma unroll
        for (int v = 0; v < 4; ++v)
            *reinterpret_cast<f32x4 *>(&sh.o[turn][r16][64 * hh + 16 * kq + 4 * v]) =
                f32x4{o[4 * hh][v] * f, o[4 * hh + 1][v] * f, o[4 * hh + 2][v] * f, o[4 * hh + 3][v] * f};
    __syncthreads();
    return store_rows<D, PARTIAL>(p, it, h, sh) ? 0 : 1;
}

// ---------------------------------------------------------------- all heads of a KV group, on bf16 matrix instructions
// An fp32 value is the sum of three bf16 ones, to the last bit: x = x1 + x2 + x3, each the rounding of what the ones before
// leave; the second is at most 2^-8 of x, the third 2^-17.  A product is then x1 y1 + (x1 y2 + x2 y1) + (x1 y3 + x2 y2 + x3 y1), bf16
// products that are exact in fp32, but for x2 y3 + x3 y2 + x3 y3: 2^-24 of it at most, 2^-27 root mean square.
//
// x3 reaches down to the last bit of x, which bf16 does not hold as a normal number where x is below 2^-103.  Values and weights are
// therefore taken kLift times as large, down to the smallest denormal (what then overflows does not come out finite).  Of keys
// below 2^-103 up to 2^-126 is lost, which takes a query above kLargeQuery to be seen in a score; such rows, and those of a query
// with numbers below kSmallQuery, are done again from the fp32 values.
constexpr float kLift = 0x1p24f, kSmallQuery = 0x1p-100f, kLargeQuery = 0x1p80f;
struct Planes {
    u32x4 x[3];  // eight values each
};
__device__ __forceinline__ Planes split8(const f32x4 &a, const f32x4 &b)
{
    Planes r;
    float x[8] = {a[0], a[1], a[2], a[3], b[0], b[1], b[2], b[3]};
#pragma unroll
    for (int n = 0; n < 3; ++n)
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            const uint32_t u = weight_pair(x[2 * w], x[2 * w + 1]);
            r.x[n][w] = u;
            if (n < 2) {
                x[2 * w] -= __uint_as_float(u << 16);
                x[2 * w + 1] -= __uint_as_float(u & 0xffff0000u);
            }
        }
    return r;
}
__device__ __forceinline__ f32x16 mfma_bf16(const u32x4 &a, const u32x4 &b, const f32x16 &c)
{
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}

constexpr int kGroupColumns = 128;  // (row, head) pairs of a workgroup, 32 to a wavefront
constexpr int kGroupKeys = 32;      // keys of a tile
template <int D>
union F32GroupShared {
    struct {
        uint8_t k[3][kGroupKeys * D * 2], v[3][kGroupKeys * D * 2];  // the planes of a tile, laid out as a bf16 tile
        u32x4 q3[NW][D / 16][64];                                    // third planes of the queries
    };
    struct {
        float o[kGroupColumns][D + 4];  // rows on their way out
        F32Row<D> row[NW];
    };
};
static_assert(2 * sizeof(F32GroupShared<128>) <= 160 * 1024, "two workgroups on a compute unit");

// One work item for 128 of its (row, head) pairs, head fastest (16 rows of up to 8 heads: all of them).  A tile's K is split
// behind the values of the tile before, its V behind its scores; the two workgroups of a compute unit take matrix
// instructions and splitting in an order of their own.
template <int D, bool PARTIAL>
__device__ __forceinline__ void attn_f32_group(const AttnParams &p, const pevlm_work_item &it, int32_t g, int32_t inner, int32_t turn, F32GroupShared<D> &sh)
{
    using C = TileCfg<D>;
    constexpr int KT = kGroupKeys, ROWB = C::ROWB, CH = C::CH, KS = C::KSTEPS, DBLK = C::DBLK, VSW = C::VSW;
    constexpr int THREADS = NW * 64, NCH = KT * CH / THREADS;  // chunks of 8 values that a lane stages of a tile
    const int32_t tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int32_t l32 = lane & 31, g32 = lane >> 5;
    const int32_t Hq = p.n_q_heads, Hkv = p.n_kv_heads, G = Hq / Hkv;
    const int32_t n_pairs = it.q_rows * G, pair0 = inner * kGroupColumns, col0 = pair0 + (wave + turn) % NW * 32;
    if (pair0 >= n_pairs) return;  // an item with fewer rows than the launch's longest
    const bool active = col0 < n_pairs;
    const int32_t my_row = it.q_start + min(col0 + l32, n_pairs - 1) / G;
    const int32_t w_lo = it.q_start + min(col0, n_pairs - 1) / G, w_hi = it.q_start + min(col0 + 31, n_pairs - 1) / G;

    // a lane's fragment of k-step kk, or of block b of head_dim: the swizzle's exclusive or goes over bits that the row leaves free
    const uint32_t k_at = (uint32_t)(l32 * ROWB + ((g32 ^ (l32 & (CH - 1))) << 4));
    const uint32_t v_at = (uint32_t)((g32 * 4 + ((lane & 15) >> 2)) * ROWB + (lane & 1) * 8 + ((((lane >> 2) & VSW) * 4 + ((lane >> 4) & 1) * 2 + ((lane & 3) >> 1)) << 4));

    const int32_t n_full = ceil_div(it.full_len, KT);
    const int32_t wg_hi = it.q_start + min(pair0 + kGroupColumns - 1, n_pairs - 1) / G;
    const int32_t n_diag = wg_hi >= it.diag_start ? min(ceil_div(it.diag_len, KT), (wg_hi - it.diag_start) / KT + 1) : 0;
    const int32_t n_tiles = n_full + n_diag;
    auto tile_range = [&](int32_t t, int32_t &k0, int32_t &kend) {
        const bool own = t >= n_full;
        k0 = own ? it.diag_start + (t - n_full) * KT : it.full_start + t * KT;
        kend = own ? it.diag_start + it.diag_len : it.full_start + it.full_len;
    };

    // ---- staging: a lane reads 8 values of a row (keys past the range repeat its last one) and writes 16 bytes of each plane
    const int32_t ch = tid % CH, srow = tid / CH;
    f32x4 raw[NCH][2];
    auto load_raw = [&](const void *base, int32_t t) {
        int32_t k0, kend;
        tile_range(t, k0, kend);
        const char *const first = (const char *)base + ((int64_t)k0 * Hkv + g) * D * 4;
        const int32_t last = min(KT, kend - k0) - 1;
#pragma unroll
        for (int j = 0; j < NCH; ++j) {
            const f32x4 *src = reinterpret_cast<const f32x4 *>(first + ((uint32_t)min(srow + j * (THREADS / CH), last) * (uint32_t)(Hkv * D * 4) + ch * 32));
            raw[j][0] = src[0];
            raw[j][1] = src[1];
        }
    };
    auto stage = [&](uint8_t (&planes)[3][KT * ROWB], bool is_v) {
#pragma unroll
        for (int j = 0; j < NCH; ++j) {
            const int32_t r = srow + j * (THREADS / CH);
            const int32_t at = r * ROWB + ((ch ^ (is_v ? (r & VSW) << 2 : r & (CH - 1))) << 4);
            const Planes x = is_v ? split8(raw[j][0] * kLift, raw[j][1] * kLift) : split8(raw[j][0], raw[j][1]);
#pragma unroll
            for (int n = 0; n < 3; ++n) *reinterpret_cast<u32x4 *>(planes[n] + at) = x.x[n];
        }
    };
    // V^T fragment: 16 keys (k-step ks) x block b of head_dim
    auto read_v = [&](const uint8_t *plane, int ks, int b) {
        union {
            s16x4 part[2];
            u32x4 all;
        } r;
#pragma unroll
        for (int tt = 0; tt < 2; ++tt) r.part[tt] = __builtin_amdgcn_ds_read_tr16_b64_v4i16(LDS_PTR(s16x4, plane + (ks * 16 + tt * 8) * ROWB + (v_at ^ (uint32_t)(b << 6))));
        return r.all;
    };
    // everybody's LDS writes have landed and everybody has read what comes next to be overwritten
    auto barrier = [] { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); };

    // ---- queries: planes 1 and 2 in registers, plane 3 in LDS
    u32x4 q1[KS], q2[KS];
    const float c_log2 = p.scale * 1.4426950408889634f;
    uint64_t extreme;
    if (n_tiles > 0) load_raw(p.k, 0);
    {
        const int32_t head = p.heads.head_order[g * G + min(col0 + l32, n_pairs - 1) % G];
        const f32x4 *q = reinterpret_cast<const f32x4 *>((const float *)p.q + ((int64_t)my_row * Hq + head) * D + 8 * g32);
        uint32_t least = 0xffffffffu;  // twice the bits of the smallest number but 0, less one
        float most = 0.f;
#pragma unroll
        for (int kk = 0; kk < KS; ++kk) {
            const Planes x = split8(q[kk * 4], q[kk * 4 + 1]);
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const float a = q[kk * 4 + j / 4][j % 4];
                least = min(least, (__float_as_uint(a) << 1) - 1u);
                most = fmaxf(most, fabsf(a));
            }
            q1[kk] = x.x[0];
            q2[kk] = x.x[1];
            sh.q3[wave][kk][lane] = x.x[2];
        }
        extreme = __ballot(least < (__float_as_uint(kSmallQuery) << 1) - 1u || !(most * c_log2 < kLargeQuery));
    }
    if (n_tiles > 0) {
        stage(sh.k, false);
        load_raw(p.v, 0);
    }
    barrier();

    float m = -INFINITY, l = 0.f;
    f32x16 o[DBLK];
#pragma unroll
    for (int b = 0; b < DBLK; ++b)
#pragma unroll
        for (int i = 0; i < 16; ++i) o[b][i] = 0.f;
    const f32x16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    for (int32_t t = 0; t < n_tiles; ++t) {
        int32_t k0, kend;
        tile_range(t, k0, kend);
        const bool causal = t >= n_full, work = active && !(causal && k0 > w_hi);
        // ---- scores; V of this tile goes to LDS.  The products of second and third planes are summed by themselves.
        f32x16 s = zero;
        if (work) {
            f32x16 lo = zero;
#pragma unroll
            for (int kk = 0; kk < KS; ++kk) {
                const uint32_t at = k_at ^ (uint32_t)(kk << 5);
                const u32x4 k1 = *reinterpret_cast<const u32x4 *>(sh.k[0] + at), k2 = *reinterpret_cast<const u32x4 *>(sh.k[1] + at);
                const u32x4 k3 = *reinterpret_cast<const u32x4 *>(sh.k[2] + at), q3 = sh.q3[wave][kk][lane];
                s = mfma_bf16(k1, q1[kk], s);
                lo = mfma_bf16(k1, q2[kk], lo);
                lo = mfma_bf16(k2, q1[kk], lo);
                lo = mfma_bf16(k2, q2[kk], lo);
                lo = mfma_bf16(k1, q3, lo);
                lo = mfma_bf16(k3, q1[kk], lo);
            }
            s += lo;
        }
        stage(sh.v, true);
        if (t + 1 < n_tiles) load_raw(p.k, t + 1);
        barrier();
        // ---- weights and values; K of the next tile goes to LDS
        if (work) {
            if (k0 + KT > kend || (causal && k0 + KT - 1 > w_lo)) {  // the range ends in the tile, or the diagonal runs through it
                const int32_t lim = (causal && my_row < kend - 1 ? my_row : kend - 1) - k0 - 4 * g32;
#pragma unroll
                for (int v = 0; v < 16; ++v) s[v] = (v & 3) + 8 * (v >> 2) <= lim ? s[v] : -INFINITY;
            }
            float psum = 0.f;
            f32x16 w;
            if (t > 0) {
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    w[v] = weight_of(s[v] - m, c_log2);  // no key seen yet: m = -inf makes the sum inf or invalid
                    psum += w[v];
                }
            }
            const int32_t up = t == 0 || !(psum < kSumBound) || m == -INFINITY;
            if (__any(up)) {
                float mx = s[0];
#pragma unroll
                for (int v = 1; v < 16; ++v) mx = fmaxf(mx, s[v]);
                mx = fmaxf(mx, other_half(mx));
                const float m_new = up | __shfl_xor(up, 32) ? fmaxf(m, mx) : m;
                const float m_use = m_new == -INFINITY ? 0.f : m_new;  // no visible key yet: all weights come out 0
                psum = 0.f;
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    w[v] = weight_of(s[v] - m_use, c_log2);
                    psum += w[v];
                }
                if (t > 0) {
                    const float alpha = weight_of(m - m_use, c_log2);  // m = -inf gives 0
                    l *= alpha;
#pragma unroll
                    for (int b = 0; b < DBLK; ++b)
#pragma unroll
                        for (int i = 0; i < 16; ++i) o[b][i] *= alpha;
                }
                m = m_new;
            }
            l += psum;
            // A tile's values are summed from zero and added to those before: one rounding at their size a tile instead of twelve.
            Planes w8[2];
#pragma unroll
            for (int ks = 0; ks < 2; ++ks)
                w8[ks] = split8(f32x4{w[8 * ks], w[8 * ks + 1], w[8 * ks + 2], w[8 * ks + 3]} * kLift,
                                f32x4{w[8 * ks + 4], w[8 * ks + 5], w[8 * ks + 6], w[8 * ks + 7]} * kLift);
#pragma unroll
            for (int b = 0; b < DBLK; ++b) {
                f32x16 sum = zero;
#pragma unroll
                for (int ks = 0; ks < 2; ++ks) {
                    u32x4 v[3];
#pragma unroll
                    for (int n = 0; n < 3; ++n) v[n] = read_v(sh.v[n], ks, b);
                    sum = mfma_bf16(v[0], w8[ks].x[0], sum);
                    sum = mfma_bf16(v[0], w8[ks].x[1], sum);
                    sum = mfma_bf16(v[1], w8[ks].x[0], sum);
                    sum = mfma_bf16(v[1], w8[ks].x[1], sum);
                    sum = mfma_bf16(v[0], w8[ks].x[2], sum);
                    sum = mfma_bf16(v[2], w8[ks].x[0], sum);
                }
                o[b] += sum;
            }
        }
        if (t + 1 < n_tiles) {
            stage(sh.k, false);
            load_raw(p.v, t + 1);
        }
        barrier();
    }

    // ---- rows out through LDS, D/4 lanes a row.  The lane's pair once more, from a lane number that the compiler takes for
    // another: the registers are full through the loop.
    int32_t out_lane = lane;
    asm volatile("" : "+v"(out_lane));
    const int32_t out32 = out_lane & 31, half = out_lane >> 5;
    const int32_t my_pair = min(col0 + out32, n_pairs - 1), my_head = p.heads.head_order[g * G + my_pair % G];
    l += other_half(l);
    const bool live = col0 + out32 < n_pairs;
    const float inv = (PARTIAL ? 1.f : 1.f / l) * (1.f / (kLift * kLift));
    float wrong = 0.f;  // stays 0 while every value is finite
#pragma unroll
    for (int b = 0; b < DBLK; ++b)
#pragma unroll
        for (int i4 = 0; i4 < 4; ++i4) {
            f32x4 x = {o[b][i4 * 4], o[b][i4 * 4 + 1], o[b][i4 * 4 + 2], o[b][i4 * 4 + 3]};
            x *= inv;
#pragma unroll
            for (int j = 0; j < 4; ++j) wrong = fmaf(x[j], 0.f, wrong);
            *reinterpret_cast<f32x4 *>(&sh.o[wave * 32 + out32][b * 32 + i4 * 8 + half * 4]) = x;
        }
    // Columns whose rows are to be done again: by this wavefront, and not stored before.
    const uint64_t marked = __ballot(live && wrong != 0.f) | (extreme & __ballot(live));
    uint32_t again = (uint32_t)(marked | marked >> 32);
    const int64_t slot = (int64_t)((PARTIAL ? it.reserved : it.q_start) + my_pair / G) * Hq + my_head;
    if (live && half == 0 && !(again >> out32 & 1)) {
        if (PARTIAL) {
            p.part_ml[slot * 2] = m;
            p.part_ml[slot * 2 + 1] = l;
        } else if (p.lse) {
            p.lse[slot] = m * p.scale + logf(l);
        }
    }
    barrier();
    constexpr int LPR = D / 4;
#pragma unroll
    for (int j = 0; j < 32; j += 64 / LPR) {
        const int32_t c = j + out_lane / LPR, c_slot_lo = __shfl((int32_t)(uint32_t)slot, c), c_slot_hi = __shfl((int32_t)(slot >> 32), c);
        const int64_t row = ((int64_t)c_slot_hi << 32) | (uint32_t)c_slot_lo;
        if (col0 + c < n_pairs && !(again >> c & 1))
            *reinterpret_cast<f32x4 *>((PARTIAL ? p.part_acc : (float *)p.out) + row * D + out_lane % LPR * 4) = *reinterpret_cast<const f32x4 *>(&sh.o[wave * 32 + c][out_lane % LPR * 4]);
    }
    for (; again; again &= again - 1) {
        const int32_t pair = col0 + __builtin_ctz(again);
        attn_f32_row<D, PARTIAL>(p, it, pair / G, p.heads.head_order[g * G + pair % G], g, sh.row[wave]);
    }
}

}  // namespace

// how a launch's items are shared out
struct F32Shares {
    int32_t items;      // items of a workgroup (a batch): more than one where a group has few heads
    int32_t step;       // list distance of items that may continue each other: a question's splits lie between its row tiles
    int32_t n_batches, units, stride, cus_per_xcd;
};

// Logical workgroup ids run over (KV head, batch of items, unit of the KV head's query heads), and every XCD (workgroup b
// runs on XCD b % 8) gets one contiguous run of them, so that its L2 holds the keys it works on.  Items
// are taken last first (the later tiles of a block are the longer ones), and where several XCDs share a KV
// head, every `stride`-th item in turn, so that each gets as many long ones.  The runs start at eighths of the ids (rounded
// up to a common length, a KV head's longest items ended up on the XCD of the one before: one region of 1100 rows x 28/4
// heads, 69 batches, 166 us, 120 now; 2000 x 14/2 heads x 64 124 and 94).  Units: one head each, or (GROUP) 128 (row, head) pairs.
template <int D, bool PARTIAL, bool GROUP>
__global__ __launch_bounds__(256, 2) void attn_f32_kernel(AttnParams p, int32_t n_logical, F32Shares gs)
{
    __shared__ __attribute__((aligned(1024))) std::conditional_t<GROUP, F32GroupShared<D>, F32Shared<D>> sh;
    const int32_t xcd = blockIdx.x & 7, eighth = n_logical >> 3, over = n_logical & 7;
    const int32_t first = xcd * eighth + (xcd * over >> 3), per_xcd = (xcd + 1) * eighth + ((xcd + 1) * over >> 3) - first;
    int32_t place = blockIdx.x >> 3;
    if (place >= per_xcd) return;
    const int32_t layer = place / gs.cus_per_xcd;  // the compute units get their first workgroups in layers: a long and a short one
    if (GROUP && layer == 1) place = gs.cus_per_xcd + min(2 * gs.cus_per_xcd, per_xcd) - 1 - place;
    const int32_t logical = first + place;
    const int32_t u = logical % gs.units, outer = logical / gs.units;  // outer: (group of units, item or items)
    const int32_t group = outer / gs.n_batches, j = outer % gs.n_batches;
    // dealt out in `stride` runs, run r from ceil(r n / stride) on; a left-over one, of the shortest, goes where two XCDs meet in it
    const int32_t run = j * gs.stride / gs.n_batches, start = (run * gs.n_batches + gs.stride - 1) / gs.stride, len = gs.n_batches / gs.stride;
    const int32_t batch = gs.n_batches - 1 - (j - start < len ? (j - start) * gs.stride + run : len * (gs.stride - run) + start);
    auto item = [&](int32_t idx) {
        if (!p.inline_items.mode) return p.items[idx];
        const pevlm_work_item it = inline_item(p.inline_items, idx);
        if (group == 0 && u == 0 && threadIdx.x == 0) p.items[idx] = it;
        return it;
    };
    if constexpr (GROUP) {
        // the items of the batch, those that continue each other in one go: a region's rows, or a question's for the same keys
        int32_t idx = batch % gs.step + batch / gs.step * gs.step * gs.items;
        pevlm_work_item next = item(idx);
        for (int32_t left = gs.items; left > 0;) {
            pevlm_work_item it = next;
            while (--left > 0 && (idx += gs.step) < p.n_items) {
                next = item(idx);
                if (next.q_start != it.q_start + it.q_rows || next.diag_start != it.diag_start || next.full_start != it.full_start || next.full_len != it.full_len) break;
                it.q_rows += next.q_rows;
                it.diag_len = next.diag_len;
            }
            attn_f32_group<D, PARTIAL>(p, it, group, u, 2 * layer, sh);
            if (idx >= p.n_items) break;
            if (left > 0) __syncthreads();
        }
    } else {
        const pevlm_work_item it = item(batch);
        const int32_t h = p.heads.head_order[group * gs.units + u], g = p.heads.kv_of_q[h];
        if (attn_f32_single<D, PARTIAL>(p, it, h, g, u, sh)) {  // the wavefront's four rows, of which none was stored
            const int32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
            for (int32_t rr = wave * kRowsPerWave; rr < it.q_rows && rr < (wave + 1) * kRowsPerWave; ++rr) attn_f32_row<D, PARTIAL>(p, it, rr, h, g, sh.row[wave]);
        }
    }
}

hipError_t launch_attn_f32(const AttnParams &p, int32_t D, bool partial, int32_t compute_units, hipStream_t stream)
{
    const int32_t G = p.n_q_heads / p.n_kv_heads;
    bool uniform = true;
    for (int32_t i = 0; i < p.n_q_heads; ++i)
        if (p.heads.kv_of_q[p.heads.head_order[i]] != i / G) uniform = false;
    F32Shares gs;
    gs.cus_per_xcd = std::max(1, compute_units / 8);
    gs.step = p.num_splits;
    gs.items = 1;
    // All heads of a group together, and for small groups as many items as columns go, while that leaves every compute unit
    // a workgroup and half of them a second one (111 items x 32/8 heads: two together 107 us, one by one 136).  With fewer
    // workgroups than compute units one head at a time has the shorter chain (us, all heads against one: 28/4 heads, 84
    // workgroups 24.5 / 18.4, 168 40.1 / 36.1, 284 58.7 / 70.0; 14/2 x 64, 142 31.3 / 24.2, 222 60.0 / 60.4, 346 82 / 99),
    // and with less than half of the columns filled it does more per instruction.
    const int64_t cus = compute_units;
    const auto batches = [&](int32_t items) { return ceil_div(p.n_items / gs.step, items) * gs.step; };
    while (kRows * G * gs.items * 2 <= kGroupColumns && 2 * (int64_t)batches(gs.items * 2) * p.n_kv_heads >= 3 * cus) gs.items *= 2;
    const int32_t group_units = ceil_div(kRows * G * gs.items, kGroupColumns);
    const bool groups = uniform && G > 1 && kRows * G * gs.items >= kGroupColumns / 2 && (int64_t)batches(gs.items) * group_units * p.n_kv_heads >= cus;
    if (!groups) gs.items = 1;
    gs.n_batches = batches(gs.items);
    gs.units = groups ? group_units : (uniform ? G : p.n_q_heads);  // per KV head, or per item if their groups differ
    const int32_t n_logical = gs.n_batches * gs.units * (uniform ? p.n_kv_heads : 1);
    gs.stride = uniform && p.n_kv_heads <= 4 ? std::min(8 / p.n_kv_heads, gs.n_batches) : 1;
    const dim3 grid((n_logical + 7) / 8 * 8);
#define PEVLM_F32_LAUNCH(DD, PP)                                                                                                  \
    do {                                                                                                                          \
        if (groups) hipLaunchKernelGGL((attn_f32_kernel<DD, PP, true>), grid, dim3(256), 0, stream, p, n_logical, gs);            \
        else hipLaunchKernelGGL((attn_f32_kernel<DD, PP, false>), grid, dim3(256), 0, stream, p, n_logical, gs);                  \
    } while (0)
    if (D == 128) { if (partial) PEVLM_F32_LAUNCH(128, true); else PEVLM_F32_LAUNCH(128, false); }
    else { if (partial) PEVLM_F32_LAUNCH(64, true); else PEVLM_F32_LAUNCH(64, false); }
#undef PEVLM_F32_LAUNCH
    return hipGetLastError();
}

}  // namespace pevlm
