// fp32 attention kernel on the fp32 matrix cores (fp32 products and sums): the numerical anchor of the
// library and the path taken for fp32 tensors.
//
// A workgroup takes one work item (<= 16 query rows) for one or two heads of a KV group; its 4 wavefronts
// take the item's key tiles in turn, each with an online softmax of its own, and are joined at the end
// by the log-sum-exp identity.  So an item of a few hundred keys is a chain of one or two tiles, and a
// short prompt, which has few items, still spreads over the chip.
//
// Two heads: the 32 columns (row, head) fill v_mfma_f32_32x32x2_f32, which sustains 153 TFLOP/s from
// registers; one head (the odd one of a group, or a grid that would not fill the chip): 16 columns on
// v_mfma_f32_16x16x4_f32, which sustains 102.
//
// Scores are formed transposed, S^T = K Q^T (A: keys, B: query rows): what a lane then holds of a query row is
// the B operand of O^T += V^T P^T as it stands.  The order of a contraction and of the output rows is free, and
// is chosen so that a lane feeds 4 MFMA steps from one 16-byte load.  K and V go from global memory to
// registers: the four SIMDs of a compute unit ask its L1 for 16 bytes a cycle, a quarter of what it
// delivers, so nothing is staged in LDS and the tile loop has no barrier.
//
// Bound: the fp32 matrix rate.  Prefill of 2304 rows (sink 256, two blocks of 1024, 28/4 heads x 128): 0.268 ms,
// 86 TFLOP/s useful, of which the matrix instructions alone would take 0.166 ms; what is left is the uneven
// number of tiles per wavefront, the chain before an item's first tile and its join.  (One row per
// wavefront with plain multiply-adds, keys over lanes: 4.59 ms.)
//
// A key that a row must not see enters its value MFMAs with the weight 0, which hides every finite value but not an
// infinite or invalid one.  Such a value leaves a NaN in the row, so rows that do not come out finite are done again
// over the keys that they see and no others (attn_f32_rows).
#include <algorithm>

#include "common.h"

namespace pevlm {

typedef __attribute__((ext_vector_type(2))) float f32x2;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(16))) float f32x16;

namespace {

constexpr int kRows = 16;  // query rows of an item
constexpr int NW = 4;      // wavefronts of a workgroup

template <int D>
struct F32Shared {
    float ml[NW][2][kRows][2];        // per wavefront, head and row: maximum of the raw scores, sum of the weights
    float o[NW][kRows][D + 4];        // one head at a time: values of every wavefront, scaled to the common maximum
    union {
        f32x4 q[D / 8][64];           // two heads: the B fragments of Q K^T, the same for every wavefront
        struct { float q[D], w[64]; } row[NW];  // attn_f32_rows: a wavefront's query row and weights of 64 keys
    };
};

// exp(d * scale) for c = scale * log2(e): two instructions where expf takes twelve, which is what the vector ALU had to do
// between the matrix instructions (fp32 ones leave it no cycles of their own).  The product is rounded once, as the argument of
// expf was.
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
// workgroup, and where the tiles do not divide by four that one had the most to do.  The row decides, so that a row's
// result does not depend on the launch.
__device__ __forceinline__ int32_t first_tile(const pevlm_work_item &it, int32_t u, int32_t wave) { return (wave + u + (it.q_start >> 4) + (it.q_start >> 7)) % NW; }

// Rows of one head (number n of the workgroup's heads): the wavefronts' values in sh.o, already scaled to
// the row's common maximum, are added and stored, four rows by a wavefront.  Returns false, with none of the
// wavefront's rows stored, if one of them is not finite.
constexpr int kRowsPerWave = kRows / NW;
template <int D, bool PARTIAL>
__device__ __forceinline__ bool store_rows(const AttnParams &p, const pevlm_work_item &it, int32_t head, int32_t n, const F32Shared<D> &sh)
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
    for (int w = 0; w < NW; ++w) M = fmaxf(M, sh.ml[w][n][orow][0]);
#pragma unroll
    for (int w = 0; w < NW; ++w) {
        const float mw = sh.ml[w][n][orow][0];
        L += mw == -INFINITY ? 0.f : sh.ml[w][n][orow][1] * expf((mw - M) * p.scale);
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

// The same four rows with plain multiply-adds, over the keys that a row sees and no others: one row after the other, lanes
// over the keys for the scores and over head_dim for the values.  Taken where infinite or invalid numbers are about.
template <int D, bool PARTIAL>
__device__ __forceinline__ void attn_f32_rows(const AttnParams &p, const pevlm_work_item &it, int32_t h, int32_t g, F32Shared<D> &sh)
{
    constexpr int DV = D / 64;
    const int32_t lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int32_t Hq = p.n_q_heads, Hkv = p.n_kv_heads;
    const float *Q = (const float *)p.q, *K = (const float *)p.k, *V = (const float *)p.v;
    float *const q_s = sh.row[wave].q, *const w_s = sh.row[wave].w;
    auto exchanged = [] {  // what a lane has written to the wavefront's own LDS is read by its other lanes
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    };
    for (int32_t rr = wave * kRowsPerWave; rr < it.q_rows && rr < (wave + 1) * kRowsPerWave; ++rr) {
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
}

// Two heads h[0], h[1] of KV head g; returns the heads (bit 0, bit 1) whose rows of this wavefront are still to be done.  Column c = lane % 32: row c % 16 of head c / 16; the lane's half (lane / 32)
// is the k index.  Step j of group i of Q K^T contracts head_dim 8 i + 4 half + j; the lane's score v belongs
// to key (v & 3) + 8 (v >> 2) + 4 half of the tile; row r of block b of O^T is head_dim DB r + b.
template <int D, bool PARTIAL>
__device__ __forceinline__ int32_t attn_f32_pair(const AttnParams &p, const pevlm_work_item &it, const int32_t (&h)[2], int32_t g, int32_t u, F32Shared<D> &sh)
{
    constexpr int KT = 32, KI = D / 8, DB = D / 32;
    typedef __attribute__((ext_vector_type(DB))) float f32xdb;
    const int32_t tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int32_t r16 = lane & 15, mine = (lane >> 4) & 1, half = lane >> 5;
    const int32_t Hq = p.n_q_heads, Hkv = p.n_kv_heads;
    const int32_t row = it.q_start + (r16 < it.q_rows ? r16 : it.q_rows - 1);
    const float *const q = (const float *)p.q + ((int64_t)row * Hq + (mine ? h[1] : h[0])) * D + 4 * half;
    // a lane's address inside a tile is a 32-bit byte offset from the tile's first row (at most 32 rows further)
    const uint32_t kv_row = (uint32_t)(Hkv * D * 4);

#pragma unroll
    for (int i = 0; i < KI / NW; ++i) sh.q[wave * (KI / NW) + i][lane] = *reinterpret_cast<const f32x4 *>(q + 8 * (wave * (KI / NW) + i));
    float m = -INFINITY, l = 0.f;
    f32x16 o[DB];
#pragma unroll
    for (int b = 0; b < DB; ++b)
#pragma unroll
        for (int i = 0; i < 16; ++i) o[b][i] = 0.f;

    // A tile is four stages of 32 MFMAs: the two halves of K's head_dim, the two halves of the keys of V.  The loads
    // of a stage are issued before the MFMAs of the stage ahead of it (the first one's during the last stage
    // of the tile before), into the buffer that the stage before that has left.
    constexpr int KH = KI / 2;
    f32x4 kbuf[2][KH];
    f32xdb vbuf[2][8];
    const int32_t n_full = ceil_div(it.full_len, KT), n_tiles = n_full + ceil_div(it.diag_len, KT);
    int32_t k0 = 0, last = 0;  // first key of the tile, its last key relative to that
    const char *kt = nullptr, *vt = nullptr;  // row k0 of the KV head
    auto tile_range = [&](int32_t t) {
        const bool own = t >= n_full;
        k0 = own ? it.diag_start + (t - n_full) * KT : it.full_start + t * KT;
        const int32_t kend = own ? it.diag_start + it.diag_len : it.full_start + it.full_len;
        last = (kend - k0 < KT ? kend - k0 : KT) - 1;
        kt = (const char *)p.k + ((int64_t)k0 * Hkv + g) * D * 4;
        vt = (const char *)p.v + ((int64_t)k0 * Hkv + g) * D * 4;
    };
    auto load_k = [&](int hf) {
        const uint32_t off = (uint32_t)((lane & 31) < last ? lane & 31 : last) * kv_row + 16 * half;
#pragma unroll
        for (int i = 0; i < KH; ++i) kbuf[hf][i] = *reinterpret_cast<const f32x4 *>(kt + (off + (hf * KH + i) * 32));
    };
    auto load_v = [&](int hf) {
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int32_t kl = (u & 3) + 8 * (2 * hf + (u >> 2)) + 4 * half;
            vbuf[hf][u] = *reinterpret_cast<const f32xdb *>(vt + ((uint32_t)(kl < last ? kl : last) * kv_row + 4 * DB * (lane & 31)));
        }
    };
    const int32_t t_first = first_tile(it, u, wave);
    const float c_log2 = p.scale * 1.4426950408889634f;
    if (t_first < n_tiles) {
        tile_range(t_first);
        load_k(0);
    }
    __syncthreads();  // the queries are in LDS
    for (int32_t t = t_first; t < n_tiles; t += NW) {
        const bool causal = t >= n_full;
        f32x16 s = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f}, s2 = s;
        auto scores = [&](int hf) {
#pragma unroll
            for (int i = 0; i < KH; ++i) {
                const f32x4 qf = sh.q[hf * KH + i][lane];
                s = __builtin_amdgcn_mfma_f32_32x32x2f32(kbuf[hf][i][0], qf[0], s, 0, 0, 0);
                s2 = __builtin_amdgcn_mfma_f32_32x32x2f32(kbuf[hf][i][1], qf[1], s2, 0, 0, 0);
                s = __builtin_amdgcn_mfma_f32_32x32x2f32(kbuf[hf][i][2], qf[2], s, 0, 0, 0);
                s2 = __builtin_amdgcn_mfma_f32_32x32x2f32(kbuf[hf][i][3], qf[3], s2, 0, 0, 0);
            }
        };
        load_k(1);
        __builtin_amdgcn_sched_barrier(0);
        scores(0);
        load_v(0);
        __builtin_amdgcn_sched_barrier(0);
        scores(1);
        load_v(1);
        __builtin_amdgcn_sched_barrier(0);
        s += s2;
        if (last < KT - 1 || (causal && k0 + KT - 1 > it.q_start)) {  // the range ends in the tile, or the diagonal runs through it
            const int32_t lim = (causal && row - k0 < last ? row - k0 : last) - 4 * half;
#pragma unroll
            for (int v = 0; v < 16; ++v) s[v] = (v & 3) + 8 * (v >> 2) <= lim ? s[v] : -INFINITY;
        }
        float psum = 0.f;
        f32x16 w;
        if (t != t_first) {
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                w[v] = weight_of(s[v] - m, c_log2);  // no key seen yet: m = -inf makes the sum inf or invalid
                psum += w[v];
            }
        }
        const int32_t up = t == t_first || !(psum < kSumBound) || m == -INFINITY;
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
            if (t != t_first) {
                const float alpha = weight_of(m - m_use, c_log2);  // m = -inf gives 0
                l *= alpha;
#pragma unroll
                for (int b = 0; b < DB; ++b)
#pragma unroll
                    for (int i = 0; i < 16; ++i) o[b][i] *= alpha;
            }
            m = m_new;
        }
        l += psum;
#pragma unroll
        for (int u = 0; u < 8; ++u)
#pragma unroll
            for (int b = 0; b < DB; ++b) o[b] = __builtin_amdgcn_mfma_f32_32x32x2f32(vbuf[0][u][b], w[u], o[b], 0, 0, 0);
        if (t + NW < n_tiles) {
            tile_range(t + NW);
            load_k(0);
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int u = 0; u < 8; ++u)
#pragma unroll
            for (int b = 0; b < DB; ++b) o[b] = __builtin_amdgcn_mfma_f32_32x32x2f32(vbuf[1][u][b], w[8 + u], o[b], 0, 0, 0);
    }

    // ---- join the wavefronts: common maximum per row, values scaled to it and added through LDS
    l += __shfl_xor(l, 32);
    if (half == 0) {
        sh.ml[wave][mine][r16][0] = m;
        sh.ml[wave][mine][r16][1] = l;
    }
    __syncthreads();
    float M = -INFINITY;
#pragma unroll
    for (int w = 0; w < NW; ++w) M = fmaxf(M, sh.ml[w][mine][r16][0]);
    const float f = m == -INFINITY ? 0.f : expf((m - M) * p.scale);
    int32_t left = 0;
#pragma unroll
    for (int n = 0; n < 2; ++n) {
        if (mine == n) {
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                f32xdb x;
#pragma unroll
                for (int b = 0; b < DB; ++b) x[b] = o[b][v] * f;
                *reinterpret_cast<f32xdb *>(&sh.o[wave][r16][DB * ((v & 3) + 8 * (v >> 2) + 4 * half)]) = x;
            }
        }
        __syncthreads();
        if (!store_rows<D, PARTIAL>(p, it, h[n], n, sh)) left |= 1 << n;
        if (n == 0) __syncthreads();
    }
    return left;
}

// One head on 16 columns: lane % 16 is the row, lane / 16 the k index; step j of group i of Q K^T contracts
// head_dim 16 i + 4 kq + j, the lane's score v of a block of 16 keys is that of key 4 kq + v, row r of
// block 4 hh + b of O^T is head_dim 64 hh + 4 r + b.
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
    for (int32_t t = first_tile(it, u, wave); t < n_tiles; t += NW) {
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
                f32x4 a[KI];
#pragma unroll
                for (int i = 0; i < KI; ++i) a[i] = *reinterpret_cast<const f32x4 *>(kp + 16 * i);
#pragma unroll
                for (int i = 0; i < KI; ++i)
#pragma unroll
                    for (int j = 0; j < 4; ++j) s[b] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[i][j], qf[i][j], s[b], 0, 0, 0);
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
        sh.ml[wave][0][r16][0] = m;
        sh.ml[wave][0][r16][1] = l;
    }
    __syncthreads();
    float M = -INFINITY;
#pragma unroll
    for (int w = 0; w < NW; ++w) M = fmaxf(M, sh.ml[w][0][r16][0]);
    const float f = m == -INFINITY ? 0.f : expf((m - M) * p.scale);
#pragma unroll
    for (int hh = 0; hh < VH; ++hh)
#pragma unroll
        for (int v = 0; v < 4; ++v)
            *reinterpret_cast<f32x4 *>(&sh.o[wave][r16][64 * hh + 16 * kq + 4 * v]) =
                f32x4{o[4 * hh][v] * f, o[4 * hh + 1][v] * f, o[4 * hh + 2][v] * f, o[4 * hh + 3][v] * f};
    __syncthreads();
    return store_rows<D, PARTIAL>(p, it, h, 0, sh) ? 0 : 1;
}

}  // namespace

// Logical workgroup ids run over (KV head, item, unit of the KV head's query heads), and every XCD (workgroup b
// runs on XCD b % 8) gets one contiguous run of them, so that its L2 holds the keys it works on.  Items
// are taken last first (the later tiles of a block are the longer ones), and where several XCDs share a KV
// head, every `stride`-th item in turn, so that each gets as many long ones.  With pairs != 0 unit u takes query
// heads 2u and 2u + 1 (the last one alone if their number is odd), which share every K and V load; otherwise
// one head each.
template <int D, bool PARTIAL>
__global__ __launch_bounds__(256, 2) void attn_f32_kernel(AttnParams p, int32_t n_logical, int32_t units, int32_t pairs,
                                                          int32_t stride)
{
    __shared__ F32Shared<D> sh;
    const int32_t logical = (int32_t)(blockIdx.x & 7) * (int32_t)(gridDim.x >> 3) + (int32_t)(blockIdx.x >> 3);
    if (logical >= n_logical) return;
    const int32_t u = logical % units, outer = logical / units;  // outer: (group of units, item)
    const int32_t group = outer / p.n_items, j = outer % p.n_items;
    const int32_t full = p.n_items / stride * stride;  // items dealt out in `stride` runs; the few others come last
    const int32_t idx = p.n_items - 1 - (j < full ? j % (full / stride) * stride + j / (full / stride) : j);
    pevlm_work_item it;
    if (p.inline_items.mode) {
        it = inline_item(p.inline_items, idx);
        if (group == 0 && u == 0 && threadIdx.x == 0) p.items[idx] = it;
    } else {
        it = p.items[idx];
    }
    // Each kind of workgroup keeps its own branch to the end: with the rows that are left joined behind both, the compiler
    // makes the one-head kernel slower (842 tokens x 4/1 heads x 128: 24 us, 13 as here).
    if (pairs) {
        const int32_t G = p.n_q_heads / p.n_kv_heads;
        const int32_t h[2] = {p.heads.head_order[group * G + 2 * u], p.heads.head_order[group * G + (2 * u + 1 < G ? 2 * u + 1 : 2 * u)]};
        int32_t left;
        if (2 * u + 1 < G) left = attn_f32_pair<D, PARTIAL>(p, it, h, group, u, sh);
        else left = attn_f32_single<D, PARTIAL>(p, it, h[0], group, u, sh);
        for (int32_t n = 0; left >> n; ++n)
            if (left >> n & 1) attn_f32_rows<D, PARTIAL>(p, it, n ? h[1] : h[0], group, sh);
    } else {
        const int32_t h = p.heads.head_order[group * units + u], g = p.heads.kv_of_q[h];
        if (attn_f32_single<D, PARTIAL>(p, it, h, g, u, sh)) attn_f32_rows<D, PARTIAL>(p, it, h, g, sh);
    }
}

hipError_t launch_attn_f32(const AttnParams &p, int32_t D, bool partial, int32_t compute_units, hipStream_t stream)
{
    // Two heads per workgroup halve the K and V traffic and use the faster instruction; one head per workgroup
    // has the shorter chain (104 tokens, 2 heads: 5.4 us against 6.7), and is taken where that alone leaves
    // the chip unfilled.
    const int32_t G = p.n_q_heads / p.n_kv_heads;
    bool uniform = true;
    for (int32_t i = 0; i < p.n_q_heads; ++i)
        if (p.heads.kv_of_q[p.heads.head_order[i]] != i / G) uniform = false;
    const int32_t pairs = uniform && G > 1 && (int64_t)p.n_items * p.n_q_heads > 2 * (int64_t)compute_units;
    const int32_t units = pairs ? (G + 1) / 2 : (uniform ? G : p.n_q_heads);  // per KV head, or per item if their groups differ
    const int32_t n_logical = p.n_items * units * (pairs || uniform ? p.n_kv_heads : 1);
    const int32_t stride = uniform && p.n_kv_heads <= 4 ? std::min(8 / p.n_kv_heads, p.n_items) : 1;
    const dim3 grid((n_logical + 7) / 8 * 8), block(256);
#define PEVLM_F32_LAUNCH(DD, PP) hipLaunchKernelGGL((attn_f32_kernel<DD, PP>), grid, block, 0, stream, p, n_logical, units, pairs, stride)
    if (D == 128) { if (partial) PEVLM_F32_LAUNCH(128, true); else PEVLM_F32_LAUNCH(128, false); }
    else { if (partial) PEVLM_F32_LAUNCH(64, true); else PEVLM_F32_LAUNCH(64, false); }
#undef PEVLM_F32_LAUNCH
    return hipGetLastError();
}

}  // namespace pevlm
