// Tile-level building blocks of the bf16 MFMA attention kernels (gfx950): staging layout of a key
// tile in LDS, S^T = K Q^T and O^T += V^T P^T on v_mfma_f32_32x32x16_bf16, masks, the weights of the
// online softmax.  Shared by the one-item-per-workgroup kernel and the streaming kernel.
#pragma once
#include "bf16_device.h"
#include "rope_math.h"

namespace pevlm {

template <int D>
struct TileCfg {
    static constexpr int KT = kKeyTile;        // keys per staged tile
    static constexpr int ROWB = D * 2;         // bytes per K/V row
    static constexpr int CH = D / 8;           // 16-byte chunks per row
    static constexpr int NLD = KT * CH / 256;  // 16-byte loads each wavefront issues per tensor per tile
    static constexpr int KSTEPS = D / 16;      // MFMA k-steps of Q K^T
    static constexpr int DBLK = D / 32;        // 32-wide blocks of head_dim in O^T
    static constexpr int VSW = CH / 4 - 1;     // V swizzle mask (64-byte granules per row - 1)
    static constexpr int TILEB = KT * ROWB;    // bytes of one staged K (or V) tile
    static constexpr int RPI = 1024 / ROWB;    // rows one wavefront-wide 16-byte-per-lane load covers
};

// per-lane LDS offsets (the XOR swizzles depend on the lane only)
struct LaneOff {
    int32_t k_row_off, k_swz, v_row_off, v_ch_lo, v_swz, g32;
};

// Global->LDS loads a wavefront slips between the MFMAs of a tile (its share of a later K tile
// during the score MFMAs, of a V tile during the value MFMAs): a wavefront-uniform base
// address, per-lane byte offsets and the LDS address of the wave's first 1 KB piece; four wavefronts share a
// tile, so its j-th piece lies 4 KB after its (j-1)-th.
template <int NLD>
struct TileLoads {
    const void *base;
    uint32_t off[NLD];
    uint32_t lds;
    __device__ __forceinline__ void issue(int j) const { load_lds_16_base(base, off[j], lds + j * 4096); }
};

constexpr float kRescaleStep = 8.f;  // log2 units the row maximum may outgrow the reference maximum

// S^T = K Q^T for the 64 keys of a staged tile: two independent accumulation chains (one per
// 32-key chunk) issued alternately; A fragments (16 bytes per lane) are fetched PF k-steps ahead of their MFMAs.
// `ld.issue(j)` requests the wavefront's j-th piece (of NL) of a later K tile.  `pre` runs while the first fragments
// are under way (scalar set-up of the tile: in front of them it delays both wavefronts of the SIMD, which
// leave the barrier together), `post` before the last pair of MFMAs (first reads of what follows them).
template <int D, bool LOADS, int NL, int PF = 2, class LD, class Pre, class Post>
__device__ __forceinline__ void qk_tile(const uint8_t *tk, const LaneOff &L, const bf16x8 (&qf)[D / 16], f32x16 (&s)[2],
                                        const LD &ld, Pre pre, Post post)
{
    using C = TileCfg<D>;
    constexpr int KS = C::KSTEPS, HK = KS / 2;
    const f32x16 init = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    bf16x8 a0[KS], a1[KS];
#define PEVLM_KFRAG(kc, kk) \
    (*reinterpret_cast<const bf16x8 *>(tk + (kc) * 32 * C::ROWB + L.k_row_off + ((((kk) * 2 + L.g32) ^ L.k_swz) << 4)))
#pragma unroll
    for (int kk = 0; kk < PF; ++kk) {
        a0[kk] = PEVLM_KFRAG(0, kk);
        a1[kk] = PEVLM_KFRAG(1, kk);
    }
    __builtin_amdgcn_sched_barrier(0);
    pre();
#pragma unroll
    for (int kk = 0; kk < KS; ++kk) {
        if (kk == KS - 1) post();
        s[0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a0[kk], qf[kk], kk == 0 ? init : s[0], 0, 0, 0);
        if (kk + PF < KS) a0[kk + PF] = PEVLM_KFRAG(0, kk + PF);
        s[1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a1[kk], qf[kk], kk == 0 ? init : s[1], 0, 0, 0);
        if (kk + PF < KS) a1[kk + PF] = PEVLM_KFRAG(1, kk + PF);
        if (LOADS && kk >= HK && kk - HK < NL) ld.issue(kk - HK);  // one 1 KB piece of a later K tile per pair of MFMAs
        __builtin_amdgcn_sched_barrier(0);
    }
#undef PEVLM_KFRAG
}

// V^T fragments of 16 keys (k-step ks of the staged tile) for every 32-wide block of head_dim
template <int D>
__device__ __forceinline__ void read_v(const uint8_t *tv, const LaneOff &L, int ks, bf16x8 (&dst)[D / 32])
{
    using C = TileCfg<D>;
#pragma unroll
    for (int b = 0; b < C::DBLK; ++b)
#pragma unroll
        for (int tt = 0; tt < 2; ++tt) {
            const uint8_t *ptr = tv + (ks * 16 + tt * 8) * C::ROWB + L.v_row_off + (((b ^ L.v_swz) * 4 + L.v_ch_lo) << 4);
            const s16x4 r = __builtin_amdgcn_ds_read_tr16_b64_v4i16(LDS_PTR(s16x4, ptr));
            const bf16x4 rb = __builtin_bit_cast(bf16x4, r);
            dst[b][tt * 4 + 0] = rb[0]; dst[b][tt * 4 + 1] = rb[1];
            dst[b][tt * 4 + 2] = rb[2]; dst[b][tt * 4 + 3] = rb[3];
        }
}

// entries a row must not see: beyond the key range, or (causal range) keys after the row.  Key
// k0 + c is visible iff c <= min(kend - 1, causal ? my_row : inf) - k0; c = const + 4*g32 per entry,
// so each entry costs one compare against a per-lane limit and one select.
__device__ __forceinline__ void mask_tile(f32x16 (&s)[2], int32_t k0, int32_t kend, bool causal, int32_t my_row, int32_t g32)
{
    int32_t last = kend - 1;
    if (causal) last = my_row < last ? my_row : last;
    const int32_t lim = last - k0 - g32 * 4;
#pragma unroll
    for (int kc = 0; kc < 2; ++kc)
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            const int32_t c = kc * 32 + (i >> 2) * 8 + (i & 3);
            s[kc][i] = c <= lim ? s[kc][i] : -INFINITY;
        }
}

// maximum over the 64 keys of the tile for this lane's row (both lanes of a row end up with it)
__device__ __forceinline__ float row_max(const f32x16 (&s)[2])
{
    // max3f is an instruction that the compiler does not know (it quiets the operands of its own): no wait for matrix results
    // is added in front of it.  The first maximum is one that it knows, and the others come after it.
    float mx = fmaxf(s[0][0], s[0][1]);
#pragma unroll
    for (int i = 2; i < 32; i += 2) mx = max3f(mx, s[i >> 4][i & 15], s[(i + 1) >> 4][(i + 1) & 15]);
    const auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(mx), __float_as_uint(mx), false, false);
    return fmaxf(__uint_as_float(sw[0]), __uint_as_float(sw[1]));
}

// weights p = exp2(c s - m) of the tile (c = scale*log2(e), m = the row's reference maximum in
// base-2 units): bf16 pairs (B fragments of the value MFMAs) and their sum over this lane's 32 keys.  Weights
// are non-negative, so a sum below 2^kRescaleStep bounds every one of them; an overflowed or invalid weight makes
// the sum inf or nan.
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
typedef __attribute__((ext_vector_type(2))) uint32_t u32x2;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;

// fused in every place (left to the compiler it is in some): a row's weights are formed in one or the other as the rows beside
// it need it, and come out the same
__device__ __forceinline__ float weight(float s, float c_log2, float mref) { return __builtin_amdgcn_exp2f(__builtin_fmaf(s, c_log2, -mref)); }

__device__ __forceinline__ uint32_t weight_pair(float p0, float p1)
{
    bf16x2 pr;
    pr[0] = (__bf16)p0;
    pr[1] = (__bf16)p1;
    return __builtin_bit_cast(uint32_t, pr);
}

// Adds four pairs of rounded weights to the lane's fp32 sum.  v_mfma_f32_4x4x4 with a block of ones adds the four
// values that a lane supplies to the lane's own accumulators (all four end up alike): 8 cycles for two words.
// v_dot2_f32_bf16 with (1, 1) is as exact and one instruction a word, but does not run beside an MFMA of
// either wavefront of the SIMD (four of them between two MFMAs: 28.4 ns a round where four multiply-adds,
// exponentials or conversions leave it at the 17.8 ns of the bare MFMAs); unpacking to fp32 costs 4 vector
// instructions a word (5 % of the 64K prefill).
__device__ __forceinline__ void add_weights(const u32x4 &pairs, f32x4 &sum)
{
    const s16x4 ones = {0x3f80, 0x3f80, 0x3f80, 0x3f80};
    const u32x2 a = {pairs[0], pairs[1]}, b = {pairs[2], pairs[3]};
    sum = __builtin_amdgcn_mfma_f32_4x4x4bf16_1k(ones, __builtin_bit_cast(s16x4, a), sum, 0, 0, 0);
    sum = __builtin_amdgcn_mfma_f32_4x4x4bf16_1k(ones, __builtin_bit_cast(s16x4, b), sum, 0, 0, 0);
}

__device__ __forceinline__ void weights(const f32x16 (&s)[2], float c_log2, float mref, float &psum, u32x4 (&pf)[4])
{
    f32x4 sum = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int j = 0; j < 4; ++j) {
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            const int kc = j >> 1, i = (j & 1) * 8 + w * 2;
            pf[j][w] = weight_pair(weight(s[kc][i], c_log2, mref), weight(s[kc][i + 1], c_log2, mref));
        }
        add_weights(pf[j], sum);
    }
    psum = sum[0];
}

// true unless this lane's sum of weights proves that all of them stayed below 2^kRescaleStep
__device__ __forceinline__ bool sum_reached_step(float psum) { return !(psum < 256.f); }
static_assert(kRescaleStep == 8.f, "sum_reached_step compares with 2^kRescaleStep");
// the row sum moved to a new reference: a product that is not fused with the addition after it in one kernel and not in another
__device__ __forceinline__ float rounded_product(float a, float b)
{
#pragma clang fp contract(off)
    return a * b;
}

// The weights of a tile are first formed against the reference maximum the row already has (m_ref, base-2 units; -inf: none yet).
// Only if a lane's weights may have reached 2^kRescaleStep (or a row has no reference yet) is the
// row maximum of the tile computed, the reference raised, o and l scaled down and the tile's weights formed
// again: weights stay below 2^kRescaleStep, which fp32 sums and bf16 weights carry without loss,
// and on almost every tile the vector ALU only does exp2, convert and sum.  A row is raised for its own weights
// only: its result does not depend on which rows share its wavefront, which the kernels, the calls with
// RoPE folded in and a prefill in pieces choose differently.
__device__ __forceinline__ float reference_of(float m_ref) { return m_ref == -INFINITY ? 0.f : m_ref; }
template <int DBLK>
__device__ __forceinline__ void raise_reference(const f32x16 (&s)[2], float c_log2, float &m_ref, float &l_run, float &psum, u32x4 (&pf)[4],
                                                f32x16 (&o)[DBLK])
{
    const int32_t up = sum_reached_step(psum) || m_ref == -INFINITY;
    if (__any(up)) {
        const float mx = row_max(s) * c_log2;
        const bool has = m_ref != -INFINITY;
        const float m_new = up | __shfl_xor(up, 32) ? fmaxf(m_ref, mx) : m_ref;
        const float alpha = has ? __builtin_amdgcn_exp2f(m_ref - m_new) : 1.f;
        m_ref = m_new;
        psum = 0.f;
        weights(s, c_log2, reference_of(m_ref), psum, pf);
        if (__any(has)) {
            l_run = rounded_product(l_run, alpha);
#pragma unroll
            for (int b = 0; b < DBLK; ++b)
#pragma unroll
                for (int i = 0; i < 16; ++i) o[b][i] *= alpha;
        }
    }
}

// A lane's query fragments turned by its row's (cos, sin) pairs, with pevlm_rope_seq's arithmetic: it holds dims
// kk*16 + g32*8 + e of its row, pair index i < D/2 in qf[kk], its partner i + D/2 in qf[kk + KSTEPS/2]
template <int KSTEPS>
__device__ __forceinline__ void rotate_query(bf16x8 (&qf)[KSTEPS], const f32x4 (&rope_cs)[KSTEPS / 2][4])
{
#pragma unroll
    for (int kk = 0; kk < KSTEPS / 2; ++kk) {
        const f32x4 *cs = rope_cs[kk];
        const u32x4 lo = __builtin_bit_cast(u32x4, qf[kk]), hi = __builtin_bit_cast(u32x4, qf[kk + KSTEPS / 2]);
        u32x4 rl, rh;
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            const float a0 = __uint_as_float(lo[w] << 16), a1 = __uint_as_float(lo[w] & 0xffff0000u);
            const float b0 = __uint_as_float(hi[w] << 16), b1 = __uint_as_float(hi[w] & 0xffff0000u);
            float r0, r1, t0, t1;
            rope_rotate(a0, b0, cs[w][0], cs[w][1], r0, t0);
            rope_rotate(a1, b1, cs[w][2], cs[w][3], r1, t1);
            rl[w] = rope_pack_bf16(r0, r1);
            rh[w] = rope_pack_bf16(t0, t1);
        }
        qf[kk] = __builtin_bit_cast(bf16x8, rl);
        qf[kk + KSTEPS / 2] = __builtin_bit_cast(bf16x8, rh);
    }
}

// A lane's share of a (row, head) pair of a split: unnormalised values, maximum and sum
template <int DBLK>
__device__ __forceinline__ void store_partial(const AttnParams &p, int64_t slot, const f32x16 (&o)[DBLK], int32_t g32, float m_ref, float c_log2, float l_tot)
{
    float *acc = p.part_acc + slot * (DBLK * 32);
#pragma unroll
    for (int b = 0; b < DBLK; ++b)
#pragma unroll
        for (int i4 = 0; i4 < 4; ++i4) {
            const f32x4 v4 = {o[b][i4 * 4], o[b][i4 * 4 + 1], o[b][i4 * 4 + 2], o[b][i4 * 4 + 3]};
            *reinterpret_cast<f32x4 *>(acc + b * 32 + i4 * 8 + g32 * 4) = v4;
        }
    if (g32 == 0) {
        p.part_ml[slot * 2] = m_ref / c_log2;  // back to raw score units (-inf stays)
        p.part_ml[slot * 2 + 1] = l_tot;
    }
}

// O^T += V^T P^T for a staged V tile (16 MFMAs per 32 values of head_dim ... 4 k-steps x DBLK blocks)
template <int D>
__device__ __forceinline__ void pv_tile(const uint8_t *tv, const LaneOff &L, const u32x4 (&pf)[4], f32x16 (&o)[D / 32])
{
    using C = TileCfg<D>;
    bf16x8 va[C::DBLK], vb[C::DBLK];
    read_v<D>(tv, L, 0, va);
#pragma unroll
    for (int ks = 0; ks < 4; ks += 2) {
        read_v<D>(tv, L, ks + 1, vb);
#pragma unroll
        for (int b = 0; b < C::DBLK; ++b) o[b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(va[b], __builtin_bit_cast(bf16x8, pf[ks]), o[b], 0, 0, 0);
        if (ks + 2 < 4) read_v<D>(tv, L, ks + 2, va);
#pragma unroll
        for (int b = 0; b < C::DBLK; ++b) o[b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vb[b], __builtin_bit_cast(bf16x8, pf[ks + 1]), o[b], 0, 0, 0);
    }
}

// One V^T fragment: 16 keys (k-step ks) x the b-th 32-wide block of head_dim
template <int D>
__device__ __forceinline__ bf16x8 read_v_one(const uint8_t *tv, const LaneOff &L, int ks, int b)
{
    using C = TileCfg<D>;
    bf16x8 dst;
#pragma unroll
    for (int tt = 0; tt < 2; ++tt) {
        const uint8_t *ptr = tv + (ks * 16 + tt * 8) * C::ROWB + L.v_row_off + (((b ^ L.v_swz) * 4 + L.v_ch_lo) << 4);
        const s16x4 r = __builtin_amdgcn_ds_read_tr16_b64_v4i16(LDS_PTR(s16x4, ptr));
        const bf16x4 rb = __builtin_bit_cast(bf16x4, r);
        dst[tt * 4 + 0] = rb[0]; dst[tt * 4 + 1] = rb[1];
        dst[tt * 4 + 2] = rb[2]; dst[tt * 4 + 3] = rb[3];
    }
    return dst;
}

// V^T fragments of the first value MFMAs of a tile
constexpr int kValuesAhead = 3;
template <int D>
__device__ __forceinline__ void first_v(const uint8_t *tv, const LaneOff &L, bf16x8 (&vf)[kValuesAhead])
{
#pragma unroll
    for (int n = 0; n < kValuesAhead; ++n) vf[n] = read_v_one<D>(tv, L, n / TileCfg<D>::DBLK, n % TileCfg<D>::DBLK);
}

// The pipelined step: O^T += V^T P^T of the previous tile (matrix cores) issued one MFMA at a time,
// each followed by the vector-ALU work for a pair (or two) of weights of the current tile, so that
// both pipes of the SIMD run from one instruction stream.  V^T fragments are read kValuesAhead MFMAs ahead, the first
// ones by the caller.  The four words of weights that a k-step of value MFMAs has used are rewritten with those of the
// current tile right after it (formed in other registers, all 16 words are copied on every tile).
// `ld.issue(j)` requests the wavefront's j-th piece (of NL) of a later V tile.
template <int D, int NL, class LD>
__device__ __forceinline__ void pv_prev_weights_cur(const uint8_t *tv_prev, const LaneOff &L, u32x4 (&pf)[4], f32x16 (&o)[D / 32],
                                                    const f32x16 (&s)[2], float c_log2, float mref, float &psum, const LD &ld,
                                                    const bf16x8 (&vfirst)[kValuesAhead])
{
    using C = TileCfg<D>;
    constexpr int PF = kValuesAhead;
    constexpr int NM = 4 * C::DBLK;  // MFMAs of the tile
    constexpr int PPM = 16 / NM;     // weight pairs formed per MFMA
    f32x4 sum = {0.f, 0.f, 0.f, 0.f};
    bf16x8 vf[NM];
    float e[8];
#pragma unroll
    for (int n = 0; n < PF; ++n) vf[n] = vfirst[n];
#pragma unroll
    for (int n = 0; n < NM; ++n) {
        const int ks = n / C::DBLK, b = n % C::DBLK;
        if (n + PF < NM) vf[n + PF] = read_v_one<D>(tv_prev, L, (n + PF) / C::DBLK, (n + PF) % C::DBLK);
        o[b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf[n], __builtin_bit_cast(bf16x8, pf[ks]), o[b], 0, 0, 0);
        if (n % 4 == 0 && n / 4 < NL) ld.issue(n / 4);
#pragma unroll
        for (int x = 0; x < PPM; ++x) {
            const int pi = n * PPM + x, kc = pi >> 3, i = (pi & 7) * 2;
            float &e0 = e[(pi & 3) * 2], &e1 = e[(pi & 3) * 2 + 1];
            e0 = weight(s[kc][i], c_log2, mref);
            e1 = weight(s[kc][i + 1], c_log2, mref);
            asm volatile("" : "+v"(e0), "+v"(e1));  // here, not after the last MFMA
        }
        if (b == C::DBLK - 1) {
#pragma unroll
            for (int w = 0; w < 4; ++w) pf[ks][w] = weight_pair(e[w * 2], e[w * 2 + 1]);
            add_weights(pf[ks], sum);
            asm volatile("" : "+v"(pf[ks]));
        }
        __builtin_amdgcn_sched_barrier(0);
    }
    psum = sum[0];
}

}  // namespace pevlm
