// Split-KV attention of a short question for gfx950 (CDNA4), bf16: the (row, head) pairs of one KV head fit one workgroup.
//
// Same work items, tile arithmetic and partials as the one-item kernel (attn_bf16.hip), bit for bit, under another schedule.
// That one has a tile and a half under way per workgroup of 4 wavefronts, and above 128 pairs two workgroups that read the same
// keys.  This one has one workgroup of 8 wavefronts to a compute unit, three LDS stages per tensor, K two tiles and V one and a
// half ahead of the arithmetic: 64 KB under way, and the keys are staged once for up to 256 pairs.  Attention and merge,
// 65 K keys: 20 rows x 28/4 heads 46.1 -> 41.8 us, x 32/8 60.9 -> 53.3, 36 rows x 32/8 76.4 -> 71.3.  What bounds it now: the 140
// pairs of 20 rows x 7 heads are five wavefronts on four SIMDs, 2 us a tile; 16 rows (four) take 36.3 us.
//
// Waits.  Loads into LDS complete in issue order per wavefront, and every wavefront issues the same number in every tile
// (past the last tile the last one again, into a stage that nobody reads): the top of a tile waits until only those of the
// tile before are outstanding.
#include "attn_bf16_tile.h"

namespace pevlm {

namespace {
constexpr int NW = kQuestionWaves;
constexpr int NST = 3;

// where the rotation of the queries comes from
constexpr int kRotated = 0, kTable = 1, kAngles = 2;

template <int NL>
struct QuestionLoads {
    const void *base;
    uint32_t off[NL];
    uint32_t lds;
    __device__ __forceinline__ void issue(int j) const { load_lds_16_base(base, off[j], lds + j * NW * 1024); }
};
}  // namespace

template <int D, int ROPE>
__global__ __launch_bounds__(NW * 64, 2) void attn_bf16_question_kernel(AttnParams p, int32_t n_logical, uint32_t group_rcp, RopeAngles angles)
{
    using C = TileCfg<D>;
    constexpr int KT = C::KT, ROWB = C::ROWB, CH = C::CH, KSTEPS = C::KSTEPS, DBLK = C::DBLK;
    constexpr int VSW = C::VSW, TILEB = C::TILEB, RPI = C::RPI, NL = KT * CH / (64 * NW), WSLICE = 32 * ROWB;
    __shared__ __attribute__((aligned(1024))) uint8_t lds[2 * NST * TILEB + NW * WSLICE];
    const int32_t per_xcd = gridDim.x >> 3, logical = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
    if (logical >= n_logical) return;
    const int32_t g = logical / p.n_items, item_idx = p.n_items - 1 - logical % p.n_items;
    const int32_t Hq = p.n_q_heads, Hkv = p.n_kv_heads, G = Hq / Hkv;
    pevlm_work_item it;
    if (p.inline_items.mode) {
        it = inline_item(p.inline_items, item_idx);
        if (g == 0 && threadIdx.x == 0) p.items[item_idx] = it;
    } else {
        it = p.items[item_idx];
    }
    const int32_t n_pairs = it.q_rows * G;

    const int32_t tid = threadIdx.x, lane = tid & 63;
    const int32_t wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int32_t l32 = lane & 31, g32 = lane >> 5;
    const uint16_t *Q = (const uint16_t *)p.q, *K = (const uint16_t *)p.k, *V = (const uint16_t *)p.v;

    LaneOff L;
    L.g32 = g32;
    L.k_row_off = l32 * ROWB;
    L.k_swz = l32 & (CH - 1);
    L.v_row_off = (g32 * 4 + ((lane & 15) >> 2)) * ROWB + (lane & 1) * 8;
    L.v_ch_lo = ((lane >> 4) & 1) * 2 + ((lane & 3) >> 1);
    L.v_swz = (lane >> 2) & VSW;

    const int32_t wave_pair0 = wave * 32;
    const bool wave_active = wave_pair0 < n_pairs;
    const int32_t my_pair = wave_pair0 + l32 < n_pairs ? wave_pair0 + l32 : n_pairs - 1;
    const int32_t row_in_item = div_by(my_pair, group_rcp), my_row = it.q_start + row_in_item;
    const int32_t wr_lo = it.q_start + div_by(wave_active ? wave_pair0 : n_pairs - 1, group_rcp);
    const int32_t wr_hi = it.q_start + div_by(wave_pair0 + 31 < n_pairs ? wave_pair0 + 31 : n_pairs - 1, group_rcp);
    const int32_t wg_hi = it.q_start + it.q_rows - 1;
    const int32_t n_full_tiles = (it.full_len + KT - 1) / KT, n_diag_tiles = (it.diag_len + KT - 1) / KT;
    const int32_t wg_diag = wg_hi >= it.diag_start ? (wg_hi - it.diag_start) / KT + 1 : 0;
    const int32_t n_tiles = n_full_tiles + (wg_diag < n_diag_tiles ? wg_diag : n_diag_tiles);
    int32_t n_w = 0;  // tiles that this wavefront computes
    if (wave_active) {
        const int32_t nd = wr_hi >= it.diag_start ? (wr_hi - it.diag_start) / KT + 1 : 0;
        n_w = n_full_tiles + (nd < n_diag_tiles ? nd : n_diag_tiles);
    }
    const uint32_t lds_k_addr = (uint32_t)(size_t)LDS_PTR(void, lds), lds_v_addr = lds_k_addr + NST * TILEB;
    uint8_t *const lds_k = lds, *const lds_v = lds + NST * TILEB, *const slice = lds + 2 * NST * TILEB + wave * WSLICE;
    const uint32_t slice_addr = lds_k_addr + 2 * NST * TILEB + wave * WSLICE;

    auto tile_range = [&](int32_t t, int32_t &k0, int32_t &kend) {
        const bool own = t >= n_full_tiles;
        k0 = own ? it.diag_start + (t - n_full_tiles) * KT : it.full_start + t * KT;
        kend = own ? it.diag_start + it.diag_len : it.full_start + it.full_len;
        return own;
    };
    // Loads of a tile: per-lane offsets are fixed but for a tile that runs past its range, whose rows repeat the last key
    // (their scores are masked, their values stay finite).
    QuestionLoads<NL> ldk, ldv;
    auto set_loads = [&](QuestionLoads<NL> &ld, const uint16_t *T, bool is_v, uint32_t lds_addr, int32_t t, int32_t stage) {
        t = t < n_tiles ? t : n_tiles - 1;
        int32_t k0, kend;
        tile_range(t, k0, kend);
        const int32_t last = kend - k0 < KT ? kend - k0 - 1 : KT - 1;
#pragma unroll
        for (int j = 0; j < NL; ++j) {
            const int32_t row = (j * NW + wave) * RPI + lane / CH, cpos = lane % CH;
            const int32_t key = row < last ? row : last;
            ld.off[j] = (uint32_t)((key * Hkv * D + ((cpos ^ (is_v ? (row & VSW) << 2 : row & (CH - 1))) << 3)) * 2);
        }
        ld.base = uniform_ptr(T + ((int64_t)k0 * Hkv + g) * D);
        ld.lds = lds_addr + stage * TILEB + wave * 1024;
    };
    auto burst = [&](const QuestionLoads<NL> &ld) {
#pragma unroll
        for (int j = 0; j < NL; ++j) ld.issue(j);
    };

    f32x4 rope_cs[ROPE != kRotated ? KSTEPS / 2 : 1][4];
    if (n_tiles > 0) {
        set_loads(ldk, K, false, lds_k_addr, 0, 0);
        burst(ldk);
        set_loads(ldv, V, true, lds_v_addr, 0, 0);
        burst(ldv);
        set_loads(ldk, K, false, lds_k_addr, 1, 1);
        burst(ldk);
    }
    {
        // query rows, whole rows through the wavefront's slice
        const uint16_t *qbase = uniform_ptr(Q + ((int64_t)it.q_start * Hq + (int64_t)g * G) * D);
#pragma unroll
        for (int j = 0; j < WSLICE / 1024; ++j) {
            const int32_t rl = j * RPI + lane / CH, pair = wave_pair0 + rl < n_pairs ? wave_pair0 + rl : n_pairs - 1;
            const int32_t r = div_by(pair, group_rcp);
            load_lds_16_base(qbase, (uint32_t)((r * Hq + pair - r * G) * ROWB + (((lane % CH) ^ (rl & (CH - 1))) << 4)), slice_addr + j * 1024);
        }
    }
    auto read_table = [&](const float *table, int64_t entry) {
        const f32x4 *tab = reinterpret_cast<const f32x4 *>(table + entry * D) + g32 * 4;
#pragma unroll
        for (int kk = 0; kk < KSTEPS / 2; ++kk)
#pragma unroll
            for (int j = 0; j < 4; ++j) rope_cs[kk][j] = tab[kk * 8 + j];
    };
    if (ROPE == kTable) read_table(p.rope_tab, it.reserved % p.rope_compact_rows + row_in_item);
    if (ROPE == kAngles) {
        // The item's (cos, sin) pairs, as the table kernel forms them, into the stages of V(1) and V(2) while the first tiles
        // are under way: a launch before this one takes 4.7 us (20 rows x 28/4 heads over 65 K keys, the call 48.3 -> 46.0).
        static_assert(kAngleRows * D * 4 <= 2 * TILEB, "the stages of V(1) and V(2) hold the pairs");
        float2 *const table = reinterpret_cast<float2 *>(lds_v + TILEB);
        const int32_t first_row = it.reserved % p.rope_compact_rows, i = tid % (D / 2);
        const double inv_freq = angles.freq.inv_freq[i];
        int32_t s = 0;
        while (s + 1 < angles.num_seqs && first_row >= angles.first[s + 1]) ++s;
        const int32_t pos0 = first_row - angles.first[s] + angles.pos[s];
        for (int32_t r = tid / (D / 2); r < it.q_rows; r += NW * 64 / (D / 2)) {
            float2 cs;
            rope_cos_sin<false>((double)(pos0 + r), inv_freq, cs.x, cs.y);
            table[r * (D / 2) + i] = cs;
        }
    }
    __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0)
    asm volatile("" ::: "memory");
    if (ROPE == kAngles) {
        __syncthreads();
        read_table(reinterpret_cast<const float *>(lds_v + TILEB), row_in_item);
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // read before the next barrier, behind which V(1) is loaded
    }
    bf16x8 qf[KSTEPS];
#pragma unroll
    for (int kk = 0; kk < KSTEPS; ++kk) qf[kk] = *reinterpret_cast<const bf16x8 *>(slice + l32 * ROWB + (((kk * 2 + g32) ^ (l32 & (CH - 1))) << 4));
    if constexpr (ROPE != kRotated) rotate_query(qf, rope_cs);

    const float c_log2 = p.scale * 1.4426950408889634f;
    float m_ref = -INFINITY, l_run = 0.f, psum = 0.f;
    f32x16 o[DBLK], s[2];
#pragma unroll
    for (int b = 0; b < DBLK; ++b)
#pragma unroll
        for (int i = 0; i < 16; ++i) o[b][i] = 0.f;
    u32x4 pf[4];
    auto mask = [&](int32_t t) {
        int32_t k0, kend;
        const bool causal = tile_range(t, k0, kend);
        if ((k0 + KT > kend) || (causal && (k0 + KT - 1 > wr_lo))) mask_tile(s, k0, kend, causal, my_row, g32);
    };
    const auto next = [](int32_t st) { return st + 1 < NST ? st + 1 : 0; };
    const auto before = [](int32_t st) { return st > 0 ? st - 1 : NST - 1; };
    // loads of tile t's step: K(t + 2) into the stage of K(t - 1), V(t + 1) into that of V(t - 2); st = t % NST
    auto prepare = [&](int32_t t, int32_t st) {
        set_loads(ldk, K, false, lds_k_addr, t + 2, before(st));
        set_loads(ldv, V, true, lds_v_addr, t + 1, next(st));
    };
    auto top = [&] {
        asm volatile("s_waitcnt vmcnt(%0)" ::"n"(2 * NL) : "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
    };
    int32_t st = 0;  // t % NST of the tile at hand
    if (n_tiles > 0) {
        __builtin_amdgcn_s_barrier();  // K(0), V(0) and K(1) of every wavefront have landed
        asm volatile("" ::: "memory");
        prepare(0, 0);
        burst(ldk);
        burst(ldv);
    }
    if (n_w > 0) {
        qk_tile<D, false, NL>(lds_k, L, qf, s, ldk, [] {}, [] {});
        mask(0);
        psum = 0.f;
        raise_reference(s, c_log2, m_ref, l_run, psum, pf, o);
        l_run += psum;
        for (int32_t t = 1; t < n_w; ++t) {
            st = next(st);
            top();
            const uint8_t *const tv = lds_v + before(st) * TILEB;
            bf16x8 vfirst[kValuesAhead];
            qk_tile<D, true, NL>(lds_k + st * TILEB, L, qf, s, ldk, [&] { prepare(t, st); }, [&] { first_v<D>(tv, L, vfirst); });
            mask(t);
            psum = 0.f;
            pv_prev_weights_cur<D, NL>(tv, L, pf, o, s, c_log2, reference_of(m_ref), psum, ldv, vfirst);
            raise_reference(s, c_log2, m_ref, l_run, psum, pf, o);
            l_run += psum;
        }
    }
    // Every wavefront passes the tops of all tiles and one barrier behind them.  The values of the last tile that a wavefront
    // computed are added behind the next one, where they have landed.
    const int32_t last_st = st;
    bool pending = n_w > 0;
    for (int32_t t = n_w > 0 ? n_w : 1; t < n_tiles; ++t) {
        st = next(st);
        top();
        prepare(t, st);
        burst(ldk);
        burst(ldv);
        if (pending) {
            pv_tile<D>(lds_v + last_st * TILEB, L, pf, o);
            pending = false;
        }
    }
    __builtin_amdgcn_s_waitcnt(0x0F70);
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    if (pending) pv_tile<D>(lds_v + last_st * TILEB, L, pf, o);

    // ---- partials of the split
    int32_t out_lane = lane;
    asm volatile("" : "+v"(out_lane));
    const int32_t out_pair = wave_pair0 + (out_lane & 31);
    const float l_tot = l_run + __shfl_xor(l_run, 32);
    if (out_pair >= n_pairs) return;
    const int32_t out_row = div_by(out_pair, group_rcp);
    const int64_t slot = ((int64_t)it.reserved + out_row) * Hq + g * G + out_pair - out_row * G;
    store_partial(p, slot, o, g32, m_ref, c_log2, l_tot);
}

// This kernel takes a compute unit per (KV head, split), so there must not be more of those.  Up to 128 pairs a workgroup
// of the one-item kernel has one too (16 rows x 28/4 heads over 65 K keys, 24 / 48 / 64 splits: 56.2 -> 51.2, 40.9 -> 36.3,
// 38.6 -> 36.3 us; 1 row 50.8 -> 46.5, 34.3 -> 32.2, 31.3 -> 31.9); above that it has two, which need not share
// a compute unit while there are few (20 rows, 192 of 256 compute units 49.8 -> 45.9, 128 48.3 -> 57.5).  Short splits do not
// make up for its longer start: 8 rows x 14/2 heads x 64, 10 tiles a split 16.7 -> 16.9, 5 tiles 14.6 -> 15.7; 28/4 heads, 13
// tiles 24.7 -> 23.2, 5 20.4 -> 20.7; the line is 8.
bool is_short_question(const AttnParams &p, int32_t split_keys, int32_t compute_units)
{
    if (split_keys < 512) return false;
    if (p.n_q_heads % p.n_kv_heads != 0) return false;
    const int32_t G = p.n_q_heads / p.n_kv_heads, pairs = p.max_item_rows * G;
    for (int32_t i = 0; i < p.n_q_heads; ++i)
        if (p.heads.head_order[i] != i || p.heads.kv_of_q[i] != i / G) return false;
    const int64_t wgs = (int64_t)p.n_items * p.n_kv_heads;
    return pairs <= 32 * kQuestionWaves && wgs <= compute_units && (pairs <= 128 || 4 * wgs >= 3 * (int64_t)compute_units);
}

hipError_t launch_attn_bf16_question(const AttnParams &p, int32_t D, const RopeAngles *angles, hipStream_t stream)
{
    static const RopeAngles none = {};
    const int32_t n_logical = p.n_items * p.n_kv_heads;
    const dim3 grid((n_logical + 7) / 8 * 8), block(NW * 64);
    const uint32_t rcp = reciprocal_of(p.n_q_heads / p.n_kv_heads);
#define PEVLM_QUESTION_LAUNCH(DD)                                                                                                       \
    do {                                                                                                                                \
        if (angles) hipLaunchKernelGGL((attn_bf16_question_kernel<DD, kAngles>), grid, block, 0, stream, p, n_logical, rcp, *angles);    \
        else if (p.rope_tab) hipLaunchKernelGGL((attn_bf16_question_kernel<DD, kTable>), grid, block, 0, stream, p, n_logical, rcp, none); \
        else hipLaunchKernelGGL((attn_bf16_question_kernel<DD, kRotated>), grid, block, 0, stream, p, n_logical, rcp, none);             \
    } while (0)
    if (D == 128) PEVLM_QUESTION_LAUNCH(128);
    else PEVLM_QUESTION_LAUNCH(64);
#undef PEVLM_QUESTION_LAUNCH
    return hipGetLastError();
}

}  // namespace pevlm
