// bf16 flash-style attention kernel for gfx950 (CDNA4): bf16 MFMA for Q K^T and P V with fp32
// accumulation, fp32 online softmax.  Serves the block-parallel prefill (sink rows, Eq. 3, and
// context-block rows, Eq. 4: a work item names a tile of query rows plus the sink key range and the
// own-block key range up to the diagonal, nothing else) and, in partial mode, the split-KV question
// attention (Eq. 5).
//
// Tiling.  A workgroup of 4 wavefronts owns 128 (query row, head) pairs of one work item (<= 128 query rows)
// and KV head; wave w owns pairs 32w..32w+31; two workgroups share a compute unit (two wavefronts per SIMD).  Keys are
// staged 64 at a time in LDS (K and V tiles, XOR-swizzled 16-byte chunks, direct global->LDS loads,
// two stages each).  Scores are formed transposed, S^T = K Q^T, with v_mfma_f32_32x32x16_bf16: in
// the accumulator layout a lane then holds 16 keys of ONE query (column = lane % 32), so the softmax
// row reduction is in-lane max3/add chains and a single exchange with lane ^ 32.  The same
// registers, converted to bf16, are directly the B operand of O^T += V^T P^T; V^T fragments come
// from LDS through the transposing read ds_read_b64_tr_b16.
//
// Schedule inside a wavefront (software pipeline over key tiles): the value MFMAs of tile t-1 are
// issued interleaved with the vector-ALU work that turns the scores of tile t into weights, so the
// matrix cores and the vector ALU of a SIMD overlap within one instruction stream as well as
// across the two resident wavefronts; the wavefront's share of the next K tile and of the current V
// tile is requested piecewise between those MFMAs.
//
// Softmax.  Weights of a tile are formed against the reference maximum the row already has; the
// row maximum is only computed (and the reference raised, accumulators rescaled) when a lane's sum
// of weights shows that one of them may have reached 2^8, or on the row's first tile.
//
// Variants: PARTIAL writes un-normalised fp32 partials (question attention, merged afterwards);
// ROPEQ rotates the query rows in registers from a (cos, sin) table instead of expecting rotated
// queries; MAPPED takes a head map other than the default one.
#include <algorithm>
#include <type_traits>

#include "attn_bf16_tile.h"
#include "rope_math.h"

namespace pevlm {

// ROPEQ: q holds un-rotated queries; each wavefront rotates its 32 rows once, right after loading
// them, from the (cos, sin) table of the call (the sequential positions of Sec. "Position Encoding").
//
// The rows of an item and the query heads of a KV group form one list of (row, head) pairs, head fastest; a
// workgroup takes 128 consecutive pairs, a wavefront 32.  So a wavefront's MFMA columns are filled whatever
// the number of rows (1 question row x 7 heads: one wavefront instead of seven with one column each; K and V are
// then read once per KV head), and the pairs of a workgroup lie within 128/G + 1 rows of each other: it stages
// the tiles up to its own last row, not up to the item's.  `logical` indexes (KV head group, item,
// workgroup of the item).  Where heads are not in equal groups every head is a group of its own, and the groups run
// inside the item, so that heads on one KV head find its keys in L2 (64/8 heads on a map, 12 K tokens in blocks of
// 152: 242 us, 320 with the items inside the head).  Against one head
// per wavefront group (two or four heads together for items of <= 64 or <= 32 rows): question of 20 rows x 28/4
// heads over 65 K keys 60 -> 45 us at the same 64 splits, block prefill of 16 K tokens 210 -> 208 us, 100 K
// tokens in blocks of 3136 with the rotation folded in 3.40 -> 3.28 ms.
template <int D, bool PARTIAL, bool ROPEQ, bool MAPPED>
__device__ __forceinline__ void attn_item(const AttnParams &p, int32_t logical, const HeadGroups &hg, uint8_t *lds_k, uint8_t *lds_v)
{
    using C = TileCfg<D>;
    constexpr int KT = C::KT, ROWB = C::ROWB, CH = C::CH, NLD = C::NLD, KSTEPS = C::KSTEPS, DBLK = C::DBLK;
    constexpr int VSW = C::VSW, TILEB = C::TILEB, RPI = C::RPI;
    int32_t inner, rest, group;
    if (!MAPPED || hg.groups_inside == 1) {
        inner = logical % hg.wgs_per_item;
        rest = logical / hg.wgs_per_item;
        group = rest / p.n_items;
    } else {
        inner = logical % (hg.wgs_per_item * hg.groups_inside);
        rest = logical / (hg.wgs_per_item * hg.groups_inside);
        group = inner / hg.wgs_per_item;
        inner %= hg.wgs_per_item;
    }
    // last item first: within a context block the later tiles are the longer ones, and a launch that
    // ends on short items has a shorter tail; where the items are dealt, the XCDs that share a group
    // take them in turn
    int32_t in_order = rest % p.n_items;
    if (!PARTIAL && hg.deal_runs > 1) {
        // run r has the positions from ceil(r n / runs) on; what is left over goes, a shortest item each, where two XCDs
        // meet inside an item
        const int32_t run = in_order * hg.deal_runs / p.n_items, start = (run * p.n_items + hg.deal_runs - 1) / hg.deal_runs;
        const int32_t nth = in_order - start;
        in_order = nth < hg.deal_len ? nth * hg.deal_runs + run : hg.deal_len * (hg.deal_runs - run) + start;
    }
    const int32_t item_idx = p.n_items - 1 - in_order;
    const int32_t G = hg.heads_per_group;
    pevlm_work_item it;
    if (p.inline_items.mode) {
        it = inline_item(p.inline_items, item_idx);
        if (group == 0 && inner == 0 && threadIdx.x == 0) p.items[item_idx] = it;
    } else {
        it = p.items[item_idx];
    }
    const int32_t n_pairs = it.q_rows * G, pair0 = inner * 128;
    if (pair0 >= n_pairs) return;  // an item with fewer rows than the launch's longest
    // With the default head map (query head h on KV head h / G) the indices are plain arithmetic; the tables
    // live in kernel-argument memory and looking them up costs two dependent memory round trips before the
    // first query row can be requested.  Under another map of equal groups lane j holds the group's j-th head.
    const int32_t head0 = !MAPPED ? group * G : __builtin_amdgcn_readfirstlane((int32_t)p.heads.head_order[group * G]);
    const int32_t g = !MAPPED ? group : __builtin_amdgcn_readfirstlane((int32_t)p.heads.kv_of_q[head0]);
    const int32_t Hq = p.n_q_heads, Hkv = p.n_kv_heads;

    const int32_t tid = threadIdx.x, lane = tid & 63;
    const int32_t wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int32_t l32 = lane & 31, g32 = lane >> 5;
    const uint16_t *Q = (const uint16_t *)p.q, *K = (const uint16_t *)p.k, *V = (const uint16_t *)p.v;
    const bool listed = MAPPED && G > 1;  // otherwise the group's heads are head0, head0 + 1, ...
    const int32_t head_base = listed ? 0 : head0;
    // the j-th head of the group, relative to head_base; the list is fetched again for the output rows
    const auto head_list = [&](int32_t ln) { return listed ? (int32_t)p.heads.head_order[group * G + (ln < G ? ln : 0)] : 0; };
    const auto head_of = [&](int32_t list, int32_t j) { return listed ? __shfl(list, j) : j; };
    const int32_t heads = head_list(lane);

    LaneOff L;
    L.g32 = g32;
    L.k_row_off = l32 * ROWB;
    L.k_swz = l32 & (CH - 1);
    L.v_row_off = (g32 * 4 + ((lane & 15) >> 2)) * ROWB + (lane & 1) * 8;
    L.v_ch_lo = ((lane >> 4) & 1) * 2 + ((lane & 3) >> 1);
    L.v_swz = (lane >> 2) & VSW;

    // ---- this lane's query row and head, and the rows of the wavefront and of the workgroup
    const int32_t wave_pair0 = pair0 + wave * 32;
    const bool wave_active = wave_pair0 < n_pairs;
    const int32_t my_pair = wave_pair0 + l32 < n_pairs ? wave_pair0 + l32 : n_pairs - 1;
    const int32_t row_in_item = div_by(my_pair, hg.group_rcp);
    const int32_t my_row = it.q_start + row_in_item;
    const int32_t wr_lo = it.q_start + div_by(wave_active ? wave_pair0 : n_pairs - 1, hg.group_rcp);
    const int32_t wr_hi = it.q_start + div_by(wave_pair0 + 31 < n_pairs ? wave_pair0 + 31 : n_pairs - 1, hg.group_rcp);
    const int32_t wg_hi = it.q_start + div_by(pair0 + 127 < n_pairs ? pair0 + 127 : n_pairs - 1, hg.group_rcp);

    // (cos, sin) of this lane's row for the fused query rotation: fetched first, so that the loads
    // are in flight together with the Q rows
    f32x4 rope_cs[ROPEQ ? KSTEPS / 2 : 1][4];
    if (ROPEQ) {
        int64_t entry = my_row;
        if (p.rope_compact_rows > 0) entry = it.reserved % p.rope_compact_rows + row_in_item;
        const f32x4 *tab = reinterpret_cast<const f32x4 *>(p.rope_tab + entry * D) + g32 * 4;
#pragma unroll
        for (int kk = 0; kk < KSTEPS / 2; ++kk)
#pragma unroll
            for (int j = 0; j < 4; ++j) rope_cs[kk][j] = tab[kk * 8 + j];
    }
    const uint32_t lds_k_addr = (uint32_t)(size_t)LDS_PTR(void, lds_k);
    const uint32_t lds_v_addr = (uint32_t)(size_t)LDS_PTR(void, lds_v);
    // Q rows of the wave are fetched with whole-row (coalesced) direct-to-LDS loads into a
    // wave-private slice of LDS stage 1 (unused until the first tile is being consumed), then read
    // back as MFMA B fragments.  Same 16-byte-chunk XOR swizzle as the K tile.
    constexpr int WSLICE = 32 * ROWB;  // bytes of 32 rows
    uint8_t *const wave_slice = (wave < 2 ? lds_k : lds_v) + TILEB + (wave & 1) * WSLICE;
    const uint32_t wave_slice_addr = (wave < 2 ? lds_k_addr : lds_v_addr) + TILEB + (wave & 1) * WSLICE;

    // tiles the workgroup stages, and tiles this wave computes: all fully visible ones, and the causal ones
    // that start at or before its last row (the rest is masked for every row)
    const int32_t n_full_tiles = (it.full_len + KT - 1) / KT;
    const int32_t n_diag_tiles = (it.diag_len + KT - 1) / KT;
    const int32_t wg_diag = wg_hi >= it.diag_start ? (wg_hi - it.diag_start) / KT + 1 : 0;
    const int32_t n_tiles = n_full_tiles + (wg_diag < n_diag_tiles ? wg_diag : n_diag_tiles);
    int32_t n_w = 0;
    if (wave_active) {
        const int32_t nd = wr_hi >= it.diag_start ? (wr_hi - it.diag_start) / KT + 1 : 0;
        n_w = n_full_tiles + (nd < n_diag_tiles ? nd : n_diag_tiles);
    }

    // ---- K/V tiles go straight from global memory into LDS (16 bytes per lane): a wavefront
    // instruction fills 1 KB of contiguous LDS, i.e. RPI whole rows; the XOR swizzle is applied by
    // choosing which 16-byte chunk of the row each lane fetches.  Two LDS stages per tensor: K(t+1)
    // and V(t) stream in while tile t's scores and tile t-1's values are computed.  Rows past the
    // key range repeat its last key (their scores are masked, their values stay finite).
#define PEVLM_TILE_RANGE(t, k0, kend, causal)                 \
    do {                                                      \
        if ((t) < n_full_tiles) {                             \
            k0 = it.full_start + (t) * KT;                    \
            kend = it.full_start + it.full_len;               \
            causal = false;                                   \
        } else {                                              \
            k0 = it.diag_start + ((t) - n_full_tiles) * KT;   \
            kend = it.diag_start + it.diag_len;               \
            causal = true;                                    \
        }                                                     \
    } while (0)
    // Per-lane byte offsets of the NLD loads inside a tile are fixed (row within the tile, swizzled
    // chunk); a tile that lies wholly inside its key range only needs a new uniform base address.
    uint32_t koff[NLD], voff[NLD];
#pragma unroll
    for (int j = 0; j < NLD; ++j) {
        const int32_t row = (j * 4 + wave) * RPI + lane / CH, cpos = lane % CH;
        koff[j] = (uint32_t)((row * Hkv * D + ((cpos ^ (row & (CH - 1))) << 3)) * 2);
        voff[j] = (uint32_t)((row * Hkv * D + ((cpos ^ ((row & VSW) << 2)) << 3)) * 2);
    }
#define PEVLM_ISSUE(T, toff, swz_expr, lds_base_addr, t, stage)                                       \
    do {                                                                                              \
        int32_t pk0, pkend;                                                                           \
        bool pcausal;                                                                                 \
        PEVLM_TILE_RANGE(t, pk0, pkend, pcausal);                                                     \
        (void)pcausal;                                                                                \
        if (pk0 + KT <= pkend) {                                                                      \
            const uint16_t *tb = uniform_ptr(T + ((int64_t)pk0 * Hkv + g) * D);                       \
            _Pragma("unroll") for (int j = 0; j < NLD; ++j)                                           \
                load_lds_16_base(tb, toff[j], lds_base_addr + (stage) * TILEB + (j * 4 + wave) * RPI * ROWB); \
        } else {                                                                                      \
            _Pragma("unroll") for (int j = 0; j < NLD; ++j) {                                         \
                const int32_t rbase = (j * 4 + wave) * RPI;                                           \
                const int32_t row = rbase + lane / CH, cpos = lane % CH;                              \
                int32_t key = pk0 + row;                                                              \
                key = key < pkend ? key : pkend - 1;                                                  \
                load_lds_16(T + ((int64_t)key * Hkv + g) * D + ((cpos ^ (swz_expr)) << 3),            \
                            lds_base_addr + (stage) * TILEB + rbase * ROWB);                          \
            }                                                                                         \
        }                                                                                             \
    } while (0)
#define PEVLM_ISSUE_K(t) PEVLM_ISSUE(K, koff, (row & (CH - 1)), lds_k_addr, t, (t) & 1)
#define PEVLM_ISSUE_V(t) PEVLM_ISSUE(V, voff, ((row & VSW) << 2), lds_v_addr, t, (t) & 1)
    // top of tile t: K(t) and V(t-1) have landed for everybody, everybody is done with K(t-1) and
    // V(t-2); then K(t+1) and V(t) are put in flight
#define PEVLM_TOP(t)                                                   \
    do {                                                               \
        __builtin_amdgcn_s_waitcnt(0x0F70); /* vmcnt(0) */             \
        __syncthreads();                                               \
        if ((t) + 1 < n_tiles) PEVLM_ISSUE_K((t) + 1);                 \
        PEVLM_ISSUE_V(t);                                              \
    } while (0)

    // Inside the pipelined loop the loads of a tile are not issued in one burst behind the barrier
    // (the wavefront would sit in the memory-instruction queue while its MFMAs wait) but one at a
    // time between MFMAs.  PEVLM_SET_LOADS prepares them: base address of tile tl, LDS destination in
    // `stage`, and, for a tile that runs past the end of its key range, per-lane offsets clamped to
    // the last valid key (put back to the plain ones on the next use).
#define PEVLM_SET_LOADS(ld, T, toff, modified, swz_expr, lds_base_addr, tl, stage)                      \
    do {                                                                                              \
        int32_t pk0, pkend;                                                                           \
        bool pcausal;                                                                                 \
        PEVLM_TILE_RANGE(tl, pk0, pkend, pcausal);                                                    \
        (void)pcausal;                                                                                \
        const bool edge = pk0 + KT > pkend;                                                           \
        if (edge || modified) {                                                                       \
            const int32_t last = edge ? pkend - 1 - pk0 : KT - 1;                                     \
            _Pragma("unroll") for (int j = 0; j < NLD; ++j) {                                         \
                const int32_t row = (j * 4 + wave) * RPI + lane / CH, cpos = lane % CH;               \
                const int32_t key = row < last ? row : last;                                          \
                toff[j] = (uint32_t)((key * Hkv * D + ((cpos ^ (swz_expr)) << 3)) * 2);               \
            }                                                                                         \
            modified = edge;                                                                          \
        }                                                                                             \
        ld.base = uniform_ptr(T + ((int64_t)pk0 * Hkv + g) * D);                                      \
        ld.lds = lds_base_addr + (stage) * TILEB + wave * 1024;                                       \
        _Pragma("unroll") for (int j = 0; j < NLD; ++j) ld.off[j] = toff[j];                          \
    } while (0)

    // First the K and V tiles of tile 0 (stage 0; they usually come from L2), then the query rows
    // (first touch: from HBM), so that all three are in flight together.
    if (n_tiles > 0) {
        PEVLM_ISSUE_K(0);
        PEVLM_ISSUE_V(0);
    }
    // Walk of a lane over the wavefront's pairs, RPI at a time: byte offset of the pair's row from the item's first
    // one, advanced without a division (an integer product costs as much as four additions).
    const uint32_t row_bytes = (uint32_t)(Hq * ROWB), step_bytes = (uint32_t)hg.step_rows * row_bytes;
    const int64_t item_off = ((int64_t)it.q_start * Hq + head_base) * D;  // elements
#define PEVLM_PAIR_WALK_BEGIN()                                              \
    int32_t walk_v = wave_pair0 + lane / CH, walk_h;                          \
    uint32_t walk_row;                                                        \
    {                                                                         \
        const int32_t r_ = div_by(walk_v, hg.group_rcp);                      \
        walk_h = walk_v - r_ * G;                                             \
        walk_row = (uint32_t)r_ * row_bytes;                                  \
    }
    // LISTED is settled outside the loops over rows: a branch in each step keeps their reads and stores from running together
#define PEVLM_PAIR_WALK_OFF(LISTED, list) (walk_row + (uint32_t)((LISTED ? __shfl(list, walk_h) : walk_h) * ROWB))
#define PEVLM_PAIR_WALK_NEXT()                                               \
    do {                                                                      \
        walk_v += RPI;                                                        \
        walk_h += hg.step_heads;                                              \
        walk_row += step_bytes;                                               \
        if (walk_h >= G) {                                                    \
            walk_h -= G;                                                      \
            walk_row += row_bytes;                                            \
        }                                                                     \
    } while (0)
    {
        const int32_t last_row = div_by(n_pairs - 1, hg.group_rcp);
        const uint32_t last_off = (uint32_t)last_row * row_bytes + (uint32_t)(head_of(heads, n_pairs - 1 - last_row * G) * ROWB);
        const uint16_t *qbase = uniform_ptr(Q + item_off);
        const auto rows_in = [&](auto listed_tag) {
            PEVLM_PAIR_WALK_BEGIN();
#pragma unroll
            for (int j = 0; j < WSLICE / 1024; ++j) {
                const int32_t rl = j * RPI + lane / CH;
                const uint32_t walk_off = PEVLM_PAIR_WALK_OFF(decltype(listed_tag)::value, heads);
                const uint32_t off = walk_v < n_pairs ? walk_off : last_off;  // pairs past the item repeat its last one
                load_lds_16_base(qbase, off + (uint32_t)(((lane % CH) ^ (rl & (CH - 1))) << 4), wave_slice_addr + j * 1024);
                PEVLM_PAIR_WALK_NEXT();
            }
        };
        if (MAPPED && listed) rows_in(std::true_type());
        else rows_in(std::false_type());
    }
    __builtin_amdgcn_s_waitcnt(0x0F70);
    asm volatile("" ::: "memory");
    const float c_log2 = p.scale * 1.4426950408889634f;
    bf16x8 qf[KSTEPS];
#pragma unroll
    for (int kk = 0; kk < KSTEPS; ++kk)
        qf[kk] = *reinterpret_cast<const bf16x8 *>(wave_slice + l32 * ROWB + (((kk * 2 + g32) ^ (l32 & (CH - 1))) << 4));
    if constexpr (ROPEQ) rotate_query(qf, rope_cs);

    // m_ref: reference maximum of this lane's row in base-2 units, c_log2 * score (-inf: none yet)
    float m_ref = -INFINITY, l_run = 0.f;
    f32x16 o[DBLK];
#pragma unroll
    for (int b = 0; b < DBLK; ++b)
#pragma unroll
        for (int i = 0; i < 16; ++i) o[b][i] = 0.f;

    // entries of tile t that a row must not see (tiles that touch the diagonal or the end of their range)
#define PEVLM_MASK(k0, kend, causal)                                                      \
    do {                                                                                  \
        if ((k0 + KT > kend) || (causal && (k0 + KT - 1 > wr_lo)))                        \
            mask_tile(s, k0, kend, causal, my_row, g32);                                  \
    } while (0)
    f32x16 s[2];
    u32x4 pf[4];  // weights of the last tile whose scores are known, bf16 pairs
    float psum;
    TileLoads<NLD> ldk, ldv;
    bool k_mod = false, v_mod = false;
    int32_t k0, kend;
    bool causal;
    if (n_tiles > 0) {  // top of tile 0 for every wavefront
        __syncthreads();  // K(0), V(0) of every wavefront have landed; the query slices in stage 1 have been read
        if (1 < n_tiles) PEVLM_ISSUE_K(1);
    }
    if (n_w > 0) {
        qk_tile<D, false, NLD>(lds_k, L, qf, s, ldk, [] {}, [] {});
        PEVLM_TILE_RANGE(0, k0, kend, causal);
        PEVLM_MASK(k0, kend, causal);
        psum = 0.f;  // no row has a reference yet: the first tile always takes the exact path
        raise_reference(s, c_log2, m_ref, l_run, psum, pf, o);
        l_run += psum;
        for (int32_t t = 1; t < n_w; ++t) {
            // top of tile t as in PEVLM_TOP, but K(t+1) and V(t) are fetched piecewise between the
            // MFMAs below; after the last tile the K loads repeat that tile into the stage nobody
            // reads any more, which keeps the loop body free of branches
            __builtin_amdgcn_s_waitcnt(0x0F70);
            __syncthreads();
            const uint8_t *const tv = lds_v + ((t - 1) & 1) * TILEB;
            bf16x8 vfirst[kValuesAhead];
            qk_tile<D, true, NLD>(
                lds_k + (t & 1) * TILEB, L, qf, s, ldk,
                [&] {
                    const int32_t tk = t + 1 < n_tiles ? t + 1 : n_tiles - 1;
                    PEVLM_SET_LOADS(ldk, K, koff, k_mod, (row & (CH - 1)), lds_k_addr, tk, (t + 1) & 1);
                    PEVLM_SET_LOADS(ldv, V, voff, v_mod, ((row & VSW) << 2), lds_v_addr, t, t & 1);
                    PEVLM_TILE_RANGE(t, k0, kend, causal);
                },
                [&] { first_v<D>(tv, L, vfirst); });
            PEVLM_MASK(k0, kend, causal);
            // values of tile t-1 (matrix cores) under the weights of tile t (vector ALU)
            psum = 0.f;
            pv_prev_weights_cur<D, NLD>(tv, L, pf, o, s, c_log2, reference_of(m_ref), psum, ldv, vfirst);
            raise_reference(s, c_log2, m_ref, l_run, psum, pf, o);
            l_run += psum;
        }
    }
    // the burst loads below use the plain per-lane offsets
    if (k_mod) {
#pragma unroll
        for (int j = 0; j < NLD; ++j) {
            const int32_t row = (j * 4 + wave) * RPI + lane / CH, cpos = lane % CH;
            koff[j] = (uint32_t)((row * Hkv * D + ((cpos ^ (row & (CH - 1))) << 3)) * 2);
        }
    }
    if (v_mod) {
#pragma unroll
        for (int j = 0; j < NLD; ++j) {
            const int32_t row = (j * 4 + wave) * RPI + lane / CH, cpos = lane % CH;
            voff[j] = (uint32_t)((row * Hkv * D + ((cpos ^ ((row & VSW) << 2)) << 3)) * 2);
        }
    }
    // Every wavefront passes the top of all n_tiles tiles and one final barrier.  The values of the
    // last tile a wave computed are added once their V tile is known to be in LDS.
    int32_t t_rest = n_w > 0 ? n_w : (n_tiles > 0 ? 1 : 0);  // the top of tile 0 is behind every wavefront
    bool synced = false;
    if (n_w > 0 && n_w < n_tiles) {
        PEVLM_TOP(n_w);
        t_rest = n_w + 1;
    } else if (n_w == n_tiles) {
        __builtin_amdgcn_s_waitcnt(0x0F70);
        __syncthreads();
        synced = true;
    }
    if (n_w > 0) pv_tile<D>(lds_v + ((n_w - 1) & 1) * TILEB, L, pf, o);
    for (int32_t t = t_rest; t < n_tiles; ++t) PEVLM_TOP(t);
    if (!synced) {
        __builtin_amdgcn_s_waitcnt(0x0F70);
        __syncthreads();
    }

    // ---- epilogue: the lane's pair once more, from a lane number that the compiler takes for another (a register held
    // through the tile loop costs 64-wide heads the third wavefront on a SIMD)
    int32_t out_lane = lane;
    asm volatile("" : "+v"(out_lane));
    const int32_t heads_again = head_list(out_lane);
    const int32_t out_pair = wave_pair0 + (out_lane & 31);
    const bool pair_valid = out_pair < n_pairs;
    const int32_t out_row = div_by(pair_valid ? out_pair : n_pairs - 1, hg.group_rcp);
    const int32_t out_head = head_base + head_of(heads_again, (pair_valid ? out_pair : n_pairs - 1) - out_row * G);
    const float l_tot = l_run + __shfl_xor(l_run, 32);
    if (PARTIAL) {
        if (!pair_valid) return;
        const int64_t slot = ((int64_t)it.reserved + out_row) * Hq + out_head;
        store_partial(p, slot, o, g32, m_ref, c_log2, l_tot);
    } else {
        // O^T fragments -> wave-private LDS slice (row-major bf16, swizzled), then whole-row 16-byte
        // stores.  The slice lies in the stage the last tile does not use: a wavefront may still be
        // adding the values of the last tile out of the other stage.
        const float inv = 1.f / l_tot;
        uint8_t *const oslice = (wave < 2 ? lds_k : lds_v) + (n_tiles & 1) * TILEB + (wave & 1) * WSLICE;
#pragma unroll
        for (int b = 0; b < DBLK; ++b)
#pragma unroll
            for (int i4 = 0; i4 < 4; ++i4) {
                bf16x4 v4;
                v4[0] = (__bf16)(o[b][i4 * 4] * inv);
                v4[1] = (__bf16)(o[b][i4 * 4 + 1] * inv);
                v4[2] = (__bf16)(o[b][i4 * 4 + 2] * inv);
                v4[3] = (__bf16)(o[b][i4 * 4 + 3] * inv);
                *reinterpret_cast<bf16x4 *>(oslice + l32 * ROWB + (((b * 4 + i4) ^ (l32 & (CH - 1))) << 4) + g32 * 8) = v4;
            }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        uint16_t *const obase = (uint16_t *)p.out;
        // Rows leave as non-temporal stores: nothing here reads them again, and the lines stay free for keys and values
        // (16 K tokens, rotation and question included: 279 -> 272 us; dense 16 K 2139 -> 2122 us).
        uint8_t *const ob = (uint8_t *)(obase + item_off);
        const auto rows_out = [&](auto listed_tag) {
            PEVLM_PAIR_WALK_BEGIN();
#pragma unroll
            for (int j = 0; j < WSLICE / 1024; ++j) {
                const int32_t rl = j * RPI + lane / CH, cpos = lane % CH;
                const uint4 val = *reinterpret_cast<const uint4 *>(oslice + rl * ROWB + ((cpos ^ (rl & (CH - 1))) << 4));
                const uint32_t walk_off = PEVLM_PAIR_WALK_OFF(decltype(listed_tag)::value, heads_again);
                if (walk_v < n_pairs) __builtin_nontemporal_store(__builtin_bit_cast(u32x4, val), reinterpret_cast<u32x4 *>(ob + (walk_off + (uint32_t)(cpos << 4))));
                PEVLM_PAIR_WALK_NEXT();
            }
        };
        if (MAPPED && listed) rows_out(std::true_type());
        else rows_out(std::false_type());
        if (p.lse && g32 == 0 && pair_valid) p.lse[(int64_t)(it.q_start + out_row) * Hq + out_head] = (m_ref + __log2f(l_tot)) * 0.69314718056f;
    }
}

// One workgroup per logical id.  Consecutive workgroup ids land on different XCDs (8 of them, each
// with its own L2); every XCD gets one contiguous run of logical ids so that the heads of a GQA
// group working on the same context block share that XCD's L2.  The runs differ by one id at most and start at
// eighths of the ids, so that two, four or eight XCDs end where their KV head does.
template <int D, bool PARTIAL, bool ROPEQ, bool MAPPED>
__global__ __launch_bounds__(256, 2) void attn_bf16_kernel(AttnParams p, int32_t n_logical, HeadGroups hg)
{
    __shared__ __attribute__((aligned(1024))) uint8_t lds_k[2 * TileCfg<D>::TILEB];
    __shared__ __attribute__((aligned(1024))) uint8_t lds_v[2 * TileCfg<D>::TILEB];
    const int32_t xcd = blockIdx.x & 7, eighth = n_logical >> 3, over = n_logical & 7;
    const int32_t logical = xcd * eighth + (xcd * over >> 3) + (blockIdx.x >> 3);
    if (logical >= (xcd + 1) * eighth + ((xcd + 1) * over >> 3)) return;
    attn_item<D, PARTIAL, ROPEQ, MAPPED>(p, logical, hg, lds_k, lds_v);
}

hipError_t launch_attn_bf16(const AttnParams &p, int32_t D, bool partial, int32_t compute_units, hipStream_t stream)
{
    // heads that share a KV head are taken together when the groups are equal (and a wavefront's lanes can hold the group)
    const int32_t G = p.n_q_heads / p.n_kv_heads;
    bool uniform = true, identity = true;
    for (int32_t i = 0; i < p.n_q_heads; ++i) {
        if (p.heads.kv_of_q[p.heads.head_order[i]] != i / G) uniform = false;
        if (p.heads.head_order[i] != i || p.heads.kv_of_q[i] != i / G) identity = false;
    }
    const bool together = uniform && (identity || G <= 64);
    HeadGroups hg;
    hg.heads_per_group = together ? G : 1;
    hg.group_rcp = reciprocal_of(hg.heads_per_group);
    hg.groups_inside = together ? 1 : p.n_q_heads;
    const int32_t rows_per_load = 512 / D;  // rows one wavefront-wide 16-byte-per-lane load covers
    hg.step_rows = rows_per_load / hg.heads_per_group;
    hg.step_heads = rows_per_load % hg.heads_per_group;
    hg.wgs_per_item = ceil_div(p.max_item_rows * hg.heads_per_group, 128);
    // Each XCD takes one contiguous run of (group, item), so with 4, 2 or 1 KV heads 2, 4 or 8 of them share a group and cut
    // its items into runs.  Runs of many blocks weigh the same and keep a block's keys in one L2 (65 K tokens in blocks of
    // 1024, 8/1 heads: 224 us, 302 dealt out).  Where one region fills the runs the first has its long rows and the last its
    // short ones (dense attention over 16 K tokens x 28/4 heads: 165 against 57 ms of workgroup time), and the XCDs take the
    // items in turn instead: 2171 -> 1656 us, 8 K tokens 555 -> 421, 2 K 45.3 -> 39.8, 8 K x 14/2 heads x 64 233 -> 137.
    // The lines.  Some compute unit has two workgroups (280 of 28/4 heads 25.5 -> 24.2 us; 224 of 16/2 heads 29.3 -> 30.3).
    // Between more than two XCDs the longest region has three runs (16/2 heads, blocks of 3136, 3.2 runs: 66.0 -> 58.2 us;
    // 2.0 runs 0.89 to 1.27 times).  Between two it has nearly a run and they meet in its later part, so that one of
    // them would take its longest rows last (28/4 heads, blocks of 2048: a sink of 256 and two blocks 99 -> 73, one block and
    // 1700 rows 69 -> 52; meeting where a block starts, two blocks 65.0 and 67.5 dealt, in its first rows 65.0 and 70.3).
    // Where all workgroups are resident at once the order matters less (16/4 heads x 64: 1.06 runs 30.8 -> 34.6, 1.15 31.7 -> 29.3).
    const int32_t n_logical = p.n_items * hg.wgs_per_item * (together ? p.n_kv_heads : p.n_q_heads);
    hg.deal_runs = 1;
    hg.deal_len = p.n_items;
    if (!partial && n_logical > compute_units && together && p.n_kv_heads < 8 && 8 % p.n_kv_heads == 0) {
        const int32_t runs = 8 / p.n_kv_heads;
        const int64_t region = (int64_t)p.max_region_items * runs, n = p.n_items;  // region / n: in runs
        const bool late = 5 * (int64_t)p.middle_half_items >= 4 * (int64_t)p.max_region_items;
        const bool pays = runs > 2 ? region >= 3 * n : late && (n_logical > 2 * compute_units ? 10 * region >= 9 * n : 20 * region >= 23 * n);
        if (p.n_items >= runs && pays) {
            hg.deal_runs = runs;
            hg.deal_len = p.n_items / runs;
        }
    }
    const dim3 grid((n_logical + 7) / 8 * 8), block(256);
#define PEVLM_ATTN_LAUNCH(DD, PP, RR)                                                                             \
    do {                                                                                                          \
        if (identity) hipLaunchKernelGGL((attn_bf16_kernel<DD, PP, RR, false>), grid, block, 0, stream, p, n_logical, hg); \
        else hipLaunchKernelGGL((attn_bf16_kernel<DD, PP, RR, true>), grid, block, 0, stream, p, n_logical, hg);           \
    } while (0)
    const bool rope = p.rope_tab != nullptr;
    if (D == 128) {
        if (partial) { if (rope) PEVLM_ATTN_LAUNCH(128, true, true); else PEVLM_ATTN_LAUNCH(128, true, false); }
        else { if (rope) PEVLM_ATTN_LAUNCH(128, false, true); else PEVLM_ATTN_LAUNCH(128, false, false); }
    } else {
        if (partial) { if (rope) PEVLM_ATTN_LAUNCH(64, true, true); else PEVLM_ATTN_LAUNCH(64, true, false); }
        else { if (rope) PEVLM_ATTN_LAUNCH(64, false, true); else PEVLM_ATTN_LAUNCH(64, false, false); }
    }
#undef PEVLM_ATTN_LAUNCH
    return hipGetLastError();
}

}  // namespace pevlm
