// Hierarchical mask estimation for single-query decode in bf16 (paper Alg. 2: one run of
// Alg. 1 per step over the current context, with bq = 1).
//
// With one query row the branch scoring is vector x gathered-rows work: bandwidth bound, no
// use for the matrix cores.  Three forms (template parameter WS, chosen by the number of problems): one
// WORKGROUP of sixteen or four waves per (sequence, query head), or one WAVE per problem with the four waves of a
// workgroup being the query heads of one KV group when Hq/Hkv = 4.  Either way the heads of a KV group run next to each other, so in
// the first round, where they score the same representative blocks, their loads meet in the L1/L2 instead of
// going to HBM four times.
//   * a table in LDS names the blocks to score (first key of each, -1: none); a lane group finds the blocks of a stage with one
//     read, and a block's score replaces its entry;
//   * a key row is read by D/8 lanes, 16 bytes each (a full 128-bit coalesced row segment), and multiplied with
//     v_dot2_f32_bf16; the ROWS partial sums of a lane are then added up over the lanes of the group by halving: at
//     each step a lane gives half of its sums away and adds the other half to what it gets, so that a lane ends up with
//     one row (or a copy of it) and everything after - maximum over the block's rows, bounds, the write - is done once
//     for all the rows of a stage instead of row by row;
//   * two stages of ROWS row loads per lane alternate, so up to 16 KB per wave are in flight;
//   * scores -> ordered threshold selection by up to four waves, a lane holding nodes with both of their scores -> the next
//     node list and the next table (two tables take turns);
//   * a branch whose representative block was scored in an earlier round keeps that score (known_branches in common.h): with
//     the first or the last block as representative one child of every node, from the second round on; with the centre
//     most branches of the last two rounds (where nodes hand on their own scores alone, see kOwnAlone: right halves of the last).  Such a branch has no entry in the table, and where a node has at most one branch to
//     score the table has one entry a node.  (Before, only the right halves of two-block nodes in the last round: 1024 problems of
//     128k tokens 264 -> 252 us, 4096 of 20k 583 -> 510, 8960 of 12k over pages 752 -> 653; 32 problems level.)
// Ragged lengths (kv_lens) and a page table are handled per row.
// Measured against the form before (nodes looked up and sums taken row by row, the selection run by eight waves of sixteen; half
// of a round was vector issue): 32 problems of 32768 tokens, d = 128, k = 512, bk = 2 50.6 -> 37.2 us, bk = 1 92 -> 50; 320 problems
// 104 -> 72; 1024 problems of k/bk = 512 331 -> 270, with 64 channels over pages 434 -> 305; 3072 problems 583 -> 555.
#pragma once
#include "common.h"
#include "launch.h"
#include <type_traits>

namespace hipattn {

// WS waves share a problem.
// WS = 1 : one wave per (sequence, head), four independent problems per workgroup.
// WS = 4 : one workgroup per (sequence, head); the four waves score a quarter of the branches each (stage i goes to
//          wave i % 4), meet at a barrier, run the selection redundantly and write a quarter of the survivors each.
// WS = 16: the same with sixteen waves, of which four (one per SIMD) run the selection: for so few problems
//          that each has a compute unit to itself, where the chain of latencies in a round is the time.
// MODE 0: contiguous keys, a (sequence, kv head) slice below 2 GB, addressed as a buffer that ends with the last key (a load past
//         it returns 0, so nothing is clamped); MODE 1: paged pool; MODE 2: contiguous, any size (64-bit row addresses).
//
// Nodes hand on the keys of their own and of their first block's score in every round (HAND_ON), or their own alone, and only to a round with
// one entry a node: with up to 64 nodes, whose rounds are so short that first blocks' keys cost what they save (64 channels, k/bk = 32, the
// first block as representative: 1920 problems 48.0 us handing both on, 45.4 so; 6 problems 16.1 / 15.0), and, as kOwnAlone, for up to 256 nodes
// of four and sixteen waves with the first or last block as representative, where no round asks for a first block's key (both / own, us, first
// block: 32 problems of 32k tokens, 128 channels, k/bk = 128 22.7 / 21.8, 64 channels 20.9 / 19.5; 1024 of 12k, 64 channels 31.5 / 30.7).
// Their own alone also with sixteen waves, eight rows a block and more than 256 nodes: handing both on spills 33 registers over contiguous keys and
// 34 over pages instead of 6 and 21.  Both / own, us, bk = 8, 128 channels: k/bk = 300, 32 problems of 32k tokens over pages 74.6 / 73.2, 256 123.5 /
// 119.7, of 8000 tokens 40.5 / 39.7, contiguous 37.7 / 36.0, k/bk = 512 33.7 / 32.7, 64 channels 24.3 / 22.8; only 256 problems of 32k tokens
// with k/bk = 512, whose last round scores nothing then, 149.6 / 157.
constexpr int kOwnAlone = 4;

// Waves per SIMD that the registers are laid out for.  With up to 64 nodes five fit (96 registers), where that spills nothing or one: the
// keys that nodes hand on took most of these kernels to four (104 registers).  us, four / five waves: 4096 problems of 8192 tokens, k/bk = 64,
// bk = 1, 64 channels 83.6 / 76.6, first block as representative 80.5 / 73.8; 128 channels 114.7 / 109.6, 94.2 / 87.2; 9600 problems of 4096
// tokens over pages, 64 channels 115 / 110.  Four stay for four waves a problem over pages (2 to 5 spilled) and for 128 channels with two
// or four rows a block (one spilled: 4096 problems, k/bk = 64 174 / 181, 9600 276 / 294).  More than 512 nodes: two; asked for one, a wave a problem
// takes 258 registers (16384 problems of 4096 tokens, k/bk = 1024, two / one: 1001 / 1498, over pages 1618 / 2956).
constexpr int decode_waves(int E, int BK, int D, int MODE, int WS)
{
    const bool five = E == 2 && (WS == 1 || (MODE != 1 && (D == 64 || BK == 1 || BK == 8)));
    return WS == 16 ? 4 : five ? 5 : E <= 8 ? 4 : E == 16 ? 3 : 2;
}
// FORM: MODE, or MODE + kOwnAlone.
template <int E, int BK, int D, int ROWS, int FORM, int WS>
__global__ __launch_bounds__(WS == 16 ? 1024 : kThreads, decode_waves(E, BK, D, FORM, WS)) void mask_decode_kernel(KParams p, int xcd_map)
{
    constexpr int MODE = FORM % kOwnAlone;
    constexpr bool SPLIT = WS > 1, PAGED = MODE == 1, HAND_ON = E > 2 && FORM < kOwnAlone && !(E == 16 && ROWS == 8 && WS == 16);
    constexpr int WGT = WS == 16 ? 1024 : kThreads;   // threads of the workgroup
    constexpr int NB = 64 * E, H = E / 2;
    constexpr int LPR = D / 8;        // lanes per key row
    constexpr int RPW = 64 / LPR;     // rows (= branches) per wave-wide load
    constexpr int U = ROWS / BK;      // branches per lane group and stage: ROWS row loads per lane, two stages in flight
    constexpr int COPIES = LPR / ROWS; // lanes that end up with the same row
    static_assert(ROWS <= LPR && U >= 1 && E % 2 == 0, "stage shape");
    constexpr int SW = WS < 4 ? 1 : WS == 4 ? 4 : (H < 4 ? H : 4);   // waves that select
    typedef uint32_t stage_t __attribute__((ext_vector_type(4 * ROWS)));
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
    constexpr int NW = SPLIT ? 1 : 4;  // private copies of the per-problem LDS state
    // Entry i of a table: first key of the i-th block to score, -1 if there is none, until the block's score (the bits of
    // the float; -1 stays) replaces it.
    __shared__ __attribute__((aligned(16))) uint32_t tab_s[NW][2][NB];
    // Nodes, sorted by position.  All of a round's nodes are m_len or m_len + 1 blocks long (chunks differ by one, and so do
    // halves of lengths that differ by one), so a node is its first block and one bit.
    __shared__ uint32_t node_s[NW][NB / 2];
    // What each node knows: the keys of its own score (entry j) and of its first block's (entry kb + j), for this round and the
    // next.  A wave with a problem of its own keeps them in the table that is not being scored.
    __shared__ uint32_t known_s[2][SPLIT ? NB : 1];

    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);  // (uniform: what follows from it stays in scalar registers)
    const int grp = lane / LPR, lc = lane % LPR;
    const int own = SPLIT ? 0 : wave;  // which LDS copy
    int64_t wg;
    if (SPLIT) {
        // keep the query heads of a KV group on one XCD (blockIdx.x % 8), next to each other in time
        const int64_t bid = blockIdx.x;
        if (xcd_map) {
            const int64_t seq = bid >> 3, gi = (bid & 7) + 8 * (seq / p.g);
            wg = gi * p.g + seq % p.g;  // = (b * hkv + hk) * g + head in group = b * hq + h
        } else {
            wg = bid;
        }
    } else {
        wg = (int64_t)blockIdx.x * 4 + wave;
    }
    if (wg >= (int64_t)p.batch * p.hq) return;
    const int b = (int)(wg / p.hq), h = (int)(wg % p.hq), hk = h / p.g;
    const int kb = p.kb;
    const int kv_len = p.kv_lens ? p.kv_lens[b] : p.max_kv_len;
    int32_t *out = p.idx_out + wg * kb;

    // BK = key rows scored per block; with a key sampling stride the block itself is bk = BK * b_sk keys
    const int bsk = p.b_sk, bk = BK * bsk;
    const int Tb = kv_len > 0 ? (kv_len + bk - 1) / bk : 0;
    if (Tb <= kb) {
        for (int j = SPLIT ? (int)threadIdx.x : lane; j < kb; j += SPLIT ? WGT : 64) out[j] = j < Tb ? j * bk : kSentinel;
        return;
    }
    // all waves of a problem hold identical copies of its state when SPLIT
    auto sync_problem = [&]() __attribute__((always_inline)) {
        if (SPLIT) __syncthreads(); else wave_lds_sync();
    };
    const int tix = SPLIT ? (int)threadIdx.x : lane, tn = SPLIT ? WGT : 64;

    const uint4 qv = *(const uint4 *)((const bf16_t *)p.Q + (int64_t)b * p.qs_b + (int64_t)h * p.qs_h + lc * 8);
    uint32_t *nodes = node_s[own];
    const RepRule rule = rep_rule(p.rep_pos);
    const bool first_rule = p.rep_pos == 1;
    auto first_key = [&](int blk) __attribute__((always_inline)) { return MODE == 0 ? (int)__umul24((uint32_t)blk, (uint32_t)bk) : blk * bk; };
    auto touch = [&](int t0) __attribute__((always_inline)) { if (PAGED && p.touched && t0 >= 0) touch_page(p, b, t0); };
    auto put_pair = [&](uint32_t *tab, int j, int tl, int tr) __attribute__((always_inline)) {
        *(uint2 *)(tab + 2 * j) = make_uint2((uint32_t)tl, (uint32_t)tr);
        touch(tl);
        touch(tr);
    };
    // the two branches of node [s, e): left [s, mid) (empty for a one-block node), right [mid, e)
    auto put_branches = [&](uint32_t *tab, int j, int s, int e) __attribute__((always_inline)) {
        const int mid = s + ((e - s) >> 1);
        put_pair(tab, j, mid > s ? first_key(rep_block(s, mid, rule)) : -1, first_key(rep_block(mid, e, rule)));
    };
    int m_len = Tb / kb;
    {
        const int r = Tb % kb;
        for (int j = tix; j < kb; j += tn) {
            const int s = chunk_bound(j, m_len, r, kb, p.kb_magic), e = chunk_bound(j + 1, m_len, r, kb, p.kb_magic);
            nodes[j] = (uint32_t)(s << 1 | (e - s - m_len));
            put_branches(tab_s[own][0], j, s, e);
            if (HAND_ON) {
                uint32_t *known = SPLIT ? known_s[0] : tab_s[own][1];
                known[j] = known[kb + j] = 0u;
            }
        }
        for (int i = 2 * kb + tix; i < NB; i += tn) tab_s[own][0][i] = tab_s[own][1][i] = 0xffffffffu;
    }
    sync_problem();

    const bf16_t *Kbase = (const bf16_t *)p.K;
    const int64_t back_delta = (const bf16_t *)p.Kback - Kbase;  // elements from the resident pool to the backing pool
    const uint32_t row_bytes = (uint32_t)p.ks_r * 2u;
    const __amdgpu_buffer_rsrc_t srd = __builtin_amdgcn_make_buffer_rsrc(
        (void *)(Kbase + (int64_t)b * p.ks_b + (int64_t)hk * p.ks_h), 0,
        MODE == 0 ? (int)((uint32_t)(kv_len - 1) * row_bytes + 2u * D) : 0, 0x00020000);

    const bool selects = !SPLIT || wave < SW;   // (uniform) nodes i * 64 + lane and what becomes of them: wave i % SW
    uint32_t nd[H];
    if (selects) {
#pragma unroll
        for (int i = 0; i < H; ++i) nd[i] = nodes[i * 64 + lane];
    }
    int cur = 0;
    bool knows = false, one_each = false;  // a round that knows scores (never the first), with one entry a node
    // ensemble sample: the round whose selection compares perturbed scores (-1: none)
    const int ens_round = ens_round_of(p.ens_sample, (Tb + kb - 1) / kb);
    const uint32_t ens_hash = ens_round >= 0 ? ens_unit_hash(p.ens_seed, p.ens_sample, b, h, 0) : 0u;
    int round = 0;
    for (int maxlen = (Tb + kb - 1) / kb; maxlen > 1; maxlen = (maxlen + 1) >> 1, ++round) {
        const int n_items = one_each ? kb : 2 * kb;   // entries to score
        uint32_t *tab = tab_s[own][cur], *next_tab = tab_s[own][cur ^ 1];

        // one stage = U blocks per lane group: the entries, then the (unconditional) loads of their BK rows
        auto fetch = [&](int base, stage_t &kv) __attribute__((always_inline)) {
            int t0[U], pg[U];
            const int at = base + grp * U;
            if constexpr (U % 4 == 0) {
#pragma unroll
                for (int u = 0; u < U; u += 4) {
                    const int4 v = *(const int4 *)(tab + at + u);
                    t0[u] = v.x; t0[u + 1] = v.y; t0[u + 2] = v.z; t0[u + 3] = v.w;
                }
            } else if constexpr (U == 2) {
                const int2 v = *(const int2 *)(tab + at);
                t0[0] = v.x; t0[1] = v.y;
            } else t0[0] = (int)tab[at];
#pragma unroll
            for (int u = 0; u < U; ++u) t0[u] = at + u < n_items ? t0[u] : -1;
#pragma unroll
            for (int u = 0; u < U; ++u) pg[u] = page_of_row<PAGED>(p, b, max(t0[u], 0));  // all page lookups of the stage first
#pragma unroll
            for (int u = 0; u < U; ++u) {
                if constexpr (MODE == 0) {
                    // (an empty entry: far past the end)
                    const uint32_t off = (t0[u] < 0 ? 0x80000000u : __umul24((uint32_t)t0[u], row_bytes)) + (uint32_t)lc * 16u;
#pragma unroll
                    for (int n = 0; n < BK; ++n) {
                        const u32x4 x = __builtin_amdgcn_raw_buffer_load_b128(srd, (int)(off + (uint32_t)(n * bsk) * row_bytes), 0, 0);
                        const int q4 = 4 * (u * BK + n);
                        kv[q4] = x[0]; kv[q4 + 1] = x[1]; kv[q4 + 2] = x[2]; kv[q4 + 3] = x[3];
                    }
                } else {
                    const int t = max(t0[u], 0);
                    // (a negative page-table entry names a page of the backing pool)
                    const bf16_t *src = Kbase + row_offset_bank<PAGED>(p, b, hk, t, pg[u], back_delta) + lc * 8;
#pragma unroll
                    for (int n = 0; n < BK; ++n) {
                        // rows past the end of the sequence re-read its last row and are ignored below
                        const uint4 x = *(const uint4 *)(src + (int64_t)min(n * bsk, kv_len - 1 - t) * p.ks_r);
                        const int q4 = 4 * (u * BK + n);
                        kv[q4] = x.x; kv[q4 + 1] = x.y; kv[q4 + 2] = x.z; kv[q4 + 3] = x.w;
                    }
                }
            }
        };
        auto score = [&](int base, const stage_t &kv) __attribute__((always_inline)) {
            float v[ROWS];
#pragma unroll
            for (int r = 0; r < ROWS; ++r) v[r] = dot8_bf16(qv, make_uint4(kv[4 * r], kv[4 * r + 1], kv[4 * r + 2], kv[4 * r + 3]));
            // the row this lane ends up with, and its block's entry
            const int row = lc / COPIES, at = base + grp * U + row / BK;
            const int t0 = (int)tab[at];
            // Sums over the lanes of the group.  Exchanges from the farthest lane to the nearest: the mirrors (lane i with 15 - i,
            // then 7 - i) also flip the lower bits of the lane number, which do not matter before they tell rows apart.
            constexpr int HALVINGS = ROWS == 8 ? 3 : ROWS == 4 ? 2 : ROWS == 2 ? 1 : 0;
            constexpr int STEPS = LPR == 16 ? 4 : 3;
            auto exchange = [&](float x, int bit) __attribute__((always_inline)) {
                return bit == 8 ? dpp_f<0x140>(x) : bit == 4 ? dpp_f<0x141>(x) : bit == 2 ? dpp_f<0x4E>(x) : dpp_f<0xB1>(x);
            };
#pragma unroll
            for (int st = 0; st < STEPS; ++st) {
                const int bit = LPR >> (st + 1);
                if (st < HALVINGS) {
                    const int n = ROWS >> (st + 1);
                    const bool up = lc & bit;
#pragma unroll
                    for (int k = 0; k < n; ++k) {
                        const float a = v[k], b = v[k + n];   // (values, not places: a choice of places would be indexed)
                        v[k] = (up ? b : a) + exchange(up ? a : b, bit);
                    }
                } else {
                    v[0] += exchange(v[0], bit);
                }
            }
            // maximum over the rows of the block that exist (rows of a block: neighbouring lanes; copies hold the same value, so
            // the mirrors serve here as well)
            float best = t0 + (row % BK) * bsk < kv_len ? v[0] : -INFINITY;
#pragma unroll
            for (int w = COPIES; w < COPIES * BK; w <<= 1) best = fmaxf(best, exchange(best, w));
            if (lc % (COPIES * BK) == 0 && at < n_items && t0 >= 0) tab[at] = score_bits(best);
        };

        constexpr int STEP = RPW * U;   // branches per stage
        constexpr int STRIDE = WS * STEP;  // distance between two stages of the same wave
        stage_t ka, kbuf;
        const int first = SPLIT ? wave * STEP : 0;
        if (first < n_items) fetch(first, ka);
        for (int base = first; base < n_items; base += 2 * STRIDE) {
            const bool has_b = base + STRIDE < n_items;
            if (has_b) fetch(base + STRIDE, kbuf);
            score(base, ka);
            if (has_b) {
                if (base + 2 * STRIDE < n_items) fetch(base + 2 * STRIDE, ka);
                score(base + STRIDE, kbuf);
            }
        }
        // What the nodes know.  (A wave with a problem of its own: in registers, the selection overwrites them.)
        const uint32_t *known = SPLIT ? known_s[cur] : next_tab;
        uint32_t own_key[SPLIT ? 1 : H], beg_key[SPLIT ? 1 : H];
        if constexpr (!SPLIT) {
#pragma unroll
            for (int i = 0; i < H; ++i) {
                own_key[i] = known[i * 64 + lane];
                beg_key[i] = HAND_ON ? known[kb + i * 64 + lane] : 0u;
            }
        }
        auto own_of = [&](int i) __attribute__((always_inline)) { return SPLIT ? known[i * 64 + lane] : own_key[SPLIT ? 0 : i]; };
        auto beg_of = [&](int i) __attribute__((always_inline)) { return !HAND_ON ? 0u : SPLIT ? known[kb + i * 64 + lane] : beg_key[SPLIT ? 0 : i]; };
        sync_problem();

        const int m_next = m_len >> 1;
        // (with the first or last block every node has one branch at most to score, with the centre nodes of one or two blocks)
        const bool last = maxlen <= 2, next_one = p.rep_pos != 0 || ((maxlen + 1) >> 1) == 2, next_knows = HAND_ON ? round_knows_scores(p.rep_pos, m_next) : next_one;
        if (selects) {
            uint32_t kl[H], kr[H];   // keys of the left and the right branch of node i * 64 + lane
            if (one_each) {
#pragma unroll
                for (int i = 0; i < H; ++i) {
                    if constexpr (HAND_ON) {
                        kl[i] = kr[i] = score_key_bits(tab[i * 64 + lane]);
                    } else {
                        // the branch that was scored, if the node has two, and the one that has the node's own score
                        int j = i * 64 + lane;
                        asm volatile("" : "+v"(j));   // (addresses kept through the loads are registers that spill)
                        const uint32_t own = j < kb ? (SPLIT ? known[j] : own_key[SPLIT ? 0 : i]) : 0u, scored = j < kb ? score_key_bits(tab[j]) : 0u;
                        const bool left_is_own = first_rule && m_len + (int)(nd[i] & 1) > 1;
                        kl[i] = left_is_own ? own : scored;
                        kr[i] = left_is_own ? scored : own;
                    }
                }
            } else {
#pragma unroll
                for (int i = 0; i < H; ++i) {
                    const uint2 x = *(const uint2 *)(tab + 2 * (i * 64 + lane));
                    kl[i] = score_key_bits(x.x);
                    kr[i] = score_key_bits(x.y);
                }
            }
            if (HAND_ON && knows) {
#pragma unroll
                for (int i = 0; i < H; ++i) {
                    uint32_t left, right;
                    bool need_l, need_r;
                    known_branches(rule, i * 64 + lane < kb ? m_len + (int)(nd[i] & 1) : 0, own_of(i), beg_of(i), left, right, need_l, need_r);
                    if (!need_l) kl[i] = left;
                    if (!need_r) kr[i] = right;
                }
            }
            const bool odd = m_len & 1;
            uint32_t *next_known = SPLIT ? known_s[cur ^ 1] : tab;
            // (three forms, so that the survivors' code has few branches: a round to come scores every branch, it knows some, or any of the two.
            // After the last round, which without HAND_ON takes the first or the second, no table is written: 32 problems of 8192 tokens over
            // pages, 128 channels, k/bk = 32 16.9 us writing one, 16.7 so)
            auto keep_one = [&](auto form, int d, uint32_t child, uint32_t own, uint32_t beg) __attribute__((always_inline)) {
                constexpr bool all = decltype(form)::value == 0, any = decltype(form)::value == 2;
                nodes[d] = child;
                if ((!all || !HAND_ON) && last) return;
                if (!all || HAND_ON) next_known[d] = own;
                if (HAND_ON && (all || rule.beg_left)) next_known[kb + d] = beg;
                const int s = (int)(child >> 1), len = m_next + (int)(child & 1), mid = s + (len >> 1);
                if (all || (any && !next_knows)) {
                    put_branches(next_tab, d, s, s + len);
                    return;
                }
                if constexpr (!HAND_ON) {
                    // (the block at the split with the first one as representative, else the block before it)
                    const int t0 = len > 1 ? first_key(mid) - (first_rule ? 0 : bk) : -1;
                    next_tab[d] = (uint32_t)t0;
                    touch(t0);
                    return;
                }
                uint32_t left, right;
                bool need_l, need_r;
                known_branches(rule, len, own, beg, left, right, need_l, need_r);
                const int tl = need_l ? first_key(rep_block(s, mid, rule)) : -1, tr = need_r ? first_key(rep_block(mid, s + len, rule)) : -1;
                if (next_one) {
                    next_tab[d] = (uint32_t)max(tl, tr);
                    touch(max(tl, tr));
                } else {
                    put_pair(next_tab, d, tl, tr);
                }
            };
            auto keep_child = [&](auto form, int i, bool keep_l, int dl, bool keep_r, int dr) __attribute__((always_inline)) {
                if (SPLIT && i % SW != wave) return;
                // a node of `len` blocks: len / 2 to the left, the rest to the right; m_len / 2 or one more
                const uint32_t bit = nd[i] & 1u, s2 = nd[i] & ~1u, len = (uint32_t)m_len + bit;
                const uint32_t own = HAND_ON ? own_of(i) : 0u, beg = beg_of(i);   // (own: what a right half begins with)
                if (keep_l) keep_one(form, dl, s2 | (odd ? bit : 0u), kl[i], beg);
                if (keep_r) keep_one(form, dr, (s2 + (len & ~1u)) | (odd ? 1u : bit), kr[i], own);
            };
            auto keep_all = [&](int i, bool keep_l, int dl, bool keep_r, int dr) __attribute__((always_inline)) { keep_child(std::integral_constant<int, 0>{}, i, keep_l, dl, keep_r, dr); };
            auto keep_own = [&](int i, bool keep_l, int dl, bool keep_r, int dr) __attribute__((always_inline)) { keep_child(std::integral_constant<int, 1>{}, i, keep_l, dl, keep_r, dr); };
            auto keep_any = [&](int i, bool keep_l, int dl, bool keep_r, int dr) __attribute__((always_inline)) { keep_child(std::integral_constant<int, 2>{}, i, keep_l, dl, keep_r, dr); };
            // four waves or one, E = 8: the registers that settling equal scores takes are the fourth wave of a SIMD (1024 paged
            // problems of k/bk = 256: 302 us with them, 247 without, 252 with the bits)
            constexpr int SEARCH = WS != 16 && E == 8 ? kInterpolate : default_search(E);
            if (round == ens_round) {
                // the selection sees the perturbed scores; kl and kr keep the true ones (they are what a later round carries)
                uint32_t pl[H], pr[H];
#pragma unroll
                for (int i = 0; i < H; ++i) {
                    const int s = (int)(nd[i] >> 1), e = s + m_len + (int)(nd[i] & 1), mid = s + ((e - s) >> 1);
                    pl[i] = ens_key(kl[i], ens_hash, rep_block(s, mid, rule), p.ens_r);
                    pr[i] = ens_key(kr[i], ens_hash, rep_block(mid, e, rule), p.ens_r);
                }
                select_topk_pairs<H, SEARCH>(pl, pr, kb, keep_any);
            } else if (next_knows) {   // (HAND_ON: also after the last round)
                if constexpr (HAND_ON) select_topk_pairs<H, SEARCH>(kl, kr, kb, keep_any);
                else select_topk_pairs<H, SEARCH>(kl, kr, kb, keep_own);
            } else {
                select_topk_pairs<H, SEARCH>(kl, kr, kb, keep_all);
            }
        }
        m_len = m_next;
        cur ^= 1;
        knows = next_knows;
        one_each = next_one;
        sync_problem();
        if (selects) {
#pragma unroll
            for (int i = 0; i < H; ++i) nd[i] = nodes[i * 64 + lane];
        }
    }

    for (int j = tix; j < kb; j += tn) out[j] = first_key((int)(nodes[j] >> 1));
}

// contiguous keys of a (sequence, kv head) within the reach of 24-bit row numbers and 31-bit offsets
static inline bool narrow_slice(const KParams &p)
{
    return !p.page_table && p.max_kv_len < (1 << 24) && p.ks_r * 2 < (1 << 24) && (int64_t)p.max_kv_len * p.ks_r * 2 < (1LL << 31);
}

template <int BK, int D, int ROWS, int WS>
static hipError_t launch_r(const KParams &p, dim3 grid, int xcd_map, hipStream_t st)
{
    dim3 block(WS == 16 ? 1024 : kThreads);
    const bool narrow = narrow_slice(p);
#define HIPATTN_LAUNCH_FORM(EV, OWN)                                                                        \
    do {                                                                                                    \
        if (p.page_table) hipLaunchKernelGGL((mask_decode_kernel<EV, BK, D, ROWS, 1 + OWN, WS>), grid, block, 0, st, p, xcd_map);  \
        else if (narrow) hipLaunchKernelGGL((mask_decode_kernel<EV, BK, D, ROWS, 0 + OWN, WS>), grid, block, 0, st, p, xcd_map);   \
        else if constexpr (WS > 1) hipLaunchKernelGGL((mask_decode_kernel<EV, BK, D, ROWS, 2 + OWN, WS>), grid, block, 0, st, p, xcd_map); \
        else return hipErrorInvalidValue;   /* (decode_mask_waves takes such a slice to four waves) */                \
    } while (0)
#define HIPATTN_LAUNCH(EV)                                                                                  \
    do {                                                                                                    \
        constexpr bool both = WS > 1 && (EV == 4 || EV == 8);                                                \
        if (both && p.rep_pos != 0) HIPATTN_LAUNCH_FORM(EV, (both ? kOwnAlone : 0));                          \
        else HIPATTN_LAUNCH_FORM(EV, 0);                                                                     \
    } while (0)
    // E registers of 64 branch slots: every count of the selection is a compare and a ballot per register, whether the
    // slots are in use or not (k/bk = 32, both with the bit search, four registers / two: 1024 problems of 65536 tokens
    // 54.2 / 48.8 us, 4096 of 8192 144 / 133)
    if (p.kb <= 64) HIPATTN_LAUNCH(2);
    else if (p.kb <= 128) HIPATTN_LAUNCH(4);
    else if (p.kb <= 256) HIPATTN_LAUNCH(8);
    else if (WS == 16 || p.kb <= 512) HIPATTN_LAUNCH(16);   // (sixteen waves: k/bk <= 512, 32 keys a lane do not fit their 128 registers)
    else if constexpr (WS != 16) HIPATTN_LAUNCH(32);
#undef HIPATTN_LAUNCH
#undef HIPATTN_LAUNCH_FORM
    return hipGetLastError();
}

template <int BK, int D>
static hipError_t launch_e(const KParams &p, hipStream_t st)
{
    const int64_t problems = (int64_t)p.batch * p.hq;
    const int64_t groups = (int64_t)p.batch * p.hkv;
    const int xcd_map = groups % 8 == 0 ? 1 : 0;
    const dim3 grid((unsigned)problems);
    constexpr int ROWS = BK < 4 ? 4 : BK, STEP = 512 / D * (ROWS / BK);   // branches per stage of a wave
    const Slice slice = p.page_table ? Slice::paged : narrow_slice(p) ? Slice::narrow : Slice::wide;
    const int waves = decode_mask_waves(problems, p.kb, D, STEP, 512 / D * (8 / BK), slice);
    if (waves == 16) return launch_r<BK, D, ROWS, 16>(p, grid, xcd_map, st);
    if (waves == 4) return launch_r<BK, D, 8, 4>(p, grid, xcd_map, st);
    return launch_r<BK, D, 8, 1>(p, dim3((unsigned)((problems + 3) / 4)), 0, st);
}

// One translation unit per (head dim, block width) instantiates this: WIDE = 4 or 8 scored rows per block, else 1 or 2.
template <int D, bool WIDE> hipError_t launch_mask_decode_variant(const KParams &p, hipStream_t st)
{
    if ((int64_t)p.batch * p.hq == 0) return hipSuccess;
    const int rows = p.bk / p.b_sk;
    if constexpr (WIDE) return rows == 4 ? launch_e<4, D>(p, st) : launch_e<8, D>(p, st);
    else return rows == 1 ? launch_e<1, D>(p, st) : launch_e<2, D>(p, st);
}

}  // namespace hipattn
