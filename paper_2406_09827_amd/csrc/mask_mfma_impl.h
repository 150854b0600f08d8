// Hierarchical mask estimation for bf16 prefill on CDNA4 matrix cores
// (paper Alg. 1; the block approximation of Sec. 3.2 is what makes the branch scoring a
// dense query-block x gathered-key-rows contraction).
//
// Work item = one WAVE = one (sequence, query head, query block), four per workgroup; with few work items a workgroup.
//   * The query block (<= 64 rows) sits in registers as the MFMA A operand.
//   * A round scores 2*kb branches = 2*kb*bk gathered key rows in tiles of 32 rows.  The rows go from memory
//     straight into LDS (buffer_load ... lds), COALESCED (a row = D/8 consecutive lanes x 16 bytes, so the address unit sees
//     whole cache lines instead of 64 separate ones), with an XOR swizzle applied to the chunk a lane fetches, and are
//     read back in the MFMA B-operand layout (lane l: row l % 32, 16-byte chunk l / 32 of each 32-byte step) without
//     bank conflicts.  A loading lane finds the rows it loads with ONE read of the table of blocks to score (its
//     rows belong to consecutive entries), issued a tile ahead, so no LDS round trip sits between two tiles.
//   * Sampling strides b_sq / b_sk (powers of two) shrink the operand tiles: only the sampled query
//     rows are loaded into the A operand, only the sampled key rows of a block are gathered.
//   * v_mfma_f32_32x32x16_bf16 gives a 32(query) x 32(key) score tile; the branch score is
//     the max over the admissible query rows (in-lane, then lanes l and l+32) and over the
//     bk keys of the block (neighbouring lanes, DPP).
//   * A block's score replaces its table entry, so a wave's whole state is the table (2 KB for 512 branches) and a tile.
//     With that and 128 registers four waves fit a SIMD, which is what the loop lives on: a wave has one tile in flight,
//     and its own chain (operands from LDS, multiplies one after the other, reduction) is long.
//   * A branch whose representative block was scored in an earlier round keeps that score (known_branches in common.h): with the centre as
//     representative most branches of the last round, and those of two or three blocks in the one before it; with the first or last block
//     one child of every node in every round after the first.  Such rounds score what is left from a compact list.  (Before, only the right halves
//     of two-block nodes in the last round did: 32k tokens 1.57 -> 1.36 ms, 128k 14.05 -> 12.2, a million 376 -> 343, 32 draft
//     rows over 12k tokens 96 times 0.59 -> 0.51.)
//   * A lane holds nodes and their two scores each; the wave runs the ordered threshold selection, writes the surviving
//     nodes compacted to LDS and, per surviving node, the representative blocks of its two branches into the table.
// Nodes are ranges of block indices; the list stays sorted by position throughout, which
// is why the result needs no sort.
// Measured, 32 query heads over 8 kv heads, d = 128, k = 512, bq = 32, bk = 2, against the form before (registers and
// ds_write, or straight into LDS with three waves a SIMD): 8k tokens 245 -> 217 us, 32k 1742 -> 1568; k = 2048 5929 -> 3864; bq = 64
// 1701 -> 1076; 16 heads of 64 channels, 16k tokens, bq = 64, bk = 4 159 -> 106.  By the clock, 32k tokens, sixteen waves a
// compute unit: 60000 clocks for the 32 tiles of a full round (1870 a tile; the multiplies take 256 of a SIMD's for each of its four waves),
// 45000 for the shared first one, 3000 each for the last two, 8500 for a round's selection and survivors.
#pragma once
#include "common.h"
#include "launch.h"

namespace hipattn {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float f32x16;

// max over lanes l and l ^ 32 (both get it)
__device__ __forceinline__ float max_half_swap(float v)
{
    const unsigned u = __float_as_uint(v);
    auto r = __builtin_amdgcn_permlane32_swap(u, u, false, false);
    return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}

// MT = 32-row query tiles (1 or 2), E = branch slots / 64, D = head dim,
// LB = log2(key rows scored per block) = log2(bk / b_sk)
// WPI: waves per work item.  1: four work items per workgroup, a wave each.  4: the workgroup takes ONE work item; its
// waves share the node state, score a quarter of the tiles each and run the selection redundantly (for launches
// with too few work items to fill the GPU wave by wave)
// SHARE (with WPI = 1): the four waves of a workgroup are four query heads of ONE (sequence, kv head, query block).  In
// the first round they all score the same representative blocks (the initial nodes depend on the lengths only), so they
// go through that round in step: every tile is loaded once, a quarter of it by each wave, and read by all of them.
// HAND_ON: nodes hand on what they know of their own and of their first block's score in every round; without it a node's own score alone, and
// only to a round with one branch a node to score (below).
template <int MT, int E, int D, bool PAGED, int LB, int WPI, bool SHARE, bool HAND_ON>
__device__ __forceinline__ void mask_mfma_body(const KParams &p, int xcd_map)
{
    static_assert(WPI == 1 || (WPI == 4 && !SHARE), "a wave or a workgroup per work item");
    static_assert(!(SHARE && PAGED), "shared first round: contiguous keys");
    constexpr bool SPLIT = WPI > 1;
    constexpr int NB = 64 * E;     // branch slots
    constexpr int KS = D / 16;     // MFMA k-steps per key row
    constexpr int BK = 1 << LB;    // key rows scored per representative block
    constexpr int EPT = 32 >> LB;  // table entries (blocks) per tile
    constexpr int CPR = D / 8;     // 16-byte chunks per key row
    constexpr int RPI = 64 / CPR;  // rows per wave-wide load
    constexpr int NLD = 32 / RPI;  // rows (= loads) per lane and tile
    constexpr int SPL = NLD > BK ? NLD >> LB : 1; // table entries a loading lane's rows belong to
    constexpr int ROWB = D * 2;    // bytes per row
    constexpr int TILEB = 32 * ROWB;
    constexpr int NS = SPLIT ? 1 : 4;  // copies of the per-work-item state
    // LDS, carved by hand: the tile buffers come first (the LDS address of a direct load travels in M0 and stays below
    // 64 KB), then per work item the table and, over a paged pool, the page of every entry's block.  The nodes lie over
    // the wave's tile buffer between two rounds and in registers during one (SPLIT: in an array of their own, with two more for
    // what they know).
    constexpr int kOffTab = 4 * TILEB, kOffPg = kOffTab + NS * NB * 4, kOffNode = kOffPg + (PAGED ? NS * NB * 4 : 0);
    __shared__ __attribute__((aligned(1024))) char lds[kOffNode + (SPLIT ? NB * (HAND_ON ? 6 : 2) : 0)];
    static_assert(4 * TILEB <= 65536 && NB * 2 <= TILEB, "LDS layout");

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int col = lane & 31, hh = lane >> 5;

    // ---- which (sequence, head, query block) this wave owns.  With `xcd_map` the workgroups an
    // XCD receives (blockIdx.x % 8) all read the same KV head; query blocks go from the longest
    // prefix down, the query heads of a KV group are adjacent.
    const uint32_t groups = (uint32_t)p.batch * (uint32_t)p.hkv;
    const uint32_t per_group = (uint32_t)p.g * (uint32_t)p.nqb;
    uint32_t group, o;
    if (!place_item(xcd_map, blockIdx.x, SPLIT ? 1 : 4, SPLIT ? 0 : wave, per_group, groups, group, o)) return;
    const uint32_t oq = o / (uint32_t)p.g;
    const int qb = p.nqb - 1 - (int)oq;
    const int b = (int)(group / (uint32_t)p.hkv), hk = (int)(group - (uint32_t)b * (uint32_t)p.hkv);
    const int h = hk * p.g + (int)(o - oq * (uint32_t)p.g);
    const int kb = p.kb;
    // sampling strides of the block score are powers of two here: key row n of a block is its key
    // n << ks (ks = log2 b_sk), query row i of the operand is row i << qs of the block (qs = log2 b_sq)
    const int ks = __builtin_ctz(p.b_sk), qs = __builtin_ctz(p.b_sq);
    const int lbk = LB + ks;  // log2(bk)

    const int kv_len = p.kv_lens ? p.kv_lens[b] : p.max_kv_len;
    const int row0 = qb * p.bq;
    const int n_rows = min(p.bq, p.q_len - row0);
    const int n_eff = (n_rows + p.b_sq - 1) >> qs;  // sampled query rows
    const int pos0 = kv_len - p.q_len + row0;
    const int L = min(kv_len, pos0 + n_rows);
    int32_t *out = p.idx_out + (((int64_t)b * p.hq + h) * p.nqb + qb) * kb;

    const int Tb = L > 0 ? (L + p.bk - 1) >> lbk : 0;
    const int tix = SPLIT ? tid : lane;
    constexpr int TN = SPLIT ? kThreads : 64;
    if (Tb <= kb) {
        for (int j = tix; j < kb; j += TN) out[j] = j < Tb ? j << lbk : kSentinel;
        return;
    }

    // query block as MFMA A operand: lane holds row (lane % 32) [+32], 8 channels per k-step.  Operand rows past the sampled rows of the
    // block repeat the last one: a repeated row cannot change a maximum, so tiles that need no causal masking take the short
    // reduction whatever the number of rows.  One tile travels like a key tile, through the wave's tile buffer, and lands while
    // the initial nodes are laid out, where that is the faster way (straight into registers, a row a lane, each of its
    // loads is 64 cache accesses).  Measured, 32 heads, bk = 2, registers / buffer, us: a workgroup per item, the last 256 rows of 4
    // sequences over pages, k/bk = 256 54.4 / 52.1; a wave per item, 3k tokens: 64 channels, k/bk = 64 25.4 / 24.5 (16-row blocks 37.7 /
    // 33.5); 128 channels, k/bk = 256 50.1 / 49.0, but 32 27.4 / 28.1, 64 32.1 / 32.7 (16-row blocks 56.8 / 61.4), 512 57.7 / 58.1, 1024 99.5 / 102.2.
    constexpr bool QLDS = MT == 1 && (SPLIT || PAGED || D == 64 || E == 8);
    const int lg = lane / CPR, lc = lane % CPR;  // loading role: tile rows lg*NLD .. +NLD-1, chunk lc
    const uint32_t chunk0 = (uint32_t)((lc ^ ((lg * NLD) & (CPR - 1))) << 4);
    const uint32_t ring0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char *)lds, ring = ring0 + wave * TILEB;
    bf16x8 qf[MT][KS];
    {
        const bf16_t *Qb = (const bf16_t *)p.Q + (int64_t)b * p.qs_b + (int64_t)h * p.qs_h + (int64_t)row0 * p.qs_r;
        if constexpr (QLDS) {
#pragma unroll
            for (int j = 0; j < NLD; ++j) {
                const char *src = (const char *)(Qb + (int64_t)(min(lg * NLD + j, n_eff - 1) << qs) * p.qs_r) + (chunk0 ^ (uint32_t)(j << 4));
                const uint32_t dst = __builtin_amdgcn_readfirstlane(ring + j * 1024);
                asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off" :: "v"(src), "s"(dst) : "memory", "m0");
            }
        } else {
#pragma unroll
            for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                for (int kk = 0; kk < KS; ++kk) {
                    const uint4 v = *(const uint4 *)(Qb + (int64_t)(min(mt * 32 + col, n_eff - 1) << qs) * p.qs_r + kk * 16 + hh * 8);
                    qf[mt][kk] = __builtin_bit_cast(bf16x8, v);
                }
        }
    }

    char *tile_s = lds + wave * TILEB;
    // The table.  While a round is scored, entry i is the first key of the i-th block to score (-1: none); the score of a
    // block replaces its entry (as the bits of the float; an empty entry stays -1, which score_key_bits maps to 0).
    uint32_t *tab = (uint32_t *)(lds + kOffTab) + (SPLIT ? 0 : wave) * NB;
    int *tpg = (int *)(lds + kOffPg) + (SPLIT ? 0 : wave) * NB;
    // Nodes, sorted by position.  All of a round's nodes are m or m + 1 blocks long (chunks differ by one, and so do
    // halves of lengths that differ by one: the next m is m / 2), so a node is its first block and one bit.
    uint32_t *nodes = SPLIT ? (uint32_t *)(lds + kOffNode) : (uint32_t *)tile_s;
    // (page sizes are powers of two here)
    const int *ptab = PAGED ? p.page_table + (int64_t)b * p.max_pages : nullptr;
    const int pg0 = PAGED ? ptab[0] : 0;  // empty entries load key 0
    auto set_entry = [&](int i, int t0) __attribute__((always_inline)) {
        tab[i] = (uint32_t)t0;
        if (PAGED) tpg[i] = t0 >= 0 ? ptab[t0 >> p.page_shift] : pg0;
        if (PAGED && p.touched && t0 >= 0) touch_page(p, b, t0);
    };
    // the waves of a work item meet here (SPLIT); otherwise the point only orders one wave's LDS traffic
    auto sync_unit = [&]() __attribute__((always_inline)) {
        if (SPLIT) __syncthreads(); else wave_lds_sync();
    };
    // the two branches of node [s, e): left [s, mid) (empty for a one-block node), right [mid, e)
    const RepRule rule = rep_rule(p.rep_pos);
    auto put_branches = [&](int j, int s, int e) __attribute__((always_inline)) {
        const int mid = s + ((e - s) >> 1);
        set_entry(2 * j, mid > s ? rep_block(s, mid, rule) << lbk : -1);
        set_entry(2 * j + 1, rep_block(mid, e, rule) << lbk);
    };
    int m_len = Tb / kb;
    uint32_t nd[E / 2];  // the nodes, in registers while the tiles pass through the buffers
    {
        const int r = Tb % kb;
        auto first_node = [&](int j) __attribute__((always_inline)) {
            const int s = chunk_bound(j, m_len, r, kb, p.kb_magic), e = chunk_bound(j + 1, m_len, r, kb, p.kb_magic);
            put_branches(j, s, e);
            return (uint32_t)(s << 1 | (e - s - m_len));
        };
        if constexpr (SPLIT) {
            for (int j = tix; j < kb; j += TN) {
                nodes[j] = first_node(j);
                if (HAND_ON) nodes[NB / 2 + j] = nodes[NB + j] = 0u;   // (own_s, beg_s)
            }
        } else {
#pragma unroll
            for (int i = 0; i < E / 2; ++i) nd[i] = i * 64 + lane < kb ? first_node(i * 64 + lane) : 0u;
        }
        for (int i = 2 * kb + tix; i < NB; i += TN) set_entry(i, -1);
    }
    sync_unit();

    // Contiguous keys: row 0 of this sequence / kv head as a buffer whose size ends with the last key.  A load past it (an
    // empty entry, a row past the end in the last block) is dropped by the address unit, so the loop has no clamps.
    // The slice address is the same in every lane; saying so (readfirstlane) makes it scalar (the launcher checks that
    // rows and row pitch fit 24 bits and the slice 31).
    const uint32_t row_bytes = (uint32_t)p.ks_r * 2u;
    const int64_t slice = ((int64_t)b * p.ks_b + (int64_t)hk * p.ks_h) * 2;  // bytes
    const uint64_t kbase = (uint64_t)((const char *)p.K + slice);
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
    const u32x4 srd = {(uint32_t)__builtin_amdgcn_readfirstlane((int)kbase), (uint32_t)__builtin_amdgcn_readfirstlane((int)(kbase >> 32)) & 0xffffu,
                       (uint32_t)__builtin_amdgcn_readfirstlane((int)((uint32_t)(kv_len - 1) * row_bytes + (uint32_t)ROWB)), 0x00020000u};
    // paged layout: this kv head's rows of page 0, and the pitch of a page
    const int64_t head_off = (int64_t)hk * p.ks_h * 2;
    const char *Kpool = (const char *)p.K + (((int64_t)__builtin_amdgcn_readfirstlane((int)(head_off >> 32)) << 32) |
                                             (uint32_t)__builtin_amdgcn_readfirstlane((int)head_off));
    const char *Kpool_back = (const char *)p.Kback + (Kpool - (const char *)p.K);
    const uint32_t page_bytes = (uint32_t)p.ks_b * 2u;

    // What a loading lane has to know of a tile: its table entries and, with a page table, their pages.
    struct meta_t { int m[SPL]; int pg[PAGED ? SPL : 1]; };
    auto read_entries = [&](const int *src, int (&m)[SPL]) __attribute__((always_inline)) {
        if (SPL == 1) m[0] = src[0];
        else if (SPL == 2) { const int2 v = *(const int2 *)src; m[0] = v.x; m[1 % SPL] = v.y; }
        else {
#pragma unroll
            for (int i = 0; i < SPL; i += 4) {
                const int4 v = *(const int4 *)(src + i);
                m[i % SPL] = v.x; m[(i + 1) % SPL] = v.y; m[(i + 2) % SPL] = v.z; m[(i + 3) % SPL] = v.w;
            }
        }
    };
    auto read_meta = [&](int tile, meta_t &mt_) __attribute__((always_inline)) {
        const int at = tile * EPT + ((lg * NLD) >> LB);
        read_entries((const int *)tab + at, mt_.m);
        if constexpr (PAGED) read_entries(tpg + at, mt_.pg);
    };
    // Load j of a tile: memory straight into LDS (lane l's 16 bytes land at M0 + 16 l, no staging register, no ds_write).
    // It fills LDS rows RPI j .. RPI j + RPI - 1; lane group lg supplies tile row lg * NLD + j (the rows a lane loads belong
    // to consecutive table entries), so tile row r sits in LDS row RPI (r % NLD) + r / NLD, and the XOR swizzle that
    // keeps the operand reads free of bank conflicts is applied to the global chunk a lane fetches.  The loads and their
    // waits are inline assembly: the compiler neither sees that they write LDS nor counts them, and no other vector
    // memory instruction is issued inside a tile loop.  (M0 is a reserved register: the compiler warns that it does not
    // track the clobber.  It is written and consumed inside one asm statement, and nothing else in these kernels uses M0.)
    const int last = kv_len - 1;
    auto issue_row = [&](const meta_t &mt_, uint32_t buf, int j) __attribute__((always_inline)) {
        const int i = SPL == 1 ? 0 : j >> LB;
        const int rho = lg * NLD + j, n = rho & (BK - 1);
        uint32_t chunk = chunk0;
        asm volatile("" : "+v"(chunk));   // (not a register per load)
        chunk ^= (uint32_t)(j << 4);
        const uint32_t dst = __builtin_amdgcn_readfirstlane(buf + j * 1024);
        if constexpr (PAGED) {
            // page base (the resident pool, or the backing pool for a negative entry) plus a 32-bit offset inside the page
            const int tf = max(mt_.m[i], 0);
            const uint32_t r = (uint32_t)((tf & (p.page_size - 1)) + min(tf + (n << ks), last) - tf);
            const char *src = (mt_.pg[i] < 0 ? Kpool_back : Kpool) + (uint64_t)(uint32_t)page_in_pool(mt_.pg[i]) * page_bytes +
                              (__umul24(r, row_bytes) + chunk);
            asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off"
                         :: "v"(src), "s"(dst) : "memory", "m0");
        } else {
            // an empty entry becomes an offset far past the end whatever the row pitch
            const uint32_t off = mt_.m[i] < 0 ? 0x80000000u : __umul24((uint32_t)mt_.m[i], row_bytes);
            const uint32_t voff = off + __umul24((uint32_t)(n << ks), row_bytes) + chunk;
            asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tbuffer_load_dwordx4 %0, %1, 0 offen lds"
                         :: "v"(voff), "s"(srd), "s"(dst) : "memory", "m0");
        }
    };
    // operands of the tile in `buf` (aligned to ROWB): tile row `col` sits in LDS row RPI (col % NLD) + col / NLD
    typedef __attribute__((address_space(3))) const u32x4 *lds_u32x4_ptr;
    const uint32_t op0 = (uint32_t)((RPI * (col % NLD) + col / NLD) * ROWB + ((hh ^ (col & (CPR - 1))) << 4));
    auto read_operands = [&](uint32_t buf, u32x4 (&kv)[KS]) __attribute__((always_inline)) {
        uint32_t base = buf + op0;
        asm volatile("" : "+v"(base));   // (one register and eight exclusive-ors instead of eight registers)
#pragma unroll
        for (int kk = 0; kk < KS; ++kk) kv[kk] = *(lds_u32x4_ptr)(uintptr_t)(base ^ (uint32_t)(kk << 5));
    };

    // Branch score from a tile of products: max over the admissible query rows of this lane's key column, then over the
    // block's columns; t0 is the block's first key (-1: empty), `at` its table entry.
    const uint32_t first_masked = (uint32_t)max(pos0 + 1, 0);  // keys from here on lie in some row's future
    const bool writes = hh == 0 && (col & (BK - 1)) == 0;
    auto score_finish = [&](const f32x16 (&acc)[MT], int t0, uint32_t *at) __attribute__((always_inline)) {
        const int t = t0 + ((col & (BK - 1)) << ks);
        float v;
        const bool masked = __ballot((uint32_t)t >= first_masked) != 0;   // (also an empty entry: its first lane has t = -1)
        if (!masked) {
            float w[MT][4];
#pragma unroll
            for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                for (int g = 0; g < 4; ++g) w[mt][g] = fmaxf(fmaxf(acc[mt][4 * g], acc[mt][4 * g + 1]), fmaxf(acc[mt][4 * g + 2], acc[mt][4 * g + 3]));
            v = fmaxf(fmaxf(w[0][0], w[0][1]), fmaxf(w[0][2], w[0][3]));
            if constexpr (MT == 2) v = fmaxf(v, fmaxf(fmaxf(w[MT - 1][0], w[MT - 1][1]), fmaxf(w[MT - 1][2], w[MT - 1][3])));
        } else {
            // operand rows below lo would look into the future, those from hi on repeat another (register r: row
            // 8 (r / 4) + r % 4 + 4 hh)
            const int lo = ((t - pos0 + p.b_sq - 1) >> qs) - 4 * hh, hi = n_eff - 4 * hh;
            v = -INFINITY;
#pragma unroll
            for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const int i = mt * 32 + (r >> 2) * 8 + (r & 3);
                    if (i >= lo && i < hi) v = fmaxf(v, acc[mt][r]);
                }
            if (t > last) v = -INFINITY;
        }
        v = max_half_swap(v);
        if (LB >= 1) v = fmaxf(v, dpp_f<0xB1>(v));  // lane ^ 1
        if (LB >= 2) v = fmaxf(v, dpp_f<0x4E>(v));  // lane ^ 2
        if (LB >= 3) v = fmaxf(v, dpp_f<0x141>(v)); // lane i <-> 7 - i of each 8 lanes: the other quad (quads are uniform by now)
        if (writes) *at = masked && t0 < 0 ? 0xffffffffu : score_bits(v);
    };

    static_assert(NLD == KS, "one load per k-step");
    const f32x16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    if constexpr (QLDS) {
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        u32x4 qv[KS];
        read_operands(ring, qv);
#pragma unroll
        for (int kk = 0; kk < KS; ++kk) qf[0][kk] = __builtin_bit_cast(bf16x8, qv[kk]);
    }
    // The query loads end here, where the compiler can see it: it does not count the loads that the tile loop
    // issues from inline assembly, and a wait for a query fragment left inside that loop would wait for them.
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int kk = 0; kk < KS; ++kk) asm volatile("" :: "v"(qf[mt][kk]));

    // Scores of earlier rounds: with a node go the keys of its own and its first block's score (known_branches).  A round that
    // profits from them runs from a compact list of what is left to score, node by node, left before right.  (Survivors take the
    // two along through the table, which is free while they are written; SPLIT: in arrays of their own.)
    // Not HAND_ON: with the first (last) block as representative every round after the first is a list of the right (left) branches of
    // nodes of two blocks and more, with the centre the last one, of left halves.  What a node knows is the score of its other branch, or of
    // itself alone; it lies in the upper half of the table, since the list has an entry a node.
    uint32_t *own_s = !HAND_ON ? tab + NB / 2 : SPLIT ? nodes + NB / 2 : tab, *beg_s = SPLIT ? own_s + NB / 2 : tab + kb;
    const bool first_rule = p.rep_pos == 1;
    bool list = false;
    int n_entries = 2 * kb;
    // ensemble sample: the round whose selection compares perturbed scores (-1: none)
    const int ens_round = ens_round_of(p.ens_sample, (Tb + kb - 1) / kb);
    const uint32_t ens_hash = ens_round >= 0 ? ens_unit_hash(p.ens_seed, p.ens_sample, b, h, qb) : 0u;
    int round = 0;
    constexpr bool IN_REGS = HAND_ON && !SPLIT;
    uint32_t own[IN_REGS ? E / 2 : 1], beg[IN_REGS ? E / 2 : 1];
#pragma unroll
    for (int i = 0; i < E / 2; ++i) {
        if constexpr (SPLIT) nd[i] = nodes[i * 64 + lane];
        if constexpr (IN_REGS) own[i] = beg[i] = 0u;
    }
    auto own_of = [&](int i) __attribute__((always_inline)) { return IN_REGS ? own[IN_REGS ? i : 0] : own_s[i * 64 + lane]; };
    auto beg_of = [&](int i) __attribute__((always_inline)) { return IN_REGS ? beg[IN_REGS ? i : 0] : beg_s[i * 64 + lane]; };
    auto known = [&](int i, uint32_t &left, uint32_t &right, bool &need_l, bool &need_r) __attribute__((always_inline)) {
        const int len = i * 64 + lane < kb ? m_len + (int)(nd[i] & 1) : 0;
        known_branches(rule, len, own_of(i), beg_of(i), left, right, need_l, need_r);
        return len;
    };
    for (int maxlen = (Tb + kb - 1) / kb; maxlen > 1; maxlen = (maxlen + 1) >> 1, ++round) {
        asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
        const int n_tiles = __builtin_amdgcn_readfirstlane((n_entries + EPT - 1) / EPT);
        if (SHARE && round == 0) {
            // Shared first round: every wave loads a quarter of tile t + 3 while tile t is scored.  One barrier per tile:
            // it says that tile t has landed (every wave waited for its share) and that every wave has the operands of
            // tile t - 1 in registers, so that its buffer may be refilled.  (Waves hold equal tables here.)
            constexpr int SH = NLD / 4;
            asm volatile("s_barrier" ::: "memory");   // every wave has its query tile out of its buffer, which the others now load into
            auto issue_share = [&](int t) __attribute__((always_inline)) {
                // load j = SH * wave + jj: the lane's row of load j
#pragma unroll
                for (int jj = 0; jj < SH; ++jj) {
                    const int j = SH * wave + jj, rho = lg * NLD + j;
                    const int t0 = (int)tab[t * EPT + (rho >> LB)];
                    const uint32_t chunk = (uint32_t)((lc ^ (rho & (CPR - 1))) << 4);
                    const uint32_t dst = __builtin_amdgcn_readfirstlane(ring0 + (t & 3) * TILEB + j * 1024);
                    const uint32_t off = t0 < 0 ? 0x80000000u : __umul24((uint32_t)(t0 + ((rho & (BK - 1)) << ks)), row_bytes);
                    const uint32_t voff = off + chunk;
                    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tbuffer_load_dwordx4 %0, %1, 0 offen lds"
                                 :: "v"(voff), "s"(srd), "s"(dst) : "memory", "m0");
                }
            };
            for (int t = 0; t < min(3, n_tiles); ++t) issue_share(t);
            for (int t = 0; t < n_tiles; ++t) {
                // the shares of tiles t+1 and t+2 may still be on their way
                if (t + 2 < n_tiles) asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" :: "i"(2 * SH) : "memory");
                else if (t + 1 < n_tiles) asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" :: "i"(SH) : "memory");
                else asm volatile("s_waitcnt vmcnt(0)\n\ts_barrier" ::: "memory");
                u32x4 kv[KS];
                read_operands(ring0 + (t & 3) * TILEB, kv);
                uint32_t *at = tab + t * EPT + (col >> LB);
                const int t0 = (int)*at;
                if (t + 3 < n_tiles) issue_share(t + 3);
                asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // (before the next barrier lets the buffer be refilled)
                f32x16 acc[MT];
#pragma unroll
                for (int kk = 0; kk < KS; ++kk)
#pragma unroll
                    for (int mt = 0; mt < MT; ++mt)
                        acc[mt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(qf[mt][kk], __builtin_bit_cast(bf16x8, kv[kk]), kk == 0 ? zero : acc[mt], 0, 0, 0);
                score_finish(acc, t0, at);
            }
            // the nodes go back into the tile buffers next: not before every wave has read its last tiles
            asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
        } else {
            // SPLIT: wave w takes tiles w, w + 4, ...
            const int first_tile = SPLIT ? wave : 0;
            constexpr int STEP = SPLIT ? 4 : 1;
            if (first_tile < n_tiles) {
                // One buffer per wave: as soon as a tile's operands are in registers the buffer is refilled with the next
                // tile, which lands while this one is multiplied and scored.  The order is pinned: multiply k, then load k.
                meta_t ml;
                read_meta(first_tile, ml);
#pragma unroll
                for (int j = 0; j < NLD; ++j) issue_row(ml, ring, j);
                read_meta(min(first_tile + STEP, n_tiles - 1), ml);
                auto step = [&](int tile, bool more) __attribute__((always_inline)) {
                    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // the tile has landed
                    u32x4 kv[KS];
                    read_operands(ring, kv);
                    uint32_t *at = tab + tile * EPT + (col >> LB);
                    const int t0 = (int)*at;
                    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // operands are in registers: the buffer may be refilled
                    __builtin_amdgcn_sched_barrier(0);
                    f32x16 acc[MT];
#pragma unroll
                    for (int kk = 0; kk < KS; ++kk) {
#pragma unroll
                        for (int mt = 0; mt < MT; ++mt)
                            acc[mt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(qf[mt][kk], __builtin_bit_cast(bf16x8, kv[kk]), kk == 0 ? zero : acc[mt], 0, 0, 0);
                        if (more) issue_row(ml, ring, kk);
                        __builtin_amdgcn_sched_barrier(0);
                    }
                    if (more) read_meta(min(tile + 2 * STEP, n_tiles - 1), ml);
                    score_finish(acc, t0, at);
                };
                int tile = first_tile;
                for (; tile + STEP < n_tiles; tile += STEP) {
                    // The four heads stay together, so that their rows meet in the L2: they still share half of the nodes in
                    // the second round.  (32 heads, without / with the barrier: 4k tokens 78.1 / 77.8 us, 32k 1582 / 1581, 48k 2883 /
                    // 2852, 64k 4705 / 4533, 128k 15.0 / 14.3 ms; 64 channels, 128k 5935 / 5888)
                    if (SHARE && (tile & 7) == 0 && !list) asm volatile("s_barrier" ::: "memory");
                    step(tile, true);
                }
                step(tile, false);
            }
        }
        sync_unit();  // every score of the round is in place
        // Lane j % 64 holds node j and the scores of its two branches.
        const bool odd = m_len & 1;
        auto child_of = [&](uint32_t w, int &len, uint32_t &left, uint32_t &right) __attribute__((always_inline)) {
            // a node of `len` blocks: len / 2 to the left, the rest to the right; m_len / 2 or one more
            const uint32_t bit = w & 1u, s2 = w & ~1u;
            len = m_len + (int)bit;
            left = s2 | (odd ? bit : 0u);
            right = (s2 + (uint32_t)(len & ~1)) | (odd ? 1u : bit);
        };
        uint32_t kl[E / 2], kr[E / 2];   // keys of the left and the right branch
        if (list) {
            int n_before = 0;
#pragma unroll
            for (int i = 0; i < E / 2; ++i) {
                if constexpr (!HAND_ON) {
                    const int j = i * 64 + lane;
                    const bool two = j < kb && m_len + (int)(nd[i] & 1) > 1;
                    const uint64_t b2 = __ballot(two);
                    kr[i] = j < kb ? own_s[j] : 0u;
                    kl[i] = two ? score_key_bits(tab[n_before + lane_prefix_count(b2)]) : 0u;
                    if (first_rule && two) { const uint32_t x = kr[i]; kr[i] = kl[i]; kl[i] = x; }
                    n_before += __popcll(b2);
                    continue;
                }
                bool need_l, need_r;
                known(i, kl[i], kr[i], need_l, need_r);
                const uint64_t bl = __ballot(need_l), br = __ballot(need_r);
                const int at = n_before + lane_prefix_count(bl) + lane_prefix_count(br);
                if (need_l) kl[i] = score_key_bits(tab[at]);
                if (need_r) kr[i] = score_key_bits(tab[at + (need_l ? 1 : 0)]);
                n_before += __popcll(bl) + __popcll(br);
            }
        } else {
#pragma unroll
            for (int i = 0; i < E / 2; ++i) {
                const uint2 x = *(const uint2 *)(tab + 2 * (i * 64 + lane));
                kl[i] = score_key_bits(x.x);
                kr[i] = score_key_bits(x.y);
            }
        }
        // SPLIT: what the nodes know whose survivors this wave writes, before they are overwritten
        uint32_t own_w[(E / 2 + 3) / 4], beg_w[(E / 2 + 3) / 4];
        if constexpr (SPLIT && HAND_ON) {
#pragma unroll
            for (int i = 0; i < (E / 2 + 3) / 4; ++i) {
                const int j = min((i * 4 + wave) * 64 + lane, NB / 2 - 1);
                own_w[i] = own_s[j];
                beg_w[i] = beg_s[j];
            }
        }
        const bool next_list = HAND_ON ? round_knows_scores(p.rep_pos, m_len >> 1) : p.rep_pos != 0 || ((maxlen + 1) >> 1) == 2;
        sync_unit();   // (every wave has the scores)
        // Ordered top-kb selection; survivors go to their places in the node array, with the keys they know.
        auto keep_child = [&](int i, bool kl_, int dl, bool kr_, int dr) __attribute__((always_inline)) {
            if (SPLIT && i % WPI != wave) return;
            int len;
            uint32_t left, right;
            child_of(nd[i], len, left, right);
            if constexpr (!HAND_ON) {
                if (kl_) { nodes[dl] = left; if (next_list) own_s[dl] = kl[i]; }
                if (kr_) { nodes[dr] = right; if (next_list) own_s[dr] = kr[i]; }
                return;
            }
            const uint32_t o = SPLIT ? own_w[i / 4] : own[IN_REGS ? i : 0], f = SPLIT ? beg_w[i / 4] : beg[IN_REGS ? i : 0];
            if (kl_) { nodes[dl] = left; own_s[dl] = kl[i]; beg_s[dl] = f; }
            if (kr_) { nodes[dr] = right; own_s[dr] = kr[i]; beg_s[dr] = o; }
        };
        if (round == ens_round) {
            // the selection sees the perturbed scores; kl and kr keep the true ones (they are what a later round carries)
            uint32_t pl[E / 2], pr[E / 2];
#pragma unroll
            for (int i = 0; i < E / 2; ++i) {
                const int s = (int)(nd[i] >> 1), e = s + m_len + (int)(nd[i] & 1), mid = s + ((e - s) >> 1);
                pl[i] = ens_key(kl[i], ens_hash, rep_block(s, mid, rule), p.ens_r);
                pr[i] = ens_key(kr[i], ens_hash, rep_block(mid, e, rule), p.ens_r);
            }
            select_topk_pairs<E / 2>(pl, pr, kb, keep_child);
        } else {
            select_topk_pairs<E / 2>(kl, kr, kb, keep_child);
        }
        m_len >>= 1;
        sync_unit();
#pragma unroll
        for (int i = 0; i < E / 2; ++i) {
            nd[i] = nodes[i * 64 + lane];
            if constexpr (IN_REGS) { own[i] = own_s[i * 64 + lane]; beg[i] = beg_s[i * 64 + lane]; }
        }
        if (maxlen <= 2) break;   // every node is one block
        if constexpr (HAND_ON) wave_lds_sync();   // (they are in registers: the table's entries may be written)
        // the blocks that the next round scores
        if (!next_list) {
#pragma unroll
            for (int i = 0; i < E / 2; ++i) {
                const int j = i * 64 + lane, s = (int)(nd[i] >> 1);
                if (j < kb && (!SPLIT || i % WPI == wave)) put_branches(j, s, s + m_len + (int)(nd[i] & 1));
            }
            // (entries from 2 kb on have stayed empty)
        } else {
            int n_todo = 0;
#pragma unroll
            for (int i = 0; i < E / 2; ++i) {
                if constexpr (!HAND_ON) {
                    const int s = (int)(nd[i] >> 1), len = m_len + (int)(nd[i] & 1);
                    const bool two = i * 64 + lane < kb && len > 1;
                    const uint64_t b2 = __ballot(two);
                    if (two && (!SPLIT || i % WPI == wave)) set_entry(n_todo + lane_prefix_count(b2), (s + (len >> 1) - (first_rule ? 0 : 1)) << lbk);
                    n_todo += __popcll(b2);
                    continue;
                }
                uint32_t left, right;
                bool need_l, need_r;
                const int len = known(i, left, right, need_l, need_r);
                const uint64_t bl = __ballot(need_l), br = __ballot(need_r);
                const int at = n_todo + lane_prefix_count(bl) + lane_prefix_count(br);
                const int s = (int)(nd[i] >> 1), mid = s + (len >> 1);
                if (!SPLIT || i % WPI == wave) {
                    if (need_l) set_entry(at, rep_block(s, mid, rule) << lbk);
                    if (need_r) set_entry(at + (need_l ? 1 : 0), rep_block(mid, s + len, rule) << lbk);
                }
                n_todo += __popcll(bl) + __popcll(br);
            }
            // the rest of the last tile
            n_todo = __builtin_amdgcn_readfirstlane(n_todo);
            const int fill = n_todo + lane;
            if (lane < EPT && fill < ((n_todo + EPT - 1) & ~(EPT - 1))) set_entry(fill, -1);
            list = true;
            n_entries = n_todo;
        }
        sync_unit();
    }

#pragma unroll
    for (int i = 0; i < E / 2; ++i) {
        const int j = i * 64 + lane;
        if (j < kb && (!SPLIT || i % WPI == wave)) out[j] = (int)(nd[i] >> 1) << lbk;
    }
}

// Waves per SIMD that LDS and registers are laid out for: 10 KB of LDS per wave with up to 512 branch slots (8 KB of it the
// tile at head dim 128), which makes four; 1024 slots or a table of pages three, 2048 slots or 1024 with a table two.
// Two query tiles at head dim 128 and three waves spill.  64-row blocks, three waves / two without spills, us:
//   a workgroup per item over pages (1 to 6 registers with 256 slots, 3 to 13 with 512, 10 to 24 with 1024), the last 256 rows of 32 heads over 16k
//     tokens, bk = 4, k/bk = 512 124 / 74 (2048 rows 309 / 211), bk = 1 74 / 63, bk = 2 71 / 67, k/bk = 128 38.5 / 37.7: two;
//   a wave per item over pages (up to 12 with 256 slots, 11 to 22 with 512), the last 4096 rows of 4 sequences of 16k tokens, k/bk = 100 bk = 1
//     286 / 298, bk = 2 357 / 373, bk = 4 490 / 505, 256 445 / 453, 609 / 614, 858 / 865 (1024 slots: two fit): three;
//   contiguous, 512 slots (up to 11), 32 heads of 16k tokens in groups of four, k/bk = 256 bk = 1 282 / 291, bk = 2 376 / 391, bk = 4 527 / 553, without
//     groups 304 / 311, 424 / 425, 574 / 575: three;
//   contiguous, 1024 slots, k/bk = 512: in groups of four (28 to 40) bk = 1 457 / 424 (40k tokens 1494 / 1453), but bk = 2 557 / 573, bk = 4 721 / 749,
//     bk = 8 858 / 887: two for bk = 1; without groups (14 to 22) bk = 1 500 / 461, bk = 2 606 / 608, bk = 4 799 / 791, bk = 8 991 / 999, 24 heads of 12k
//     tokens in groups of three 267 / 238, 318 / 315, 439 / 384, 8 heads of 16k 169 / 134, 187 / 178, 238 / 234, 309 / 311: two.
// One tile, bk = 1 and 512 slots over pages, a workgroup per item spills 4 at four waves: 1024 rows 70 us, at three waves 89 (2 spilled then).
constexpr int mask_waves(int MT, int E, int D, bool PAGED, int LB, bool SPLIT, bool SHARE, bool HAND_ON)
{
    const int lds_wave = 32 * D * 2 + (SPLIT ? 64 * E : 256 * E) * (PAGED ? 2 : 1) + (SPLIT ? (HAND_ON ? 96 : 32) * E : 0);
    const int by_lds = (160 << 10) / (4 * lds_wave), by_regs = MT == 2 && D == 128 ? (E >= 32 || (PAGED && SPLIT) || (E == 16 && !SPLIT && (LB == 0 || !SHARE)) ? 2 : 3) : E >= 32 ? 2 : E >= 16 ? 3 : 4;
    return by_lds < by_regs ? by_lds : by_regs;
}
template <int MT, int E, int D, bool PAGED, int LB, int WPI, bool SHARE, bool HAND_ON>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(mask_waves(MT, E, D, PAGED, LB, WPI > 1, SHARE, HAND_ON)))) void mask_mfma_kernel(KParams p, int xcd_map)
{
    mask_mfma_body<MT, E, D, PAGED, LB, WPI, SHARE, HAND_ON>(p, xcd_map);
}

template <int MT, int E, int D, int LB, bool HAND_ON>
static hipError_t launch_mask_mfma_e(const KParams &p, int xcd_map, dim3 grid, bool split, bool one_sequence_per_workgroup, hipStream_t st)
{
    // (the four work items of a workgroup are then four heads of one query block: they share the first round's tiles)
    const bool share = one_sequence_per_workgroup && p.g % 4 == 0 && !p.page_table && !(p.flags & 2);
    const int per_cu = mask_workgroups_per_cu(p.max_kv_len, D, p.kv_lens == nullptr);
    const auto launch = [&](auto kernel, bool paged, bool split_) {
        const int lds = (split_ ? 1 : 4) * 256 * E * (paged ? 2 : 1) + 4 * 64 * D + (split_ ? (HAND_ON ? 384 : 128) * E : 0);
        const int pad = per_cu && !split_ ? (160 << 10) / per_cu - lds : 0;
        hipLaunchKernelGGL(kernel, grid, dim3(kThreads), (unsigned)(pad > 0 ? pad & ~1023 : 0), st, p, xcd_map);
        return hipGetLastError();
    };
    // the page-table variant is a separate instantiation: a table read in the row-offset code
    // would otherwise put a full memory wait into the contiguous path's load pipeline
    if (split) return p.page_table ? launch(mask_mfma_kernel<MT, E, D, true, LB, 4, false, HAND_ON>, true, true)
                                   : launch(mask_mfma_kernel<MT, E, D, false, LB, 4, false, HAND_ON>, false, true);
    if (p.page_table) {
        if constexpr (E < 32 || D == 64) return launch(mask_mfma_kernel<MT, E, D, true, LB, 1, false, HAND_ON>, true, false);
        return hipErrorInvalidValue;
    }
    return share ? launch(mask_mfma_kernel<MT, E, D, false, LB, 1, true, HAND_ON>, false, false)
                 : launch(mask_mfma_kernel<MT, E, D, false, LB, 1, false, HAND_ON>, false, false);
}
template <int MT, int D, int LB>
static hipError_t launch_mask_mfma_d(const KParams &p, int xcd_map, dim3 grid, bool split, bool one_seq, hipStream_t st)
{
    if (p.kb <= 128) return mask_hands_on(p.kb, D, 1 << LB, MT == 2, p.rep_pos) ? launch_mask_mfma_e<MT, 4, D, LB, true>(p, xcd_map, grid, split, one_seq, st)
                                                           : launch_mask_mfma_e<MT, 4, D, LB, false>(p, xcd_map, grid, split, one_seq, st);
    if (p.kb <= 256) return launch_mask_mfma_e<MT, 8, D, LB, true>(p, xcd_map, grid, split, one_seq, st);
    if (p.kb <= 512) return launch_mask_mfma_e<MT, 16, D, LB, true>(p, xcd_map, grid, split, one_seq, st);
    return launch_mask_mfma_e<MT, 32, D, LB, true>(p, xcd_map, grid, split, one_seq, st);
}

// One translation unit per key-block size instantiates this.
template <int LB> hipError_t launch_mask_mfma_lb(const KParams &p, hipStream_t st)
{
    const int64_t groups = (int64_t)p.batch * p.hkv;
    const int64_t per_group = (int64_t)p.g * p.nqb;
    const int64_t units = groups * per_group;
    if (units == 0) return hipSuccess;
    const bool one_tile = (p.bq + p.b_sq - 1) / p.b_sq <= 32;
    // groups worked on at a time: as many as keep the key rows in flight inside the memory-side cache
    const int gc = groups_at_a_time_of(groups, (int64_t)p.max_kv_len * p.d * 2, 160LL << 20);
    const bool split = mask_item_per_workgroup(units, p.kb, p.d, !one_tile, p.page_table != nullptr, groups, gc, p.max_kv_len);
    // Measured, 32 heads' worth of rows over 32k tokens, in linear order / so many groups at a time: three sequences of 2 kv heads (two at a
    // time) 383 / 316 us, six (four) 454 / 318, 12 heads in threes over 24 groups 956 / 574, over pages 915 / 613; but a wave per item
    // over pages, two of six at a time 294 / 318 (16k tokens): linear.
    const int xcd_map = !split && p.page_table && gc == 2 && groups > 2 ? 0 : gc;
    dim3 grid((unsigned)placed_workgroups(xcd_map, split ? 1 : 4, per_group, groups));
    // the four work items of a workgroup are consecutive items of one (sequence, kv head) group
    const bool one_seq = !split && per_group % 4 == 0;
    if constexpr (LB <= 2) {
        if (p.d == 64) return one_tile ? launch_mask_mfma_d<1, 64, LB>(p, xcd_map, grid, split, one_seq, st) : launch_mask_mfma_d<2, 64, LB>(p, xcd_map, grid, split, one_seq, st);
    }
    return one_tile ? launch_mask_mfma_d<1, 128, LB>(p, xcd_map, grid, split, one_seq, st) : launch_mask_mfma_d<2, 128, LB>(p, xcd_map, grid, split, one_seq, st);
}

}  // namespace hipattn
