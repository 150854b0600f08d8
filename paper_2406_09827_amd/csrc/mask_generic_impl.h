// Hierarchical mask estimation for any shape (paper Alg. 1, block form of Sec. 3.2): fp32, and the bf16 shapes the
// tuned kernels (mask_mfma_impl.h, mask_decode_impl.h) leave out.  Any bq <= 64, bk <= 16, k/bk <= 1024, sampling
// stride and representative, contiguous or paged K with any page size, prefill or decode.
//
// One workgroup (4 waves) per (sequence, query head, query block).  The block score is a contraction in fp32 as well,
// so it runs on the matrix cores: v_mfma_f32_16x16x4_f32 multiplies full fp32 operands into fp32 sums (bf16:
// v_mfma_f32_16x16x32_bf16).  In fp32 the matrix pipe (64 flop per clock and SIMD, twice the vector unit's
// rate without packed instructions) is the busiest unit, 52 % of the clocks by counter at 4096 tokens; a wave waits 80 % of its
// time, for it and for the gathered rows, which three waves per SIMD do not cover.  Everything else keeps off its way:
//   * The sampled query rows sit in registers as MT operand tiles of 16 rows (small query blocks do not pay for 32).
//   * The branches that need a score are put on a list (LDS: block position, row offset, branch slot); a child whose
//     representative is its node's own representative has the node's score and is not listed.  The key rows of the list
//     are gathered in tiles of 8 KB per wave: loaded coalesced one tile ahead into registers, written to the wave's LDS
//     tile with an XOR swizzle and read back as matrix operands (lane l: row l % 16, 16-byte chunk l / 16 of each
//     64 bytes; the order of the channels inside the contraction is free, so a chunk feeds four fp32 steps).
//   * A row's maximum over the admissible query rows goes to its branch's key with an LDS atomic maximum, which takes
//     any number of rows per block.
//   * Selection: the ordered threshold selection of common.h, run redundantly by the four waves.
// Measured, fp32, 32 query heads over 8 kv heads, T = 4096, k = 512, bq = 32, bk = 2, d = 128: 11.77 ms with
// vector-unit dot products and a shuffle per (row, key) before, 0.58 ms now = 99 TFLOP/s of the 152 a large fp32 matrix
// product reaches; T = 1024, one head, k = 128, bq = 16, d = 64: 187 -> 18 us (64 workgroups: latency; 20 us each with a
// pause between launches).
#pragma once
#include "mfma_generic.h"
#include "launch.h"

namespace hipattn {

// (waves per SIMD: two query tiles of 128 fp32 channels and k/bk <= 256 spill 4 to 8 registers at three waves; at two, with
// none spilled, 4096 tokens of 32 heads, k/bk = 256 take 636 us instead of 582, k/bk = 64 404 instead of 360)
template <typename T, int D, int E, int MT>
__global__ __launch_bounds__(kThreads, E > 16 ? 1 : (E > 8 || MT > 2) ? 2 : 3) void mask_generic_kernel(KParams p, int xcd_map, uint32_t rows_magic)
{
    constexpr int NB = 64 * E;             // branch slots (two per node)
    constexpr int ROWB = D * (int)sizeof(T);
    constexpr int CPR = ROWB / 16;         // 16-byte chunks per key row = lanes per row of a coalesced load
    constexpr int RPW = 64 / CPR;          // rows per wave-wide load
    constexpr int TILE = 8192 / ROWB;      // key rows per tile
    constexpr int KT = TILE / 16, CS = CPR / 4;
    typedef uint32_t stage_t __attribute__((ext_vector_type(32)));
    constexpr int SW = (CPR < 16 ? CPR : 16) - 1;
    __shared__ __attribute__((aligned(16))) uint4 tile_s[4][512];
    __shared__ int64_t loff[NB];           // list entry: element offset of its block's first row in K
    __shared__ int lt0[NB];                // ... position of that row
    __shared__ int lslot[NB];              // ... branch slot
    __shared__ uint32_t keys[NB];
    __shared__ int nds_s[2][NB / 2], nde_s[2][NB / 2];  // nodes [s, e) of this round and of the next
    __shared__ uint32_t ndk_s[2][NB / 2];  // ... score key of the branch that became the node
    __shared__ int n_list_s;

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r16 = lane & 15, lg = lane >> 4;
    const uint32_t groups = (uint32_t)p.batch * (uint32_t)p.hkv, per_group = (uint32_t)p.g * (uint32_t)p.nqb;
    uint32_t group, o;
    if (!place_item(xcd_map, blockIdx.x, 1, 0, per_group, groups, group, o)) return;
    const uint32_t oq = o / (uint32_t)p.g;
    const int qb = p.nqb - 1 - (int)oq;  // the longest prefix first
    const int b = (int)(group / (uint32_t)p.hkv), hk = (int)(group - (uint32_t)b * (uint32_t)p.hkv);
    const int h = hk * p.g + (int)(o - oq * (uint32_t)p.g);
    const int kb = p.kb, bk = p.bk, bsk = p.b_sk, bsq = p.b_sq;
    const int rpb = bk / bsk;              // key rows scored per block

    const int kv_len = p.kv_lens ? p.kv_lens[b] : p.max_kv_len;
    const int row0 = qb * p.bq;
    const int n_rows = min(p.bq, p.q_len - row0);
    const int n_eff = (n_rows + bsq - 1) / bsq;  // sampled query rows
    const int pos0 = kv_len - p.q_len + row0;
    const int L = min(kv_len, pos0 + n_rows);  // visible prefix of this query block
    int32_t *out = p.idx_out + (((int64_t)b * p.hq + h) * p.nqb + qb) * kb;

    const int Tb = L > 0 ? (L + bk - 1) / bk : 0;
    if (Tb <= kb) {  // nothing to prune: every visible block is selected
        for (int j = tid; j < kb; j += kThreads) out[j] = j < Tb ? j * bk : kSentinel;
        return;
    }

    // sampled query rows as A operands; rows past the last one repeat it (that cannot change a maximum)
    uint4 qf[MT][CS];
    {
        const T *Qb = (const T *)p.Q + (int64_t)b * p.qs_b + (int64_t)h * p.qs_h + (int64_t)row0 * p.qs_r;
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) {
            const char *src = (const char *)(Qb + (int64_t)(min(mt * 16 + r16, n_eff - 1) * bsq) * p.qs_r) + lg * 16;
#pragma unroll
            for (int cs = 0; cs < CS; ++cs) qf[mt][cs] = *(const uint4 *)(src + cs * 64);
        }
    }

    // initial nodes: kb chunks of [0, Tb) with rounded bounds; all non-empty because Tb > kb
    const int a = Tb / kb, r = Tb % kb;
    for (int j = tid; j < kb; j += kThreads) {
        nds_s[0][j] = chunk_bound(j, a, r, kb);
        nde_s[0][j] = chunk_bound(j + 1, a, r, kb);
    }
    if (tid == 0) n_list_s = 0;
    for (int i = 2 * kb + tid; i < NB; i += kThreads) keys[i] = 0u;
    __syncthreads();

    const T *Kbase = (const T *)p.K;
    const int64_t back_delta = (const T *)p.Kback - Kbase;  // elements from the resident pool to the backing pool
    char *tile = (char *)tile_s[wave];

    // ensemble sample: the round whose selection compares perturbed scores (-1: none)
    const int ens_round = ens_round_of(p.ens_sample, a + (r ? 1 : 0));
    const uint32_t ens_hash = ens_round >= 0 ? ens_unit_hash(p.ens_seed, p.ens_sample, b, h, qb) : 0u;
    int round = 0;
    // maxlen bounds the longest node
    for (int maxlen = a + (r ? 1 : 0); maxlen > 1; maxlen = (maxlen + 1) >> 1, ++round) {
        const int *nd_s = nds_s[round & 1], *nd_e = nde_s[round & 1];
        const uint32_t *nd_key = ndk_s[round & 1];
        // split every node into its left and right branch (slots 2j, 2j+1; left may be empty) and list the blocks to score
        for (int base = wave * 64; base < 2 * kb; base += kThreads) {
            const int slot = base + lane;
            bool todo = false;
            int blk = 0;
            if (slot < 2 * kb) {
                const int s = nd_s[slot >> 1], e = nd_e[slot >> 1], mid = s + ((e - s) >> 1);
                const int bs = (slot & 1) ? mid : s, be = (slot & 1) ? e : mid;
                uint32_t k0 = 0u;  // an empty branch
                if (be > bs) {
                    blk = rep_block(bs, be, p.rep_pos);
                    todo = round == 0 || blk != rep_block(s, e, p.rep_pos);
                    // a real branch starts at "-inf" (it may end up without an admissible pair)
                    k0 = todo ? kKeyNegInf : nd_key[slot >> 1];
                }
                keys[slot] = k0;
            }
            const uint64_t m = __ballot(todo);
            int at = 0;
            if (lane == 0) at = atomicAdd(&n_list_s, __popcll(m));
            at = __builtin_amdgcn_readfirstlane(at) + lane_prefix_count(m);
            if (todo) {
                const int t0 = blk * bk;
                bool miss;
                const int64_t off = kv_row_offset(p, b, hk, t0, miss);
                loff[at] = off + (miss ? back_delta : 0);
                lt0[at] = t0;
                lslot[at] = slot;
                if (p.touched) touch_page(p, b, t0);
            }
        }
        __syncthreads();
        const int n_list = __builtin_amdgcn_readfirstlane(n_list_s);
        const int n_tiles = (n_list * rpb + TILE - 1) / TILE;

        stage_t stage;  // one vector value, so that it stays in registers
        auto load_tile = [&](int t) __attribute__((always_inline)) {
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const int rr = t * TILE + j * RPW + lane / CPR;
                const int li0 = div_small(rr, rows_magic), li = min(li0, n_list - 1), n = li0 < n_list ? rr - li0 * rpb : 0;
                const int dn = min(n * bsk, kv_len - 1 - lt0[li]);  // rows past the end re-read the last one and are dropped
                const uint4 x = *(const uint4 *)((const char *)(Kbase + loff[li] + (int64_t)dn * p.ks_r) + (lane % CPR) * 16);
                stage[4 * j] = x.x; stage[4 * j + 1] = x.y; stage[4 * j + 2] = x.z; stage[4 * j + 3] = x.w;
            }
        };
        if (wave < n_tiles) load_tile(wave);
        for (int t = wave; t < n_tiles; t += 4) {
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const int row = j * RPW + lane / CPR;
                *(uint4 *)(tile + row * ROWB + (((lane % CPR) ^ (row & SW)) << 4)) =
                    make_uint4(stage[4 * j], stage[4 * j + 1], stage[4 * j + 2], stage[4 * j + 3]);
            }
            load_tile(min(t + 4, n_tiles - 1));
            wave_lds_sync();
            gen_f32x4 acc[KT][MT];
#pragma unroll
            for (int kt = 0; kt < KT; ++kt)
#pragma unroll
                for (int mt = 0; mt < MT; ++mt) acc[kt][mt] = gen_f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int cs = 0; cs < CS; ++cs)
#pragma unroll
                for (int kt = 0; kt < KT; ++kt) {
                    const uint4 kv = *(const uint4 *)(tile + (kt * 16 + r16) * ROWB + (((cs * 4 + lg) ^ (r16 & SW)) << 4));
#pragma unroll
                    for (int mt = 0; mt < MT; ++mt) acc[kt][mt] = mfma_chunk<T>(qf[mt][cs], kv, acc[kt][mt]);
                }
            wave_lds_sync();  // the operands are read: the tile may be overwritten
            // lane: key row kt*16 + r16 of the tile, query rows mt*16 + 4*lg + {0..3}
#pragma unroll
            for (int kt = 0; kt < KT; ++kt) {
                const int rr = t * TILE + kt * 16 + r16;
                const int li = div_small(rr, rows_magic);
                const bool listed = li < n_list;
                const int tk = listed ? lt0[li] + (rr - li * rpb) * bsk : kv_len;
                const int lo = tk - pos0;  // block rows below lo would look into the future
                float v = -INFINITY;
#pragma unroll
                for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const int i = min(mt * 16 + lg * 4 + e, n_eff - 1);  // (a repeated row counts as the row it repeats)
                        if (i * bsq >= lo) v = fmaxf(v, acc[kt][mt][e]);
                    }
                auto s16 = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
                v = fmaxf(__uint_as_float(s16[0]), __uint_as_float(s16[1]));
                auto s32 = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
                v = fmaxf(__uint_as_float(s32[0]), __uint_as_float(s32[1]));
                if (lg == 0 && tk < kv_len && v > -INFINITY) atomicMax(&keys[lslot[li]], score_key(v));
            }
        }
        __syncthreads();

        // every wave selects redundantly; wave (i % 4) writes the survivors of register i
        uint32_t ksel[E];
#pragma unroll
        for (int i = 0; i < E; ++i) ksel[i] = keys[i * 64 + lane];
        auto branch_of = [&](int slot, int &s, int &e) __attribute__((always_inline)) {
            s = nd_s[slot >> 1], e = nd_e[slot >> 1];
            const int mid = s + ((e - s) >> 1);
            if (slot & 1) s = mid; else e = mid;
        };
        if (round == ens_round) {  // the perturbed scores decide; keys[] keeps the true ones, which a later round may carry
#pragma unroll
            for (int i = 0; i < E; ++i) {
                if (ksel[i] == 0u) continue;
                int s, e;
                branch_of(i * 64 + lane, s, e);
                ksel[i] = ens_key(ksel[i], ens_hash, rep_block(s, e, p.rep_pos), p.ens_r);
            }
        }
        int *ns2 = nds_s[(round & 1) ^ 1], *ne2 = nde_s[(round & 1) ^ 1];
        uint32_t *nk2 = ndk_s[(round & 1) ^ 1];
        select_topk_visit<E>(ksel, kb, [&](int i, bool kept, int dest) __attribute__((always_inline)) {
            if ((i & 3) != wave || !kept) return;
            int s, e;
            branch_of(i * 64 + lane, s, e);
            ns2[dest] = s;
            ne2[dest] = e;
            nk2[dest] = keys[i * 64 + lane];
        });
        if (tid == 0) n_list_s = 0;
        __syncthreads();
    }

    for (int j = tid; j < kb; j += kThreads) out[j] = nds_s[round & 1][j] * bk;
}

template <typename T, int D, int MT>
static hipError_t launch_mask_generic_e(const KParams &p, int xcd_map, dim3 grid, uint32_t magic, hipStream_t st)
{
    dim3 block(kThreads);
    if (p.kb <= 64) hipLaunchKernelGGL((mask_generic_kernel<T, D, 2, MT>), grid, block, 0, st, p, xcd_map, magic);
    else if (p.kb <= 256) hipLaunchKernelGGL((mask_generic_kernel<T, D, 8, MT>), grid, block, 0, st, p, xcd_map, magic);
    else if (p.kb <= 512) hipLaunchKernelGGL((mask_generic_kernel<T, D, 16, MT>), grid, block, 0, st, p, xcd_map, magic);
    else hipLaunchKernelGGL((mask_generic_kernel<T, D, 32, MT>), grid, block, 0, st, p, xcd_map, magic);
    return hipGetLastError();
}

template <typename T, int D>
static hipError_t launch_mask_generic_d(const KParams &p, hipStream_t st)
{
    const int64_t groups = (int64_t)p.batch * p.hkv, per_group = (int64_t)p.g * p.nqb;
    if (groups * per_group == 0) return hipSuccess;
    const int xcd_map = groups % 8 == 0 ? 8 : 0;
    dim3 grid((unsigned)placed_workgroups(xcd_map, 1, per_group, groups));
    const uint32_t magic = div_magic(p.bk / p.b_sk);
    const int rows = (p.bq + p.b_sq - 1) / p.b_sq;
    if (rows <= 16) return launch_mask_generic_e<T, D, 1>(p, xcd_map, grid, magic, st);
    if (rows <= 32) return launch_mask_generic_e<T, D, 2>(p, xcd_map, grid, magic, st);
    return launch_mask_generic_e<T, D, 4>(p, xcd_map, grid, magic, st);
}

}  // namespace hipattn
