// Hierarchical mask estimation for any shape (paper Alg. 1, block form of Sec. 3.2): fp32, and the bf16 shapes the
// tuned kernels (mask_mfma_impl.h, mask_decode_impl.h) leave out.  Any bq <= 64, bk <= 16, k/bk <= 1024, sampling
// stride and representative, contiguous or paged K with any page size, prefill or decode.
//
// One workgroup (4 waves) per (sequence, query head, query block).  The block score is a contraction, so it runs on the
// matrix cores (v_mfma_f32_16x16x32_bf16); fp32 operands go in as three bf16 planes (mfma_generic.h): six products at
// 16 times the rate of the fp32 instruction, and a third of its error.  What bounds the kernel then are the gathered rows: the
// wide tiles load them straight as operands, 64 cache accesses an instruction: the address unit is busy 82 % of the
// clocks, the return path 93 %, vector issue 51 %, the matrix pipe 32 % (4096 tokens, by counter).
//   * The sampled query rows are MT operand tiles of 16 rows (small query blocks do not pay for 32), in registers, or their
//     planes in LDS where two tiles of them would leave two waves per SIMD instead of three (4096 tokens: 398 us with the
//     planes in registers, 389 so).  fp32 blocks of more than 32 rows: two waves share a tile, each with half of the rows.
//   * The branches that need a score are put on a list (LDS: block position, row offset, branch slot); a branch whose
//     representative block was scored in an earlier round has that score and is not listed (known_branches in common.h; fp32, 4096 tokens
//     of 32 heads 389 -> 367 us against right halves in the last round alone).  The key rows of the list are
//     gathered in tiles of 8 KB per wave, one tile ahead (the order of the channels inside the contraction is free).  Coalesced
//     and through the wave's LDS tile (XOR swizzle; lane l: row l % 16, chunk l / 16 of each 64 bytes) for bf16 and for one fp32
//     query tile, whose matrix work is too short to hide the accesses (16-row blocks, 4096 tokens of 32 heads 580 us, straight
//     735); straight for two query tiles (389 us, through LDS 435) and for k/bk above 512, where the LDS tiles cost a
//     workgroup per compute unit (8000 tokens, 8 heads, d = 64, k/bk = 1024 258 us, through LDS 478).
//   * A row's maximum over the admissible query rows goes to its branch's key with an LDS atomic maximum, which takes
//     any number of rows per block.
//   * Selection: the ordered threshold selection of common.h, run redundantly by the four waves.
// Measured, fp32, 32 query heads over 8 kv heads, T = 4096, k = 512, bq = 32, bk = 2, d = 128: 576 us with the fp32 instruction
// (half of the clocks on the matrix pipe), 378 us with planes; d = 64 337 -> 224; one sequence of 1024 tokens, one head, k = 128, bq = 16, d = 64: 18.0
// -> 17.1 (64 workgroups: latency).
#pragma once
#include "mfma_generic.h"
#include "launch.h"

namespace hipattn {

// (waves per SIMD: two query tiles of 64 fp32 channels and k/bk <= 256 spill 4 to 7 registers at three waves; at two, with none
// spilled, 4096 tokens of 32 heads, k/bk = 256 take 245 us instead of 216, k/bk = 64 182 instead of 153)
template <typename T, int D, int E, int MT>
__global__ __launch_bounds__(kThreads, E > 16 ? 1 : (E > 8 || MT > 2) ? 2 : 3) void mask_generic_kernel(KParams p, int xcd_map, uint32_t rows_magic)
{
    constexpr bool F32 = sizeof(T) == 4;
    // fp32, more than 32 rows: two waves share a tile, each scores half of the rows.  Planes of two operand tiles are in LDS.
    constexpr int HALVES = F32 && MT > 2 ? 2 : 1, MW = MT / HALVES;
    constexpr bool QLDS = F32 && MW > 1;
    constexpr bool STAGED = !F32 || (MW == 1 && E <= 16);  // key rows pass through LDS, see above
    constexpr int NB = 64 * E;             // branch slots (two per node)
    constexpr int ROWB = D * (int)sizeof(T);
    constexpr int CPR = ROWB / 16;         // 16-byte chunks per key row = lanes per row of a coalesced load
    constexpr int RPW = 64 / CPR;          // rows per wave-wide load
    constexpr int TILE = 8192 / ROWB;      // key rows per tile
    constexpr int SW = (CPR < 16 ? CPR : 16) - 1;
    constexpr int KT = TILE / 16, CS = CPR / 4;
    typedef uint32_t stage_t __attribute__((ext_vector_type(32)));
    __shared__ __attribute__((aligned(16))) uint4 tile_s[STAGED ? 4 : 1][STAGED ? 512 : 1];
    __shared__ int64_t loff[NB];           // list entry: element offset of its block's first row in K
    __shared__ int lt0[NB];                // ... position of that row
    __shared__ int lslot[NB];              // ... branch slot
    __shared__ uint32_t keys[NB];
    // Nodes of this round and of the next: first block and one bit (all of a round's nodes are m_len or m_len + 1 blocks long:
    // chunks differ by one, and so do halves of lengths that differ by one)
    __shared__ uint32_t nd_s[2][NB / 2];
    __shared__ uint32_t ndk_s[2][NB / 2], ndb_s[2][NB / 2];  // ... keys of its own and its first block's score, 0: not known (known_branches)
    __shared__ __attribute__((aligned(16))) uint4 qp_s[QLDS ? MT * (CS / 2) * 192 : 1];  // [half][step][operand tile][plane][lane]
    __shared__ float tiny_s[4];
    __shared__ int n_list_s;

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r16 = lane & 15, lg = lane >> 4;
    const int half = wave & (HALVES - 1), first_tile = wave / HALVES;
    constexpr int tile_step = 4 / HALVES;
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
    const auto q_row = [&](int mt) __attribute__((always_inline)) {
        const int i = min(mt * 16 + r16, n_eff - 1) * bsq;
        return (const char *)((const T *)p.Q + (int64_t)b * p.qs_b + (int64_t)h * p.qs_h + (int64_t)(row0 + i) * p.qs_r) + lg * 16;
    };
    uint4 qf[F32 ? 1 : MT][F32 ? 1 : CS];
    Planes8 qp[F32 && !QLDS ? CS / 2 : 1][F32 && !QLDS ? MW : 1];
    QueryReach reach;
    const uint4 *q_own = qp_s + half * (CS / 2 * MW * 192) + lane;
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
        const char *src = q_row(mt);
        if constexpr (F32) {
#pragma unroll
            for (int cs = 0; cs < CS; cs += 2) {
                if (QLDS && ((mt * CS + cs) >> 1 & 3) != wave) continue;
                const uint4 x = *(const uint4 *)(src + cs * 64), y = *(const uint4 *)(src + cs * 64 + 64);
                const Planes8 pl = split_planes8(x, y);
                if constexpr (QLDS) {
                    uint4 *to = qp_s + ((mt / MW * (CS / 2) + cs / 2) * MW + mt % MW) * 192 + lane;
                    to[0] = pl.h; to[64] = pl.m; to[128] = pl.l;
                } else {
                    qp[cs / 2][mt] = pl;
                }
                reach.add(x);
                reach.add(y);
            }
        } else {
#pragma unroll
            for (int cs = 0; cs < CS; ++cs) qf[mt][cs] = *(const uint4 *)(src + cs * 64);
        }
    }
    float tiny = 0.f;  // scores this close to 0 may have lost more to the planes' range than fp32 products lose
    if constexpr (F32) {  // (whole numbers order magnitudes)
        tiny = __uint_as_float(wave_max_u32(__ballot(reach.loses_bits()) != 0 ? 0x7f800000u : reach.largest));
        if (lane == 0) tiny_s[wave] = tiny;
    }

    // initial nodes: kb chunks of [0, Tb) with rounded bounds; all non-empty because Tb > kb
    const int a = Tb / kb, r = Tb % kb;
    for (int j = tid; j < kb; j += kThreads) {
        const int s = chunk_bound(j, a, r, kb, p.kb_magic);
        nd_s[0][j] = (uint32_t)(s << 1 | (chunk_bound(j + 1, a, r, kb, p.kb_magic) - s - a));
        ndk_s[0][j] = ndb_s[0][j] = 0u;
    }
    if (tid == 0) n_list_s = 0;
    for (int i = 2 * kb + tid; i < NB; i += kThreads) keys[i] = 0u;
    __syncthreads();
    if constexpr (F32) {
        tiny = fmaxf(fmaxf(tiny_s[0], tiny_s[1]), fmaxf(tiny_s[2], tiny_s[3]));
        tiny = tiny < 0x1p-76f && tiny > 0.f ? INFINITY : tiny * D * 0x1p-100f;   // (queries of 0: scores of 0)
    }

    const T *Kbase = (const T *)p.K;
    const int64_t back_delta = (const T *)p.Kback - Kbase;  // elements from the resident pool to the backing pool

    // this lane's part of a coalesced load and of a tile in LDS (chunk c of row r is at place c ^ (r & SW) of the row), and
    // where its operands are: the steps of 4 chunks and the rows of a load only flip bits of these
    const char *kchunk = (const char *)Kbase + (lane % CPR) * 16;
    char *const tile = (char *)tile_s[STAGED ? wave : 0];
    const int put = lane / CPR * ROWB + (((lane % CPR) ^ (lane / CPR)) << 4), get = r16 * ROWB + ((lg ^ (r16 & SW)) << 4);

    // ensemble sample: the round whose selection compares perturbed scores (-1: none)
    const int ens_round = ens_round_of(p.ens_sample, a + (r ? 1 : 0));
    const uint32_t ens_hash = ens_round >= 0 ? ens_unit_hash(p.ens_seed, p.ens_sample, b, h, qb) : 0u;
    // Two tiles of 64 fp32 channels work the representative rule and the selection's LDS addresses out where they are needed: kept
    // through the tiles these are up to 9 spilled registers more (k/bk = 256, 2000 tokens of 32 heads 73.1 / 70.1 us, 4096 216 / 210; k/bk = 64 152 /
    // 148).  One tile is 2 % slower so.
    constexpr bool kAnew = F32 && D == 64 && MT == 2;
    const RepRule rule_kept = rep_rule(p.rep_pos);
    auto rule_now = [&]() __attribute__((always_inline)) {
        if constexpr (!kAnew) return rule_kept;
        int rep_pos = p.rep_pos;
        asm volatile("" : "+s"(rep_pos));
        return rep_rule(rep_pos);
    };
    int round = 0, m_len = a;
    // maxlen bounds the longest node
    for (int maxlen = a + (r ? 1 : 0); maxlen > 1; maxlen = (maxlen + 1) >> 1, ++round, m_len >>= 1) {
        const uint32_t *nd = nd_s[round & 1], *nd_own = ndk_s[round & 1], *nd_beg = ndb_s[round & 1];
        // split every node into its left and right branch (slots 2j, 2j+1; left may be empty) and list the blocks to score
        for (int base = wave * 64; base < 2 * kb; base += kThreads) {
            const int slot = base + lane;
            bool todo = false;
            int blk = 0;
            if (slot < 2 * kb) {
                const RepRule rule = rule_now();
                const int j = slot >> 1, s = (int)(nd[j] >> 1), len = m_len + (int)(nd[j] & 1), mid = s + (len >> 1);
                uint32_t left, right;
                bool need_l, need_r;
                known_branches(rule, len, nd_own[j], nd_beg[j], left, right, need_l, need_r);
                todo = (slot & 1) ? need_r : need_l;
                blk = (slot & 1) ? rep_block(mid, s + len, rule) : rep_block(s, mid, rule);
                // a branch to score starts at "-inf" (it may end up without an admissible pair)
                keys[slot] = todo ? kKeyNegInf : (slot & 1) ? right : left;
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

        struct Rows { int64_t off[KT]; int tk[KT], slot[KT]; };  // rows l % 16 of a tile, lane l: place in bytes, position, branch slot
        auto rows_of = [&](int t) __attribute__((always_inline)) {
            Rows r;
#pragma unroll
            for (int kt = 0; kt < KT; ++kt) {
                const int rr = t * TILE + kt * 16 + r16;
                const int li0 = div_small(rr, rows_magic), li = min(li0, n_list - 1), dn = li0 < n_list ? (rr - li0 * rpb) * bsk : 0;
                const int t0 = lt0[li];
                // rows past the end re-read the last one and are dropped
                r.off[kt] = (loff[li] + (int64_t)min(dn, kv_len - 1 - t0) * p.ks_r) * (int)sizeof(T);
                r.tk[kt] = li0 < n_list ? t0 + dn : kv_len;
                r.slot[kt] = lslot[li];
            }
            return r;
        };
        auto score_tile = [&](const Rows &rows, auto key_chunk) __attribute__((always_inline)) {
            gen_f32x4 acc[KT][MW];
#pragma unroll
            for (int kt = 0; kt < KT; ++kt)
#pragma unroll
                for (int mt = 0; mt < MW; ++mt) acc[kt][mt] = gen_f32x4{0.f, 0.f, 0.f, 0.f};
            if constexpr (F32) {
                gen_f32x4 low[KT][MW];
#pragma unroll
                for (int kt = 0; kt < KT; ++kt)
#pragma unroll
                    for (int mt = 0; mt < MW; ++mt) low[kt][mt] = gen_f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int cs = 0; cs < CS; cs += 2)
#pragma unroll
                    for (int kt = 0; kt < KT; ++kt) {
                        const Planes8 kp = split_planes8(key_chunk(kt, cs), key_chunk(kt, cs + 1));
                        if constexpr (QLDS) {
                            Planes8 q[MW];
#pragma unroll
                            for (int mt = 0; mt < MW; ++mt) {
                                const uint4 *from = q_own + (cs / 2 * MW + mt) * 192;
                                q[mt] = Planes8{from[0], from[64], from[128]};
                            }
                            mfma_planes<false>(kp, q, acc[kt], low[kt]);
                        } else {
                            mfma_planes<false>(kp, qp[cs / 2], acc[kt], low[kt]);
                        }
                    }
                bool again = false;
#pragma unroll
                for (int kt = 0; kt < KT; ++kt) {
                    float all = 0.f;
#pragma unroll
                    for (int mt = 0; mt < MW; ++mt)
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            acc[kt][mt][e] += low[kt][mt][e];
                            all += fabsf(acc[kt][mt][e]);
                        }
                    again |= not_finite(all) || all < tiny;
                }
                if (__builtin_expect(__ballot(again) != 0, 0)) {  // infinities, or magnitudes at the end of the range: once more, in fp32
#pragma unroll
                    for (int mt = 0; mt < MW; ++mt) {
                        const char *src = q_row(half * MW + mt);
#pragma unroll
                        for (int kt = 0; kt < KT; ++kt) acc[kt][mt] = gen_f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                        for (int cs = 0; cs < CS; ++cs) {
                            const uint4 qv = *(const uint4 *)(src + cs * 64);
#pragma unroll
                            for (int kt = 0; kt < KT; ++kt) acc[kt][mt] = mfma_chunk<float>(qv, key_chunk(kt, cs), acc[kt][mt]);
                        }
                    }
                }
            } else {
#pragma unroll
                for (int cs = 0; cs < CS; ++cs)
#pragma unroll
                    for (int kt = 0; kt < KT; ++kt)
#pragma unroll
                        for (int mt = 0; mt < MW; ++mt) acc[kt][mt] = mfma_chunk<T>(qf[mt][cs], key_chunk(kt, cs), acc[kt][mt]);
            }
            // lane: key row kt*16 + r16 of the tile, query rows mt*16 + 4*lg + {0..3}
#pragma unroll
            for (int kt = 0; kt < KT; ++kt) {
                const int tk = rows.tk[kt];
                float v = -INFINITY;
                if (__ballot(tk > pos0 && tk < kv_len) == 0) {  // no row has these keys in its future
#pragma unroll
                    for (int mt = 0; mt < MW; ++mt)
#pragma unroll
                        for (int e = 0; e < 4; ++e) v = fmaxf(v, acc[kt][mt][e]);
                } else {
                    const int lo = tk - pos0;  // block rows below lo would look into the future
#pragma unroll
                    for (int mt = 0; mt < MW; ++mt)
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            const int i = min((half * MW + mt) * 16 + lg * 4 + e, n_eff - 1);  // (a repeated row counts as the row it repeats)
                            if (i * bsq >= lo) v = fmaxf(v, acc[kt][mt][e]);
                        }
                }
                auto s16 = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
                v = fmaxf(__uint_as_float(s16[0]), __uint_as_float(s16[1]));
                auto s32 = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
                v = fmaxf(__uint_as_float(s32[0]), __uint_as_float(s32[1]));
                if (lg == 0 && tk < kv_len && v > -INFINITY) atomicMax(&keys[rows.slot[kt]], score_key(v));
            }
        };
        // the loads of a tile are in flight while another one is multiplied (the last tile's once more at the end: a load on one
        // path only would make the waits of the other wait for all)
        if constexpr (STAGED) {
            stage_t stage;  // one vector value, so that it stays in registers
            Rows next;
            auto load_tile = [&](int t) __attribute__((always_inline)) {
                next = rows_of(t);
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    const int64_t off = __shfl((long long)next.off[j * RPW / 16], j * RPW % 16 + lane / CPR, 64);
                    const uint4 x = *(const uint4 *)(kchunk + off);
                    stage[4 * j] = x.x; stage[4 * j + 1] = x.y; stage[4 * j + 2] = x.z; stage[4 * j + 3] = x.w;
                }
            };
            if (first_tile < n_tiles) load_tile(first_tile);
            for (int t = first_tile; t < n_tiles; t += tile_step) {
                const Rows rows = next;
#pragma unroll
                for (int j = 0; j < 8; ++j)
                    *(uint4 *)(tile + ((put ^ ((j * RPW & SW) << 4)) + j * RPW * ROWB)) =
                        make_uint4(stage[4 * j], stage[4 * j + 1], stage[4 * j + 2], stage[4 * j + 3]);
                load_tile(min(t + tile_step, n_tiles - 1));
                wave_lds_sync();
                score_tile(rows, [&](int kt, int cs) __attribute__((always_inline)) { return *(const uint4 *)(tile + ((get ^ (cs << 6)) + kt * 16 * ROWB)); });
                wave_lds_sync();  // the operands are read: the tile may be overwritten
            }
        } else if (first_tile < n_tiles) {
            stage_t xa, xb;
            Rows ra, rb;
            auto load_tile = [&](int t, stage_t &x, Rows &r) __attribute__((always_inline)) {
                r = rows_of(t);
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    const uint4 v = *(const uint4 *)((const char *)Kbase + r.off[i / CS] + lg * 16 + i % CS * 64);
                    x[4 * i] = v.x; x[4 * i + 1] = v.y; x[4 * i + 2] = v.z; x[4 * i + 3] = v.w;
                }
                __builtin_amdgcn_sched_barrier(0);  // (the loads go out before the multiplies)
            };
            const auto chunks = [](const stage_t &x) __attribute__((always_inline)) {
                return [&x](int kt, int cs) __attribute__((always_inline)) {
                    const int at = 4 * (kt * CS + cs);
                    return make_uint4(x[at], x[at + 1], x[at + 2], x[at + 3]);
                };
            };
            load_tile(first_tile, xa, ra);
            for (int t = first_tile;;) {
                load_tile(min(t + tile_step, n_tiles - 1), xb, rb);
                score_tile(ra, chunks(xa));
                if ((t += tile_step) >= n_tiles) break;
                load_tile(min(t + tile_step, n_tiles - 1), xa, ra);
                score_tile(rb, chunks(xb));
                if ((t += tile_step) >= n_tiles) break;
            }
        }
        __syncthreads();

        // every wave selects redundantly; wave (i % 4) writes the survivors of register i
        int lane_sel = lane;
        if constexpr (kAnew) asm volatile("" : "+v"(lane_sel));
        uint32_t ksel[E];
#pragma unroll
        for (int i = 0; i < E; ++i) ksel[i] = keys[i * 64 + lane_sel];
        auto branch_of = [&](int slot, int &s, int &e) __attribute__((always_inline)) {
            s = (int)(nd[slot >> 1] >> 1), e = s + m_len + (int)(nd[slot >> 1] & 1);
            const int mid = s + ((e - s) >> 1);
            if (slot & 1) s = mid; else e = mid;
        };
        if (round == ens_round) {  // the perturbed scores decide; keys[] keeps the true ones, which a later round may carry
#pragma unroll
            for (int i = 0; i < E; ++i) {
                if (ksel[i] == 0u) continue;
                int s, e;
                branch_of(i * 64 + lane_sel, s, e);
                ksel[i] = ens_key(ksel[i], ens_hash, rep_block(s, e, rule_now()), p.ens_r);
            }
        }
        uint32_t *nd2 = nd_s[(round & 1) ^ 1], *nk2 = ndk_s[(round & 1) ^ 1], *nb2 = ndb_s[(round & 1) ^ 1];
        select_topk_visit<E>(ksel, kb, [&](int i, bool kept, int dest) __attribute__((always_inline)) {
            if ((i & 3) != wave || !kept) return;
            int s, e;
            const int slot = i * 64 + lane_sel;
            branch_of(slot, s, e);
            nd2[dest] = (uint32_t)(s << 1 | (e - s - (m_len >> 1)));
            nk2[dest] = keys[slot];
            nb2[dest] = ((slot & 1) ? nd_own : nd_beg)[slot >> 1];   // (a right half begins with its node's centre)
        });
        if (tid == 0) n_list_s = 0;
        __syncthreads();
    }

    for (int j = tid; j < kb; j += kThreads) out[j] = (int)(nd_s[round & 1][j] >> 1) * bk;
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
