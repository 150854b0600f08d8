// Block-sparse attention over the selected key blocks for any shape (paper Eq. 2-3): fp32, and the bf16 shapes the
// tuned kernels (attn_mfma.hip, attn_decode.hip) leave out.  Scores, exponentials, probabilities and their products with the
// values are fp32 throughout: fp32 factors enter the matrix cores as three bf16 planes (mfma_generic.h), bf16 ones as they are.
//
// One workgroup (4 waves) per (sequence, query head, query block, 16 or 32 query rows); the waves take every fourth
// tile of 16 gathered keys, each with its own online softmax, and their states are merged through LDS at the end.
//   * S^T = K Q^T: A = key rows (lane l: row l % 16, 16-byte chunk l / 16 of each 64 bytes), B = the query rows (bf16: in
//     registers; fp32: planes in LDS, which their registers would take).  A lane then holds 4 consecutive keys of one query, so the
//     softmax runs along lanes l ^ 16 and l ^ 32 only;
//   * O^T += V^T P^T over the 16 keys of a tile: register r of S^T is key 4 (l / 16) + r, and a lane loads four consecutive channels
//     of its four keys, a plain coalesced row load; nothing of K or V passes through LDS.  A 16x16x32 step takes a lane's four
//     keys twice, in two planes each: three steps make the six products (bf16 values: two steps for the three).
// The values of a tile are loaded before its scores are multiplied and the next tile's keys before its values are.  The selected
// blocks' positions and row offsets (page table included) are worked out once per workgroup, in LDS.
// What bounds it: the cache's return path (keys as operands are 64 accesses an instruction), busy 75 % of the clocks, and vector
// issue (planes, softmax), 59 %; the matrix pipe is busy 30 % (4096 tokens, by counter).  Loading keys coalesced and through LDS is slower (281 us at 4096 tokens, 254 so).
// Measured, fp32, 32 query heads over 8 kv heads, T = 4096, k = 512, bq = 32, bk = 2, d = 128: 342 us with
// v_mfma_f32_16x16x4_f32, 257 us with planes; T = 1024, one head, k = 128, bq = 16, d = 64: 10.8 -> 10.8 us (64 workgroups: latency);
// bf16, 8 heads, 64-row blocks, k = 512: 65 -> 43 us.  Error against 64 bits (T = 4096): 3.3e-7 -> 1.7e-7 in norm.
#pragma once
#include "mfma_generic.h"
#include "launch.h"

namespace hipattn {

__device__ __forceinline__ void store4(float *p, float4 v) { *(float4 *)p = v; }
__device__ __forceinline__ void store4(bf16_t *p, float4 v)
{
    *(uint2 *)p = make_uint2((uint32_t)f32_to_bf16(v.x) | ((uint32_t)f32_to_bf16(v.y) << 16),
                             (uint32_t)f32_to_bf16(v.z) | ((uint32_t)f32_to_bf16(v.w) << 16));
}

// e^x for x <= 0 within two units in the last place: 2^(x log2 e) with the rounding error of the product put back.
// The error alone is bounded (that of -inf and of what overflows is NaN or infinite, and the median takes the bound for
// it), so a NaN - a NaN logit, or the difference of two infinite ones - comes out as NaN and not as probability 0.
__device__ __forceinline__ float exp_neg(float x)
{
    const float y = x * 1.44269504f, e = __builtin_amdgcn_fmed3f(fmaf(x, 1.44269504f, -y) + x * 1.92596299e-8f, -1.f, 1.f);
    const float v = __builtin_amdgcn_exp2f(y);
    return fmaf(v, e * 0.693147181f, v);
}
constexpr int kGenMaxKb = 1024;
// fp32: probabilities of the walk are 2^23 times e^(logit - reference), so that their planes hold all the bits of the smallest,
// 2^-126.  (Sums that overflow for it, of values beyond 2^90, are not finite and done again by rows.)
template <typename T> constexpr float kProbScale = sizeof(T) == 4 ? 0x1p23f : 1.f;

// One query row by one wave, one key per lane and its value by all lanes: reads of K and V, and multiplies into the row,
// only what counts for it.  The matrix-core walk gives a key that does not count for a row (one in the row's future, or of
// another of the three ranges) probability 0, and 0 * inf = NaN: a row that is not finite is done again here, so that an
// infinite or NaN value reaches the rows that attend to it and no others.  So are the rows of a query block with a block that
// does not lie in one page (here every key's page is looked up), and fp32 rows that the planes' range would show in: a channel
// that comes out small beside its weights, queries with lost bits, queries so large that those lost of a key would show.
// (A channel whose values are all below 2^-134, where nothing of them is left in the planes, comes out as 0.)
template <typename T, int D>
__device__ __forceinline__ void attend_row(const KParams &p, int b, int h, int hk, int kv_len, int row, const int32_t *idx, int lane)
{
#pragma clang fp contract(off)   // the largest logit minus itself is 0, whatever its size
    constexpr int CPL = D / 64;  // output channels per lane
    const T *q = (const T *)p.Q + (int64_t)b * p.qs_b + (int64_t)h * p.qs_h + (int64_t)row * p.qs_r;
    // the selected blocks' keys in [n_sink, w0), then the sink [0, ns), then the window [w0, vis)
    const int vis = min(kv_len - p.q_len + row + 1, kv_len), w0 = max(vis - p.n_window, 0), ns = min(p.n_sink, w0);
    const int n_sel = p.kb * p.bk, n_keys = vis > 0 ? n_sel + ns + vis - w0 : 0;
    float m_run = -INFINITY, l_run = 0.f, acc[CPL];
#pragma unroll
    for (int c = 0; c < CPL; ++c) acc[c] = 0.f;
    for (int base = 0; base < n_keys; base += 64) {
        const int ki = base + lane;
        int t = -1;  // this lane's key, -1: none
        if (ki < n_sel) {
            const int j = ki / p.bk, first = idx[j];
            if (first >= 0 && first < kv_len) t = first + ki - j * p.bk;
            if (t < p.n_sink || t >= w0) t = -1;
        } else if (ki < n_keys) {
            t = ki < n_sel + ns ? ki - n_sel : w0 + ki - n_sel - ns;
        }
        bool miss = false;
        const int64_t off = t >= 0 ? kv_row_offset(p, b, hk, t, miss) : 0;
        float x = -INFINITY;
        if (t >= 0) {
            const T *k = (const T *)(miss ? p.Kback : p.K) + off;
            float dot = 0.f;
#pragma unroll 4
            for (int c = 0; c < D; ++c) dot = fmaf(ld_f32(q + c), ld_f32(k + c), dot);
            x = dot * p.sm_scale;
        }
        float mx = x, sum;
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) mx = fmaxf(mx, __shfl_xor(mx, o, 64));
        const float m_new = fmaxf(m_run, mx), m_safe = m_new == -INFINITY ? 0.f : m_new, alpha = exp_neg(m_run - m_safe);
        const float pr = sum = t >= 0 ? exp_neg(x - m_safe) : 0.f;
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) sum += __shfl_xor(sum, o, 64);
        l_run = l_run * alpha + sum;
        m_run = m_new;
#pragma unroll
        for (int c = 0; c < CPL; ++c) acc[c] *= alpha;
        const uint64_t live = __ballot(t >= 0);
        for (int src = 0; src < 64; ++src) {
            if (!((live >> src) & 1)) continue;
            const float ps = __shfl(pr, src, 64);
            const T *v = (const T *)(__shfl((int)miss, src, 64) ? p.Vback : p.V) + __shfl((long long)off, src, 64);
#pragma unroll
            for (int c = 0; c < CPL; ++c) acc[c] = fmaf(ps, ld_f32(v + lane + 64 * c), acc[c]);
        }
    }
    const float inv = l_run > 0.f ? 1.f / l_run : 0.f;
    T *o = (T *)p.O + (int64_t)b * p.os_b + (int64_t)h * p.os_h + (int64_t)row * p.os_r;
#pragma unroll
    for (int c = 0; c < CPL; ++c) st_f32(o + lane + 64 * c, acc[c] * inv);
}

template <typename T, int D, int MT>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(2))) void attn_generic_kernel(KParams p, int mtn, int xcd_map, uint32_t bk_magic)
{
    constexpr int CS = D * (int)sizeof(T) / 64;  // 64-byte steps of a row in S^T = K Q^T
    constexpr int CQ = D / 64;                   // 64-channel groups of O^T
    constexpr bool F32 = sizeof(T) == 4;
    constexpr int VW = F32 ? 4 : 2;              // words of four channels of a value row
    constexpr int PITCH = D + 4;                 // floats per row of a merged state
    // block list and query planes while the tiles are walked, then the four waves' states
    constexpr int kWalk = kGenMaxKb * 12 + (F32 ? MT * (D / 32) * 3 * 1024 : 0), kMerge = 4 * MT * 16 * PITCH * 4;
    constexpr int kLds = kWalk > kMerge ? kWalk : kMerge;
    __shared__ __attribute__((aligned(16))) char lds[kLds];
    __shared__ float ml_s[4][2][MT * 16];
    __shared__ int n_blk_s;                      // list entries up to the last block; kCut: no walk, the rows are done one by one
    constexpr int kCut = kGenMaxKb + 1;
    int64_t *blk_off = (int64_t *)lds;           // element offset of a selected block's first row, bit 0: in the backing pools
    int *blk_pos = (int *)(lds + kGenMaxKb * 8); // its position, -1: no block

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r16 = lane & 15, lg = lane >> 4;
    const uint32_t groups = (uint32_t)p.batch * (uint32_t)p.hkv, per_group = (uint32_t)p.g * (uint32_t)p.nqb * (uint32_t)mtn;
    uint32_t group, o;
    if (!place_item(xcd_map, blockIdx.x, 1, 0, per_group, groups, group, o)) return;
    const uint32_t gm = (uint32_t)(p.g * mtn), oq = o / gm, rem = o - oq * gm;
    const int qb = p.nqb - 1 - (int)oq;
    const int b = (int)(group / (uint32_t)p.hkv), hk = (int)(group - (uint32_t)b * (uint32_t)p.hkv);
    const int hi = (int)(rem / (uint32_t)mtn), h = hk * p.g + hi, sub = (int)rem - hi * mtn;
    const int kb = p.kb, bk = p.bk;
    const int kv_len = p.kv_lens ? p.kv_lens[b] : p.max_kv_len;
    const int row0 = qb * p.bq + sub * MT * 16;
    const int n_rows = min(MT * 16, min(p.bq, p.q_len - qb * p.bq) - sub * MT * 16);
    if (n_rows <= 0) return;
    const int pos0 = kv_len - p.q_len + row0;
    const int32_t *idx = p.idx_in + (((int64_t)b * p.hq + h) * p.nqb + qb) * kb;

    if (tid == 0) n_blk_s = 0;
    __syncthreads();
    for (int j = tid; j < kb; j += kThreads) {
        const int first = idx[j];
        bool ok = first >= 0 && first < kv_len;
        if (ok && p.page_table && first - logical_page(p, first) * p.page_size + bk > p.page_size) {
            atomicMax(&n_blk_s, kCut);   // (an entry that is no multiple of bk: no walk, the rows are done below)
            ok = false;
        }
        bool miss;
        const int64_t off = kv_row_offset(p, b, hk, ok ? first : 0, miss);
        blk_pos[j] = ok ? first : -1;
        if (ok) atomicMax(&n_blk_s, j + 1);
        blk_off[j] = off | (miss ? 1 : 0);
    }

    // query rows as B operands: bf16 in registers, fp32 as planes in LDS, behind the block list (wave w splits every fourth)
    uint4 qf[F32 ? 1 : MT][F32 ? 1 : CS];
    uint4 *qp = (uint4 *)(lds + kGenMaxKb * 12) + lane;   // [mt][step][plane][lane]
    {
        QueryReach reach;
        const T *Qb = (const T *)p.Q + (int64_t)b * p.qs_b + (int64_t)h * p.qs_h + (int64_t)row0 * p.qs_r;
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) {
            const char *src = (const char *)(Qb + (int64_t)min(mt * 16 + r16, n_rows - 1) * p.qs_r) + lg * 16;
            if constexpr (F32) {
#pragma unroll
                for (int cs = 0; cs < CS; cs += 2) {
                    if (((mt * CS + cs) >> 1 & 3) != wave) continue;
                    const uint4 q0 = *(const uint4 *)(src + cs * 64), q1 = *(const uint4 *)(src + cs * 64 + 64);
                    reach.add(q0);
                    reach.add(q1);
                    const Planes8 x = split_planes8(q0, q1);
                    uint4 *to = qp + (mt * CS + cs) / 2 * 192;
                    to[0] = x.h; to[64] = x.m; to[128] = x.l;
                }
            } else {
#pragma unroll
                for (int cs = 0; cs < CS; ++cs) qf[mt][cs] = *(const uint4 *)(src + cs * 64);
            }
        }
        // (a logit has an error of 2^-133 times the sum of the magnitudes of its queries from the keys' lost bits)
        if (F32 && __ballot(reach.loses_bits() || reach.largest >= __float_as_uint(0x1p90f)) != 0 && lane == 0) atomicMax(&n_blk_s, kCut);
    }
    __syncthreads();

    const T *Kbase = (const T *)p.K, *Vbase = (const T *)p.V;
    // from an offset with bit 0 set to the row in the backing pool
    const int64_t k_back = (const T *)p.Kback - Kbase - 1, v_back = (const T *)p.Vback - Vbase - 1;
    // Key tiles: the selected blocks, then the sink keys [0, ns), then the window keys [wlo, vis_last).  For a row at
    // position q with vis = min(q + 1, kv_len) and w0 = max(vis - n_window, 0) a selected or sink key t counts iff
    // t < w0 (selected: also t >= n_sink), a window key iff w0 <= t < vis: every key counts once.
    const int n_blk = __builtin_amdgcn_readfirstlane(n_blk_s), n_keys = n_blk < kCut ? n_blk * bk : 0;
    const int vis_last = min(pos0 + n_rows, kv_len);
    const int wlo = max(min(pos0 + 1, kv_len) - p.n_window, 0);
    const int ns = min(p.n_sink, max(vis_last - p.n_window, 0));
    const int nw = p.n_window > 0 ? max(vis_last - wlo, 0) : 0;
    const int w0_last = max(vis_last - p.n_window, 0);

    typedef uint32_t keys_t __attribute__((ext_vector_type(4 * CS)));
    typedef uint32_t vals_t __attribute__((ext_vector_type(4 * VW * CQ)));
    auto load_keys = [&](int64_t off) __attribute__((always_inline)) {
        const char *src = (const char *)(Kbase + off + (-(off & 1) & k_back)) + lg * 16;
        keys_t kf;
#pragma unroll
        for (int cs = 0; cs < CS; ++cs) {
            const uint4 x = *(const uint4 *)(src + cs * 64);
            kf[4 * cs] = x.x; kf[4 * cs + 1] = x.y; kf[4 * cs + 2] = x.z; kf[4 * cs + 3] = x.w;
        }
        return kf;
    };

    float m_run[MT], l_run[MT];  // l: this lane's keys only
    gen_f32x4 acc[MT][CQ][4];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
        m_run[mt] = -INFINITY;
        l_run[mt] = 0.f;
#pragma unroll
        for (int cq = 0; cq < CQ; ++cq)
#pragma unroll
            for (int e = 0; e < 4; ++e) acc[mt][cq][e] = gen_f32x4{0.f, 0.f, 0.f, 0.f};
    }
    // This wave's share of tiles [from, to): key_of(tile, t, off) gives the position of key r16 of a tile (-1: counts
    // for no row) and where its row is; `window`: keys count from a row's window start, not up to it.
    auto walk = [&](int from, int to, bool window, auto key_of) __attribute__((always_inline)) {
        if (from + wave >= to) return;
        int t_cur;
        int64_t off_cur;
        key_of(from + wave, t_cur, off_cur);
        keys_t kf = load_keys(off_cur);
        for (int tile = from + wave; tile < to; tile += 4) {
            int tk[4];
            vals_t vf;
            gen_f32x4 s[MT];
#pragma unroll
            for (int r = 0; r < 4; ++r) {  // keys 4 lg + r: lane 4 lg + r holds position and offset
                tk[r] = __shfl(t_cur, lg * 4 + r, 64);
                const int64_t off = __shfl((long long)off_cur, lg * 4 + r, 64);
                const T *src = Vbase + off + (-(off & 1) & v_back) + r16 * 4;
#pragma unroll
                for (int cq = 0; cq < CQ; ++cq) {
                    const int at = VW * (r * CQ + cq);
                    if constexpr (F32) {
                        const uint4 x = *(const uint4 *)(src + cq * 64);
                        vf[at] = x.x; vf[at + 1] = x.y; vf[at + 2] = x.z; vf[at + 3] = x.w;
                    } else {
                        const uint2 x = *(const uint2 *)(src + cq * 64);
                        vf[at] = x.x; vf[at + 1] = x.y;
                    }
                }
            }
            __builtin_amdgcn_sched_barrier(0);  // (the loads go out before the multiplies)
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) s[mt] = gen_f32x4{0.f, 0.f, 0.f, 0.f};
            if constexpr (F32) {
                gen_f32x4 low[MT];
#pragma unroll
                for (int mt = 0; mt < MT; ++mt) low[mt] = gen_f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int cs = 0; cs < CS; cs += 2) {
                    const Planes8 kp = split_planes8(make_uint4(kf[4 * cs], kf[4 * cs + 1], kf[4 * cs + 2], kf[4 * cs + 3]),
                                                     make_uint4(kf[4 * cs + 4], kf[4 * cs + 5], kf[4 * cs + 6], kf[4 * cs + 7]));
                    Planes8 q[MT];
#pragma unroll
                    for (int mt = 0; mt < MT; ++mt) {
                        const uint4 *from = qp + (mt * CS + cs) / 2 * 192;
                        q[mt] = Planes8{from[0], from[64], from[128]};
                    }
                    mfma_planes<true>(kp, q, s, low);
                }
#pragma unroll
                for (int mt = 0; mt < MT; ++mt) s[mt] += low[mt];
            } else {
#pragma unroll
                for (int cs = 0; cs < CS; ++cs)
#pragma unroll
                    for (int mt = 0; mt < MT; ++mt)
                        s[mt] = mfma_chunk<T>(make_uint4(kf[4 * cs], kf[4 * cs + 1], kf[4 * cs + 2], kf[4 * cs + 3]), qf[mt][cs], s[mt]);
            }
            // (unconditional, the last tile again at the end: a load on one path only would make the waits below wait for all)
            key_of(min(tile + 4, to - 1), t_cur, off_cur);
            kf = load_keys(off_cur);
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) {
                const int vis = min(pos0 + mt * 16 + r16 + 1, kv_len), w0 = max(vis - p.n_window, 0);
                const int lo = window ? w0 : 0, hi_ = window ? vis : w0;
                float mx = -INFINITY, x[4];
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    x[r] = tk[r] >= lo && tk[r] < hi_ ? s[mt][r] * p.sm_scale : -INFINITY;
                    mx = fmaxf(mx, x[r]);
                }
                auto s16 = __builtin_amdgcn_permlane16_swap(__float_as_uint(mx), __float_as_uint(mx), false, false);
                mx = fmaxf(__uint_as_float(s16[0]), __uint_as_float(s16[1]));
                auto s32 = __builtin_amdgcn_permlane32_swap(__float_as_uint(mx), __float_as_uint(mx), false, false);
                mx = fmaxf(__uint_as_float(s32[0]), __uint_as_float(s32[1]));
                // the reference moves when a logit passes it by 8 or more: probabilities then reach e^8, which costs no bits,
                // and the sums are multiplied on the first tile only as a rule
                const float m_new = mx > m_run[mt] + 8.f ? mx : m_run[mt], m_safe = m_new == -INFINITY ? 0.f : m_new;
                const float alpha = exp_neg(m_run[mt] - m_safe);  // 0 on the first tile that counts
                float sum = 0.f;
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    x[r] = exp_neg(x[r] - m_safe) * kProbScale<T>;
                    sum += x[r];
                }
                s[mt] = gen_f32x4{x[0], x[1], x[2], x[3]};
                l_run[mt] = l_run[mt] * alpha + sum;
                m_run[mt] = m_new;
                if (__ballot(alpha != 1.f) != 0) {
#pragma unroll
                    for (int cq = 0; cq < CQ; ++cq)
#pragma unroll
                        for (int e = 0; e < 4; ++e) acc[mt][cq][e] *= alpha;
                }
            }
            // a 16x16x32 step takes a lane's four keys twice, in two planes each
            Planes p01[MT], p23[MT];
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) {
                p01[mt] = split_planes(s[mt][0], s[mt][1]);
                p23[mt] = split_planes(s[mt][2], s[mt][3]);
            }
#pragma unroll
            for (int cq = 0; cq < CQ; ++cq)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    if constexpr (F32) {
                        const auto v = [&](int r) __attribute__((always_inline)) { return __uint_as_float(vf[4 * (r * CQ + cq) + e]); };
                        const Planes a = split_planes(v(0), v(1)), b2 = split_planes(v(2), v(3));
                        const uint4 hm = make_uint4(a.h, b2.h, a.m, b2.m), hl = make_uint4(a.h, b2.h, a.l, b2.l);
#pragma unroll
                        for (int mt = 0; mt < MT; ++mt)
                            acc[mt][cq][e] = mfma_chunk<bf16_t>(hl, make_uint4(p01[mt].l, p23[mt].l, p01[mt].h, p23[mt].h), acc[mt][cq][e]);
#pragma unroll
                        for (int mt = 0; mt < MT; ++mt)
                            acc[mt][cq][e] = mfma_chunk<bf16_t>(hm, make_uint4(p01[mt].m, p23[mt].m, p01[mt].m, p23[mt].m), acc[mt][cq][e]);
#pragma unroll
                        for (int mt = 0; mt < MT; ++mt)
                            acc[mt][cq][e] = mfma_chunk<bf16_t>(hm, make_uint4(p01[mt].h, p23[mt].h, p01[mt].h, p23[mt].h), acc[mt][cq][e]);
                    } else {
                        const auto v = [&](int r) __attribute__((always_inline)) { return vf[2 * (r * CQ + cq) + (e >> 1)]; };
                        const uint32_t half = e & 1 ? 0x07060302u : 0x05040100u;
                        const uint32_t a = __builtin_amdgcn_perm(v(1), v(0), half), b2 = __builtin_amdgcn_perm(v(3), v(2), half);
                        const uint4 vv = make_uint4(a, b2, a, b2);
#pragma unroll
                        for (int mt = 0; mt < MT; ++mt)
                            acc[mt][cq][e] = mfma_chunk<bf16_t>(make_uint4(a, b2, 0u, 0u), make_uint4(p01[mt].l, p23[mt].l, 0u, 0u), acc[mt][cq][e]);
#pragma unroll
                        for (int mt = 0; mt < MT; ++mt)
                            acc[mt][cq][e] = mfma_chunk<bf16_t>(vv, make_uint4(p01[mt].m, p23[mt].m, p01[mt].h, p23[mt].h), acc[mt][cq][e]);
                    }
                }
        }
    };
    if (vis_last > 0) {
        walk(0, (n_keys + 15) >> 4, false, [&](int tile, int &t, int64_t &off) __attribute__((always_inline)) {
            const int ki = tile * 16 + r16, j = min(div_small(ki, bk_magic), kb - 1), n = ki - j * bk;
            const int first = blk_pos[j], x = first + n;
            const bool in = ki < n_keys && first >= 0 && x < kv_len;
            t = in && x >= p.n_sink && x < w0_last ? x : -1;
            off = blk_off[j] + (in ? (int64_t)n * p.ks_r : 0);
        });
        auto plain = [&](int x, int end, int &t, int64_t &off) __attribute__((always_inline)) {
            t = x < end ? x : -1;
            bool miss;
            off = kv_row_offset(p, b, hk, max(t, 0), miss);
            off |= miss ? 1 : 0;
        };
        if (ns > 0) walk(0, (ns + 15) >> 4, false, [&](int tile, int &t, int64_t &off) __attribute__((always_inline)) { plain(tile * 16 + r16, ns, t, off); });
        if (nw > 0) walk(0, (nw + 15) >> 4, true, [&](int tile, int &t, int64_t &off) __attribute__((always_inline)) { plain(wlo + tile * 16 + r16, vis_last, t, off); });
    }

    // ---- merge: every wave leaves its state in LDS as rows of channels; with m = the largest reference the states
    // are rescaled by exp(m_w - m) and added
    __syncthreads();  // the block list is no longer needed
    float *st = (float *)lds + wave * MT * 16 * PITCH;
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
        float l = l_run[mt];
        l += __shfl_xor(l, 16, 64);
        l += __shfl_xor(l, 32, 64);
        if (lg == 0) {
            ml_s[wave][0][mt * 16 + r16] = m_run[mt];
            ml_s[wave][1][mt * 16 + r16] = l;
        }
#pragma unroll
        for (int cq = 0; cq < CQ; ++cq)
#pragma unroll
            for (int x = 0; x < 4; ++x)  // row (4 lg + x) of the channel operand is channels 4 (4 lg + x) + {0..3}
                *(float4 *)(st + (mt * 16 + r16) * PITCH + cq * 64 + lg * 16 + x * 4) =
                    make_float4(acc[mt][cq][0][x], acc[mt][cq][1][x], acc[mt][cq][2][x], acc[mt][cq][3][x]);
    }
    __syncthreads();
    T *Ob = (T *)p.O + (int64_t)b * p.os_b + (int64_t)h * p.os_h + (int64_t)row0 * p.os_r;
    bool odd = false;  // a result of this lane is not finite, or so small that its values' planes may have left the range
    for (int i = tid; i < n_rows * (D / 4); i += kThreads) {
        const int row = i / (D / 4), c4 = (i % (D / 4)) * 4;
        float m = -INFINITY;
#pragma unroll
        for (int w = 0; w < 4; ++w) m = fmaxf(m, ml_s[w][0][row]);
        const float m_safe = m == -INFINITY ? 0.f : m;
        float l = 0.f;
        float4 sum = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            const float a = exp_neg(ml_s[w][0][row] - m_safe);
            const float4 x = *(const float4 *)((const float *)lds + (w * MT * 16 + row) * PITCH + c4);
            l = fmaf(ml_s[w][1][row], a, l);
            sum.x = fmaf(x.x, a, sum.x); sum.y = fmaf(x.y, a, sum.y); sum.z = fmaf(x.z, a, sum.z); sum.w = fmaf(x.w, a, sum.w);
        }
        const float inv = l > 0.f ? 1.f / l : 0.f;
        const auto small = [&](float s) __attribute__((always_inline)) { return fabsf(s) < 0x1p-100f * l && s != 0.f; };
        odd |= not_finite(fabsf(sum.x) + fabsf(sum.y) + fabsf(sum.z) + fabsf(sum.w) + l) ||
               (F32 && (small(sum.x) || small(sum.y) || small(sum.z) || small(sum.w)));
        store4(Ob + (int64_t)row * p.os_r + c4, make_float4(sum.x * inv, sum.y * inv, sum.z * inv, sum.w * inv));
    }
    if (__ballot(odd) != 0 || n_blk == kCut) {  // the rows that this wave stored, again
        __threadfence_block();
        for (int i = tid - lane; i < n_rows * (D / 4); i += kThreads)
            for (int row = i / (D / 4); row < min(i / (D / 4) + 256 / D, n_rows); ++row)
                attend_row<T, D>(p, b, h, hk, kv_len, row0 + row, idx, lane);
    }
}

template <typename T, int D>
static hipError_t launch_attn_generic_d(const KParams &p, hipStream_t st)
{
    const int mt = p.bq <= 16 ? 1 : 2, mtn = (p.bq + mt * 16 - 1) / (mt * 16);
    const int64_t groups = (int64_t)p.batch * p.hkv, per_group = (int64_t)p.g * p.nqb * mtn;
    if (groups * per_group == 0) return hipSuccess;
    if (groups * per_group > 0x7fffffffLL) return hipErrorInvalidValue;
    const int xcd_map = groups % 8 == 0 ? 8 : 0;
    dim3 grid((unsigned)placed_workgroups(xcd_map, 1, per_group, groups)), block(kThreads);
    const uint32_t magic = div_magic(p.bk);
    if (mt == 1) hipLaunchKernelGGL((attn_generic_kernel<T, D, 1>), grid, block, 0, st, p, mtn, xcd_map, magic);
    else hipLaunchKernelGGL((attn_generic_kernel<T, D, 2>), grid, block, 0, st, p, mtn, xcd_map, magic);
    return hipGetLastError();
}

}  // namespace hipattn
