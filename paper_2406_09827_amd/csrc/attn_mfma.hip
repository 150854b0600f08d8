// Block-sparse attention for bf16 prefill on CDNA4 matrix cores (paper Eq. 2-3; the "block sparse flash attention" of the
// appendix: online softmax over the gathered keys).
//
// Work item = one wave = one (sequence, query head, query block, 32-row query tile), four per workgroup; with few work
// items two or four waves share one (WPI).  Per tile of 32 gathered keys:
//   S^T = K_tile . Q^T     v_mfma_f32_32x32x16_bf16, A = key rows (read back from LDS one row per lane), B = the query tile
//                          held in registers.  The result has one query per lane and 16 keys in its registers, so the
//                          softmax statistics of a query are lane-local (plus one exchange with lane ^ 32) and P^T is already
//                          in B-operand layout.
//   O^T += V_tile^T . P^T  the value rows are read back channel-major with the LDS transpose read ds_read_b64_tr_b16 (the
//                          contraction runs over keys, so V has to be transposed on the way to the A operand).
// P is a single bf16 term; the row sum is taken over the ROUNDED probabilities, so numerator and denominator of the output
// carry the same weights: the rounding of P then perturbs the weights of a weighted mean by 2^-9 relative instead of adding
// an error of that size to the output.
// How a tile travels:
//   * The keys of a work item - selected blocks, sink, window - are worked out before the loop, 16 tiles of them, into a list
//     in LDS (position of every key; over a paged pool its page as well), with two bits per tile that say whether any key
//     counts and whether any needs masking.  Longer lists are refilled 8 tiles at a time.  The loop itself then only reads
//     its rows' positions.  (Any k in 72 KB of LDS, over pages 80: two workgroups to a compute unit where an index row of 1024
//     entries in LDS left one.)
//   * global_load_lds_dwordx4 delivers lane l's 16 bytes at M0 + 16 l without passing through registers or the LDS
//     instruction pipe.  Load j of a tile fills LDS rows RPI j .. RPI j + RPI - 1 (RPI = 4 rows of 256 bytes or 8 of 128); lane
//     group lg supplies gathered key NLD lg + j (a lane's rows are consecutive keys: one or two 16-byte reads of the list tell
//     it where they are), hence key x sits in LDS row RPI (x % NLD) + x / NLD.
//   * XOR swizzles, applied to the global chunk a lane fetches, keep the operand reads free of bank conflicts.  Keys: 16-byte
//     chunk c at place c ^ (x % 16), with 64 channels c ^ (x % 4 + 4 (x / 8 % 2)).  Values: 32-byte chunk pair p at place
//     p ^ rotl3(x % 8), with 64 channels p ^ 2 (x % 2): the 16 consecutive channels a transpose read takes stay together and
//     the eight 32-byte pieces that 32 lanes of it fetch fall into different banks.  With 64 channels two rows share the 256
//     bytes of all banks, so the four keys that a lane takes per read have to be two of even and two of odd rows: row r of
//     the score tile is gathered key r with bits 1 and 2 exchanged.
//   * ONE key and ONE value buffer per wave: as soon as a tile's key operands are in registers the key buffer is refilled
//     with the next tile's keys, which land while this tile is multiplied and its softmax runs; the same for the values
//     after the transpose reads.  The direct loads are inline assembly with hand-placed waits (the compiler neither knows
//     that they write LDS nor counts them) and, but for a refill of the list, the only vector memory instructions of the loop.
// Measured, 32 query heads over 8 kv heads, d = 128, k = 512, bq = 32, against the form before (metadata in the loop, the whole
// index row in LDS; 64 channels staged through registers at three waves a SIMD, now four, over pages three): 3k tokens 59.2 -> 54.3 us, 32k 553 ->
// 544, over pages 852 -> 763, d = 64 298 -> 265; k = 2048 2903 -> 1771.  By the clock, 32k tokens: a tile takes a
// wave 2850 clocks - operands read and the next keys' loads issued 760, scores and softmax 1070, values read, loads issued and
// products 930, waits for loads 110 - and an item 10100 before its first tile and 2800 after its last of sixteen.
#include "common.h"
#include "launch.h"
#include <type_traits>

namespace hipattn {

namespace {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(2 * sizeof(__bf16)))) __bf16 bf16x2;
typedef __attribute__((__vector_size__(2 * sizeof(float)))) float f32x2;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float f32x16;
typedef __attribute__((__vector_size__(4 * sizeof(short)))) short s16x4;
typedef __attribute__((address_space(3))) s16x4 *lds_s16x4_ptr;
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) const u32x4 *lds_u32x4_ptr;

__device__ __forceinline__ uint32_t pack_bf16(float lo, float hi)
{
    f32x2 x = {lo, hi};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(x, bf16x2));
}

constexpr int kListTiles = 16;   // tiles whose keys are listed; refilled by halves

}  // namespace

// MODE 0: contiguous K/V, rows within reach of a 32-bit lane offset (rows_by_lane_offset): addressed by that and a scalar
//         slice base; MODE 1: paged pool; MODE 2: contiguous, any size (64-bit row addresses).
// WPI: waves per work item.  With 2 or 4 the workgroup takes ONE work item; wave w walks key tiles w, w + WPI, ... with its own
//      softmax state and the states are merged through LDS at the end.
// Waves per SIMD: two with 128 channels; with 64 four (1 to 3 registers spilled; three waves without: 16k tokens, 32 heads 131 us, so
// 125), over pages three, which is what their LDS leaves room for.  Over pages a row's address takes 64-bit multiplies: once for its
// key and value (page sizes 16 and 64 alike; for each of them: 181 us with 64 channels, now 160; 383 with 128, now 328; as many
// waves as a target of four left, two: 229).
template <int D, int MODE, int WPI>
__global__ __launch_bounds__(WPI == 2 ? 128 : kThreads) __attribute__((amdgpu_waves_per_eu(D == 64 ? (MODE == 1 ? 3 : 4) : 2))) void attn_mfma_kernel(KParams p, int log_bk, int mtn, int xcd_map)
{
    constexpr bool PAGED = MODE == 1, SPLIT = WPI > 1;
    constexpr int W = SPLIT ? WPI : 4;   // waves of the workgroup
    constexpr int KS = D / 16;           // k-steps of S^T = K Q^T
    constexpr int CT = D / 32;           // 32-channel tiles of O^T
    constexpr int CPR = D / 8;           // 16-byte chunks per row
    constexpr int RPI = 64 / CPR;        // rows per wave-wide load
    constexpr int NLD = 32 / RPI;        // such loads per 32-row tile
    constexpr int ROWB = D * 2, TILEB = 32 * ROWB;
    constexpr int LIST = kListTiles * 32;
    // LDS: key and value buffer of every wave first (the targets of the direct loads, whose LDS address travels in M0), then
    // the lists
    constexpr int kOffList = W * 2 * TILEB, kOffPage = kOffList + W * LIST * 4;
    static_assert(kOffList <= 65536, "direct-load targets must stay below 64 KB");
    __shared__ __attribute__((aligned(1024))) char lds[kOffPage + (PAGED ? W * LIST * 4 : 0)];

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int col = lane & 31, hh = lane >> 5;
    const int lg = lane / CPR, lc = lane % CPR;  // loading role: gathered keys lg*NLD .. +NLD-1, LDS chunk place lc

    // ---- which (sequence, head, query block, query tile) this wave owns
    const uint32_t groups = (uint32_t)p.batch * (uint32_t)p.hkv;
    const uint32_t per_group = (uint32_t)p.g * (uint32_t)p.nqb * (uint32_t)mtn;
    uint32_t group, o;
    if (!place_item(xcd_map, blockIdx.x, SPLIT ? 1 : 4, SPLIT ? 0 : wave, per_group, groups, group, o)) return;
    const uint32_t gm = (uint32_t)(p.g * mtn), oq = o / gm, rem = o - oq * gm;
    const int qb = p.nqb - 1 - (int)oq;
    const int b = (int)(group / (uint32_t)p.hkv), hk = (int)(group - (uint32_t)b * (uint32_t)p.hkv);
    const int h = hk * p.g + (mtn == 2 ? (int)(rem >> 1) : (int)rem), mt = mtn == 2 ? (int)(rem & 1) : 0;

    const int kv_len = p.kv_lens ? p.kv_lens[b] : p.max_kv_len;
    const int row0 = qb * p.bq + mt * 32;
    const int n_rows = min(32, min(p.bq, p.q_len - qb * p.bq) - mt * 32);
    if (n_rows <= 0) return;
    const int pos0 = kv_len - p.q_len + row0;  // position of this tile's first query row
    const int bk = 1 << log_bk;
    // Key tiles: first the selected blocks, then the sink keys [0, ns), then the window keys
    // [wlo, vis_last).  For a row at position q with vis = min(q+1, kv_len) and
    // w0 = max(vis - n_window, 0): a selected or sink key t counts iff t < w0 (selected also
    // t >= n_sink), a window key iff w0 <= t < vis - so every key counts once.
    const int n_keys = p.kb << log_bk;
    const int vis_last = min(pos0 + n_rows, kv_len);                     // keys any row of the tile may see
    const int wlo = max(min(pos0 + 1, kv_len) - p.n_window, 0);          // window start of the first row
    const int ns = min(p.n_sink, max(vis_last - p.n_window, 0));         // sink keys some row takes as sink
    const int nw = p.n_window > 0 ? max(vis_last - wlo, 0) : 0;
    const int tiles_sel = (n_keys + 31) >> 5, tiles_sink = (ns + 31) >> 5, tiles_win = (nw + 31) >> 5;
    const int n_tiles = tiles_sel + tiles_sink + tiles_win;
    const int w0_first = wlo;                                             // smallest w0 over the rows
    const int w0_last = max(vis_last - p.n_window, 0);                    // largest w0 over the rows

    auto uniform64 = [](int64_t v) __attribute__((always_inline)) {
        return ((int64_t)__builtin_amdgcn_readfirstlane((int)(v >> 32)) << 32) | (uint32_t)__builtin_amdgcn_readfirstlane((int)v);
    };
    const bf16_t *Kbase = (const bf16_t *)p.K, *Vbase = (const bf16_t *)p.V;
    const int64_t seq_off = (int64_t)b * p.ks_b + (int64_t)hk * p.ks_h;  // contiguous layout: row 0 of this slice
    // the same in every lane: as a scalar it becomes the scalar base of the row loads
    const int64_t slice_u = uniform64(seq_off * 2);
    const char *Kseq = (const char *)p.K + slice_u, *Vseq = (const char *)p.V + slice_u;
    const uint32_t row_bytes = (uint32_t)p.ks_r * 2u;
    const int32_t *idx = p.idx_in + (((int64_t)b * p.hq + h) * p.nqb + qb) * p.kb;

    char *kt = lds + wave * 2 * TILEB, *vt = kt + TILEB;
    int *list = (int *)(lds + kOffList) + wave * LIST;     // position of every listed key, or kNoKey
    int *pages = (int *)(lds + kOffPage) + wave * LIST;    // paged pool: the page-table entry of its page
    constexpr int kNoKey = (int)0xff000000;                // negative, and row 0 to a 24-bit multiply
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char *)lds;
    const uint32_t kt_m0 = lds0 + wave * 2 * TILEB, vt_m0 = kt_m0 + TILEB;

    const float c = p.sm_scale * 1.44269504088896340736f;  // scores are kept in log2 units
    constexpr float kSlack = 8.f;
    float m_run = -INFINITY, l_run = 0.f;
    f32x16 oacc[CT];
#pragma unroll
    for (int ct = 0; ct < CT; ++ct)
#pragma unroll
        for (int r = 0; r < 16; ++r) oacc[ct][r] = 0.f;

    // this wave's tiles: all of them, or every WPI-th one
    int nt = SPLIT ? (n_tiles > wave ? (n_tiles - wave + WPI - 1) / WPI : 0) : n_tiles;

    // Lists the keys of the wave's tiles i0 .. i0 + N - 1 (N = 4, 8 or 16; i0 a multiple of 8).  Keys that do not count load
    // row 0 of the sequence (always mapped, finite) and get probability 0.  Bit i % 16 of `any`: some key of tile i may count
    // for some row; of `mask`: some (key, row) pair needs masking.
    uint32_t any = 0, mask = 0;
    const uint32_t plain = (uint32_t)max(w0_first - p.n_sink, 0);   // (w0_first <= kv_len)
    // (All index entries are read first, then all page entries: two latencies, not one per tile.)
    auto index_entry = [&](int i0, int u) __attribute__((always_inline)) {
        const int tile = SPLIT ? wave + WPI * (i0 + 2 * u + hh) : i0 + 2 * u + hh;
        return idx[min(tile * 32 + col, n_keys - 1) >> log_bk];
    };
    auto list_tiles = [&](int i0, auto count, int (&t)[kListTiles / 2]) __attribute__((always_inline)) {
        constexpr int N = decltype(count)::value;
        const uint32_t at = (uint32_t)i0 % kListTiles, bits = ((1u << N) - 1u) << at;
        any &= ~bits;
        mask &= ~bits;
#pragma unroll
        for (int u = 0; u < N / 2; ++u) {
            const int tile = SPLIT ? wave + WPI * (i0 + 2 * u + hh) : i0 + 2 * u + hh;
            const int ki = tile * 32 + col, first = t[u], tk = first + (ki & (bk - 1));
            // nearly always: 64 selected keys that all rows see
            if (__ballot((uint32_t)(tk - p.n_sink) < plain && ki < n_keys) == ~0ull) {
                t[u] = tk;
                any |= 3u << (at + 2 * u);
            } else {
                bool counts, care = true;
                if (tile < tiles_sel) {
                    t[u] = ki < n_keys && first >= 0 && first < kv_len && tk < kv_len && tk >= p.n_sink ? tk : -1;
                    counts = t[u] >= 0 && t[u] < w0_last;
                    care = t[u] < 0 || t[u] >= w0_first;
                } else {
                    const bool sink = tile < tiles_sel + tiles_sink;
                    const int te = ki - (sink ? tiles_sel * 32 : (tiles_sel + tiles_sink) * 32 - wlo);
                    t[u] = te < (sink ? ns : vis_last) ? te : -1;
                    counts = tile < n_tiles;
                }
                const uint64_t bc = __ballot(counts), bm = __ballot(care);
                any |= (((uint32_t)bc != 0 ? 1u : 0u) | ((uint32_t)(bc >> 32) != 0 ? 2u : 0u)) << (at + 2 * u);
                mask |= (((uint32_t)bm != 0 ? 1u : 0u) | ((uint32_t)(bm >> 32) != 0 ? 2u : 0u)) << (at + 2 * u);
            }
            list[(at + 2 * u) * 32 + lane] = t[u] >= 0 ? t[u] : kNoKey;
        }
        if constexpr (PAGED) {
#pragma unroll
            for (int u = 0; u < N / 2; ++u) t[u] = page_of_row<true>(p, b, max(t[u], 0));
#pragma unroll
            for (int u = 0; u < N / 2; ++u) pages[(at + 2 * u) * 32 + lane] = t[u];
        }
        any = (uint32_t)__builtin_amdgcn_readfirstlane((int)any);
        mask = (uint32_t)__builtin_amdgcn_readfirstlane((int)mask);
    };
    // Where this lane's rows of a listed tile are.  Paged: bytes from the start of the pool, once for the key and the value; bit 0: of
    // the backing pool (a negative page-table entry).
    struct rows_t { uint32_t off[PAGED ? 1 : NLD]; int64_t at[PAGED ? NLD : 1]; };
    auto read_rows = [&](int i, rows_t &R) __attribute__((always_inline)) {
        const int x = (i % kListTiles) * 32 + lg * NLD;
#pragma unroll
        for (int j = 0; j < NLD; j += 4) {
            const int4 t4 = *(const int4 *)(list + x + j);
            if constexpr (PAGED) {
                const int4 p4 = *(const int4 *)(pages + x + j);
                const int tk[4] = {t4.x, t4.y, t4.z, t4.w}, pg[4] = {p4.x, p4.y, p4.z, p4.w};
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    R.at[j + e] = row_offset_in<true>(p, b, hk, max(tk[e], 0), page_in_pool(pg[e])) * 2 + (pg[e] < 0 ? 1 : 0);
            } else {
                R.off[j] = (uint32_t)t4.x; R.off[j + 1] = (uint32_t)t4.y; R.off[j + 2] = (uint32_t)t4.z; R.off[j + 3] = (uint32_t)t4.w;
            }
        }
        if constexpr (MODE == 0) {
#pragma unroll
            for (int j = 0; j < NLD; ++j) R.off[j] = __umul24(R.off[j], row_bytes);
        }
    };
    // The direct loads of a tile's keys (VAL = false) or values (VAL = true): load j brings gathered key x = NLD lg + j to LDS
    // row RPI j + lg, this lane the 16-byte chunk that belongs at place lc of that row.  (M0 is a reserved register: the
    // compiler warns that it does not track the clobber.  It is written and consumed inside one asm statement, and nothing else
    // in this kernel uses M0.)
    // An instruction offset moves both the global and the LDS address, so one M0 serves four loads; what it adds to the global
    // address is taken off the lane's part (kRowBias bytes stand before it so that nothing gets negative).
    const uint32_t kchunk = (uint32_t)((D == 128 ? lc ^ ((lg & 1) << 3) : lc ^ ((lg & 2) << 1)) << 4), vchunk = (uint32_t)(lc << 4);
    auto issue_rows = [&](const rows_t &R, bool val) __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < NLD; ++j) {
            const int rot = D == 128 ? ((j & 3) << 1) | ((j >> 2) & 1) : (j & 1) << 1;   // value place = chunk pair ^ rot
            uint32_t chunk = val ? vchunk : kchunk;
            asm volatile("" : "+v"(chunk));   // (not a register per load)
            chunk ^= (uint32_t)(val ? rot << 5 : j << 4);
            const uint32_t dst = __builtin_amdgcn_readfirstlane((val ? vt_m0 : kt_m0) + (j & ~3) * 1024);
            const int back = (j & 3) * 1024;
            if constexpr (MODE == 0) {
                const uint32_t vo = R.off[j] + chunk + (uint32_t)(kRowBias - back);
                const char *base = (val ? Vseq : Kseq) - kRowBias;
                if (j & 3) asm volatile("global_load_lds_dwordx4 %0, %1 offset:%2" :: "v"(vo), "s"(base), "i"(back) : "memory");
                else asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1"
                                  :: "v"(vo), "s"(base), "s"(dst) : "memory", "m0");
            } else {
                const char *src;
                if constexpr (PAGED) {
                    const char *pool = (const char *)(val ? p.V : p.K), *backing = (const char *)(val ? p.Vback : p.Kback) - 1;
                    src = (R.at[j] & 1 ? backing : pool) + R.at[j] + chunk;
                } else {
                    src = (const char *)((val ? Vbase : Kbase) + seq_off + (int64_t)max((int)R.off[j], 0) * p.ks_r) + chunk;
                }
                src -= back;
                if (j & 3) asm volatile("global_load_lds_dwordx4 %0, off offset:%1" :: "v"(src), "i"(back) : "memory");
                else asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off" :: "v"(src), "s"(dst) : "memory", "m0");
            }
        }
    };
    // row r of the score tile is gathered key xkey(r)
    auto xkey = [](int r) __attribute__((always_inline)) { return D == 128 ? r : (r & 25) | ((r & 2) << 1) | ((r & 4) >> 1); };

    // (no more tiles than there are, by fours: 64 to 256 keys of 4096 query tiles, all sixteen listed / so many: 25.0 / 23.3 us, 29.4 / 27.4,
    // 39.5 / 38.1)
    // (64 channels over contiguous rows at a wave an item: the choice spills two more of the loop's registers, 36.5 -> 37.5 us at 4096
    // tiles of k = 512, and gives 0.3 us at k = 64)
    constexpr bool kChoose = D == 128 || PAGED || SPLIT;
    int entry[kListTiles / 2];
#pragma unroll
    for (int u = 0; u < kListTiles / 2; ++u) entry[u] = index_entry(0, u);
    // The query tile comes in through the key buffer by coalesced loads of RPI rows, behind the index entries that
    // the listing needs first.  (Straight into registers, a row a lane, each of eight loads
    // was 64 cache accesses, and the entries waited behind them: 11800 of an item's 61000 clocks until its first tile was there
    // at 32k tokens, now 10100; 64 channels 11600 of 64500, now 9600 of 59300.  The listing does not run under these loads: the compiler
    // does not count them, so its waits for the entries are waits for the tile too.)
    // Tiles of up to 8 or 16 rows load so many, row x to LDS row x: with all 32, as copies of the last one, 8-row blocks of 8192 tokens took 4 %
    // more (two sequences of 16 heads, k = 256: 128 channels 230 us, straight into registers 220, so 220; 64 channels 126 / 122 / 118).  Others
    // go where a key tile goes, rows NLD apart in a load: with neighbouring rows in a load 32k tokens take 1 % more (529 / 535 us).
    const bool few = n_rows <= 16;
    auto issue_query = [&](int j, int row, uint32_t chunk) __attribute__((always_inline)) {
        const char *Qb = (const char *)((const bf16_t *)p.Q + (int64_t)b * p.qs_b + (int64_t)h * p.qs_h + (int64_t)row0 * p.qs_r);
        const char *src = Qb + (int64_t)min(row, n_rows - 1) * p.qs_r * 2 + chunk;
        const uint32_t dst = __builtin_amdgcn_readfirstlane(kt_m0 + j * 1024);
        asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off" :: "v"(src), "s"(dst) : "memory", "m0");
    };
    if (!few) {
#pragma unroll
        for (int j = 0; j < NLD; ++j) issue_query(j, lg * NLD + j, kchunk ^ (uint32_t)(j << 4));
    } else {
        const uint32_t qchunk = (uint32_t)((D == 128 ? lc ^ lg : lc ^ (lg >> 1)) << 4);
        auto eight_rows = [&](auto from) __attribute__((always_inline)) {
            constexpr int j0 = decltype(from)::value / RPI;
#pragma unroll
            for (int j = j0; j < j0 + 8 / RPI; ++j) issue_query(j, RPI * j + lg, qchunk ^ (uint32_t)((D == 128 ? j & 3 : j & 1) << 6));
        };
        eight_rows(std::integral_constant<int, 0>{});
        if (n_rows > 8) eight_rows(std::integral_constant<int, 8>{});
    }
    if (kChoose && nt <= 4) list_tiles(0, std::integral_constant<int, 4>{}, entry);
    else if (kChoose && nt <= 8) list_tiles(0, std::integral_constant<int, 8>{}, entry);
    else list_tiles(0, std::integral_constant<int, kListTiles>{}, entry);
    // (the tail of a list that ends early: a prefix with fewer keys than k)
    if (nt <= kListTiles) nt = any ? 32 - __builtin_clz(any) : 0;
    wave_lds_sync();
    // query tile as B operand (lane: query col, channels kk*16 + hh*8 ..)
    bf16x8 qf[KS];
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    {
        const int sw = D == 128 ? col & 15 : few ? (col >> 1) & 7 : (col & 3) | ((col >> 1) & 4);
        const uint32_t qrow = (uint32_t)((few ? col : RPI * (col % NLD) + col / NLD) * ROWB + ((hh ^ sw) << 4)) + kt_m0;
#pragma unroll
        for (int kk = 0; kk < KS; ++kk) qf[kk] = __builtin_bit_cast(bf16x8, *(lds_u32x4_ptr)(uintptr_t)(qrow ^ (uint32_t)(kk << 5)));
        if (n_rows < 32) {   // (rows past the last one need not have been loaded)
#pragma unroll
            for (int kk = 0; kk < KS; ++kk) qf[kk] = __builtin_bit_cast(bf16x8, col < n_rows ? __builtin_bit_cast(u32x4, qf[kk]) : u32x4{0, 0, 0, 0});
        }
    }
    if (nt > 0) {
        rows_t R0;
        read_rows(0, R0);
        asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");   // nothing of the compiler's is in flight from here on
        issue_rows(R0, false);
        issue_rows(R0, true);
    }
    // Outstanding vector memory operations at the top of iteration i, oldest first: keys of tile i (NLD), values of
    // tile i (NLD).
    for (int i = 0; i < nt; ++i) {
        const bool more = i + 1 < nt;
        const uint32_t bit = 1u << (i % kListTiles);
        const bool counts = any & bit;
        if (more && i + 1 >= kListTiles && (i + 1) % (kListTiles / 2) == 0) {
            // tiles i + 1 .. i + 8 go where tiles i - 15 .. i - 8 were (this tile's keys are in the other half)
            int entry[kListTiles / 2];
#pragma unroll
            for (int u = 0; u < kListTiles / 4; ++u) entry[u] = index_entry(i + 1, u);
            list_tiles(i + 1, std::integral_constant<int, kListTiles / 2>{}, entry);
            wave_lds_sync();
        }
        // ---- keys of tile i have landed; its values may still be on their way
        asm volatile("s_waitcnt vmcnt(%0)" :: "i"(NLD) : "memory");
        u32x4 kv[KS];
        if (counts) {
            const int x = xkey(col);
            const int sw = D == 128 ? x & 15 : (x & 3) | ((x >> 1) & 4);
            uint32_t krow = (uint32_t)((RPI * (x % NLD) + x / NLD) * ROWB + ((hh ^ sw) << 4)) + kt_m0;
            asm volatile("" : "+v"(krow));   // (one register and exclusive-ors instead of a register per read)
#pragma unroll
            for (int kk = 0; kk < KS; ++kk) kv[kk] = *(lds_u32x4_ptr)(uintptr_t)(krow ^ (uint32_t)(kk << 5));
        }
        rows_t R1;
        if (more) read_rows(i + 1, R1);
        // the key operands are in registers (and this lane's rows of the next tile are known): the key buffer may be refilled
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        if (more) issue_rows(R1, false);
        // outstanding now: values of tile i [, keys of tile i+1]

        f32x16 sacc;
        bf16x8 pb[2];
        if (counts) {
            // ---- S^T = K Q^T: A = key rows (lane: key xkey(col)), B = queries
#pragma unroll
            for (int r = 0; r < 16; ++r) sacc[r] = 0.f;
#pragma unroll
            for (int kk = 0; kk < KS; ++kk)
                sacc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, kv[kk]), qf[kk], sacc, 0, 0, 0);

            // ---- online softmax for query `col` (both half-waves hold the same query)
            float s[16], mx = -INFINITY;
            if (mask & bit) {
                // positions of the 16 keys this lane holds scores for: rows 8g + 4hh + {0..3};
                // admissible range [lo, hi) of key positions for this lane's query
                const bool window = (SPLIT ? wave + WPI * i : i) >= tiles_sel + tiles_sink;
                const int visq = min(pos0 + col + 1, kv_len);
                const int w0q = max(visq - p.n_window, 0);
                const int lo = window ? w0q : 0, hi = window ? visq : w0q;
                const int *tk = list + (i % kListTiles) * 32;
#pragma unroll
                for (int g = 0; g < 4; ++g) {
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const int tkey = tk[xkey(8 * g + e) + (D == 128 ? 4 : 2) * hh];
                        s[4 * g + e] = tkey >= lo && tkey < hi ? sacc[4 * g + e] : -INFINITY;
                    }
                    asm volatile("" ::: "memory");   // (four positions in registers at a time)
                }
            } else {
#pragma unroll
                for (int r = 0; r < 16; ++r) s[r] = sacc[r];
            }
            // raw scores here; the scale (c > 0) is applied to the maximum and inside the exponent
#pragma unroll
            for (int r = 0; r < 16; ++r) mx = fmaxf(mx, s[r]);
            {   // other half of the query's keys: lane ^ 32
                const unsigned u = __float_as_uint(mx);
                auto sw = __builtin_amdgcn_permlane32_swap(u, u, false, false);
                mx = fmaxf(__uint_as_float(sw[0]), __uint_as_float(sw[1])) * c;
            }
            // The running reference m_run only has to bound the exponents, it need not be the exact
            // maximum: it moves (and the accumulators are rescaled) only when a tile's maximum exceeds
            // it by more than kSlack (log2 units; probabilities then stay below 2^kSlack, far inside
            // the range of fp32 sums and bf16 operands).  The final division by l cancels the reference.
            const float m_new = mx > m_run + kSlack ? mx : m_run;
            const float m_safe = m_new == -INFINITY ? 0.f : m_new;
            const float alpha = __builtin_amdgcn_exp2f(m_run - m_safe);
#pragma unroll
            for (int r = 0; r < 16; ++r) s[r] = __builtin_amdgcn_exp2f(fmaf(s[r], c, -m_safe));
            // P^T as B operand of the two 16-key steps (registers 8*st .. 8*st+7), rounded to bf16; the row sum runs
            // over the rounded values (v_dot2_f32_bf16 against ones, fp32 accumulation)
            float lsum = 0.f;
            {
                const bf16x2 ones = __builtin_bit_cast(bf16x2, 0x3f803f80u);
#pragma unroll
                for (int st = 0; st < 2; ++st) {
                    uint32_t hi[4];
#pragma unroll
                    for (int e2 = 0; e2 < 4; ++e2) {
                        hi[e2] = pack_bf16(s[8 * st + 2 * e2], s[8 * st + 2 * e2 + 1]);
                        lsum = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, hi[e2]), ones, lsum, false);
                    }
                    pb[st] = __builtin_bit_cast(bf16x8, make_uint4(hi[0], hi[1], hi[2], hi[3]));
                }
            }
            l_run = l_run * alpha + lsum;
            m_run = m_new;
            if (__ballot(alpha != 1.f) != 0) {
#pragma unroll
                for (int ct = 0; ct < CT; ++ct)
#pragma unroll
                    for (int r = 0; r < 16; ++r) oacc[ct][r] *= alpha;
            }
        }

        // ---- the values of tile i have landed
        if (more) asm volatile("s_waitcnt vmcnt(%0)" :: "i"(NLD) : "memory");
        else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        bf16x8 va[2][CT];
        if (counts) {
            // Value tile read back channel-major with the LDS transpose read.  ds_read_b64_tr_b16 works on blocks of
            // 16 lanes: lanes 4e .. 4e+3 of a block point at 16 consecutive bf16 of source row e (e = 0..3), and lane
            // i of the block receives element i of each of the four rows.  Block = (channel half cb, key half hh):
            // rows are score rows 16 st [+ 8] + 4 hh + e, so a lane ends up with 4 keys of its channel - half an A operand
            // per read - in the order in which P^T holds them.
            const int i16 = lane & 15, cb = (lane >> 4) & 1, e = i16 >> 2;
            const int x0 = xkey(4 * hh + e);   // (adding 8 or 16 to the row adds 8 or 16 to the key: NLD divides both)
            const int vsw = D == 128 ? 2 * e + hh : (x0 & 1) << 1;   // (x0 % 8 rotated left by one bit)
            uint32_t vrow = (uint32_t)((RPI * (x0 % NLD) + x0 / NLD) * ROWB + ((cb ^ vsw) << 5) + (i16 & 3) * 8) + vt_m0;
            asm volatile("" : "+v"(vrow));
#pragma unroll
            for (int st = 0; st < 2; ++st)
#pragma unroll
                for (int ct = 0; ct < CT; ++ct) {
                    const uint32_t place = vrow ^ (uint32_t)(ct << 6);
                    const s16x4 lo4 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_ptr)(uintptr_t)(place + (16 * st / NLD) * ROWB));
                    const s16x4 hi4 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_ptr)(uintptr_t)(place + ((16 * st + 8) / NLD) * ROWB));
                    const uint2 a = __builtin_bit_cast(uint2, lo4), c2 = __builtin_bit_cast(uint2, hi4);
                    va[st][ct] = __builtin_bit_cast(bf16x8, make_uint4(a.x, a.y, c2.x, c2.y));
                }
        }
        // the value operands are in registers: the value buffer may be refilled
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        if (more) issue_rows(R1, true);
        if (counts) {
            // ---- O^T += V^T P^T (the CT accumulators are independent)
#pragma unroll
            for (int st = 0; st < 2; ++st)
#pragma unroll
                for (int ct = 0; ct < CT; ++ct) oacc[ct] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(va[st][ct], pb[st], oacc[ct], 0, 0, 0);
        }
    }

    bf16_t *Ob = (bf16_t *)p.O + (int64_t)b * p.os_b + (int64_t)h * p.os_h + (int64_t)row0 * p.os_r;
    if constexpr (SPLIT) {
        // Every wave leaves its state (running reference, partial sum, accumulators) in its own buffers, lane-contiguous, and
        // merges a share of the channels: with m = max of the references, every state is rescaled by 2^(m_w - m) before it
        // is added (the usual merge of online-softmax states).  Nothing of a list is read any more.
        constexpr int OWN = WPI < CT ? CT / WPI : 1;   // 32-channel tiles per merging wave
        float *st = (float *)kt, *ml = (float *)list;
#pragma unroll
        for (int ct = 0; ct < CT; ++ct)
            if (ct / OWN != wave) {
#pragma unroll
                for (int r = 0; r < 16; ++r) st[(ct * 16 + r) * 64 + lane] = oacc[ct][r];
            }
        const float l_own = l_run + __shfl_xor(l_run, 32, 64);
        ml[lane] = m_run;
        ml[64 + lane] = l_own;
        __syncthreads();
        if (wave * OWN >= CT) return;
        float m = m_run, f[WPI], l = 0.f;
#pragma unroll
        for (int w = 0; w < WPI; ++w) m = fmaxf(m, ((const float *)(lds + kOffList))[w * LIST + lane]);
        const float m_safe = m == -INFINITY ? 0.f : m;
#pragma unroll
        for (int w = 0; w < WPI; ++w) {
            const float *mlw = (const float *)(lds + kOffList) + w * LIST;
            f[w] = __builtin_amdgcn_exp2f(mlw[lane] - m_safe);
            l = fmaf(mlw[64 + lane], f[w], l);
        }
        const float inv = l > 0.f ? 1.f / l : 0.f;
#pragma unroll
        for (int ct = 0; ct < CT; ++ct) {
            if (ct / OWN != wave) continue;
            float own = 0.f;
#pragma unroll
            for (int w = 0; w < WPI; ++w) own = w == wave ? f[w] : own;
            float out[16];
#pragma unroll
            for (int r = 0; r < 16; ++r) out[r] = oacc[ct][r] * own;
#pragma unroll
            for (int w = 0; w < WPI; ++w) {
                if (w == wave) continue;
                const float *sw = (const float *)(lds + w * 2 * TILEB) + ct * 16 * 64 + lane;
#pragma unroll
                for (int r = 0; r < 16; ++r) out[r] = fmaf(sw[r * 64], f[w], out[r]);
            }
            if (col < n_rows) {
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    uint2 u;
                    u.x = pack_bf16(out[4 * g + 0] * inv, out[4 * g + 1] * inv);
                    u.y = pack_bf16(out[4 * g + 2] * inv, out[4 * g + 3] * inv);
                    *(uint2 *)(Ob + (int64_t)col * p.os_r + ct * 32 + g * 8 + hh * 4) = u;
                }
            }
        }
        return;
    }

    // ---- normalise, transpose through LDS (16-byte chunk c of row r at place c ^ (r % CPR)), coalesced store
    const float l_tot = l_run + __shfl_xor(l_run, 32, 64);
    const float inv = l_tot > 0.f ? 1.f / l_tot : 0.f;
#pragma unroll
    for (int ct = 0; ct < CT; ++ct)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            uint2 u;
            u.x = pack_bf16(oacc[ct][4 * g + 0] * inv, oacc[ct][4 * g + 1] * inv);
            u.y = pack_bf16(oacc[ct][4 * g + 2] * inv, oacc[ct][4 * g + 3] * inv);
            *(uint2 *)(vt + col * ROWB + (((ct * 4 + g) ^ (col & (CPR - 1))) << 4) + hh * 8) = u;
        }
    wave_lds_sync();
#pragma unroll
    for (int i = 0; i < NLD; ++i) {
        const int row = lg + i * RPI;
        if (row < n_rows) *(uint4 *)(Ob + (int64_t)row * p.os_r + lc * 8) = *(const uint4 *)(vt + row * ROWB + ((lc ^ (row & (CPR - 1))) << 4));
    }
}

bool attn_mfma_supported(const KParams &p, bool bf16)
{
    return bf16 && p.q_len > 1 && p.bk <= 16 && (p.bk & (p.bk - 1)) == 0 && p.bq <= 64;
}

hipError_t launch_attn_mfma(const KParams &p, hipStream_t st)
{
    int log_bk = 0;
    while ((1 << log_bk) < p.bk) ++log_bk;
    const int mtn = (p.bq + 31) / 32;
    const int64_t groups = (int64_t)p.batch * p.hkv;
    const int64_t per_group = (int64_t)p.g * p.nqb * mtn;
    const int64_t waves = groups * per_group;
    if (waves == 0) return hipSuccess;
    // groups worked on at a time (measured: all eight up to 128k tokens at head dim 128, four at 256k, one at a million; as many as
    // divide their number against linear order: twelve of four heads, 32k tokens, the last 2656 rows 115.6 / 89.2 us, over pages 125.6 / 96.0;
    // 36 of three 273 / 206)
    const int gc = groups_at_a_time_of(groups, (int64_t)p.max_kv_len * p.d * 4, 768LL << 20);
    const int wpi = attn_waves_per_item(waves, p.kb * p.bk, p.d, p.page_table != nullptr, groups, gc, p.max_kv_len);
    const dim3 grid((unsigned)placed_workgroups(gc, wpi > 1 ? 1 : 4, per_group, groups)), block(wpi == 2 ? 128 : kThreads);
    const int mode = p.page_table ? 1 : rows_by_lane_offset(p.max_kv_len, p.ks_r * 2, p.d) ? 0 : 2;
    const auto launch = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, grid, block, 0, st, p, log_bk, mtn, gc);
        return hipGetLastError();
    };
#define HIPATTN_MODE(DV, WV) (mode == 0 ? launch(attn_mfma_kernel<DV, 0, WV>) : mode == 1 ? launch(attn_mfma_kernel<DV, 1, WV>) : launch(attn_mfma_kernel<DV, 2, WV>))
    if (p.d == 64) return wpi == 4 ? HIPATTN_MODE(64, 4) : wpi == 2 ? HIPATTN_MODE(64, 2) : HIPATTN_MODE(64, 1);
    return wpi == 4 ? HIPATTN_MODE(128, 4) : wpi == 2 ? HIPATTN_MODE(128, 2) : HIPATTN_MODE(128, 1);
#undef HIPATTN_MODE
}

}  // namespace hipattn
