// Rules by which the launchers choose between kernels, in plain C++ so that a host test compiles them as they stand.
#pragma once
#include <stdint.h>

namespace hipattn {

// Prefill sparse attention addresses the rows of a contiguous (sequence, kv head) slice by unsigned 32-bit byte offsets from a
// scalar base that lies kRowBias bytes before the slice: one M0 serves four loads, whose instruction offsets of up to
// kRowBias move the global address as well and are taken off the lane's part.  The largest offset is that of the last row's
// last chunk plus the bias.  Row number and pitch go through a 24-bit multiply.
constexpr int kRowBias = 3 * 1024;
inline bool rows_by_lane_offset(int64_t max_kv_len, int64_t row_bytes, int d)
{
    return max_kv_len < (1 << 24) && row_bytes < (1 << 24) && (max_kv_len - 1) * row_bytes + 2 * d + kRowBias <= (1LL << 32);
}

// Prefill mask: a workgroup per work item (its waves share the tiles and select redundantly) or a wave, by the number of work items.
// The fewer blocks a round has, the less there is to share.  Measured, 16384 tokens, 32 heads over 8 kv heads, a wave / a workgroup
// per item, us; 128 channels and bk = 2 if not said otherwise:
//   k/bk      512 items      768         1024          1504
//   32        35 / 29        36 / 34     36 / 38       41 / 58     64-row blocks, bk = 4: 52 / 37, 52 / 42, 52 / 65, 61 / 74
//   64        45 / 32        44 / 36     44 / 41       52 / 65     bk = 1: 37 / 31, 38 / 36, 37 / 40, 43 / 62
//   128       60 / 36        59 / 42     58 / 49       72 / 75     64 channels 45 / 29, 46 / 33, 46 / 37, 52 / 47
//   256       90 / 49        89 / 58     89 / 72      108 / 106    64-row blocks, bk = 4, over pages 153 / 81, 154 / 123, 157 / 149, 220 / 213
//   512      128 / 68       127 / 86    127 / 105     161 / 150    bk = 1: 105 / 61, 105 / 71, 104 / 111, 124 / 129
//   1024     172 / 91          -        174 / 163     208 / 233    16 items 205 / 66; 64-row blocks, bk = 4: 16 items 223 / 66, 512 220 / 106,
//                                                                  1024 225 / 195; 64 channels, bk = 1 132 / 73, -, 135 / 134, 146 / 191
// 2048 items, k/bk = 256, over 32k tokens 157 / 182.
// Over pages with 128 channels and k/bk above 512 a wave per item would leave one wave a SIMD, a workgroup two: a workgroup whatever
// the number (k/bk = 1024, 1024 items 210 / 184, 2048 413 / 349, 16384 2426 / 1933; 64-row blocks, bk = 4, 8192 items 1608 / 1212;
// bk = 8, 16384 items 2885 / 1982; k/bk = 600, bk = 1, 16384 items 2039 / 2059).
// What is shared inside a workgroup that holds four heads of a query block has to be found in the L2 by workgroups of a head each, so
// beyond 768 items (512 where the groups, of a sequence and kv head each, go in linear order) the keys that an XCD reads at a time must
// not be too many.  `gc` of place_item, 0 in linear order; k/bk = 256, bk = 2, a wave / a workgroup per item:
//   eight groups (gc = 8): 64k tokens 768 items 147 / 112, 1024 148 / 140, 1472 187 / 198; 128k 182 / 178, 203 / 228, 270 / 318
//   twelve (4): 16k about 900 items 104 / 87, 1400 121 / 111; 32k 128 / 130, 152 / 173; four, 64k 1024 items 149 / 156, 1472 186 / 219
//   six (2): 16k 103 / 92, 119 / 113; 32k 128 / 146, 150 / 187
//   one, three, five (0): 16k 89 / 68, 103 / 93, 105 / 111; 32k 124 / 98, 128 / 147, 132 / 159
//   over pages, where four heads of a workgroup share nothing: eight groups 128k 215 / 178, 232 / 231, 303 / 314; twelve 32k 153 /
//   130, 183 / 180; six 154 / 148, 182 / 193; three and five in linear order 153 / 148, 183 / 195, 157 / 161, 192 / 211
// (The line at 1024 is at 768 for two query tiles of 128 channels: so many workgroups run at a time.)
inline bool mask_item_per_workgroup(int64_t units, int kb, int d, bool two_tiles, bool paged, int64_t groups, int gc, int64_t max_kv_len)
{
    if (units <= 512) return true;
    if (paged && d == 128 && kb > 512) return true;   // (the kernel of the other form is not built)
    const int64_t mb = 1 << 20, key_bytes = max_kv_len * d * 2;
    const bool few = units <= (two_tiles && d == 128 ? 768 : 1024);
    if (few ? kb <= 32 : units > 1536 || kb <= 128 || kb > 512) return false;
    if (gc == 0) return key_bytes * groups <= 12 * mb;
    return paged || units <= 768 || key_bytes <= (few ? 2 : 1) * mb * gc;
}

// Prefill mask, k/bk up to 128: do nodes hand on their first blocks' scores, so that branches of the last two rounds that an earlier round
// has scored are left out, or their own scores alone (one branch a node from the second round on with the first or last block as
// representative, in the last round with the centre).  With the first or last block nothing else is known.  With the centre the rows that are
// not gathered pay for the bookkeeping but where they are 128 bytes each.  Measured, 16 heads over 4 kv heads, bq = 32, own scores alone / all, us:
//   last block as representative, 16k tokens: 128 channels, bk = 2, k/bk = 32 78.7 / 85.3, 64 100.8 / 103.2; 64 channels, bk = 1, k/bk = 16 65.4 / 72.0
//   centre, 16k tokens, bk = 1: 64 channels k/bk = 16 59.4 / 62.0 (33k tokens 112 / 120), 64 67.6 / 69.5 (135 / 142), 96 79.6 / 76.9 (159 / 160), 128
//     85.8 / 82.5; over 64-row blocks, 33k tokens, k/bk = 64 102.9 / 98.5; bk = 2, k/bk = 16 61.0 / 60.4, 48 76.7 / 72.6;
//     128 channels, bk = 1, k/bk = 16 74.4 / 73.7, 48 91.0 / 87.6; bk = 2, k/bk = 32 97.0 / 92.3, 48 120 / 111
inline bool mask_hands_on(int kb, int d, int scored_rows, bool two_tiles, int rep_pos)
{
    return rep_pos == 0 && (d == 128 || scored_rows > 1 || two_tiles || kb > 64);
}

// Workgroups of the prefill mask kernel that may share a compute unit (0: as many as fit), by the bytes of a kv head's keys.  Where
// these do not stay in the caches the kernel waits for the memory side, and what counts is how often the waves of an XCD meet in
// its L2: fewer workgroups at a time (the launch asks for LDS that it does not use) meet more often.  Measured, in ms, as many as
// fit / two / one to a compute unit; four heads a group if not said otherwise:
//   whole prompts, 32 heads, bq = 32, bk = 2, k = 512: 64k tokens (16 MB) 4.52 / 4.96 / 7.42;  128k (32 MB) 14.34 / 14.05 / 18.45,
//     stored token by token (rows 2 KB apart) 15.78 / 14.88 / 18.35;  256k (64 MB) - / 39.4 / 45.1;
//   bq = 64, bk = 4, k = 2048: 1M tokens (256 MB) - / 387.4 / 376.7;
//   no grouping, 8 heads: the last 64k rows of 128k tokens 3.10 / 2.97 / 2.80, the last 32k of 256k 2.21 / 2.10 / 2.05;
//   64 channels: the last 32k rows of 512k tokens (64 MB) 4.06 / 3.91 / 5.63, the last 16k of 1M (128 MB) 2.48 / 2.37 / 3.25.
// Where the keys do stay, two cost 10 % and one 60 %, so the cut is left out where the lengths are only known on the device
// (kv_lens): max_kv_len is then what the cache could hold.  (32k tokens in a table for 1M: 0.72 ms, one to a compute unit 1.13; what
// it would give over pages: the last 8k rows of 128k tokens 1.38 / 1.35 / 1.69, the last 4k of 256k 0.93 / 0.91 / 1.07.)
inline int mask_workgroups_per_cu(int64_t max_kv_len, int d, bool lengths_known)
{
    const int64_t key_bytes = max_kv_len * d * 2;
    if (!lengths_known || key_bytes <= (24 << 20)) return 0;
    if (d == 64) return key_bytes > (128 << 20) ? 2 : 0;
    return key_bytes > (128 << 20) ? 1 : 2;
}

// Decode mask estimation: waves per (sequence, head), by the number of problems (`step`: branches per stage of a wave,
// `step8`: with eight rows a stage, as four waves and one take them):
//   up to 256 (one per compute unit) and k/bk <= 512: sixteen, unless the branches of a round are one stage or less for each
//       of four waves.  Measured, d = 128, bk = 2, four waves / sixteen: 32 problems of 32768 tokens k/bk = 32 20.0 / 18.4 us,
//       256 42.7 / 37.5, of 65536 tokens over pages 512 119 / 86; 256 problems k/bk = 32 23.8 / 22.5, 256 55.6 / 53.6; beyond a
//       problem per compute unit 320 problems 256 72 / 99, 384 problems of 65536 tokens 512 167 / 202.  Stages of four rows (eight
//       make no difference at sixteen waves: 37.5 / 37.5 and 53.6 / 53.8 us, k/bk = 512 over pages 79 / 86, contiguous 115 / 109).
//       With eight scored rows a block and k/bk above 256 the sixteen-wave kernels spill (21 registers over pages, 6 contiguous)
//       and are mostly the better ones all the same: k/bk = 512, 32768 tokens, four / sixteen: 32
//       problems 86.9 / 67.8 us, over pages 151 / 79.6, 64 channels 48.4 / 41.8; 256 problems 140 / 159, over pages 225 / 159.
//       A contiguous slice of 2 GB or more, a million tokens stored token by token with 8 kv heads: 32 problems k/bk = 256 91.9 /
//       78.6, 128 problems 512 195 / 188.
//   up to 8192, or 16384 of 128 channels over contiguous keys with k/bk <= 256 and eight stages or more: four, so that enough loads
//       are in flight per compute unit and the selection of one problem overlaps with the loads of the others; beyond that one
//       (nothing computed twice, no barriers).  Measured with 32 query heads over 8 kv heads, four waves / one: 8192 problems of
//       8192 tokens, k/bk = 256 681 / 711 us; 16384 of 4096 849 / 893, of 8192, k/bk = 128 963 / 1007, of 3000, k/bk = 512 832 /
//       756; 32768 of 2048, k/bk = 256 944 / 928.  12288 of 4096 tokens, bk = 2: k/bk = 16 240 / 166, 32 (four stages) 263 / 248,
//       64 350 / 369, 256 642 / 673; over pages 32 322 / 255, 64 420 / 391, 256 759 / 727; with 64 channels 16 219 / 81, 64 220 /
//       184, 256 355 / 342, over pages 64 264 / 189, 256 418 / 369.  (So many problems over slices of 2 GB or more do not fit the
//       memory: there is no such kernel, they take four.)
enum class Slice { paged, narrow, wide };   // contiguous: within 32-bit offsets or not
inline int decode_mask_waves(int64_t problems, int kb, int d, int step, int step8, Slice slice)
{
    if (problems <= 256 && kb <= 512 && 2 * kb > 4 * step) return 16;
    if (problems <= 8192 || slice == Slice::wide) return 4;
    return problems <= 16384 && slice == Slice::narrow && d == 128 && kb <= 256 && 2 * kb >= 8 * step8 ? 4 : 1;
}

// Prefill sparse attention: waves per work item (query tile), by the number of items and of selected keys (32 a tile).  Measured, 16384
// tokens, one / two / four waves per item, us (11 us is what a launch takes):
//   128 channels   64 items k = 512 21.6 / 12.7 / 11.0;  512 k = 256 14.5 / 11.5 / 11.6, 512 22.4 / 16.6 / 15.4;  1024 k = 128 12.0 / 12.9 / 17.0,
//                  256 15.8 / 16.3 / 20.6, 512 23.5 / 20.9 / 27.3;  1536 512 29.9 / 34.4 / 37.6
//   over pages     64 512 31.1 / 17.9 / 12.1;  512 512 31.8 / 22.8 / 17.1;  1024 128 13.9 / 13.9 / 18.0, 256 20.1 / 18.0 / 22.2, 512 33.1 / 26.3 / 30.6;
//                  1536 512 42.9 / 45.6 / 43.2
//   64 channels    512 512 16.6 / 12.0 / 11.2;  1024 256 11.3 / 11.1 / 10.9, 512 17.3 / 13.6 / 13.3;  1536 256 13.7 / 12.5 / 15.0, 512 20.8 / 18.6 / 19.4;  4096 512
//                  34.7 / 36.7 / 40.6;  over pages 1536 512 27.5 / 21.1 / 22.5, 4096 512 48.2 / 48.1 / 50.9
// Where the groups go in linear order (an odd number: `gc` 0) the heads that share rows are on different XCDs with two waves an item: five
// groups of 16384 tokens, 900 items, one / two 28.5 / 31.7 (the keys and values of one or three fit the caches).
inline int attn_waves_per_item(int64_t items, int n_keys, int d, bool paged, int64_t groups, int gc, int64_t max_kv_len)
{
    if (items <= 512) return 4;
    if (items > 1024 || n_keys <= (d == 128 && !paged ? 256 : 128)) return 1;
    return gc == 0 && !paged && groups * max_kv_len * d * 4 > (24 << 20) ? 1 : 2;
}

}  // namespace hipattn
