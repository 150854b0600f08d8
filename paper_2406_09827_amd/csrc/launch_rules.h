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

}  // namespace hipattn
