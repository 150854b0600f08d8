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

}  // namespace hipattn
