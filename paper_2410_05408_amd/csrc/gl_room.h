// gl_room.h -- room for the network's rows of a surrogate batch (host).
#pragma once

#include <cstdint>

namespace gl {

constexpr int64_t kNetRowBytes = 2 * 16 + 8 + 8 + 4;  // features, output, scale, result

// Rows that a batch of n_out outputs gets room for, with room for `cap` there
// and `seen` the most that a pass has asked for: 16 per output up to 2^24 rows
// (872 MB), a quarter per output where that is more; the demand and a quarter
// more once it was larger than the room; at most an eighth of the device's
// memory.  Units without room are evaluated exactly, and which ones they are
// depends on the order in which workgroups run, so the room is to last: 4096
// sets of 3000 x 15 sub-samples ask for 10^5 rows under a 1 ppm gate.
inline int64_t net_rows(int64_t n_out, int64_t seen, int64_t cap, int64_t mem_total)
{
    constexpr int64_t base = (int64_t)1 << 24;
    int64_t want = n_out < base / 16 ? 16 * n_out : n_out / 4 > base ? n_out / 4 : base;
    if (seen > cap && seen + seen / 4 > want) want = seen + seen / 4;
    const int64_t most = mem_total / 8 / kNetRowBytes;
    return want < most ? want : most;
}

// New buffers of the given sizes for all of `slots`, or none: where one cannot
// be had, the old ones stay.
template <int N, class Alloc, class Free>
bool replace_all(void** const (&slots)[N], const int64_t (&bytes)[N], Alloc&& alloc, Free&& release)
{
    void* fresh[N] = {};
    for (int i = 0; i < N; ++i) {
        fresh[i] = alloc(bytes[i]);
        if (!fresh[i]) {
            for (int j = 0; j < i; ++j) release(fresh[j]);
            return false;
        }
    }
    for (int i = 0; i < N; ++i) {
        if (*slots[i]) release(*slots[i]);
        *slots[i] = fresh[i];
    }
    return true;
}

}  // namespace gl
