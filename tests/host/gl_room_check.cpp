// Host check of csrc/gl_room.h: gl_room_check rows N_OUT SEEN CAP MEM
//                               gl_room_check replace HELD FAIL_AT
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <set>

#include "gl_room.h"

int main(int argc, char** argv)
{
    if (argc == 6 && std::strcmp(argv[1], "rows") == 0) {
        std::printf("%lld\n", (long long)gl::net_rows(std::atoll(argv[2]), std::atoll(argv[3]), std::atoll(argv[4]), std::atoll(argv[5])));
        return 0;
    }
    if (argc == 4 && std::strcmp(argv[1], "replace") == 0) {
        // three buffers, held before or not; allocation FAIL_AT fails
        std::set<void*> live;
        int calls = 0;
        const int held = std::atoi(argv[2]), fail_at = std::atoi(argv[3]);
        void* b[3] = {};
        for (int i = 0; i < 3 && held; ++i) live.insert(b[i] = std::malloc(8));
        void* const old[3] = {b[0], b[1], b[2]};
        void** const slots[3] = {&b[0], &b[1], &b[2]};
        const int64_t bytes[3] = {16, 32, 48};
        bool good = true;  // nothing freed twice or that is not there
        const bool ok = gl::replace_all(
            slots, bytes,
            [&](int64_t n) {
                if (calls++ == fail_at) return (void*)nullptr;
                void* p = std::malloc((size_t)n);
                live.insert(p);
                return p;
            },
            [&](void* p) { good = good && live.erase(p) == 1; });  // (kept, so that no address comes again)
        int kept = 0, there = 0;
        for (int i = 0; i < 3; ++i) {
            kept += b[i] == old[i];
            there += b[i] && live.count(b[i]);
        }
        std::printf("%d %d %d %d %d\n", ok, good, kept, there, (int)live.size());
        return 0;
    }
    std::fprintf(stderr, "usage: gl_room_check rows N_OUT SEEN CAP MEM | replace HELD FAIL_AT\n");
    return 2;
}
