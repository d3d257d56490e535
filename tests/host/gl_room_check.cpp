// Host check of csrc/gl_room.h: gl_room_check rows N_OUT SEEN CAP MEM
#include <cstdio>
#include <cstdlib>
#include <cstring>

#include "gl_room.h"

int main(int argc, char** argv)
{
    if (argc == 6 && std::strcmp(argv[1], "rows") == 0) {
        std::printf("%lld\n", (long long)gl::net_rows(std::atoll(argv[2]), std::atoll(argv[3]), std::atoll(argv[4]), std::atoll(argv[5])));
        return 0;
    }
    std::fprintf(stderr, "usage: gl_room_check rows N_OUT SEEN CAP MEM\n");
    return 2;
}
