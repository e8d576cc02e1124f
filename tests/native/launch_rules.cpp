// The launch rules of paper_2609_18178_amd/csrc/launch.h, for tests/test_launch_shape.py:
//   tile MODE ELEMS LONGEST WORKSPACE   elements of one pass of a tile in such a call
//   dealt TILES RUN                       the tile of every block of a grid
#include <cstdio>
#include <cstdlib>
#include <cstring>

#include "launch.h"

int main(int argc, char** argv) {
    const auto arg = [&](int k) { return k < argc ? std::strtoull(argv[k], nullptr, 0) : 0ull; };
    if (argc == 6 && std::strcmp(argv[1], "tile") == 0) {
        const auto mode = static_cast<pact::Mode>(arg(2));
        std::printf("%u\n", pact::shape_of(mode, pact::form_of(mode, arg(3), arg(4), arg(5) != 0)).elems());
        return 0;
    }
    if (argc == 4 && std::strcmp(argv[1], "dealt") == 0) {
        for (uint32_t b = 0; b < arg(2); ++b) std::printf("%u\n", pact::dealt_tile(b, arg(2), arg(3)));
        return 0;
    }
    return 2;
}
