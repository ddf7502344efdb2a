// The form that runs a whole AllReduce call and its launch shape, as the rules of forms.h give them.
// Built with g++ against plan.cpp; no GPU. One line of output per call:
//   forms VARIANT SIDES PLACEMENT ELEMS [VARIANT SIDES PLACEMENT ELEMS ...]    (B 27x27 natural 4098 ...)
// with ELEMS+K for vectors that start K elements beyond a multiple of 16 bytes:
//     tile c<cells of a thread> v<vectors of a tile>
//     fold w<waves of a tile> v<vectors of a tile> one|spread [per-collective]
//     sweep o<operations of a level> c<cells of a thread> v<vectors of a tile> [loop]
//     steps
#include <cstdio>
#include <cstdlib>
#include <cstring>

#include "forms.h"
#include "plan.h"

using namespace trivance;

static uint32_t sweep_tiles(const trivance_plan_t* p, int64_t elems, const SweepShape& s) {
    uint32_t tiles = 0;
    for (int c = 0; c < p->D; ++c) {
        int64_t b, e;
        block_bounds(p, elems, c, -1, &b, &e);
        tiles += (uint32_t)(((e - b + 3) / 4 + ((int64_t)1 << s.shift) - 1) >> s.shift);
    }
    return tiles;
}

int main(int argc, char** argv) {
    for (int i = 1; i + 3 < argc; i += 4) {
        int dims[kMaxDims] = {}, D = 0, n = 1;
        for (const char* s = argv[i + 1]; *s;) {
            char* end;
            dims[D++] = (int)std::strtol(s, &end, 10);
            n *= dims[D - 1];
            s = *end ? end + 1 : end;
        }
        const int64_t elems = std::strtoll(argv[i + 3], nullptr, 10);
        const char* plus = std::strchr(argv[i + 3], '+');
        const bool aligned = !plus || std::atoi(plus + 1) % 4 == 0;
        trivance_plan_t* p = nullptr;
        if (trivance_plan_ex(n, dims, D, *argv[i] == 'L' ? TRIVANCE_LATENCY_OPT : TRIVANCE_BANDWIDTH_OPT,
                             std::strcmp(argv[i + 2], "natural") ? TRIVANCE_PLACE_BY_SCHEDULE : 0u,
                             &p) != TRIVANCE_OK)
            return 1;
        switch (whole_form(p, elems, aligned)) {
            case Form::kTile: {
                TileShape s{};
                tile_shape(p, elems, &s);
                std::printf("tile c%d v%d\n", s.cells, 1 << s.shift);
                break;
            }
            case Form::kFold: {
                const FoldShape s = fold_shape(p, elems);
                std::printf("fold w%d v%u %s%s\n", s.waves, s.lanes, s.spread ? "spread" : "one",
                            fold_together(p) ? "" : " per-collective");
                break;
            }
            case Form::kSweep: {
                SweepShape s{};
                sweep_shape(p, elems, &s);
                const uint32_t tiles = sweep_tiles(p, elems, s);
                std::printf("sweep o%d c%d v%d%s\n", s.ops, s.cells, 1 << s.shift,
                            sweep_grid(s, tiles) < tiles ? " loop" : "");
                break;
            }
            default: std::printf("steps\n");
        }
        trivance_plan_destroy(p);
    }
    return 0;
}
