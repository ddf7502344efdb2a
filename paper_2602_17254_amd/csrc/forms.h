// Which form runs a whole AllReduce call, and its launch shape. Host code without HIP, so that the
// rules can be evaluated without a GPU (tests/c/forms.cpp).
#pragma once

#include <algorithm>
#include <cstddef>
#include <cstdint>

#include "plan.h"

namespace trivance {

constexpr uint32_t kComputeUnits = 256;

// ---- small bandwidth-optimal calls: tiles in local memory (tile.hip) ----

struct TileShape {
    uint32_t shift;
    int cells;  // per thread
    int threads;
};

// Up to 24 MiB of vectors or 4096 values a rank. In us, fold.hip's waves against these tiles: 27x27
// ranks of 256 values 18 / 6, of 4096 (12 MB) 19 / 10, of 16,384 (48 MB) 23 / 40; 16x16x16 of 256
// values 107 / 22, of 4096 (67 MB) 129 / 84, of 16,384 174 / 536; rings of 64 and 243 equal at 17 MB.
// Below, a row is in flight from every thread at once and a step costs 0.4 us; above, the fold
// reads longer pieces of a row. On few ranks with long rows the line lies too high: 4 ranks of 1,048,576
// values (17 MB) take 6.6 with the fold's waves and 9.2 with the tiles that they get (the steps 15.7),
// 8 ranks 10.7 and 15.5 at 34 MB, above the line.
constexpr int64_t kTileBytes = (int64_t)24 << 20;
constexpr int64_t kTileElems = 4096;

inline bool tile_shape(const trivance_plan_t* p, int64_t elems, TileShape* s) {
    if (p->tile_masks.empty()) return false;
    if ((int64_t)p->n * elems * 4 > kTileBytes && elems > kTileElems) return false;
    // as many vectors to a tile as leave two tiles for every compute unit (27x27 ranks of 256
    // values: one 6.2 us, two 7.7, four 10.8; of 4096: one 11.7, two 9.6, four 12.2)
    const int64_t vecs = (elems + 3) / 4, most = std::max(2048, 2 * p->n);
    s->shift = 0;
    while (s->shift < 6 && vecs >= 2 * (int64_t)kComputeUnits << (s->shift + 1) &&
           ((int64_t)p->n << (s->shift + 1)) <= most)
        ++s->shift;
    const int64_t cells = (int64_t)p->n << s->shift;
    s->cells = 1;
    while (s->cells < 8 && cells > 1024 * s->cells) s->cells *= 2;
    s->threads = (int)((cells + 64 * s->cells - 1) / (64 * s->cells)) * 64;
    return cells * 16 <= 159 * 1024 && s->threads <= 1024;
}

inline bool tile_fits(const trivance_plan_t* p, int64_t elems) {
    TileShape s;
    return elems < ((int64_t)1 << 28) && tile_shape(p, elems, &s);
}

// ---- bandwidth-optimal calls: a fold over the rows (fold.hip) ----

constexpr int kStreamWaves = 4;        // tiles of a workgroup when a wave has a tile of its own
constexpr uint32_t kSpreadTile = 256;  // elements that a wave of the spread copies

struct FoldShape {
    int spread;      // 1: result to row 0, spread_kernel copies it
    int waves;       // waves per tile
    uint32_t lanes;  // column vectors of a tile
};

inline size_t fold_lds(const FoldShape& s, size_t roots, int sub_depth, int top_depth) {
    if (s.waves == 1) return (size_t)kStreamWaves * (sub_depth + top_depth) * 64 * 16;
    return (roots + 1 + (size_t)s.waves * sub_depth + top_depth) * s.lanes * 16;
}

// Fold and spread from 192 MiB of vectors on. Measured in us, one launch against two, at 134 MB
// (ring of 8) 45.7 / 46.3, at 191 MB (27x27) 68.4 / 65.9, at 255 MB (ring of 243) 88 / 81, at 268 MB
// (rings of 4 and 64) 91 / 81 and 92 / 82: below the size of the 256 MB last-level cache the writes
// of the one launch end there, and the second launch costs 3 us. These are calls on vectors that are not
// in the cache; on one set of vectors that stays there one launch is the faster up to its size (4 ranks at
// 255 MB 59 / 77).
constexpr int64_t kSpreadBytes = (int64_t)192 << 20;
// Not on two ranks, nor on three whose rows exceed that cache: the second launch reads row 0 once more,
// a fourth or a sixth on top of the call's traffic, and two launches were slower than the steps. In
// us over three sets of vectors in turn, two launches / steps / one: 2 ranks at 403 MB 143 / 141 / 130,
// at 1600 MB 611 / 598 / 509; 3 ranks at 403 MB 136 / 140 / 145, at 2400 MB 871 / 869 / 815 (as a
// torus of 1x3 887 / 869 / 799); 4 ranks at 2400 MB 848 / 1357 / 838. One launch is the slower of the two,
// though not slower than the steps, on 3 rows 16 bytes short of 1 GiB (1202 / 1350 / 1320).
constexpr int64_t kLastLevelBytes = (int64_t)256 << 20;

inline bool fold_spreads(int n, int64_t elems) {
    if (n * elems * 4 < kSpreadBytes || n == 2) return false;
    return n > 3 || elems * 4 <= kLastLevelBytes;
}

// A wave per tile from 2048 tiles of 1 KiB on (524,288 elements): it needs no local memory for the
// subtrees and no barrier. With fewer tiles that leaves compute units idle, so sixteen waves share
// one. In us, sixteen waves against one: 32x32 ranks at 524,288 elements 717 / 631, at 262,144
// 364 / 427, at 65,536 97 / 298; 16x16x16 at 524,288 3576 / 2743, at 262,144 1852 / 1957; 27x27 at
// 16,384 23 / 168.
constexpr int64_t kStreamVecs = (int64_t)2048 * 64;
// Local memory of a tile's subtrees: all of a compute unit's if need be. 32x32 ranks of 65,536
// elements took 117 us with tiles narrowed to fit 64 KiB and 97 with 156 KiB.
constexpr size_t kFoldLds = 156 * 1024;

inline FoldShape fold_shape(const trivance_plan_t* p, int64_t elems) {
    size_t roots = 0;
    int sub_depth = 0, top_depth = 0;
    for (const FoldProgram& f : p->folds) {
        roots = std::max(roots, f.roots.size());
        sub_depth = std::max(sub_depth, f.sub_depth);
        top_depth = std::max(top_depth, f.top_depth);
    }
    const int64_t vecs = (elems + 3) / 4;
    FoldShape s{fold_spreads(p->n, elems) ? 1 : 0, 1, 64};
    if (vecs >= kStreamVecs) return s;
    // with at most eight subtrees four waves share a tile (more would find none)
    s.waves = roots > 8 ? 16 : 4;
    // tiles narrow down to 64 bytes while there are fewer than one per compute unit: 27x27 ranks of
    // 4096 elements 26 us with 1 KiB tiles, 20 with 256 B and 19 with 64 B
    while (s.lanes > 4 && vecs < (int64_t)kComputeUnits * s.lanes) s.lanes /= 2;
    while (s.lanes > 4 && fold_lds(s, roots, sub_depth, top_depth) > kFoldLds) s.lanes /= 2;
    return s;
}

// Whether the programs of all collectives fit the kernel arguments of one launch (otherwise: a launch
// per collective).
inline bool fold_together(const trivance_plan_t* p) {
    size_t words = 0;
    for (const FoldProgram& f : p->folds) words += f.words();
    return words <= kMaxFoldWords;
}

// Rows below 1 GiB (32-bit offsets), and n rows of granules counted in 31 bits (the block of a column,
// and the units of the spread; 550 GB of vectors). The tiles above stay within both by their limits.
inline bool fold_fits(const trivance_plan_t* p, int64_t elems) {
    const int64_t granules = (elems + kGranule - 1) / kGranule;
    return !p->folds.empty() && elems < ((int64_t)1 << 28) &&
           (int64_t)p->n * (granules + 1) < ((int64_t)1 << 31) - 4;
}

// ---- latency-optimal calls: all steps in local memory (sweep.hip) ----

// Words of an operation in the kernel arguments, and how many words there are.
constexpr uint32_t sweep_op_words(int D) { return D <= 2 ? 8 : 12; }
constexpr uint32_t kSweepTabWords = 896;

// Tile and thread counts, measured over the plans and sizes of the tests and benchmarks:
//  * up to 64 column vectors, while at least four workgroups fit a compute unit (three up to four
//    vectors, 64 bytes of a row): ring of 81 with 16 vectors 263 us, 32 273, 8 279; ring of 729 with
//    four 389, two 537.
//  * four cells to a thread from 1024 cells on for one operation a level (ring of 81: four 263, two
//    283, one 407; of 27: two 164, four 167), two with up to four operations (ring of 64: two 265, one
//    376), one where fewer than three workgroups fit (32x32: one 665, two 782).
//  * fewer vectors to a tile while there is less than a tile per compute unit.
struct SweepShape {
    uint32_t shift;  // column vectors of a tile: 1 << shift
    int cells;       // per thread
    int ops;         // operations of a level, rounded up to a compiled size
    int threads;
    size_t lds;
    uint32_t per_cu;  // workgroups a compute unit runs
};

constexpr size_t kSweepLds = 160 * 1024 - 256;

inline bool sweep_shape(const trivance_plan_t* p, int64_t elems, SweepShape* s) {
    // one step of powers of three: a read and a write as well (ring of 3: step 63 us, tile 74)
    if (p->sweeps.empty() || (p->S == 1 && p->slots.empty())) return false;
    int ops = 0, slots = 0;
    size_t words = 1;
    for (int c = 0; c < p->D; ++c) {
        const SweepProgram& g = p->sweeps[p->sweeps.size() == 1 ? 0 : c];
        ops = std::max(ops, g.max_ops);
        slots = std::max(slots, g.slots);
        words += g.words.size() / 4;
    }
    if (ops > 12 || words * sweep_op_words(p->D) > kSweepTabWords) return false;
    s->ops = ops == 1 ? 1 : (ops <= 4 ? 4 : 12);
    const size_t col = (size_t)slots * p->n * 16;  // local memory per column vector
    const int64_t vecs = (elems + 3) / 4;
    const int most = s->ops == 1 ? 4 : (s->ops == 4 ? 2 : 1);
    s->shift = 0;
    while (s->shift < 6 && ((int64_t)p->n << (s->shift + 1)) <= 1024 * most &&
           (col << (s->shift + 1)) <= (s->shift < 2 ? kSweepLds / 3 : kSweepLds / 4))
        ++s->shift;
    while (s->shift > 0 && vecs < (int64_t)kComputeUnits << s->shift) --s->shift;
    const int64_t cells = (int64_t)p->n << s->shift;
    s->cells = s->ops == 1 ? (cells > 1024 ? 4 : 2) : s->ops == 4 && cells <= 1024 ? 2 : most;
    if (s->ops > 1 && 3 * (col << s->shift) > kSweepLds && cells <= 1024) s->cells = 1;
    s->threads = (int)((cells + 64 * s->cells - 1) / (64 * s->cells)) * 64;
    s->lds = col << s->shift;
    if (s->lds > kSweepLds || s->threads > 1024 || s->cells > most || cells > 32767) return false;
    s->per_cu = (uint32_t)std::min<size_t>(kSweepLds / s->lds, 2048 / s->threads);
    return true;
}

// Workgroups of the launch; fewer than `tiles`: each takes several.
inline uint32_t sweep_grid(const SweepShape& s, uint32_t tiles) {
    if (s.per_cu > 2 || s.cells > 1 || s.ops == 1) return tiles;
    return std::min(tiles, kComputeUnits * s.per_cu);
}

// Tiles of 16 bytes of a row (2187 ranks) read every cache line eight times, and rows a multiple of 2 MiB
// apart share their cache sets, so that few lines last until the next tile comes. On powers of three the
// steps are the faster form then, unless they would run on single elements (`aligned` 0: the vectors
// do not start at 16 bytes). In us, sweep / steps: 9x9x27 ranks of 524,288 values 13375 / 10495, of
// 1,048,576 26448 / 20881, ring of 2187 12719 / 11187 and 25182 / 22835; of 786,432 values 14635 / 15240
// and 13929 / 17049, of 524,320 6153 / 10602 and 5569 / 11535; 9x9x27 of 524,288 unaligned 14252 / 27740.
// Plans with several operations a level carry partial sums through memory in their steps and stay
// faster here (1944 ranks of 524,288 values 11906 / 19718, 2000 14304 / 35021).
constexpr int64_t kAliasElems = (int64_t)1 << 19;

inline bool sweep_fits(const trivance_plan_t* p, int64_t elems, bool aligned) {
    SweepShape s;
    if (elems >= ((int64_t)1 << 32) || !sweep_shape(p, elems, &s)) return false;
    return !(aligned && s.ops == 1 && s.shift == 0 && elems % kAliasElems == 0);
}

// ---- the choice ----

// A whole call: plans that a fold program (bandwidth-optimal, fold_plan.h) or a column program
// (latency-optimal, sweep_plan.h) fits read and write each vector once; the others run step by step.
// `aligned`: the vectors start at a multiple of 16 bytes.
enum class Form { kTile, kFold, kSweep, kSteps };

inline Form whole_form(const trivance_plan_t* p, int64_t elems, bool aligned) {
    if (tile_fits(p, elems)) return Form::kTile;
    if (fold_fits(p, elems)) return Form::kFold;
    if (sweep_fits(p, elems, aligned)) return Form::kSweep;
    return Form::kSteps;
}

}  // namespace trivance
