// Fold programs (fold_plan.h) against the schedule they replace, on the host: for every block of
// every collective the program, read as the fold kernel reads it, must visit each row exactly once
// and give the bits of the block's reduce-scatter steps run one after another on floats whose
// sums depend on the association; the trees by offset (tile.hip) likewise. Built with g++ against plan.cpp; no GPU. Exit status 0 on success.
//   fold_program SIDES...    (a ring "9", a torus "5x7")
#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <vector>

#include "plan.h"

using trivance::kMaxDims;

static int coord(const trivance_plan_t* p, int r, int d) { return r / p->strides[d] % p->dims[d]; }

// The reduce-scatter of block j, step by step over all ranks: a rank that a child sends to adds
// the child's pre-step value; `alive` ends a rank's part once it has forwarded.
static float by_steps(const trivance_plan_t* p, int c, int j, std::vector<float> x) {
    int taken[kMaxDims] = {};
    for (int t = 0; t < p->S; ++t) {
        const trivance::Pass& ps = p->passes[t];
        const int a = ps.dim[c], dist = ps.distance[c], side = p->dims[a];
        std::vector<float> y = x;
        for (int r = 0; r < p->n; ++r) {
            uint32_t flags = 0;
            bool live = true;
            for (int d = 0; d < p->D; ++d) {
                const uint32_t o = (uint32_t)((coord(p, r, d) - coord(p, j, d) + p->dims[d]) % p->dims[d]);
                if (p->tree) {
                    bool in = false;
                    for (uint32_t v : p->trees[d].alive[taken[d]]) in = in || v == o;
                    live = live && in;
                    if (d == a)
                        for (uint32_t v : p->trees[d].recv[taken[d]])
                            if ((v & 0x3FFFFFFFu) == o) flags = v & 0xC0000000u;
                } else {
                    // power of three: the blocks r keeps after the step
                    live = live && o % (uint32_t)ps.modulus[c][d] == 0;
                    flags = 0xC0000000u;
                }
            }
            if (!live || !flags) continue;
            const int xa = coord(p, r, a);
            const int l = r + ((xa - dist + side) % side - xa) * p->strides[a];
            const int q = r + ((xa + dist) % side - xa) * p->strides[a];
            float v = x[r];
            if (flags & trivance::kFromLeft) v += x[l];
            if (flags & trivance::kFromRight) v += x[q];
            y[r] = v;
        }
        x.swap(y);
        ++taken[a];
    }
    return x[j];
}

// The same from the trees by offset (tile_masks), as the tile kernel runs them.
static float by_masks(const trivance_plan_t* p, int c, int j, std::vector<float> x) {
    std::vector<uint32_t> mask(p->n);
    for (int r = 0; r < p->n; ++r) {
        uint32_t bits = 0, until = 31;
        for (int d = 0; d < p->D; ++d) {
            const int o = (coord(p, r, d) - coord(p, j, d) + p->dims[d]) % p->dims[d];
            const uint32_t w = p->tile_masks.at(p->tile_mask0.at(c * p->D + d) + o);
            bits |= w;
            until = std::min(until, w >> trivance::kTileForwardShift);
        }
        until = std::min<uint32_t>(until, trivance::kMaxTileSteps);
        mask[r] = bits & ((1u << (2 * until)) - 1u);
    }
    for (int t = 0; t < p->S; ++t) {
        const int a = p->passes[t].dim[c], dist = p->passes[t].distance[c];
        for (int r = 0; r < p->n; ++r) {
            // in place: a rank that is read in a step does not receive in it
            const uint32_t f = (mask[r] >> (2 * t)) & 3u;
            const int xa = coord(p, r, a), side = p->dims[a];
            const int l = r + ((xa - dist + side) % side - xa) * p->strides[a];
            const int q = r + ((xa + dist) % side - xa) * p->strides[a];
            if (f & 1u) x[r] += ((mask[l] >> (2 * t)) & 3u) ? NAN : x[l];
            if (f & 2u) x[r] += ((mask[q] >> (2 * t)) & 3u) ? NAN : x[q];
        }
    }
    return x[j];
}

struct Fold {
    std::vector<float> open;
    float cur = 0;
    void node(uint32_t w, float v) {
        if (w & trivance::kFoldFirst) cur = v;
        else if (w & trivance::kFoldLeaf) cur += v;
        else open.push_back(cur), cur = v;
        for (uint32_t k = (w >> trivance::kFoldPopsShift) & trivance::kFoldMaxPops; k > 0; --k) cur = open.back() + cur, open.pop_back();
    }
};

static int check(const char* text) {
    int dims[kMaxDims] = {}, D = 0, n = 1;
    for (const char* s = text; *s;) {
        char* end;
        dims[D++] = (int)std::strtol(s, &end, 10);
        n *= dims[D - 1];
        s = *end ? end + 1 : end;
    }
    trivance_plan_t* p = nullptr;
    if (trivance_plan(n, dims, D, TRIVANCE_BANDWIDTH_OPT, &p) != TRIVANCE_OK) return 1;
    int bad = p->folds.empty() || (int)p->fold_of.size() != D;
    const int bits = trivance::kFoldCoordBits / D;
    uint32_t seed = 12345;
    for (int c = 0; c < D && !bad; ++c) {
        const trivance::FoldProgram& f = p->folds[p->fold_of[c]];
        bad |= f.words() > trivance::kMaxFoldWords || f.shape.size() != f.roots.size();
        const int step = n > 300 ? n / 37 + 1 : 1;  // every block of small plans, a sample of large ones
        for (int j = 0; j < n && !bad; j += step) {
            std::vector<float> x(n);
            for (float& v : x) {
                seed = seed * 1664525u + 1013904223u;
                v = (float)(int32_t)seed / 1e6f * ((seed & 7u) ? 1.0f : 1e-3f);
            }
            std::vector<int> seen(n, 0);
            Fold top;
            size_t deepest = 0;
            for (size_t g = 0; g < f.roots.size(); ++g) {
                Fold sub;
                for (uint32_t pos = f.shape_begin[f.shape[g]];; ++pos) {
                    if (pos >= f.nodes.size()) return 2;
                    const uint32_t w = f.nodes[pos];
                    int row = 0, left = 0, right = 0;  // the node's row and its neighbours' at distance 1
                    for (int i = 0; i < D; ++i) {
                        const int d = (p->fold_dim0[c] + i) % D;
                        const uint32_t mask = (1u << bits) - 1u;
                        const int y = (int)((((f.roots[g] >> (i * bits)) & mask) + ((w >> (i * bits)) & mask) +
                                             (uint32_t)coord(p, j, d)) % (uint32_t)dims[d]);
                        row += y * p->strides[d];
                        left += (i ? y : (y + dims[d] - 1) % dims[d]) * p->strides[d];
                        right += (i ? y : (y + 1) % dims[d]) * p->strides[d];
                    }
                    ++seen[row];
                    float v = x[row];
                    if (w & trivance::kFoldLeft) ++seen[left], v += x[left];
                    if (w & trivance::kFoldRight) ++seen[right], v += x[right];
                    sub.node(w, v);
                    if ((int)sub.open.size() > f.sub_depth) return 3;
                    if (w & trivance::kFoldLast) break;
                }
                if (!sub.open.empty()) return 4;
                top.node(f.roots[g], sub.cur);
                deepest = top.open.size() > deepest ? top.open.size() : deepest;
            }
            bad |= (int)deepest > f.top_depth || !top.open.empty();
            for (int s : seen) bad |= s != 1;
            const float want = by_steps(p, c, j, x);
            bad |= std::memcmp(&want, &top.cur, sizeof(float)) != 0;
            const float tiled = p->tile_masks.empty() ? want : by_masks(p, c, j, x);
            bad |= std::memcmp(&want, &tiled, sizeof(float)) != 0;
        }
    }
    trivance_plan_destroy(p);
    return bad ? 5 : 0;
}

int main(int argc, char** argv) {
    int failures = 0;
    for (int i = 1; i < argc; ++i) {
        const int rc = check(argv[i]);
        if (rc) std::printf("%s: %d\n", argv[i], rc), ++failures;
    }
    std::printf("%d failures\n", failures);
    return failures != 0;
}
