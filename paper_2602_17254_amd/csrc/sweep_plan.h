// Column programs of the latency-optimal variant: the steps of one column over all ranks as a short
// list of sums.
//
// Every value a rank holds between steps (its window, and on sides that are not powers of three
// the partial sums beside it) is the same expression at every rank, shifted: an array over the
// ranks. A step forms new arrays by joint reductions
//     out[x] = (own[x] + left[x - d e]) + right[x + d e]
// with absent terms skipped. An output with a single term is an earlier array seen from another
// rank, so it costs nothing here: the program names it by that array and a displacement, and only
// real sums become operations. Arrays are given slots of on-chip memory by their last use; a
// level (one step) reads all its terms before it writes, so an output may take the slot of an
// array that the same level reads last.
#pragma once

#include <algorithm>
#include <array>
#include <cstdint>
#include <vector>

#include "plan.h"

namespace trivance {

inline void build_sweep_programs(trivance_plan_t* p) {
    p->sweeps.clear();
    if (p->n < 2 || p->n > kMaxSweepRanks || p->D > kMaxSweepDims || p->S < 1) return;
    const int D = p->D, S = p->S;
    const int bits = kSweepCoordBits / D;
    for (int d = 0; d < D; ++d)
        if (p->dims[d] > (1 << bits) - 1) return;
    struct Ref {
        int array;
        std::array<int, kMaxSweepDims> at;  // displacement, 0 <= at[d] < side
    };
    struct Op {
        int level;
        std::vector<Ref> src;
        int last = -1;  // level of the last use
        int slot = -1;
    };
    bool equal = true;
    for (int d = 0; d < D; ++d) equal = equal && p->dims[d] == p->dims[0];
    std::vector<SweepProgram> progs;
    for (int c = 0; c < (equal ? 1 : D); ++c) {
        std::vector<Op> ops(1);  // array 0: the rank's own vector
        ops[0].level = -1;
        std::vector<Ref> state{Ref{0, {}}};
        for (int t = 0; t < S; ++t) {
            const Pass& ps = p->passes[t];
            const int a = ps.dim[c], side = p->dims[a], dist = ps.distance[c];
            const int nout = p->slots.empty() ? 1 : p->slots[t].nout[c];
            std::vector<Ref> next;
            for (int i = 0; i < nout; ++i) {
                const int part[3] = {p->slots.empty() ? 0 : p->slots[t].own[c][i],
                                     p->slots.empty() ? 0 : p->slots[t].left[c][i],
                                     p->slots.empty() ? 0 : p->slots[t].right[c][i]};
                const int shift[3] = {0, side - dist, dist};
                Op op;
                op.level = t;
                for (int q = 0; q < 3; ++q) {
                    if (part[q] < 0) continue;
                    Ref r = state[part[q]];
                    r.at[a] = (r.at[a] + shift[q]) % side;
                    op.src.push_back(r);
                }
                if (op.src.size() == 1) {
                    next.push_back(op.src[0]);
                    continue;
                }
                ops.push_back(op);
                next.push_back(Ref{(int)ops.size() - 1, {}});
            }
            state.swap(next);
        }
        // the result: one array, of the last level, not displaced
        if (state.size() != 1 || state[0].array != (int)ops.size() - 1 || ops.back().level != S - 1)
            return;
        for (int d = 0; d < D; ++d)
            if (state[0].at[d]) return;
        // last uses, backwards from the result; unused operations drop out
        ops.back().last = S;
        for (int i = (int)ops.size() - 1; i > 0; --i)
            if (ops[i].last >= 0)
                for (const Ref& r : ops[i].src)
                    ops[r.array].last = std::max(ops[r.array].last, ops[i].level);
        SweepProgram g;
        std::vector<int> owner;  // slot -> array in it, -1 free
        auto take = [&](int array) {
            for (size_t s = 0; s < owner.size(); ++s)
                if (owner[s] < 0) {
                    owner[s] = array;
                    return (int)s;
                }
            owner.push_back(array);
            return (int)owner.size() - 1;
        };
        ops[0].slot = take(0);
        for (int t = 0; t < S; ++t) {
            g.level_begin.push_back((uint32_t)(g.words.size() / 4));
            for (int& o : owner)
                if (o >= 0 && ops[o].last <= t) o = -1;
            int count = 0;
            for (size_t i = 1; i < ops.size(); ++i) {
                if (ops[i].level != t || ops[i].last < 0) continue;
                ++count;
                ops[i].slot = t == S - 1 ? 0 : take((int)i);  // the last level's goes to memory
                for (int q = 0; q < 3; ++q) {
                    uint32_t w = kSweepNone;
                    if (q < (int)ops[i].src.size()) {
                        const Ref& r = ops[i].src[q];
                        w = (uint32_t)ops[r.array].slot << kSweepCoordBits;
                        for (int f = 0; f < D; ++f)
                            w |= (uint32_t)r.at[(c + f) % D] << (f * bits);
                    }
                    g.words.push_back(w);
                }
                g.words.push_back((uint32_t)ops[i].slot);
            }
            g.max_ops = std::max(g.max_ops, count);
        }
        g.level_begin.push_back((uint32_t)(g.words.size() / 4));
        g.slots = (int)owner.size();
        progs.push_back(g);
    }
    size_t total = 0;
    for (const SweepProgram& g : progs) total += g.words.size() + g.level_begin.size();
    if (total > kMaxSweepWords) return;
    p->sweeps.swap(progs);
}

}  // namespace trivance
