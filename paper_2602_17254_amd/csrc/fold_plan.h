// Fold programs of the bandwidth-optimal variant: the order in which one pass over the n rows adds
// up a block.
//
// The reduce-scatter reduces block j along one tree rooted at rank j (Sec. 4.1, 4.3, 4.4), and the
// tree depends on the offsets from j alone. With V(o, T) the partial that the rank at offset o
// holds before reduce-scatter step T,
//     V(o, 0) = x_o,   V(o, t + 1) = (V(o, t) + V(o - d_t, t)) + V(o + d_t, t)
// (absent terms skipped), and the block's result is V(0, S). So a node adds its children in step
// order, left before right, to its own row, and a walk of the tree in preorder with a short stack
// of open sums performs the schedule's own adds, in its own association, while it reads every row
// once. The all-gather only copies the result to every rank.
//
// The first step always joins a row with its neighbours at distance 1, so a program node stands for
// V(o, 1): up to three rows under one word.
//
// The walk is cut at one step: V(o, cut) is evaluated by the subprogram of its shape, and the
// sums of the subtrees (the "roots" of the cut, in preorder) are combined by the steps from `cut` on.
// Subtrees of one shape differ by a translation only and share one subprogram, so the program of
// n rows takes far fewer than n words and travels in the kernel arguments; subtrees are also what
// several waves can evaluate at the same time.
#pragma once

#include <algorithm>
#include <cstdint>
#include <map>
#include <vector>

#include "plan.h"

namespace trivance {

// Walks the tree of one collective: nodes in preorder with the folds that follow each.
struct FoldWalk {
    const trivance_plan_t* p;
    int c;
    // flags[d][k][o]: children of offset o in step k of dimension d's tree
    const std::vector<std::vector<std::vector<uint32_t>>>* flags;
    const Pass* rs;  // the reduce-scatter passes, step t at rs[t]

    struct Node {
        int o[kMaxFoldDims];
        bool leaf, first;
        uint32_t pops;
    };

    uint32_t children(const int* o, int t) const {
        return (*flags)[rs[t].dim[c]][rs[t].taken[c][rs[t].dim[c]]][o[rs[t].dim[c]]];
    }

    // V(o, T) over the steps [tmin, T), appended to out.
    void visit(const int* o, int tmin, int T, bool first, std::vector<Node>* out) const {
        const size_t me = out->size();
        Node node{};
        for (int d = 0; d < p->D; ++d) node.o[d] = o[d];
        node.leaf = true;
        node.first = first;
        out->push_back(node);
        for (int t = tmin; t < T; ++t) {
            const int a = rs[t].dim[c];
            const int side = p->dims[a], dist = rs[t].distance[c];
            const uint32_t f = children(o, t);
            for (int q = 0; q < 2; ++q) {
                if (!(f & (q == 0 ? kFromLeft : kFromRight))) continue;
                int child[kMaxFoldDims];
                for (int d = 0; d < p->D; ++d) child[d] = o[d];
                child[a] = (o[a] + (q == 0 ? side - dist : dist)) % side;
                (*out)[me].leaf = false;
                const size_t at = out->size();
                visit(child, tmin, t, false, out);
                // a leaf child is added to this node's sum directly; any other one leaves its own
                // sum open, folded after its last node
                if (!(*out)[at].leaf) out->back().pops += 1;
            }
        }
    }
};

inline uint32_t fold_word(const FoldWalk::Node& nd, int D, int c, const int* rel,
                          const int* dims) {
    // coordinates in the order of dimensions c, c + 1, ... (cyclic; c: that of the first step):
    // collectives of a torus with equal sides then share one program
    const int bits = kFoldCoordBits / D;
    uint32_t w = 0;
    for (int f = 0; f < D; ++f) {
        const int d = (c + f) % D;
        const int x = (nd.o[d] - rel[d] + dims[d]) % dims[d];
        w |= (uint32_t)x << (f * bits);
    }
    if (nd.leaf) w |= kFoldLeaf;
    if (nd.first) w |= kFoldFirst;
    return w | (nd.pops << kFoldPopsShift);
}

// Largest number of sums open besides the current one.
inline int fold_depth(const std::vector<FoldWalk::Node>& nodes) {
    int sp = 0, most = 0;
    for (const FoldWalk::Node& nd : nodes) {
        if (!nd.first && !nd.leaf) most = std::max(most, ++sp);
        sp -= (int)nd.pops;
    }
    return most;
}

// The program of collective c cut at step `cut`; false if it does not fit.
// With `uniform` (every side a power of three) all subtrees have the first one's shape.
inline bool fold_program(const FoldWalk& w, int S, int cut, bool uniform, FoldProgram* out) {
    const trivance_plan_t* p = w.p;
    const int zero[kMaxFoldDims] = {};
    std::vector<FoldWalk::Node> top, sub;
    w.visit(zero, cut, S, true, &top);
    *out = FoldProgram();
    if ((int)top.size() > kMaxFoldRoots) return false;
    out->cut = cut;
    const int dim0 = w.rs[0].dim[w.c];
    out->top_depth = fold_depth(top);
    std::map<std::vector<uint32_t>, int> seen;
    for (const FoldWalk::Node& r : top) {
        if (r.pops > kFoldMaxPops) return false;
        out->roots.push_back(fold_word(r, p->D, dim0, zero, p->dims));
        if (uniform && !out->shape.empty()) {
            out->shape.push_back(0u);
            continue;
        }
        sub.clear();
        w.visit(r.o, 1, cut, true, &sub);
        std::vector<uint32_t> words;
        for (const FoldWalk::Node& nd : sub) {
            if (nd.pops > kFoldMaxPops) return false;
            const uint32_t f = w.children(nd.o, 0);
            words.push_back(fold_word(nd, p->D, dim0, r.o, p->dims) |
                            (f & kFromLeft ? kFoldLeft : 0u) | (f & kFromRight ? kFoldRight : 0u));
        }
        words.back() |= kFoldLast;
        const auto ins = seen.emplace(words, (int)out->shape_begin.size());
        if (ins.second) {
            out->sub_depth = std::max(out->sub_depth, fold_depth(sub));
            out->shape_begin.push_back((uint32_t)out->nodes.size());
            out->nodes.insert(out->nodes.end(), words.begin(), words.end());
            if (out->words() > kMaxFoldWords) return false;
        }
        out->shape.push_back((uint32_t)ins.first->second);
    }
    return out->words() <= kMaxFoldWords;
}

// The trees by offset (kMaxTileSteps in plan.h); none if they do not fit.
inline void build_tile_masks(trivance_plan_t* p, const std::vector<DimTree>& trees,
                             const std::vector<Pass>& rs) {
    p->tile_masks.clear();
    p->tile_mask0.clear();
    if (p->S > kMaxTileSteps) return;
    std::vector<uint32_t> words, first;
    std::map<std::vector<uint32_t>, uint32_t> seen;
    for (int c = 0; c < p->D; ++c)
        for (int d = 0; d < p->D; ++d) {
            std::vector<uint32_t> w(p->dims[d], 31u << kTileForwardShift);
            for (int t = 0; t < p->S; ++t) {
                if (rs[t].dim[c] != d) continue;
                const int k = rs[t].taken[c][d];
                for (uint32_t r : trees[d].recv[k]) {
                    const uint32_t o = r & ~(kFromLeft | kFromRight);
                    if (r & kFromLeft) w[o] |= 1u << (2 * t);
                    if (r & kFromRight) w[o] |= 2u << (2 * t);
                }
                // forwarded in step k: there before it and not after
                std::vector<bool> after(p->dims[d], false);
                for (uint32_t o : trees[d].alive[k + 1]) after[o] = true;
                for (uint32_t o : trees[d].alive[k])
                    if (!after[o])
                        w[o] = (w[o] & ((1u << kTileForwardShift) - 1u)) | (uint32_t)t << kTileForwardShift;
            }
            const auto ins = seen.emplace(w, (uint32_t)words.size());
            if (ins.second) words.insert(words.end(), w.begin(), w.end());
            first.push_back(ins.first->second);
        }
    if (words.size() > kMaxTileWords) return;
    p->tile_masks.swap(words);
    p->tile_mask0.swap(first);
}

// Builds the fold programs of a bandwidth-optimal plan of S reduce-scatter steps. A plan they do not
// fit (more ranks or dimensions, sides that do not fit a word's fields, too many words) keeps
// none and runs step by step.
inline void build_fold_programs(trivance_plan_t* p, const std::vector<DimTree>& trees) {
    p->folds.clear();
    if (p->n < 2 || p->n > kMaxFoldRanks || p->D > kMaxFoldDims || p->S < 1) return;
    for (int d = 0; d < p->D; ++d)
        if (p->dims[d] > (1 << (kFoldCoordBits / p->D)) - 1) return;
    std::vector<std::vector<std::vector<uint32_t>>> flags(p->D);
    for (int d = 0; d < p->D; ++d) {
        flags[d].assign(trees[d].S, std::vector<uint32_t>(p->dims[d], 0u));
        for (int k = 0; k < trees[d].S; ++k)
            for (uint32_t r : trees[d].recv[k])
                flags[d][k][r & ~(kFromLeft | kFromRight)] = r & (kFromLeft | kFromRight);
    }
    // steps taken before, per dimension (the power-of-three passes do not carry them)
    std::vector<Pass> rs(p->passes.begin(), p->passes.begin() + p->S);
    for (int c = 0; c < p->D; ++c) {
        if (rs[0].distance[c] != 1) return;
        int count[kMaxDims] = {};
        for (int t = 0; t < p->S; ++t) {
            for (int d = 0; d < p->D; ++d) rs[t].taken[c][d] = count[d];
            count[rs[t].dim[c]] += 1;
        }
    }
    build_tile_masks(p, trees, rs);
    bool equal = true, uniform = true;
    for (int d = 0; d < p->D; ++d) {
        equal = equal && p->dims[d] == p->dims[0];
        int v = p->dims[d];
        while (v % 3 == 0) v /= 3;
        uniform = uniform && v == 1;
    }
    // The cut: the same step for every collective, from 1 to half of them the one with the fewest
    // words in all. Any cut gives the same adds; near the middle there are few roots and few nodes per
    // shape. On equal sides every collective has the first one's program (its dimensions renamed).
    const int ncoll = equal ? 1 : p->D;
    std::vector<FoldProgram> best;
    size_t best_words = 0;
    for (int cut = 1; cut <= (p->S + 1) / 2; ++cut) {
        std::vector<FoldProgram> progs(ncoll);
        size_t total = 0;
        bool ok = true;
        for (int c = 0; c < ncoll && ok; ++c) {
            ok = fold_program(FoldWalk{p, c, &flags, rs.data()}, p->S, cut, uniform, &progs[c]);
            total += progs[c].words();
        }
        if (ok && (best.empty() || total < best_words)) {
            best.swap(progs);
            best_words = total;
        }
    }
    if (best.empty()) return;
    p->folds.swap(best);
    for (int c = 0; c < p->D; ++c) {
        p->fold_of.push_back(equal ? 0 : c);
        p->fold_dim0.push_back(rs[0].dim[c]);
    }
}

}  // namespace trivance
