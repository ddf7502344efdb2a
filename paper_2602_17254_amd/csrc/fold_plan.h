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
#include <utility>
#include <vector>

#include "plan.h"

namespace trivance {

// The tree of one dimension by offset, and what the choice of the cut needs to know of it.
struct OffsetTree {
    int side = 1, S = 0;
    std::vector<uint32_t> kids;            // offset -> bits 2 k and 2 k + 1: children of step k, left and right
    std::vector<int> forward;              // offset -> the step in which it forwards (the owner: S)
    std::vector<uint32_t> alive;           // k -> offsets not forwarded in steps < k
    // Subtrees of an offset over the steps < k that differ by a translation only are one shape:
    // k -> offset -> shape (of the offsets alive), and the number of shapes.
    std::vector<std::vector<uint32_t>> shape;
    std::vector<uint32_t> shapes;
    // k -> nodes of all shapes, and the same without the children of step 0
    std::vector<uint64_t> nodes, nodes_after0;
};

// `t`: the dimension's tree, or nullptr for a side of 3^S, where offset o has both children in step k
// if 3^(k+1) divides it (the closed form of Sec. 4.3).
inline OffsetTree offset_tree(int side, const DimTree* t) {
    OffsetTree r;
    r.side = side;
    r.kids.assign(side, 0u);
    r.forward.assign(side, 0);
    std::vector<int> dist;
    if (t) {
        r.S = t->S;
        dist = t->dist;
        for (int k = 0; k < r.S; ++k)
            for (uint32_t v : t->recv[k]) r.kids[v & ~(kFromLeft | kFromRight)] |= (v >> 30) << (2 * k);
        for (int k = 0; k <= r.S; ++k)
            for (uint32_t o : t->alive[k]) r.forward[o] = k;
    } else {
        for (int m = 1; m < side; m *= 3, ++r.S) {
            dist.push_back(m);
            for (int o = 0; o < side; o += 3 * m) {
                r.kids[o] |= 3u << (2 * r.S);
                r.forward[o] = r.S + 1;
            }
        }
    }
    r.alive.assign(r.S + 1, 0u);
    for (int o = 0; o < side; ++o) ++r.alive[r.forward[o]];
    for (int k = r.S - 1; k >= 0; --k) r.alive[k] += r.alive[k + 1];
    if (!t) {
        // every subtree over the steps < k has 3^k nodes and the same shape
        uint64_t m = 1;
        for (int k = 0; k <= r.S; ++k, m *= 3) {
            r.shapes.push_back(1u);
            r.nodes.push_back(m);
            r.nodes_after0.push_back(k ? m / 3 : 1);
        }
        return r;
    }
    // a shape over the steps <= k: that of the same offset over the steps < k and those of its children
    r.shape.assign(r.S + 1, std::vector<uint32_t>(side, 0u));
    r.shapes.push_back(1u);
    std::vector<uint64_t> count{1}, after0{1};
    r.nodes.push_back(1);
    r.nodes_after0.push_back(1);
    for (int k = 0; k < r.S; ++k) {
        std::map<uint64_t, uint32_t> seen;
        std::vector<uint64_t> next, next0;
        uint64_t all = 0, all0 = 0;
        for (uint32_t o : t->alive[k + 1]) {
            const uint32_t f = (r.kids[o] >> (2 * k)) & 3u;
            const uint32_t own = r.shape[k][o];
            uint64_t key = own, n = count[own], n0 = after0[own];
            for (int q = 0; q < 2; ++q) {
                uint32_t s = 0xFFFFu;  // no child; a side is at most kMaxFoldRanks, so are the shapes
                if (f & (1u << q)) {
                    s = r.shape[k][(o + (q ? dist[k] : side - dist[k])) % side];
                    n += count[s];
                    n0 += k ? after0[s] : 0;
                }
                key = key << 16 | s;
            }
            const auto ins = seen.emplace(key, (uint32_t)next.size());
            if (ins.second) {
                next.push_back(n);
                next0.push_back(n0);
                all += n;
                all0 += n0;
            }
            r.shape[k + 1][o] = ins.first->second;
        }
        count.swap(next);
        after0.swap(next0);
        r.shapes.push_back((uint32_t)count.size());
        r.nodes.push_back(all);
        r.nodes_after0.push_back(all0);
    }
    return r;
}

// Walks the tree of one collective: nodes in preorder with the folds that follow each.
struct FoldWalk {
    struct Node {
        int o[kMaxFoldDims];
        bool leaf, first;
        uint32_t pops;
    };
    struct Step {
        int dim, dist, k;  // k: steps the collective took in `dim` before
    };

    int D;
    const int* dims;
    const OffsetTree* const* trees;
    std::vector<Step> steps;

    uint32_t children(const int* o, int t) const {
        const Step& st = steps[t];
        return (trees[st.dim]->kids[o[st.dim]] >> (2 * st.k)) & 3u;
    }

    // V(o, T) over the steps [tmin, T), appended to out.
    void visit(const int* o, int tmin, int T, bool first, std::vector<Node>* out) const {
        const size_t me = out->size();
        Node node{};
        for (int d = 0; d < D; ++d) node.o[d] = o[d];
        node.leaf = true;
        node.first = first;
        out->push_back(node);
        for (int t = tmin; t < T; ++t) {
            const uint32_t f = children(o, t);
            if (!f) continue;
            const int a = steps[t].dim, side = dims[a], dist = steps[t].dist;
            for (int q = 0; q < 2; ++q) {
                if (!(f & (1u << q))) continue;
                int child[kMaxFoldDims];
                for (int d = 0; d < D; ++d) child[d] = o[d];
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

    // Steps taken in dimension d before step `cut`.
    int taken(int d, int cut) const {
        int n = 0;
        for (int t = 0; t < cut; ++t) n += steps[t].dim == d;
        return n;
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

// Words of the program cut at step `cut`, and its roots, counted without writing it (subtrees whose words
// come out the same although their steps differ count apart).
inline uint64_t fold_size(const FoldWalk& w, int cut, uint64_t* roots) {
    uint64_t nodes = 1;
    *roots = 1;
    for (int d = 0; d < w.D; ++d) {
        const OffsetTree& t = *w.trees[d];
        const int k = w.taken(d, cut);
        *roots *= t.alive[k];
        nodes *= d == w.steps[0].dim ? t.nodes_after0[k] : t.nodes[k];
    }
    return *roots + (*roots + 1) / 2 + nodes;
}

// The program cut at step `cut`; false if it does not fit.
inline bool fold_program(const FoldWalk& w, int cut, FoldProgram* out) {
    const int zero[kMaxFoldDims] = {};
    const int dim0 = w.steps[0].dim;
    std::vector<FoldWalk::Node> top, sub;
    w.visit(zero, cut, (int)w.steps.size(), true, &top);
    *out = FoldProgram();
    out->top_depth = fold_depth(top);
    // a subtree's words depend on its shape along every dimension only: each is written once
    uint32_t radix[kMaxFoldDims], combined = 1;
    int k[kMaxFoldDims];
    for (int d = 0; d < w.D; ++d) {
        k[d] = w.taken(d, cut);
        radix[d] = combined;
        combined *= w.trees[d]->shapes[k[d]];
    }
    std::vector<int> known(combined, -1);
    std::map<std::vector<uint32_t>, int> seen;
    for (const FoldWalk::Node& r : top) {
        if (r.pops > kFoldMaxPops) return false;
        out->roots.push_back(fold_word(r, w.D, dim0, zero, w.dims));
        uint32_t which = 0;
        for (int d = 0; d < w.D; ++d)
            if (!w.trees[d]->shape.empty()) which += radix[d] * w.trees[d]->shape[k[d]][r.o[d]];
        if (known[which] < 0) {
            sub.clear();
            w.visit(r.o, 1, cut, true, &sub);
            std::vector<uint32_t> words;
            for (const FoldWalk::Node& nd : sub) {
                if (nd.pops > kFoldMaxPops) return false;
                const uint32_t f = w.children(nd.o, 0);
                words.push_back(fold_word(nd, w.D, dim0, r.o, w.dims) |
                                (f & 1u ? kFoldLeft : 0u) | (f & 2u ? kFoldRight : 0u));
            }
            words.back() |= kFoldLast;
            const auto ins = seen.emplace(words, (int)out->shape_begin.size());
            if (ins.second) {
                out->sub_depth = std::max(out->sub_depth, fold_depth(sub));
                out->shape_begin.push_back((uint32_t)out->nodes.size());
                out->nodes.insert(out->nodes.end(), words.begin(), words.end());
                if (out->words() > kMaxFoldWords) return false;
            }
            known[which] = ins.first->second;
        }
        out->shape.push_back((uint32_t)known[which]);
    }
    return out->words() <= kMaxFoldWords;
}

// The trees by offset (kMaxTileSteps in plan.h); none if they do not fit.
inline void build_tile_masks(trivance_plan_t* p, const OffsetTree* const* trees,
                             const std::vector<FoldWalk>& walks) {
    p->tile_masks.clear();
    p->tile_mask0.clear();
    if (p->S > kMaxTileSteps) return;
    for (int d = 0; d < p->D; ++d)
        if ((size_t)p->dims[d] > kMaxTileWords) return;
    std::vector<uint32_t> words, first;
    std::map<std::vector<uint32_t>, uint32_t> seen;
    for (int c = 0; c < p->D; ++c)
        for (int d = 0; d < p->D; ++d) {
            std::vector<int> at(trees[d]->S + 1, 31);  // the collective's step of the tree's step k
            for (int t = 0; t < p->S; ++t)
                if (walks[c].steps[t].dim == d) at[walks[c].steps[t].k] = t;
            std::vector<uint32_t> w(p->dims[d]);
            for (int o = 0; o < p->dims[d]; ++o) {
                w[o] = (uint32_t)at[trees[d]->forward[o]] << kTileForwardShift;
                for (int k = 0; k < trees[d]->S; ++k)
                    w[o] |= ((trees[d]->kids[o] >> (2 * k)) & 3u) << (2 * at[k]);
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
// none and runs step by step. Every plan pays for this, also one that only the cost model reads. So the
// words of every cut are counted and one program is written: plans of a ring of 243 / a ring of 6561 /
// 32x32 / 16x16x16 / 16x18x20 ranks take 4 / 19 / 18 / 33 / 70 us, with every cut's program written
// to compare them 27 / 1090 / 105 / 311 / 854, with none 1 / 1 / 9 / 7 / 6.
inline void build_fold_programs(trivance_plan_t* p) {
    p->folds.clear();
    if (p->n < 2 || p->n > kMaxFoldRanks || p->D > kMaxFoldDims || p->S < 1) return;
    for (int d = 0; d < p->D; ++d)
        if (p->dims[d] > (1 << (kFoldCoordBits / p->D)) - 1) return;
    for (int c = 0; c < p->D; ++c)
        if (p->passes[0].distance[c] != 1) return;
    OffsetTree built[kMaxFoldDims];
    const OffsetTree* trees[kMaxFoldDims];
    for (int d = 0; d < p->D; ++d) {
        int e = 0;  // the first dimension of this side
        while (p->dims[e] != p->dims[d]) ++e;
        if (e == d) built[d] = offset_tree(p->dims[d], p->tree ? &p->trees[d] : nullptr);
        trees[d] = &built[e];
    }
    std::vector<FoldWalk> walks(p->D);
    bool equal = true;
    for (int c = 0; c < p->D; ++c) {
        walks[c] = FoldWalk{p->D, p->dims, trees, {}};
        int count[kMaxDims] = {};
        for (int t = 0; t < p->S; ++t) {
            const int a = p->passes[t].dim[c];
            walks[c].steps.push_back({a, p->passes[t].distance[c], count[a]++});
        }
        equal = equal && p->dims[c] == p->dims[0];
    }
    build_tile_masks(p, trees, walks);
    // The cut: the same step for every collective, from 1 to half of them the one with the fewest
    // words in all. Any cut gives the same adds; near the middle there are few roots and few nodes per
    // shape. On equal sides every collective has the first one's program (its dimensions renamed).
    const int ncoll = equal ? 1 : p->D;
    std::vector<std::pair<uint64_t, int>> cuts;
    for (int cut = 1; cut <= (p->S + 1) / 2; ++cut) {
        uint64_t total = 0, roots = 0, most = 0;
        for (int c = 0; c < ncoll; ++c) {
            total += fold_size(walks[c], cut, &roots);
            most = std::max(most, roots);
        }
        if (most <= (uint64_t)kMaxFoldRoots) cuts.emplace_back(total, cut);
    }
    std::sort(cuts.begin(), cuts.end());
    std::vector<FoldProgram> progs(ncoll);
    for (const auto& cut : cuts) {
        bool ok = true;
        for (int c = 0; c < ncoll && ok; ++c) ok = fold_program(walks[c], cut.second, &progs[c]);
        if (!ok) continue;
        p->folds.swap(progs);
        for (int c = 0; c < p->D; ++c) {
            p->fold_of.push_back(equal ? 0 : c);
            p->fold_dim0.push_back(walks[c].steps[0].dim);
        }
        return;
    }
}

}  // namespace trivance
