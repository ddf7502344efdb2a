// Whole bandwidth-optimal AllReduce for gfx950: each vector is read once and written once. The fold
// kernel adds up every column over the rows in the order of the block's reduction tree (the
// programs come from fold_plan.h), so the results are the step kernels', bit for bit; the
// result goes to every row, as the all-gather's copies would carry it.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>
#include <cstring>

#include "calls.h"
#include "device.h"
#include "forms.h"
#include "plan.h"

namespace trivance {
namespace {

// What the split and the layout rest on (MI355X, 16x16x16 ranks of 4 MiB unless said otherwise).
// One read and one write of every vector at the rate of a plain copy (6.76 TB/s) take 5.08 ms; the
// 18 step launches took 22.4 ms, fold and spread take 4.98 (less than
// the copy's: see the rates of pure reads and pure writes below).
//  * Two launches. Waves that read their column of all rows and then write it to all rows drift
//    apart, and with reads and writes of many rows mixed the memory gave 4.9-5.3 TB/s on 240 rows
//    of 32 MiB and 4.6-5.9 on 16 of 256 MiB, over nine store policies, occupancies, batches,
//    barriers and pipelined waves. Reads alone reach 6.7-7.2, and one-store waves that walk the
//    rows in address order 7.0-7.4. So the fold only writes row 0, and spread_kernel copies it. The
//    one-launch form stays for the calls that fold_spreads (forms.h) names.
//  * The scalar unit bounds the reads next: a wave's kibibyte may take 91 cycles of its compute
//    unit, and decoding one row per program word took about as many. One word for the up to
//    three rows of V(o, 1) cut the read part from 3.58 to 2.69 ms.
//  * Three nodes (up to nine loads) in flight per wave: two or four measured the same, six 18%
//    slower (128 instead of 96 registers). Where several waves share a tile, five or six gained
//    1% at 16x16x16 ranks of 64 Ki values and lost 27% at 64 ranks of 400000.
constexpr int kFoldBatch = 3;

struct FoldArgs {
    int64_t elems;
    int64_t seg_g[kMaxFoldDims + 1];
    uint32_t n;
    uint32_t side[kMaxFoldDims], stride[kMaxFoldDims];
    FastDiv32 f_side[kMaxFoldDims];
    FastDiv32 f_gc[kMaxFoldDims];        // granules of segment c
    uint32_t tile_end[kMaxFoldDims];     // segment c owns tiles [tile_end[c-1], tile_end[c])
    uint32_t tail_tile;                  // the tile of the last elems % 4 columns (or beyond all)
    uint32_t nroots[kMaxFoldDims];       // per collective: its program in tab
    uint32_t root0[kMaxFoldDims], start0[kMaxFoldDims], node0[kMaxFoldDims];
    uint32_t dim0[kMaxFoldDims];         // dimension of the collective's first step
    uint32_t steps;                      // placed plans: reduce-scatter steps
    uint32_t pdim[kMaxFoldDims];         // and the dimension of step t in bits 4 t .. 4 t + 3
    int placed;
    int sub_depth, top_depth;
    uint32_t lanes;                      // column vectors of a tile
    uint32_t wg_base;
    int spread;                          // 1: the result goes to row 0 only (spread_kernel follows)
    uint32_t tab[kMaxFoldWords];
};
static_assert(sizeof(FoldArgs) <= 4096, "fold kernel arguments above 4 KiB");

// One tile: `lanes` column vectors of every row. P waves evaluate the subtrees of the cut (P = 1:
// a wave of its own, which also combines them as it goes).
template <typename T, int VEC, int D, int P>
__device__ __forceinline__ void fold_tile(T* __restrict__ buf, const FoldArgs& a, uint32_t tile,
                                          uint32_t wave, Vec<T, VEC>* lds) {
    using V = Vec<T, VEC>;
    const uint32_t lane = threadIdx.x & 63;
    int c = 0;
#pragma unroll
    for (int i = 0; i < D - 1; ++i)
        if (tile >= a.tile_end[i]) c = i + 1;
    const int64_t E = a.elems;
    const int64_t seg_b = a.seg_g[c] * kGranule;
    const int64_t seg_e = imin64(a.seg_g[c + 1] * kGranule, E);
    const uint32_t W = a.lanes;
    // the tile's columns; the tail tile holds the columns after the last whole vector
    const int64_t col0 = VEC == 1 ? E / 4 * 4
                                  : seg_b + (int64_t)(tile - (c ? a.tile_end[c - 1] : 0u)) * W * VEC;
    const uint32_t nvec = (uint32_t)imin64((seg_e - col0) / VEC, W);
    // lanes without a column of their own repeat the last one and store nothing
    const uint32_t cl = lane < nvec ? lane : nvec - 1;
    const T* const col = buf + col0 + (int64_t)cl * VEC;

    // the block of this lane's columns and its coordinates
    const uint32_t gr = (uint32_t)((col0 - seg_b + (int64_t)cl * VEC) / kGranule);
    uint32_t j = fdiv32((gr + 1) * a.n - 1, a.f_gc[c]);
    uint32_t y[D] = {};
    if (a.placed) {
        // j is the block's position: its base-3 digits, the last step's lowest
        for (int t = (int)a.steps - 1; t >= 0; --t) {
            const uint32_t j3 = __umulhi(j, 0xAAAAAAABu) >> 1;
            const uint32_t dim = (a.pdim[c] >> (4 * t)) & 15u;
            const uint32_t digit = j - 3u * j3;
#pragma unroll
            for (int d = 0; d < D; ++d)
                if (dim == (uint32_t)d) y[d] = 3u * y[d] + digit;
            j = j3;
        }
    } else {
#pragma unroll
        for (int d = 0; d < D; ++d) {
            const uint32_t q = d + 1 < D ? fdiv32(j, a.f_side[d]) : 0u;
            y[d] = j - q * a.side[d];
            j = q;
        }
    }
    // in the order of dimensions dim0, dim0 + 1, ... (cyclic), as in the program
    uint32_t x[D], side[D], stride[D];
#pragma unroll
    for (int f = 0; f < D; ++f) {
        const uint32_t d = a.dim0[c] + f < (uint32_t)D ? a.dim0[c] + f : a.dim0[c] + f - D;
        side[f] = a.side[d];
        stride[f] = a.stride[d];
        x[f] = y[0];
#pragma unroll
        for (int q = 1; q < D; ++q)
            if ((uint32_t)q == d) x[f] = y[q];
    }
    constexpr int kBits = kFoldCoordBits / D;
    constexpr uint32_t kMask = (1u << kBits) - 1u;
    const uint64_t row_bytes = (uint64_t)E * sizeof(T);

    // the wave's part of the local memory: sums open below the current one
    V* const sub = lds + (P == 1 ? 0u : (a.nroots[c] + 1u + wave * (uint32_t)a.sub_depth) * W);
    const uint32_t SW = P == 1 ? 64u : W;          // vectors of one open sum
    const uint32_t sl = P == 1 ? lane : (lane < W ? lane : W - 1);
    V* const top = P == 1 ? sub + a.sub_depth * 64 : lds + (a.nroots[c] + 1u + P * (uint32_t)a.sub_depth) * W;
    V cur, tcur;
#pragma unroll
    for (int i = 0; i < VEC; ++i) cur.v[i] = tcur.v[i] = (T)0;
    int sp = 0, tp = 0;
    auto add_root = [&](uint32_t rw, const V& val) {
        if (rw & kFoldFirst) {
            tcur = val;
        } else if (rw & kFoldLeaf) {
            tcur = vadd(tcur, val);
        } else {
            top[tp * SW + sl] = tcur;
            ++tp;
            tcur = val;
        }
        for (uint32_t k = (rw >> kFoldPopsShift) & kFoldMaxPops; k > 0; --k) {
            --tp;
            tcur = vadd(top[tp * SW + sl], tcur);
        }
    };

    const uint32_t nroots = a.nroots[c];
    const uint32_t* const roots = a.tab + a.root0[c];
    const uint32_t* const starts = a.tab + a.start0[c];
    const uint32_t* const nodes = a.tab + a.node0[c];
    uint32_t g = P == 1 ? 0u : wave;
    uint32_t rw = 0, pos = 0, xr[D];  // the open subtree: its word, its next node, its root's coordinates
    auto wrap = [](uint32_t v, uint32_t n) {  // v mod n for v < 2 n
        const uint32_t z = v - n;
        return v < z ? v : z;  // z wraps around when v < n
    };
    auto open_root = [&]() {
        rw = roots[g];
        pos = (starts[g >> 1] >> (16 * (g & 1u))) & 0xFFFFu;
#pragma unroll
        for (int f = 0; f < D; ++f) xr[f] = wrap(x[f] + ((rw >> (f * kBits)) & kMask), side[f]);
    };
    if (g < nroots) open_root();
    while (g < nroots) {
        V vo[kFoldBatch], vl[kFoldBatch], vr[kFoldBatch];
        uint32_t w[kFoldBatch], rws[kFoldBatch], gs[kFoldBatch];
        int live = 0;
#pragma unroll
        for (int u = 0; u < kFoldBatch; ++u) {
            if (g < nroots) {
                live = u + 1;
                w[u] = nodes[pos];
                rws[u] = rw;
                gs[u] = g;
                uint32_t z[D], rest = 0;
#pragma unroll
                for (int f = 0; f < D; ++f) {
                    z[f] = wrap(xr[f] + ((w[u] >> (f * kBits)) & kMask), side[f]);
                    if (f) rest += z[f] * stride[f];
                }
                auto at = [&](uint32_t z0) {
                    return ld_any<T, VEC, true>(reinterpret_cast<const T*>(
                        reinterpret_cast<const char*>(col) + (rest + z0 * stride[0]) * row_bytes));
                };
                vo[u] = at(z[0]);
                if (w[u] & kFoldLeft) vl[u] = at(wrap(z[0] + side[0] - 1u, side[0]));
                if (w[u] & kFoldRight) vr[u] = at(wrap(z[0] + 1u, side[0]));
                if (w[u] & kFoldLast) {
                    g += P;
                    if (g < nroots) open_root();
                } else {
                    ++pos;
                }
            }
        }
#pragma unroll
        for (int u = 0; u < kFoldBatch; ++u) {
            if (u >= live) break;
            V val = vo[u];
            if (w[u] & kFoldLeft) val = vadd(val, vl[u]);
            if (w[u] & kFoldRight) val = vadd(val, vr[u]);
            if (w[u] & kFoldFirst) {
                cur = val;
            } else if (w[u] & kFoldLeaf) {
                cur = vadd(cur, val);
                for (uint32_t k = (w[u] >> kFoldPopsShift) & kFoldMaxPops; k > 0; --k) {
                    --sp;
                    cur = vadd(sub[sp * SW + sl], cur);
                }
            } else {
                sub[sp * SW + sl] = cur;
                ++sp;
                cur = val;
            }
            if (w[u] & kFoldLast) {
                if constexpr (P == 1) add_root(rws[u], cur);
                else lds[gs[u] * W + sl] = cur;
            }
        }
    }
    // every row has been read: the result goes to all of them
    if constexpr (P == 1) {
        const uint32_t nbytes = nvec * VEC * (uint32_t)sizeof(T);
        const uint32_t off = lane * VEC * (uint32_t)sizeof(T);
        T* out = buf + col0;
        const uint32_t rows = a.spread ? 1u : a.n;
        for (uint32_t r = 0; r < rows; ++r, out += E)
            st_out_as<1>(buffer_rsrc(out, nbytes), off, tcur);
    } else {
        __syncthreads();
        V* const res = lds + nroots * W;
        if (wave == 0) {
            for (uint32_t k = 0; k < nroots; ++k) add_root(roots[k], lds[k * W + sl]);
            res[sl] = tcur;
        }
        __syncthreads();
        // a store instruction covers 64 / W rows
        const uint32_t per = 64u / W, lr = lane / W, lc = lane - lr * W;
        const V val = res[lc];
        const uint32_t off = (uint32_t)(lr * row_bytes) + lc * VEC * (uint32_t)sizeof(T);
        const uint32_t rows = a.spread ? 1u : a.n;
        for (uint32_t r = wave * per; r < rows; r += P * per)
            if (lc < nvec && r + lr < rows)
                st_out_as<1>(buffer_rsrc(buf + col0 + (int64_t)r * E, 0xFFFFFFFFu), off, val);
    }
}

template <typename T, int D, int P>
__global__ __launch_bounds__(64 * (P == 1 ? kStreamWaves : P)) void fold_kernel(T* __restrict__ buf,
                                                                                FoldArgs a) {
    extern __shared__ __align__(16) char lds[];
    const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t wg = a.wg_base + xcd_contiguous(blockIdx.x, gridDim.x);
    const uint32_t tile = P == 1 ? wg * kStreamWaves + wave : wg;
    if (tile >= a.tile_end[D - 1]) return;
    // waves with a tile of their own: a part of the local memory each, of the size of whole vectors
    // also where the tile is the tail
    char* const mine = P == 1 ? lds + wave * (uint32_t)(a.sub_depth + a.top_depth) * 64u * 16u : lds;
    if (tile == a.tail_tile)
        fold_tile<T, 1, D, P>(buf, a, tile, wave, reinterpret_cast<Vec<T, 1>*>(mine));
    else
        fold_tile<T, 4, D, P>(buf, a, tile, wave, reinterpret_cast<Vec<T, 4>*>(mine));
}

// Copies row 0 to every other row. One wave stores up to 64 vectors of one row; consecutive waves
// walk the tiles of one panel of a row, then the next row, then the next panel.
//  * One store per wave, in address order: 7.0-7.4 TB/s where the all-gather steps' two stores per
//    load gave 6.2; three or more rows per wave gave 5.5-6.4.
//  * A panel of 4096 tiles (4 MiB of row 0) stays in the L2 caches while all rows are written, and
//    a multiple of 8 workgroups per panel row keeps each XCD on its own eighth of it. Panels of
//    0.5, 1 and 2 MiB measured 25, 16 and 7% slower on the 9x9x9 torus at 8 MiB, 8 MiB the same,
//    64 MiB 10% slower on the ring of 8.
//  * A row whose length is no multiple of 128 bytes starts inside a cache line. Its tiles are
//    shifted so that every store but the row's first and last ones covers whole lines.
struct SpreadArgs {
    int64_t elems;
    uint32_t n1;          // rows to write: n - 1
    uint32_t tiles;       // per row
    uint32_t panel;       // tiles of a panel
    uint32_t units;       // n1 * tiles
    FastDiv32 f_full;     // panel * n1
    FastDiv32 f_panel, f_last;  // panel, tiles of the last one
    uint32_t wg_base;
    int shifted;
};
constexpr uint32_t kSpreadPanel = 4096;
constexpr int kSpreadWaves = 4;

template <typename T>
__global__ __launch_bounds__(64 * kSpreadWaves) void spread_kernel(T* __restrict__ buf,
                                                                   SpreadArgs a) {
    const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t lane = threadIdx.x & 63;
    const uint32_t unit = (a.wg_base + blockIdx.x) * kSpreadWaves + wave;
    if (unit >= a.units) return;
    const uint32_t p = fdiv32(unit, a.f_full);
    const uint32_t rest = unit - p * a.panel * a.n1;
    const bool last = (p + 1) * a.panel > a.tiles;
    const uint32_t width = last ? a.tiles - p * a.panel : a.panel;
    const uint32_t r = fdiv32(rest, last ? a.f_last : a.f_panel);
    const int64_t E = a.elems;
    T* const dst = buf + (int64_t)(r + 1) * E;
    int64_t col = (int64_t)(p * a.panel + (rest - r * width)) * kSpreadTile + lane * 4;
    // elements of the row before its first whole cache line: tile 0 ends there
    if (a.shifted)
        col -= kSpreadTile - ((0u - (uint32_t)(reinterpret_cast<uintptr_t>(dst) / sizeof(T))) & 31u);
    const BufI4 rs = buffer_rsrc(dst, (uint32_t)(E * (int64_t)sizeof(T)));
    if (col >= 0 && col + 4 <= E) {
        st_out_as<0>(rs, (uint32_t)col * (uint32_t)sizeof(T), ld_any<T, 4, false>(buf + col));
    } else {
        for (int i = 0; i < 4; ++i)
            if (col + i >= 0 && col + i < E)
                st_out_as<0>(rs, (uint32_t)(col + i) * (uint32_t)sizeof(T), Vec<T, 1>{{buf[col + i]}});
    }
}

template <typename T>
hipError_t launch_spread(T* buf, int64_t elems, const trivance_plan_t* p, const Exec& x) {
    SpreadArgs a;
    std::memset(&a, 0, sizeof(a));
    a.elems = elems;
    a.n1 = (uint32_t)p->n - 1;
    a.shifted = elems % 32 != 0 || (uintptr_t)buf % 128 != 0 ? 1 : 0;
    a.tiles = (uint32_t)((elems + kSpreadTile - 1) / kSpreadTile) + (a.shifted ? 1u : 0u);
    a.panel = std::min(kSpreadPanel, a.tiles);
    a.units = a.n1 * a.tiles;
    a.f_full = make_fastdiv32(a.panel * a.n1);
    a.f_panel = make_fastdiv32(a.panel);
    a.f_last = make_fastdiv32(a.tiles % a.panel ? a.tiles % a.panel : a.panel);
    hipError_t err = hipSuccess;
    for_each_dispatch(((uint64_t)a.units + kSpreadWaves - 1) / kSpreadWaves, 64 * kSpreadWaves,
                      x.items, [&](uint32_t first, uint32_t count) {
        a.wg_base = first;
        hipLaunchKernelGGL((spread_kernel<T>), dim3(count), dim3(64 * kSpreadWaves), 0, x.stream,
                           buf, a);
        err = hipGetLastError();
        return err == hipSuccess;
    });
    return err;
}

template <typename T, int D, int P>
hipError_t launch_fold(T* buf, FoldArgs a, uint64_t grid, size_t lds, const Exec& x) {
    hipError_t err = hipSuccess;
    constexpr int threads = 64 * (P == 1 ? kStreamWaves : P);
    for_each_dispatch(grid, threads, x.items, [&](uint32_t first, uint32_t count) {
        a.wg_base = first;
        hipLaunchKernelGGL((fold_kernel<T, D, P>), dim3(count), dim3(threads), lds, x.stream, buf,
                           a);
        err = hipGetLastError();
        return err == hipSuccess;
    });
    return err;
}

template <typename T, int D>
int run_fold_dims(T* buf, int64_t elems, const trivance_plan_t* p, hipStream_t stream) {
    const Exec x{stream, p->dispatch_items};
    const FoldShape s = fold_shape(p, elems);
    FoldArgs a;
    std::memset(&a, 0, sizeof(a));
    a.elems = elems;
    a.n = (uint32_t)p->n;
    a.lanes = s.lanes;
    a.spread = s.spread;
    a.placed = p->placed ? 1 : 0;
    a.steps = (uint32_t)p->S;
    const int64_t G = (elems + kGranule - 1) / kGranule;
    for (int c = 0; c <= D; ++c) a.seg_g[c] = (int64_t)c * G / D;
    for (int c = 0; c < D; ++c) {
        a.f_gc[c] = make_fastdiv32((uint32_t)std::max<int64_t>(1, a.seg_g[c + 1] - a.seg_g[c]));
        a.side[c] = (uint32_t)p->dims[c];
        a.stride[c] = (uint32_t)p->strides[c];
        a.f_side[c] = make_fastdiv32((uint32_t)p->dims[c]);
        if (p->placed)
            for (int t = 0; t < p->S; ++t) a.pdim[c] |= (uint32_t)p->passes[t].dim[c] << (4 * t);
    }
    // programs: all in one launch, or one launch per collective
    const bool together = fold_together(p);
    for (int c0 = 0; c0 < D; c0 += together ? D : 1) {
        const int c1 = together ? D : c0 + 1;
        uint32_t used = 0;
        a.sub_depth = a.top_depth = 0;
        size_t most_roots = 0;
        uint32_t at[kMaxFoldDims];
        for (size_t f = 0; f < p->folds.size(); ++f) {
            const FoldProgram& fp = p->folds[f];
            if (!together && (int)f != p->fold_of[c0]) continue;
            at[f] = used;
            for (uint32_t w : fp.roots) a.tab[used++] = w;
            for (size_t r = 0; r < fp.roots.size(); r += 2)
                a.tab[used++] = fp.shape_begin[fp.shape[r]] |
                                (r + 1 < fp.roots.size() ? fp.shape_begin[fp.shape[r + 1]] << 16 : 0u);
            for (uint32_t w : fp.nodes) a.tab[used++] = w;
            a.sub_depth = std::max(a.sub_depth, fp.sub_depth);
            a.top_depth = std::max(a.top_depth, fp.top_depth);
            most_roots = std::max(most_roots, fp.roots.size());
        }
        uint32_t tiles = 0;
        a.tail_tile = ~0u;
        for (int c = 0; c < D; ++c) {
            if (c >= c0 && c < c1) {
                const FoldProgram& fp = p->folds[p->fold_of[c]];
                a.dim0[c] = (uint32_t)p->fold_dim0[c];
                a.nroots[c] = (uint32_t)fp.roots.size();
                a.root0[c] = at[p->fold_of[c]];
                a.start0[c] = a.root0[c] + a.nroots[c];
                a.node0[c] = a.start0[c] + (a.nroots[c] + 1) / 2;
                const int64_t len = std::min(a.seg_g[c + 1] * kGranule, elems) - a.seg_g[c] * kGranule;
                tiles += (uint32_t)((len / 4 + s.lanes - 1) / s.lanes);
                if (len % 4) a.tail_tile = tiles++;
            }
            a.tile_end[c] = tiles;
        }
        if (tiles == 0) continue;
        const size_t lds = fold_lds(s, most_roots, a.sub_depth, a.top_depth);
        hipError_t err;
        if (s.waves == 1)
            err = launch_fold<T, D, 1>(buf, a, (tiles + kStreamWaves - 1) / kStreamWaves, lds, x);
        else if (s.waves == 4)
            err = launch_fold<T, D, 4>(buf, a, tiles, lds, x);
        else
            err = launch_fold<T, D, 16>(buf, a, tiles, lds, x);
        if (err != hipSuccess) return TRIVANCE_EHIP;
    }
    if (s.spread && launch_spread(buf, elems, p, x) != hipSuccess) return TRIVANCE_EHIP;
    return TRIVANCE_OK;
}

template <typename T>
int run_fold(T* buf, int64_t elems, const trivance_plan_t* p, hipStream_t stream) {
    switch (p->D) {
        case 1: return run_fold_dims<T, 1>(buf, elems, p, stream);
        case 2: return run_fold_dims<T, 2>(buf, elems, p, stream);
        case 3: return run_fold_dims<T, 3>(buf, elems, p, stream);
        default: return run_fold_dims<T, 4>(buf, elems, p, stream);
    }
}

}  // namespace

int run_fold_call(float* buf, int64_t elems, const trivance_plan_t* p, hipStream_t stream) {
    return run_fold(buf, elems, p, stream);
}

int run_fold_call(int* buf, int64_t elems, const trivance_plan_t* p, hipStream_t stream) {
    return run_fold(buf, elems, p, stream);
}

}  // namespace trivance
