// Whole bandwidth-optimal AllReduce in one launch, for gfx950: the fold kernel and its launcher. The
// fold programs come from fold_plan.h.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>
#include <cstring>
#ifdef FOLD_TUNE
#include <cstdlib>
#endif

#include "device.h"
#include "plan.h"

namespace trivance {
namespace {

constexpr int kFoldBatch = 8;  // rows whose loads a wave issues together
constexpr int kStreamWaves = 4;

struct FoldArgs {
    int64_t elems;
    int64_t seg_g[kMaxFoldDims + 1];
    uint32_t n;
    int narrow;                          // 1 if n * (granules of a segment + 1) < 2^31
    uint32_t side[kMaxFoldDims], stride[kMaxFoldDims];
    FastDiv32 f_side[kMaxFoldDims];
    FastDiv32 f_gc[kMaxFoldDims];        // granules of segment c
    uint32_t tile_end[kMaxFoldDims];     // segment c owns tiles [tile_end[c-1], tile_end[c])
    uint32_t tail_tile;                  // the tile of the last elems % 4 columns (or beyond all)
    uint32_t nroots[kMaxFoldDims];       // per collective: its program in tab
    uint32_t root0[kMaxFoldDims], start0[kMaxFoldDims], node0[kMaxFoldDims];
    uint32_t steps;                      // placed plans: reduce-scatter steps
    uint32_t pdim[kMaxFoldDims];         // and the dimension of step t in bits 4 t .. 4 t + 3
    int placed;
    int sub_depth, top_depth;
    uint32_t lanes;                      // column vectors of a tile
    uint32_t wg_base;
    int keep;
    uint32_t tab[kMaxFoldWords];
};
static_assert(sizeof(FoldArgs) <= 4096, "fold kernel arguments above 4 KiB");

// Rows whose length is no multiple of 16 bytes are read with 16-byte loads all the same: the
// instructions need 4-byte alignment.
template <typename T, int VEC>
__device__ __forceinline__ Vec<T, VEC> ld_row(const T* p) {
    Vec<T, VEC> r;
    if constexpr (VEC == 4) {
        typedef T U __attribute__((ext_vector_type(4), aligned(4)));
        const U x = __builtin_nontemporal_load(reinterpret_cast<const U*>(p));
#pragma unroll
        for (int i = 0; i < 4; ++i) r.v[i] = x[i];
    } else {
        r.v[0] = __builtin_nontemporal_load(p);
    }
    return r;
}

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

    // the block of this lane's columns and its coordinates, in the order of dimensions c, c + 1, ...
    const uint32_t gr = (uint32_t)((col0 - seg_b + (int64_t)cl * VEC) / kGranule);
    uint32_t j;
    if (a.narrow) {
        j = fdiv32((gr + 1) * a.n - 1, a.f_gc[c]);
    } else {
        j = (uint32_t)(((uint64_t)(gr + 1) * a.n - 1) / (uint64_t)(a.seg_g[c + 1] - a.seg_g[c]));
    }
    uint32_t x[D], side[D], stride[D];
    if (a.placed) {
        // j is the block's position: its base-3 digits, the last step's lowest
        uint32_t y[D] = {};
        for (int t = (int)a.steps - 1; t >= 0; --t) {
            const uint32_t j3 = __umulhi(j, 0xAAAAAAABu) >> 1;
            const uint32_t dim = (a.pdim[c] >> (4 * t)) & 15u;
            const uint32_t digit = j - 3u * j3;
#pragma unroll
            for (int d = 0; d < D; ++d)
                if (dim == (uint32_t)d) y[d] = 3u * y[d] + digit;
            j = j3;
        }
#pragma unroll
        for (int f = 0; f < D; ++f) {
            const int d = c + f < D ? c + f : c + f - D;
#pragma unroll
            for (int q = 0; q < D; ++q)
                if (q == d) x[f] = y[q];
        }
    } else {
        uint32_t y[D];
#pragma unroll
        for (int d = 0; d < D; ++d) {
            const uint32_t q = d + 1 < D ? fdiv32(j, a.f_side[d]) : 0u;
            y[d] = j - q * a.side[d];
            if (d + 1 == D) y[d] = j;
            j = q;
        }
#pragma unroll
        for (int f = 0; f < D; ++f) {
            const int d = c + f < D ? c + f : c + f - D;
#pragma unroll
            for (int q = 0; q < D; ++q)
                if (q == d) x[f] = y[q];
        }
    }
#pragma unroll
    for (int f = 0; f < D; ++f) {
        const int d = c + f < D ? c + f : c + f - D;
        side[f] = a.side[d];
        stride[f] = a.stride[d];
    }
    constexpr int kBits = kFoldCoordBits / D;
    constexpr uint32_t kMask = (1u << kBits) - 1u;
    const uint64_t row_bytes = (uint64_t)E * sizeof(T);

    // the wave's part of the local memory: sums open below the current one
    V* const sub = lds + (P == 1 ? wave * (uint32_t)(a.sub_depth + a.top_depth) * 64u
                                 : (a.nroots[c] + 1u + wave * (uint32_t)a.sub_depth) * W);
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
        for (uint32_t k = rw >> kFoldPopsShift; k > 0; --k) {
            --tp;
            tcur = vadd(top[tp * SW + sl], tcur);
        }
    };

    const uint32_t nroots = a.nroots[c];
    const uint32_t* const roots = a.tab + a.root0[c];
    const uint32_t* const starts = a.tab + a.start0[c];
    const uint32_t* const nodes = a.tab + a.node0[c];
    uint32_t g = P == 1 ? 0u : wave;
    uint32_t rw = 0, pos = 0, r0[D];
    auto open_root = [&]() {
        rw = roots[g];
        pos = (starts[g >> 1] >> (16 * (g & 1u))) & 0xFFFFu;
#pragma unroll
        for (int f = 0; f < D; ++f) r0[f] = (rw >> (f * kBits)) & kMask;
    };
    if (g < nroots) open_root();
    while (g < nroots) {
        V v[kFoldBatch];
        uint32_t w[kFoldBatch], rws[kFoldBatch], gs[kFoldBatch];
#pragma unroll
        for (int u = 0; u < kFoldBatch; ++u) {
            w[u] = kFoldLast | kFoldFirst | kFoldLeaf;
            rws[u] = gs[u] = ~0u;
            if (g < nroots) {
                w[u] = nodes[pos];
                rws[u] = rw;
                gs[u] = g;
                uint32_t row = 0;
#pragma unroll
                for (int f = 0; f < D; ++f) {
                    uint32_t s = r0[f] + ((w[u] >> (f * kBits)) & kMask);
                    s = s >= side[f] ? s - side[f] : s;
                    const uint32_t y = x[f] + s;
                    const uint32_t z = y - side[f];
                    row += (y < z ? y : z) * stride[f];  // z wraps around when y < side
                }
                v[u] = ld_row<T, VEC>(reinterpret_cast<const T*>(
                    reinterpret_cast<const char*>(col) + row * row_bytes));
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
            if (gs[u] == ~0u) continue;
            if (w[u] & kFoldFirst) {
                cur = v[u];
            } else if (w[u] & kFoldLeaf) {
                cur = vadd(cur, v[u]);
                for (uint32_t k = w[u] >> kFoldPopsShift; k > 0; --k) {
                    --sp;
                    cur = vadd(sub[sp * SW + sl], cur);
                }
            } else {
                sub[sp * SW + sl] = cur;
                ++sp;
                cur = v[u];
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
        for (uint32_t r = 0; r < a.n; ++r, out += E)
            st_out<T, VEC>(buffer_rsrc(out, nbytes), off, tcur, a.keep);
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
        for (uint32_t r = wave * per; r < a.n; r += P * per)
            if (lc < nvec && r + lr < a.n)
                st_out<T, VEC>(buffer_rsrc(buf + col0 + (int64_t)r * E, 0xFFFFFFFFu), off, val,
                               a.keep);
    }
}

template <typename T, int D, int P>
__global__ __launch_bounds__(64 * (P == 1 ? kStreamWaves : P)) void fold_kernel(T* __restrict__ buf,
                                                                                FoldArgs a) {
    extern __shared__ __align__(16) char lds[];
    const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t wg = a.wg_base + blockIdx.x;
    const uint32_t tile = P == 1 ? wg * kStreamWaves + wave : wg;
    if (tile >= a.tile_end[D - 1]) return;
    if (tile == a.tail_tile)
        fold_tile<T, 1, D, P>(buf, a, tile, wave, reinterpret_cast<Vec<T, 1>*>(lds));
    else
        fold_tile<T, 4, D, P>(buf, a, tile, wave, reinterpret_cast<Vec<T, 4>*>(lds));
}

struct FoldShape {
    int waves;       // waves per tile
    uint32_t lanes;  // column vectors of a tile
};

inline FoldShape fold_shape(const trivance_plan_t* p, int64_t elems) {
    FoldShape s{1, 64};
    const int64_t tiles = (elems + 255) / 256;
    if (tiles < 2048) s = FoldShape{16, 64};
    if (tiles < 256) s = FoldShape{16, 16};
#ifdef FOLD_TUNE
    if (const char* e = std::getenv("FOLD_P")) s.waves = std::atoi(e);
    if (const char* e = std::getenv("FOLD_W")) s.lanes = (uint32_t)std::atoi(e);
#endif
    if (s.waves > 1)
        while (s.lanes > 4 && p->folds[0].roots.size() * s.lanes * 16 > 56 * 1024) s.lanes /= 4;
    return s;
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
    a.placed = p->placed ? 1 : 0;
    a.steps = (uint32_t)p->S;
    a.keep = 2 * (int64_t)p->n * elems * 4 <= kKeepPassBytes ? 1 : 0;
    const int64_t G = (elems + kGranule - 1) / kGranule;
    int64_t max_gc = 0;
    for (int c = 0; c <= D; ++c) a.seg_g[c] = (int64_t)c * G / D;
    for (int c = 0; c < D; ++c) {
        max_gc = std::max(max_gc, a.seg_g[c + 1] - a.seg_g[c]);
        a.f_gc[c] = make_fastdiv32((uint32_t)std::max<int64_t>(1, a.seg_g[c + 1] - a.seg_g[c]));
        a.side[c] = (uint32_t)p->dims[c];
        a.stride[c] = (uint32_t)p->strides[c];
        a.f_side[c] = make_fastdiv32((uint32_t)p->dims[c]);
        if (p->placed)
            for (int t = 0; t < p->S; ++t) a.pdim[c] |= (uint32_t)p->passes[t].dim[c] << (4 * t);
    }
    a.narrow = (int64_t)p->n * (max_gc + 1) < ((int64_t)1 << 31) ? 1 : 0;
    // programs: all in one launch, or one launch per collective
    size_t words = 0;
    for (const FoldProgram& f : p->folds) words += f.words();
    const bool together = words <= kMaxFoldWords;
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
        size_t lds;
        hipError_t err;
        if (s.waves == 1) {
            lds = (size_t)kStreamWaves * (a.sub_depth + a.top_depth) * 64 * 16;
            err = launch_fold<T, D, 1>(buf, a, (tiles + kStreamWaves - 1) / kStreamWaves, lds, x);
        } else {
            lds = (most_roots + 1 + (size_t)s.waves * a.sub_depth + a.top_depth) * s.lanes * 16;
            if (s.waves == 4) err = launch_fold<T, D, 4>(buf, a, tiles, lds, x);
            else err = launch_fold<T, D, 16>(buf, a, tiles, lds, x);
        }
        if (err != hipSuccess) return TRIVANCE_EHIP;
    }
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

bool fold_fits(const trivance_plan_t* p, int64_t elems) {
    return !p->folds.empty() && elems < ((int64_t)1 << 28);
}

int run_fold_call(float* buf, int64_t elems, const trivance_plan_t* p, hipStream_t stream) {
    return run_fold(buf, elems, p, stream);
}

int run_fold_call(int* buf, int64_t elems, const trivance_plan_t* p, hipStream_t stream) {
    return run_fold(buf, elems, p, stream);
}

}  // namespace trivance
