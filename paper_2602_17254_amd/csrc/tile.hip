// Small bandwidth-optimal AllReduces for gfx950: the whole call in one launch, a workgroup holding a
// tile of columns of all n rows in local memory. The adds are the reduce-scatter steps' own, so the
// results are theirs, bit for bit. Latency bounds it: one round trip to memory for all rows of the
// tile, one barrier per step, one store.
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

struct TileArgs {
    int64_t elems;
    int64_t seg_g[kMaxFoldDims + 1];
    uint32_t n;
    uint32_t side[kMaxFoldDims], stride[kMaxFoldDims];
    FastDiv32 f_side[kMaxFoldDims];
    FastDiv32 f_gc[kMaxFoldDims];        // granules of segment c
    uint32_t tile_end[kMaxFoldDims];     // segment c owns tiles [tile_end[c-1], tile_end[c])
    uint32_t mask0[kMaxFoldDims][kMaxFoldDims];  // first entry of (collective, dimension) in tab
    uint32_t steps;
    uint32_t step[kMaxFoldDims][kMaxTileSteps];  // dimension in the low 2 bits, distance above
    int placed;
    uint32_t shift;                      // 1 << shift column vectors of a tile
    uint32_t cells;                      // n << shift
    uint32_t wg_base;
    uint32_t tab[kMaxTileWords];
};
static_assert(sizeof(TileArgs) <= 4096, "tile kernel arguments above 4 KiB");
static_assert(2 * kMaxTileSteps == kTileForwardShift, "two bits a step below the forwarding step");

// A thread owns CELLS (rank, column vector) cells. A rank's part in the tree of its column's block
// depends on its offset from the block's owner: one word per dimension (tile_masks) holds the
// steps in which it receives, and from which sides, and the step in which it forwards. In one step
// a rank that receives is read by nobody and a rank that is read does not receive, so a step needs
// one barrier.
template <typename T, int D, int CELLS>
__global__ __launch_bounds__(1024) void tile_kernel(T* __restrict__ buf, TileArgs a) {
    using V = Vec<T, 4>;
    extern __shared__ __align__(16) char lds[];
    const uint32_t tile = a.wg_base + xcd_contiguous(blockIdx.x, gridDim.x);
    int c = 0;
#pragma unroll
    for (int i = 0; i < D - 1; ++i)
        if (tile >= a.tile_end[i]) c = i + 1;
    const int64_t E = a.elems;
    const int64_t seg_b = a.seg_g[c] * kGranule;
    const int64_t col0 = seg_b + ((int64_t)(tile - (c ? a.tile_end[c - 1] : 0u)) << a.shift) * 4;
    const int64_t left = imin64(a.seg_g[c + 1] * kGranule, E) - col0;
    const uint32_t wv = 1u << a.shift;

    V cur[CELLS];
    uint32_t z[CELLS][D], owner[CELLS], mask[CELLS], rank[CELLS], vec[CELLS];
    bool mine[CELLS];
#pragma unroll
    for (int k = 0; k < CELLS; ++k) {
        const uint32_t i = threadIdx.x + k * blockDim.x;
        mine[k] = i < a.cells;
        rank[k] = (mine[k] ? i : 0u) >> a.shift;
        vec[k] = i & (wv - 1);
        const T* const q = buf + (int64_t)rank[k] * E + col0 + vec[k] * 4;
        const int64_t l = mine[k] ? left - (int64_t)vec[k] * 4 : 0;
        if (l >= 4) {
            cur[k] = ld_any<T, 4, true>(q);
        } else {
#pragma unroll
            for (int i2 = 0; i2 < 4; ++i2) cur[k].v[i2] = i2 < l ? q[i2] : (T)0;
        }
    }
#pragma unroll
    for (int k = 0; k < CELLS; ++k) {
        // the block of the cell's columns (columns past the segment's end take its last block)
        const int64_t in = imin64(col0 - seg_b + vec[k] * 4, col0 - seg_b + left - 1);
        const uint32_t gr = (uint32_t)(in / kGranule);
        uint32_t j = fdiv32((gr + 1) * a.n - 1, a.f_gc[c]);
        uint32_t y[D] = {};
        if (a.placed) {
            // j is the block's position: its base-3 digits, the last step's lowest
            for (int t = (int)a.steps - 1; t >= 0; --t) {
                const uint32_t j3 = __umulhi(j, 0xAAAAAAABu) >> 1;
                const uint32_t dim = a.step[c][t] & 3u;
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
        // the cell's coordinates, here and not before the row loads (0.1 us of 7.6 on 9x9x9 ranks of
        // 1000 values)
        uint32_t r = rank[k];
#pragma unroll
        for (int d = 0; d < D; ++d) {
            const uint32_t q = d + 1 < D ? fdiv32(r, a.f_side[d]) : 0u;
            z[k][d] = r - q * a.side[d];
            r = q;
        }
        uint32_t own = 0, bits = 0, until = 31;
#pragma unroll
        for (int d = 0; d < D; ++d) {
            const uint32_t o = z[k][d] >= y[d] ? z[k][d] - y[d] : z[k][d] + a.side[d] - y[d];
            const uint32_t w = a.tab[a.mask0[c][d] + o];
            bits |= w;
            until = min(until, w >> kTileForwardShift);
            own += y[d] * a.stride[d];
        }
        owner[k] = own;
        if (until > (uint32_t)kMaxTileSteps) until = kMaxTileSteps;
        mask[k] = mine[k] ? bits & ((1u << (2 * until)) - 1u) : 0u;
    }
#pragma unroll
    for (int k = 0; k < CELLS; ++k)
        if (mine[k]) st<T, 4>(reinterpret_cast<T*>(lds + (threadIdx.x + k * blockDim.x) * 16), cur[k]);
    __syncthreads();
    for (uint32_t t = 0; t < a.steps; ++t) {
        const uint32_t dim = a.step[c][t] & 3u, dist = a.step[c][t] >> 2;
        const uint32_t span = a.side[dim] * (a.stride[dim] << a.shift);
        const uint32_t by = dist * (a.stride[dim] << a.shift);
#pragma unroll
        for (int k = 0; k < CELLS; ++k) {
            const uint32_t f = (mask[k] >> (2 * t)) & 3u;
            if (f) {
                const uint32_t i = threadIdx.x + k * blockDim.x;
                uint32_t x = z[k][0];
#pragma unroll
                for (int d = 1; d < D; ++d)
                    if ((uint32_t)d == dim) x = z[k][d];
                if (f & 1u)
                    cur[k] = vadd(cur[k], ld<T, 4>(reinterpret_cast<const T*>(
                                              lds + (i - by + (x < dist ? span : 0u)) * 16)));
                if (f & 2u)
                    cur[k] = vadd(cur[k], ld<T, 4>(reinterpret_cast<const T*>(
                                              lds + (i + by - (x + dist >= a.side[dim] ? span : 0u)) * 16)));
                st<T, 4>(reinterpret_cast<T*>(lds + i * 16), cur[k]);
            }
        }
        __syncthreads();
    }
#pragma unroll
    for (int k = 0; k < CELLS; ++k) {
        T* const q = buf + (int64_t)rank[k] * E + col0 + vec[k] * 4;
        const int64_t l = mine[k] ? left - (int64_t)vec[k] * 4 : 0;
        const V res = ld<T, 4>(reinterpret_cast<const T*>(lds + ((owner[k] << a.shift) + vec[k]) * 16));
        if (l >= 4) {
            typedef T U __attribute__((ext_vector_type(4), aligned(4)));
            U s;
#pragma unroll
            for (int i = 0; i < 4; ++i) s[i] = res.v[i];
            *reinterpret_cast<U*>(q) = s;
        } else {
#pragma unroll
            for (int i = 0; i < 3; ++i)
                if (i < l) q[i] = res.v[i];
        }
    }
}

template <typename T, int D, int CELLS>
hipError_t launch_tile(T* buf, TileArgs a, uint32_t grid, int threads, const Exec& x) {
    hipError_t err = hipSuccess;
    for_each_dispatch(grid, threads, x.items, [&](uint32_t first, uint32_t count) {
        a.wg_base = first;
        hipLaunchKernelGGL((tile_kernel<T, D, CELLS>), dim3(count), dim3(threads),
                           (size_t)a.cells * 16, x.stream, buf, a);
        err = hipGetLastError();
        return err == hipSuccess;
    });
    return err;
}

template <typename T, int D>
int run_tile_dims(T* buf, int64_t elems, const trivance_plan_t* p, hipStream_t stream) {
    const Exec x{stream, p->dispatch_items};
    TileShape s;
    if (!tile_shape(p, elems, &s)) return TRIVANCE_EUNSUPPORTED;
    TileArgs a;
    std::memset(&a, 0, sizeof(a));
    a.elems = elems;
    a.n = (uint32_t)p->n;
    a.placed = p->placed ? 1 : 0;
    a.steps = (uint32_t)p->S;
    a.shift = s.shift;
    a.cells = (uint32_t)p->n << s.shift;
    const int64_t G = (elems + kGranule - 1) / kGranule;
    for (int c = 0; c <= D; ++c) a.seg_g[c] = (int64_t)c * G / D;
    uint32_t tiles = 0;
    for (int c = 0; c < D; ++c) {
        const int64_t gc = a.seg_g[c + 1] - a.seg_g[c];
        a.f_gc[c] = make_fastdiv32((uint32_t)std::max<int64_t>(1, gc));
        a.side[c] = (uint32_t)p->dims[c];
        a.stride[c] = (uint32_t)p->strides[c];
        a.f_side[c] = make_fastdiv32((uint32_t)p->dims[c]);
        for (int d = 0; d < D; ++d) a.mask0[c][d] = p->tile_mask0[c * D + d];
        for (int t = 0; t < p->S; ++t)
            a.step[c][t] = (uint32_t)p->passes[t].dim[c] | (uint32_t)p->passes[t].distance[c] << 2;
        const int64_t len = std::min(a.seg_g[c + 1] * kGranule, elems) - a.seg_g[c] * kGranule;
        tiles += (uint32_t)(((len + 3) / 4 + ((int64_t)1 << s.shift) - 1) >> s.shift);
        a.tile_end[c] = tiles;
    }
    std::copy(p->tile_masks.begin(), p->tile_masks.end(), a.tab);
    hipError_t err;
    switch (s.cells) {
        case 1: err = launch_tile<T, D, 1>(buf, a, tiles, s.threads, x); break;
        case 2: err = launch_tile<T, D, 2>(buf, a, tiles, s.threads, x); break;
        case 4: err = launch_tile<T, D, 4>(buf, a, tiles, s.threads, x); break;
        default: err = launch_tile<T, D, 8>(buf, a, tiles, s.threads, x); break;
    }
    return err == hipSuccess ? TRIVANCE_OK : TRIVANCE_EHIP;
}

template <typename T>
int run_tile(T* buf, int64_t elems, const trivance_plan_t* p, hipStream_t stream) {
    switch (p->D) {
        case 1: return run_tile_dims<T, 1>(buf, elems, p, stream);
        case 2: return run_tile_dims<T, 2>(buf, elems, p, stream);
        case 3: return run_tile_dims<T, 3>(buf, elems, p, stream);
        default: return run_tile_dims<T, 4>(buf, elems, p, stream);
    }
}

}  // namespace

int run_tile_call(float* buf, int64_t elems, const trivance_plan_t* p, hipStream_t stream) {
    return run_tile(buf, elems, p, stream);
}

int run_tile_call(int* buf, int64_t elems, const trivance_plan_t* p, hipStream_t stream) {
    return run_tile(buf, elems, p, stream);
}

}  // namespace trivance
