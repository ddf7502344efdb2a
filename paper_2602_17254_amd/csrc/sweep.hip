// Whole latency-optimal AllReduce for gfx950: each vector is read once and written once. A
// workgroup holds a tile of columns of all n rows in local memory and runs every step of the
// schedule there (sweep_plan.h), so the results are the step kernels', bit for bit.
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

// An operation in the kernel arguments: per term the byte offset of the array's slot and, for every
// two dimensions, the displacements in cells (16 bits each); then the byte offset of the result's
// slot with what follows in its low bits (slots are multiples of 16 bytes).
template <int D>
struct alignas(16) SweepOp {
    static constexpr int H = (D + 1) / 2;
    uint32_t base[3];
    uint32_t dst;
    uint32_t by[3][H];
    uint32_t pad[4 - 3 * H % 4];
    static constexpr uint32_t kWords = sweep_op_words(D);
};
constexpr uint32_t kTwoTerms = 1u;   // no third term
constexpr uint32_t kLevelEnd = 2u;   // last operation of its level
constexpr uint32_t kProgramEnd = 4u;

typedef unsigned short U16x2 __attribute__((ext_vector_type(2)));
typedef uint32_t U32x4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ U16x2 as_u16x2(uint32_t w) { return __builtin_bit_cast(U16x2, w); }

struct SweepArgs {
    int64_t elems;
    int64_t seg_g[kMaxSweepDims + 1];
    uint32_t side[kMaxSweepDims], stride[kMaxSweepDims];
    FastDiv32 f_side[kMaxSweepDims];
    uint32_t tile_end[kMaxSweepDims];  // segment c owns tiles [tile_end[c-1], tile_end[c])
    uint32_t op0[kMaxSweepDims];       // per collective: its first operation in tab
    uint32_t shift;                    // 1 << shift column vectors of a tile
    uint32_t cells;                    // n << shift
    uint32_t grid;                     // workgroups of the whole launch
    uint32_t wg_base;
    U32x4 tab[kSweepTabWords / 4];
};
static_assert(sizeof(SweepArgs) <= 4096, "sweep kernel arguments above 4 KiB");

// A thread owns CELLS (rank, column vector) cells of the tile. A level of the program has up to
// OPS operations, whose results stay in registers until every thread has read its terms. LOOP: the
// workgroup takes several tiles and reads the next one's rows while it works on one.
//
// What bounds it (MI355X). Rings of powers of three: the memory, 5.2-5.7 TB/s, where probes that
// read many rows and then write them reached 4.6-5.9 (fold.hip). Ring of 81
// at 8 MiB 263 us, of which one read and one write at a copy's rate are 201; the four step launches
// took 858. With partial sums: the vector instructions that find the terms and the barriers between
// levels (ring of 64 at 8 MiB 265 us, steps 2298; 32x32 at 256 KiB 630-665, steps 4346, one
// workgroup of 147 KiB to a compute unit). Measured on the way:
//  * addresses as products of coordinates: ring of 64 313 us, 32x32 956. With the displacements
//    scaled beforehand, two dimensions to a word and the sum in one dot instruction, a term costs four
//    instructions.
//  * an operation's words one scalar load at a time, or a whole level's read ahead: 445 and 1104.
//    One record of 32 bytes, read one operation ahead, costs two loads and no wait of its own.
//  * the next tile's rows in registers cost half the waves where more than two workgroups fit a
//    compute unit (ring of 81 353 against 263), and pay below (8x8x8 354 against 428).
//  * the stores are not streamed: tiles are narrower than a cache line on the larger tori, and the
//    line is completed by the neighbours in the L2 cache.
template <typename T, int D, int CELLS, int OPS, bool LOOP>
__global__ __launch_bounds__(1024) __attribute__((amdgpu_waves_per_eu(CELLS > 2 ? 6 : 4)))
void sweep_kernel(T* __restrict__ buf, SweepArgs a) {
    using V = Vec<T, 4>;
    constexpr int H = (D + 1) / 2;
    extern __shared__ __align__(16) char lds[];
    const int64_t E = a.elems;
    const uint32_t wv = 1u << a.shift;
    uint32_t rank[CELLS], vec[CELLS], z[CELLS][D];
    bool mine[CELLS];
#pragma unroll
    for (int k = 0; k < CELLS; ++k) {
        const uint32_t i = threadIdx.x + k * blockDim.x;
        mine[k] = i < a.cells;
        uint32_t r = (mine[k] ? i : 0u) >> a.shift;
        rank[k] = r;
        vec[k] = i & (wv - 1);
#pragma unroll
        for (int d = 0; d < D; ++d) {
            const uint32_t q = d + 1 < D ? fdiv32(r, a.f_side[d]) : 0u;
            z[k][d] = r - q * a.side[d];
            r = q;
        }
    }
    auto collective = [&](uint32_t tile) {
        int c = 0;
#pragma unroll
        for (int i = 0; i < D - 1; ++i)
            if (tile >= a.tile_end[i]) c = i + 1;
        return c;
    };
    // the tile's first column, and the columns from there to the segment's end
    auto columns = [&](uint32_t tile, int64_t* left) {
        const int c = collective(tile);
        const int64_t col = a.seg_g[c] * kGranule +
                            ((int64_t)(tile - (c ? a.tile_end[c - 1] : 0u)) << a.shift) * 4;
        *left = imin64(a.seg_g[c + 1] * kGranule, E) - col;
        return col;
    };
    const uint32_t tiles = a.tile_end[D - 1];
    V x[CELLS];
    auto fetch = [&](uint32_t tile) {
        int64_t left;
        const T* const base = buf + columns(tile, &left);
#pragma unroll
        for (int k = 0; k < CELLS; ++k) {
            const T* const q = base + (int64_t)rank[k] * E + vec[k] * 4;
            const int64_t l = mine[k] ? left - (int64_t)vec[k] * 4 : 0;
            if (l >= 4) {
                x[k] = ld_any<T, 4, true>(q);
            } else {
#pragma unroll
                for (int i = 0; i < 4; ++i) x[k].v[i] = i < l ? q[i] : (T)0;
            }
        }
    };
    uint32_t tile = xcd_contiguous(a.wg_base + blockIdx.x, a.grid);
    if (tile < tiles) fetch(tile);
    if (!LOOP && tile >= tiles) return;
    do {
        if (LOOP && tile >= tiles) break;
        const int c = collective(tile);
        // a cell's place along every dimension in cells, in the order of dimensions c, c + 1, ...
        // (cyclic), as in the program; two dimensions to a word
        uint32_t u[CELLS][H], span[H] = {};
#pragma unroll
        for (int k = 0; k < CELLS; ++k)
#pragma unroll
            for (int h = 0; h < H; ++h) u[k][h] = 0;
#pragma unroll
        for (int f = 0; f < D; ++f) {
            const uint32_t d = c + f < D ? c + f : c + f - D;
            const uint32_t step = a.stride[d] << a.shift;
            span[f / 2] |= (a.side[d] * step) << (16 * (f % 2));
#pragma unroll
            for (int k = 0; k < CELLS; ++k) {
                uint32_t y = z[k][0];
#pragma unroll
                for (int q = 1; q < D; ++q)
                    if ((uint32_t)q == d) y = z[k][q];
                u[k][f / 2] |= (y * step + (f ? 0u : vec[k])) << (16 * (f % 2));
            }
        }
        if (LOOP) __syncthreads();  // the previous tile has left local memory
#pragma unroll
        for (int k = 0; k < CELLS; ++k)
            if (mine[k])
                st<T, 4>(reinterpret_cast<T*>(lds + (threadIdx.x + k * blockDim.x) * 16), x[k]);
        if (LOOP && tile + a.grid < tiles) fetch(tile + a.grid);
        __syncthreads();

        auto get = [&](const SweepOp<D>& w, int q, int k) {
            uint32_t at = w.base[q];
#pragma unroll
            for (int h = 0; h < H; ++h) {
                // (place + displacement) mod span in both halves: the difference wraps around
                // when there is nothing to subtract
                const U16x2 s = as_u16x2(u[k][h]) + as_u16x2(w.by[q][h]);
                const U16x2 y = __builtin_elementwise_min(s, (U16x2)(s - as_u16x2(span[h])));
                at = __builtin_amdgcn_udot2(y, U16x2{16, 16}, at, false);
            }
            return ld<T, 4>(reinterpret_cast<const T*>(lds + at));
        };
        V out[CELLS][OPS];
        uint32_t dst[OPS];
        // operations are read one ahead: scalar and local memory share a counter, so one that is
        // waited for on its own would cost its latency
        uint32_t at_op = a.op0[c];
        auto read_op = [&]() {
            struct {
                U32x4 v[SweepOp<D>::kWords / 4];
            } w;
#pragma unroll
            for (uint32_t i = 0; i < SweepOp<D>::kWords / 4; ++i) w.v[i] = a.tab[at_op + i];
            at_op += SweepOp<D>::kWords / 4;
            return __builtin_bit_cast(SweepOp<D>, w);
        };
        SweepOp<D> next = read_op();
        for (;;) {
            bool open = true;
            uint32_t last = 0;
#pragma unroll
            for (int o = 0; o < OPS; ++o) {
                if (open) {
                    const SweepOp<D> w = next;
                    next = read_op();  // there is one more than the program has
                    last = w.dst;
                    dst[o] = w.dst & ~15u;
                    open = !(w.dst & kLevelEnd);
                    if (w.dst & kTwoTerms) {
#pragma unroll
                        for (int k = 0; k < CELLS; ++k) out[k][o] = vadd(get(w, 0, k), get(w, 1, k));
                    } else {
#pragma unroll
                        for (int k = 0; k < CELLS; ++k)
                            out[k][o] = joint(get(w, 0, k), get(w, 1, k), get(w, 2, k));
                    }
                } else {
                    dst[o] = ~0u;
                }
            }
            if (last & kProgramEnd) break;
            __syncthreads();
#pragma unroll
            for (int o = 0; o < OPS; ++o) {
                if (dst[o] != ~0u) {
#pragma unroll
                    for (int k = 0; k < CELLS; ++k)
                        if (mine[k])
                            st<T, 4>(reinterpret_cast<T*>(lds + dst[o] +
                                                          (threadIdx.x + k * blockDim.x) * 16),
                                     out[k][o]);
                }
            }
            __syncthreads();
        }
        int64_t left;
        T* const base = buf + columns(tile, &left);
#pragma unroll
        for (int k = 0; k < CELLS; ++k) {
            T* const q = base + (int64_t)rank[k] * E + vec[k] * 4;
            const int64_t l = mine[k] ? left - (int64_t)vec[k] * 4 : 0;
            if (l >= 4) {
                typedef T U __attribute__((ext_vector_type(4), aligned(4)));
                U s;
#pragma unroll
                for (int i = 0; i < 4; ++i) s[i] = out[k][0].v[i];
                *reinterpret_cast<U*>(q) = s;
            } else {
#pragma unroll
                for (int i = 0; i < 3; ++i)
                    if (i < l) q[i] = out[k][0].v[i];
            }
        }
        tile += a.grid;
    } while (LOOP);
}

template <typename T, int D, int CELLS, int OPS, bool LOOP>
hipError_t launch_sweep(T* buf, SweepArgs a, const SweepShape& s, const Exec& x) {
    hipError_t err = hipSuccess;
    for_each_dispatch(a.grid, s.threads, x.items, [&](uint32_t first, uint32_t count) {
        a.wg_base = first;
        hipLaunchKernelGGL((sweep_kernel<T, D, CELLS, OPS, LOOP>), dim3(count), dim3(s.threads),
                           s.lds, x.stream, buf, a);
        err = hipGetLastError();
        return err == hipSuccess;
    });
    return err;
}

template <typename T, int D>
int run_sweep_dims(T* buf, int64_t elems, const trivance_plan_t* p, hipStream_t stream) {
    const Exec x{stream, p->dispatch_items};
    SweepShape s;
    if (!sweep_shape(p, elems, &s)) return TRIVANCE_EUNSUPPORTED;
    SweepArgs a;
    std::memset(&a, 0, sizeof(a));
    a.elems = elems;
    a.shift = s.shift;
    a.cells = (uint32_t)p->n << s.shift;
    const uint32_t slot_bytes = a.cells * 16;
    const int64_t G = (elems + kGranule - 1) / kGranule;
    uint32_t used = 0, tiles = 0;
    for (int c = 0; c < D; ++c) {
        a.side[c] = (uint32_t)p->dims[c];
        a.stride[c] = (uint32_t)p->strides[c];
        a.f_side[c] = make_fastdiv32((uint32_t)p->dims[c]);
    }
    for (int c = 0; c <= D; ++c) a.seg_g[c] = (int64_t)c * G / D;
    constexpr int kBits = kSweepCoordBits / D;
    static_assert(sizeof(SweepOp<D>) == 4 * SweepOp<D>::kWords, "an operation without gaps");
    SweepOp<D>* const tab = reinterpret_cast<SweepOp<D>*>(a.tab);
    for (int c = 0; c < D; ++c) {
        const SweepProgram& g = p->sweeps[p->sweeps.size() == 1 ? 0 : c];
        a.op0[c] = used * (SweepOp<D>::kWords / 4);
        size_t level = 1;
        for (size_t o = 0; o < g.words.size() / 4; ++o) {
            SweepOp<D>& op = tab[used++];
            const uint32_t* const w = &g.words[4 * o];
            for (int q = 0; q < 3; ++q) {
                if (w[q] == kSweepNone) continue;
                op.base[q] = (w[q] >> kSweepCoordBits) * slot_bytes;
                for (int f = 0; f < D; ++f)
                    op.by[q][f / 2] |= (((w[q] >> (f * kBits)) & ((1u << kBits) - 1u)) *
                                        (a.stride[(c + f) % D] << s.shift)) << (16 * (f % 2));
            }
            op.dst = w[3] * slot_bytes;
            if (w[2] == kSweepNone) op.dst |= kTwoTerms;
            if (o + 1 == g.level_begin[level]) {
                op.dst |= kLevelEnd;
                if (++level == g.level_begin.size()) op.dst |= kProgramEnd;
            }
        }
        const int64_t len = std::min(a.seg_g[c + 1] * kGranule, elems) - a.seg_g[c] * kGranule;
        tiles += (uint32_t)(((len + 3) / 4 + ((int64_t)1 << s.shift) - 1) >> s.shift);
        a.tile_end[c] = tiles;
    }
    a.grid = sweep_grid(s, tiles);
    hipError_t err = hipErrorInvalidValue;
    const bool loop = a.grid < tiles;
    if (s.ops == 1) {
        switch (s.cells) {
            case 2: err = launch_sweep<T, D, 2, 1, false>(buf, a, s, x); break;
            case 4: err = launch_sweep<T, D, 4, 1, false>(buf, a, s, x); break;
        }
    } else if (s.ops == 4) {
        if (s.cells == 2) err = launch_sweep<T, D, 2, 4, false>(buf, a, s, x);
        else if (loop) err = launch_sweep<T, D, 1, 4, true>(buf, a, s, x);
        else err = launch_sweep<T, D, 1, 4, false>(buf, a, s, x);
    } else {
        if (loop) err = launch_sweep<T, D, 1, 12, true>(buf, a, s, x);
        else err = launch_sweep<T, D, 1, 12, false>(buf, a, s, x);
    }
    return err == hipSuccess ? TRIVANCE_OK : TRIVANCE_EHIP;
}

template <typename T>
int run_sweep(T* buf, int64_t elems, const trivance_plan_t* p, hipStream_t stream) {
    switch (p->D) {
        case 1: return run_sweep_dims<T, 1>(buf, elems, p, stream);
        case 2: return run_sweep_dims<T, 2>(buf, elems, p, stream);
        case 3: return run_sweep_dims<T, 3>(buf, elems, p, stream);
        default: return run_sweep_dims<T, 4>(buf, elems, p, stream);
    }
}

}  // namespace

int run_sweep_call(float* buf, int64_t elems, const trivance_plan_t* p, hipStream_t stream) {
    return run_sweep(buf, elems, p, stream);
}

int run_sweep_call(int* buf, int64_t elems, const trivance_plan_t* p, hipStream_t stream) {
    return run_sweep(buf, elems, p, stream);
}

}  // namespace trivance
