// Column programs (sweep_plan.h) against the schedule they replace, on the host: run as the sweep
// kernel runs them, on slots of n values, they must give the bits of the latency-optimal steps
// run one after another on floats whose sums depend on the association. Built with g++ against
// plan.cpp; no GPU. Exit status 0 on success.
//   sweep_program SIDES...    (a ring "9", a torus "5x7")
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <vector>

#include "plan.h"

using trivance::kMaxDims;
typedef std::vector<float> Vec;

static int shifted(const trivance_plan_t* p, int r, int d, int by) {
    const int x = r / p->strides[d] % p->dims[d];
    return r + ((x + by + p->dims[d]) % p->dims[d] - x) * p->strides[d];
}

static Vec by_steps(const trivance_plan_t* p, int c, const Vec& x) {
    std::vector<Vec> state{x};
    for (int t = 0; t < p->S; ++t) {
        const trivance::Pass& ps = p->passes[t];
        const int nout = p->slots.empty() ? 1 : p->slots[t].nout[c];
        std::vector<Vec> next(nout, Vec(p->n));
        for (int i = 0; i < nout; ++i) {
            const int own = p->slots.empty() ? 0 : p->slots[t].own[c][i];
            const int left = p->slots.empty() ? 0 : p->slots[t].left[c][i];
            const int right = p->slots.empty() ? 0 : p->slots[t].right[c][i];
            for (int r = 0; r < p->n; ++r) {
                const int l = shifted(p, r, ps.dim[c], -ps.distance[c]);
                const int q = shifted(p, r, ps.dim[c], ps.distance[c]);
                float v = 0;
                bool any = false;
                if (own >= 0) v = state[own][r], any = true;
                if (left >= 0) v = any ? v + state[left][l] : state[left][l], any = true;
                if (right >= 0) v = any ? v + state[right][q] : state[right][q];
                next[i][r] = v;
            }
        }
        state.swap(next);
    }
    return state[0];
}

static Vec by_program(const trivance_plan_t* p, int c, const Vec& x) {
    const trivance::SweepProgram& g = p->sweeps[p->sweeps.size() == 1 ? 0 : c];
    const int bits = trivance::kSweepCoordBits / p->D;
    std::vector<Vec> lds(g.slots, Vec(p->n, NAN));
    lds[0] = x;
    for (int t = 0; t < p->S; ++t) {
        std::vector<Vec> out;
        for (uint32_t o = g.level_begin[t]; o < g.level_begin[t + 1]; ++o) {
            const uint32_t* w = &g.words[4 * o];
            Vec v(p->n);
            for (int r = 0; r < p->n; ++r)
                for (int q = 0; q < 3; ++q) {
                    if (w[q] == trivance::kSweepNone) continue;
                    int from = r;
                    for (int f = 0; f < p->D; ++f)
                        from = shifted(p, from, (c + f) % p->D, (int)((w[q] >> (f * bits)) & ((1u << bits) - 1u)));
                    const float s = lds.at(w[q] >> trivance::kSweepCoordBits)[from];
                    v[r] = q ? v[r] + s : s;
                }
            out.push_back(v);
        }
        if (t + 1 == p->S) return out.size() == 1 ? out[0] : Vec();
        for (uint32_t o = g.level_begin[t]; o < g.level_begin[t + 1]; ++o)
            lds.at(g.words[4 * o + 3]) = out[o - g.level_begin[t]];
    }
    return Vec();
}

int main(int argc, char** argv) {
    int failures = 0;
    uint32_t seed = 12345;
    for (int i = 1; i < argc; ++i) {
        int dims[kMaxDims] = {}, D = 0, n = 1;
        for (const char* s = argv[i]; *s;) {
            char* end;
            dims[D++] = (int)std::strtol(s, &end, 10);
            n *= dims[D - 1];
            s = *end ? end + 1 : end;
        }
        trivance_plan_t* p = nullptr;
        if (trivance_plan(n, dims, D, TRIVANCE_LATENCY_OPT, &p) != TRIVANCE_OK) return 1;
        bool ok = !p->sweeps.empty();
        for (int c = 0; c < D && ok; ++c) {
            Vec x(n);
            for (float& v : x) {
                seed = seed * 1664525u + 1013904223u;
                v = (float)(int32_t)seed / 1e6f * ((seed & 7u) ? 1.0f : 1e-3f);
            }
            const Vec want = by_steps(p, c, x), got = by_program(p, c, x);
            ok = got.size() == want.size() && std::memcmp(&got[0], &want[0], n * sizeof(float)) == 0;
        }
        if (!ok) std::printf("%s differs\n", argv[i]), ++failures;
        trivance_plan_destroy(p);
    }
    std::printf("%d failures\n", failures);
    return failures != 0;
}
