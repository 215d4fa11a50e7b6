// Which rows a chain's steps visit, and where a chain starts.
#pragma once
#include "device_utils.h"
#include "internal.h"

namespace wpsgd {

constexpr int kWindowParts = 4;

// Rows of a chain's steps, 64 at a time: window(w) for w = 0, 1, 2, .. in turn; past the chain's end the row of its last
// step once more (such a step adds 0 times its row, which must be a row the chain has visited: 0 times a NaN is one).
struct StepRows {
    uint32_t chain, seed_lo, seed_hi, m;
    int64_t step0, n, left;
    const uint32_t *perm;
    uint32_t lo, len, inc, pos, last;
    __device__ void init(const ChainArgs &a, int cb, int lane)
    {
        chain = (uint32_t)a.order[cb];
        seed_lo = a.seed_lo;
        seed_hi = a.seed_hi;
        m = (uint32_t)a.m;
        step0 = first_step(a, cb);
        n = a.nsteps[cb];
        left = n - lane;
        perm = a.perm;
        lo = inc = pos = last = 0;
        len = 1;
        if (perm) {
            lo = a.shard[cb];
            len = a.shard[a.k + cb];
            const uint32_t pos0 = (uint32_t)((uint64_t)step0 % len), room = len - pos0;
            inc = (uint32_t)kWave % len;
            last = (uint32_t)((uint64_t)(step0 + n - 1) % len);
            pos = (uint32_t)lane < room ? pos0 + (uint32_t)lane : ((uint32_t)lane - room) % len;
        }
    }
    // the same in kWindowParts parts, u = 0, 1, ..: the generator's ten rounds are long multiplications
    uint32_t c0, c1, c2, c3, k0, k1;
    __device__ uint32_t window_part(int u, int64_t w, int lane)
    {
        if (perm) return u == kWindowParts - 1 ? window(w, lane) : 0u;
        if (u == 0) {
            const uint64_t step = (uint64_t)(step0 + w * kWave + lane + (left > 0 ? 0 : left - 1));
            left -= kWave;
            c0 = (uint32_t)step;
            c1 = (uint32_t)(step >> 32);
            c2 = chain;
            c3 = 0u;
            k0 = seed_lo;
            k1 = seed_hi;
        }
        philox4x32_rounds(c0, c1, c2, c3, k0, k1, u < 2 ? 3 : 2);
        return mul_hi_u32(c0, m);
    }
    __device__ uint32_t window(int64_t w, int lane)
    {
        const int64_t behind = left > 0 ? 0 : left - 1;              // from the lane's step back to the chain's last
        left -= kWave;
        if (perm) {
            const uint32_t r = perm[(uint64_t)lo + (behind == 0 ? pos : last)];
            const uint32_t t = pos + inc;                 // may wrap past 2^32: then it is past the share too
            pos = (t < pos || t >= len) ? t - len : t;
            return r;
        }
        return sample_row(seed_lo, seed_hi, chain, (uint64_t)(step0 + w * kWave + lane + behind), m);
    }
    // the row of one step
    __device__ uint32_t at(int64_t t) const
    {
        if (perm) {
            uint32_t r = perm[(uint64_t)lo + (uint64_t)(step0 + t) % len];
            asm volatile("" : "+v"(r));                   // waits here: the caller's rows on their way are not waited for on the other path
            return r;
        }
        return sample_row(seed_lo, seed_hi, chain, (uint64_t)(step0 + t), m);
    }
};

// Where a chain starts: from a vector, from zero, or from the weighted sum of the models of the span before (periodic averaging),
// which every chain forms for itself, in the order and precision of combine_kernel: the same bits, without its launch between two
// spans.  What it costs is a trip to memory per kStartModels rows, whose loads are all on their way at once: none is conditional
// (with eight rows and a branch per row 16 chains, d = 64, hinge took 17.9 us a span, so 15.1).  The rule is in api.hip.
constexpr int kStartModels = 16;
template <typename TV, int N, typename F>
__device__ inline void start_values(const ChainArgs &a, TV (&v)[N], F &&column)
{
    if (!a.models) {
#pragma unroll
        for (int e = 0; e < N; ++e) v[e] = (a.w_start && column(e) < a.d) ? (TV)a.w_start[column(e)] : (TV)0;
        return;
    }
    double acc[N];
    int64_t at[N];
#pragma unroll
    for (int e = 0; e < N; ++e) {
        acc[e] = 0.0;
        at[e] = column(e) < a.d ? column(e) : 0;
    }
    // (quadruples of columns are consecutive: every caller's columns are)
    const bool quads = N % 4 == 0 && a.d % 4 == 0;
    for (int i = 0; i < a.k; i += kStartModels) {
        float x[kStartModels][N];
        double w[kStartModels];
#pragma unroll
        for (int u = 0; u < kStartModels; ++u) {
            const int r = i + u < a.k ? i + u : a.k - 1;
            w[u] = a.model_weights[r];
            const float *row = a.models + (int64_t)r * a.d;
            if (quads) {
#pragma unroll
                for (int e = 0; e + 3 < N; e += 4) {
                    const float4 q = *reinterpret_cast<const float4 *>(row + at[e]);
                    x[u][e] = q.x; x[u][e + 1] = q.y; x[u][e + 2] = q.z; x[u][e + 3] = q.w;
                }
            } else {
#pragma unroll
                for (int e = 0; e < N; ++e) x[u][e] = row[at[e]];
            }
        }
#pragma unroll
        for (int u = 0; u < kStartModels; ++u)
#pragma unroll
            for (int e = 0; e < N; ++e) {
                const double t = fma(w[u], (double)x[u][e], acc[e]);
                acc[e] = i + u < a.k ? t : acc[e];
            }
    }
#pragma unroll
    for (int e = 0; e < N; ++e) v[e] = column(e) < a.d ? (TV)(float)acc[e] : (TV)0;
}
__device__ inline float start_value(const ChainArgs &a, int column)
{
    float v[1];
    start_values(a, v, [&](int) { return column; });
    return v[0];
}

}  // namespace wpsgd
