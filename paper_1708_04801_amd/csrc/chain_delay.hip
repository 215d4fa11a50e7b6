// Delay SGD under the Check function (Section IV, Algorithms 3 and 4; Lemma 4): one workgroup is one
// server, or one of several that share its samples.  It keeps the accepted iterates w_{J-reach} .. w_J (reach = max(tau, 1)) and room for one
// candidate as a ring of fp64 vectors in the workspace.  Every thread owns the same columns of every
// vector in every pass, so the ring needs no synchronisation of its own; it is re-read every sample
// and stays in the cache of the compute unit's XCD.
//
// Per sample x (one row of the data set), one pass over the row forms beta^2 = x.x and the projections
// L_t = w_t.x of the iterates the delayed gradient spans.  From those scalars alone every thread takes
// the same decision: the slope u at w_{J-tau}, the triples of the first call of Check, and the triple
// (w_{J-1}, w_J, candidate) of the second call, whose third projection follows from the update rule,
//     L_c = L_J - eta*lambda*L_{J-tau} - eta*u*beta^2,
// so a sample that is thrown away costs no second pass.  Only an accepted candidate is written:
//     w_{J+1} = w_J - eta*lambda*w_{J-tau} - eta*u*x          (the recurrence in the proof of Lemma 4)
// together with its squared length, which later tests need for the part across a sample,
// |w|^2 - L^2/beta^2.  All arithmetic is fp64; the result is rounded to fp32 once, at the end.
//
// Four kernels.  delay_server_reg_kernel holds the ring in registers, newest iterate first, and shifts
// it when a candidate is accepted; the rows of the next samples (which do not depend on what is
// accepted) are requested PF samples ahead, so a sample costs the pass over its row, one exchange of
// sums and the decision.  It covers rows of up to 256 x EPT elements (bfloat16 ones that are not aligned by a load
// per element) and delays up to 4.  For the same delays and rows of whole 16-byte pieces,
// delay_server_batch_kernel decides B samples per exchange under the Check function, where nearly every sample is
// thrown away, with several workgroups per server while compute units are idle, and delay_server_plain_kernel takes
// tau + 1 samples per exchange without it, where the delay makes their gradients independent; both stage rows in LDS.
// delay_server_kernel keeps the ring in the workspace and covers longer rows and delays.
#include <hip/hip_ext.h>

#include <atomic>
#include <mutex>

#include "dense_rows.h"
#include "device_utils.h"
#include "internal.h"

namespace wpsgd {
namespace {

constexpr int kDelayThreads = 256;
constexpr int kDelayWaves = kDelayThreads / kWave;

template <typename TX, int VEC> struct DelayRow;
template <> struct DelayRow<float, 1> {
    double x[1];
    __device__ void load(const float *p) { x[0] = (double)p[0]; }
};
template <> struct DelayRow<float, 4> {
    double x[4];
    __device__ void load(const float *p)
    {
        const float4 q = *reinterpret_cast<const float4 *>(p);
        x[0] = (double)q.x; x[1] = (double)q.y; x[2] = (double)q.z; x[3] = (double)q.w;
    }
};
template <> struct DelayRow<uint16_t, 1> {
    double x[1];
    __device__ void load(const uint16_t *p) { x[0] = (double)bf16_one(p[0]); }
};
template <> struct DelayRow<uint16_t, 8> {
    double x[8];
    __device__ void load(const uint16_t *p)
    {
        const uint4 q = *reinterpret_cast<const uint4 *>(p);
        x[0] = (double)bf16_lo(q.x); x[1] = (double)bf16_hi(q.x); x[2] = (double)bf16_lo(q.y); x[3] = (double)bf16_hi(q.y);
        x[4] = (double)bf16_lo(q.z); x[5] = (double)bf16_hi(q.z); x[6] = (double)bf16_lo(q.w); x[7] = (double)bf16_hi(q.w);
    }
};

// A wave's COUNT sums into LDS, out[t * STEP] for value t: one by one from lane 63, or four to a register, each
// written by the first lane of the row of lanes it ends up in.
template <int COUNT, int STEP, int N>
__device__ inline void wave_sums_to_lds(const double (&v)[N], double *out, int lane)
{
    if constexpr (COUNT == 1) {
        const double t = wave_sum_lane63(v[0]);
        if (lane == kWave - 1) out[0] = t;
    } else {
        double w[COUNT], t[(COUNT + 3) / 4];
#pragma unroll
        for (int i = 0; i < COUNT; ++i) w[i] = v[i];
        wave_sums_merged(w, t);
        const int r = merged_row(lane / 16);
        if (lane % 16 == 0) {
#pragma unroll
            for (int q = 0; q < (COUNT + 3) / 4; ++q)
                if (4 * q + r < COUNT) out[(4 * q + r) * STEP] = t[q];
        }
    }
}

// One triple of Algorithm 4: the newest projection must lie between the middle one and
// Length_min = (L_b - rate*L_a)/(1 - rate), ends included, and the part of the middle iterate across
// the sample (squared length pb) must not be longer than that of the oldest (pa).
__device__ inline bool check_triple(double La, double Lb, double Lc, double pa, double pb, double rate)
{
    if (!(rate < 1.0)) return false;
    const double Lmin = (Lb - rate * La) / (1.0 - rate);
    const double lo = Lmin < Lb ? Lmin : Lb, hi = Lmin < Lb ? Lb : Lmin;
    return lo <= Lc && Lc <= hi && !(pb > pa);
}

// The two halves of that test without a division, as the register kernel takes them (rate < 1 and
// beta2 > 0 are the caller's business; only comparisons that sit within rounding of a tie can differ).
// Between L_b and Length_min: multiply the three numbers by 1 - rate > 0.
__device__ inline bool inside_interval(double La, double Lb, double Lc, double rate)
{
    const double s = 1.0 - rate;
    const double e0 = s * Lb, e1 = Lb - rate * La, c = s * Lc;
    const double lo = e1 < e0 ? e1 : e0, hi = e1 < e0 ? e0 : e1;
    return (lo <= c) & (c <= hi);
}
// |b|^2 - L_b^2/beta2 <= |a|^2 - L_a^2/beta2, multiplied by beta2.
__device__ inline bool across_does_not_grow(double La, double Lb, double na2, double nb2, double beta2)
{
    return !((nb2 - na2) * beta2 > Lb * Lb - La * La);
}

// base^(1/REACH) for the delays the register kernel covers, by square and cube roots.
template <int REACH>
__device__ inline double delay_root(double base)
{
    if constexpr (REACH == 1) return base;
    else if constexpr (REACH == 2) return sqrt(base);
    else if constexpr (REACH == 3) return cbrt(base);
    else if constexpr (REACH == 4) return sqrt(sqrt(base));
    else return pow(base, 1.0 / (double)REACH);
}

// MAXW: how many iterates one pass can project (reach + 1 are needed).
template <typename TX, int VEC, int MAXW>
__global__ __launch_bounds__(kDelayThreads) void delay_server_kernel(DelayArgs a)
{
    constexpr int NT = kDelayThreads, NW = kDelayWaves;
    __shared__ double red[2][NW][MAXW + 1];
    __shared__ double nrm[MAXW + 1];               // squared lengths of the ring's vectors, by slot

    const int tid = threadIdx.x;
    const int lane = tid & (kWave - 1);
    const int wave = tid / kWave;
    const int chain = blockIdx.x;
    const int64_t n = a.n_samples[chain];
    const int64_t d = a.d;
    const int reach = a.tau > 1 ? a.tau : 1;
    const int slots = reach + 2;
    const TX *X = static_cast<const TX *>(a.dense);
    double *ring = a.ring + (int64_t)chain * slots * d;
    const double eta = a.eta, eta_lambda = a.eta * a.lambda;
    int parity = 0;

    // sums `count` values per thread over the workgroup; every thread receives the same totals
    auto block_sums = [&](double(&v)[MAXW + 1], int count) {
#pragma unroll
        for (int t = 0; t <= MAXW; ++t)
            if (t < count) {
                const double w = wave_sum_lane63(v[t]);
                if (lane == kWave - 1) red[parity][wave][t] = w;
            }
        __syncthreads();
#pragma unroll
        for (int t = 0; t <= MAXW; ++t)
            if (t < count) {
                double sum = red[parity][0][t];
#pragma unroll
                for (int w = 1; w < NW; ++w) sum += red[parity][w][t];
                v[t] = sum;
            }
        parity ^= 1;
    };

    {   // w_0 and its squared length
        double v[MAXW + 1];
        v[0] = 0.0;
        for (int64_t col = (int64_t)tid * VEC; col < d; col += (int64_t)NT * VEC)
#pragma unroll
            for (int j = 0; j < VEC; ++j) {
                const double w = a.w_start ? (double)a.w_start[col + j] : 0.0;
                ring[col + j] = w;
                v[0] += w * w;
            }
        block_sums(v, 1);
        if (tid == 0) nrm[0] = v[0];
    }

    RowWindow win;
    win.init(a.seed_lo, a.seed_hi, (uint32_t)chain, (uint32_t)a.m);
    int64_t J = 0;                                  // accepted updates so far

    for (int64_t s = 0; s < n; ++s) {
        const uint32_t row = win.get(s);
        const TX *xr = X + (int64_t)row * a.ld;
        const double y = (double)a.y[row];
        const int64_t at = J - a.tau > 0 ? J - a.tau : 0;          // where the gradient is evaluated
        // iterates to project: w_{J-reach} .. w_J under Check, w_{J-tau} alone without it
        const int64_t first = a.check ? (J - reach > 0 ? J - reach : 0) : at;
        const int nwin = a.check ? (int)(J - first) + 1 : 1;
        int64_t off[MAXW];
#pragma unroll
        for (int t = 0; t < MAXW; ++t) off[t] = (int64_t)((first + t) % slots) * d;

        double v[MAXW + 1];                          // v[t] = w_{first+t}.x, v[MAXW] = x.x
#pragma unroll
        for (int t = 0; t <= MAXW; ++t) v[t] = 0.0;
        for (int64_t col = (int64_t)tid * VEC; col < d; col += (int64_t)NT * VEC) {
            DelayRow<TX, VEC> c;
            c.load(xr + col);
#pragma unroll
            for (int j = 0; j < VEC; ++j) v[MAXW] += c.x[j] * c.x[j];
#pragma unroll
            for (int t = 0; t < MAXW; ++t)
                if (t < nwin) {
                    const double *w = ring + off[t] + col;
#pragma unroll
                    for (int j = 0; j < VEC; ++j) v[t] += w[j] * c.x[j];
                }
        }
        // the totals are wanted in v[0..nwin) and v[MAXW]; move x.x next to the projections
        {
            const double b = v[MAXW];
#pragma unroll
            for (int t = 0; t < MAXW; ++t)
                if (t == nwin) v[t] = b;
            if (nwin == MAXW) v[MAXW] = b;
        }
        block_sums(v, nwin + 1);
        double beta2 = v[MAXW], L_new = 0.0, L_prev = 0.0;
#pragma unroll
        for (int t = 0; t < MAXW; ++t) {
            if (t == nwin) beta2 = v[t];
            if (t == nwin - 1) L_new = v[t];             // w_J.x (without Check: w_{J-tau}.x)
            if (t == nwin - 2) L_prev = v[t];            // w_{J-1}.x
        }
        const double yhat = (a.check && a.tau == 0) ? L_new : v[0];
        const double g = a.loss == kLossHinge ? loss_slope<kLossHinge>(y, yhat) : loss_slope<kLossLogistic>(y, yhat);

        bool keep = true;
        if (a.check) {
            const double base = eta_lambda + eta * beta2;
            const double rate = reach == 1 ? base : pow(base, 1.0 / (double)reach);
            auto across2 = [&](int64_t t, double L) {
                const double n2 = nrm[t % slots];
                return beta2 > 0.0 ? n2 - L * L / beta2 : n2;
            };
#pragma unroll
            for (int t = 2; t < MAXW; ++t)
                if (t < nwin && keep)
                    keep = check_triple(v[t - 2], v[t - 1], v[t], across2(first + t - 2, v[t - 2]),
                                        across2(first + t - 1, v[t - 1]), rate);
            if (keep && J >= 1) {
                const double L_cand = L_new - eta_lambda * yhat - eta * g * beta2;
                keep = check_triple(L_prev, L_new, L_cand, across2(J - 1, L_prev), across2(J, L_new), rate);
            }
        }
        if (keep) {
            const double *wj = ring + (int64_t)(J % slots) * d;
            const double *wd = ring + (int64_t)(at % slots) * d;
            double *dst = ring + (int64_t)((J + 1) % slots) * d;
            const double eg = eta * g;
            double u[MAXW + 1];
            u[0] = 0.0;
            for (int64_t col = (int64_t)tid * VEC; col < d; col += (int64_t)NT * VEC) {
                DelayRow<TX, VEC> c;
                c.load(xr + col);
#pragma unroll
                for (int j = 0; j < VEC; ++j) {
                    const double w = wj[col + j] - eta_lambda * wd[col + j] - eg * c.x[j];
                    dst[col + j] = w;
                    u[0] += w * w;
                }
            }
            block_sums(u, 1);
            ++J;
            if (tid == 0) nrm[J % slots] = u[0];
        }
    }

    const double *last = ring + (int64_t)(J % slots) * d;
    float *out = a.W + (int64_t)chain * d;
    for (int64_t col = (int64_t)tid * VEC; col < d; col += (int64_t)NT * VEC)
#pragma unroll
        for (int j = 0; j < VEC; ++j) out[col + j] = (float)last[col + j];
    if (tid == 0) a.accepted[chain] = J;
}

// The ring in registers.  R1 = max(tau, 1) + 1 iterates are kept: r[i] is w_{J-i}; before J reaches i
// the slot holds w_0, which is what an index below zero means.  n2[i] is |w_{J-i}|^2 (CHECK only).
template <typename TX, int EPT, int VEC, int R1, int PF, bool CHECK>
__global__ __launch_bounds__(kDelayThreads) void delay_server_reg_kernel(DelayArgs a)
{
    constexpr int NT = kDelayThreads, NW = kDelayWaves;
    using Frag = RowFrag<TX, NT, EPT, VEC>;
    __shared__ double red[2][NW][R1 + 1];

    const int tid = threadIdx.x;
    const int lane = tid & (kWave - 1);
    const int wave = tid / kWave;
    const int chain = blockIdx.x;
    const int64_t n = a.n_samples[chain];
    const uint32_t d = (uint32_t)a.d;
    const char *X = static_cast<const char *>(a.dense);
    const int64_t row_stride = a.ld * (int64_t)sizeof(TX);
    const uint32_t row_bytes = d * (uint32_t)sizeof(TX);
    const double eta = a.eta, eta_lambda = a.eta * a.lambda;
    const bool no_delay = R1 == 2 && a.tau == 0;    // with three or more iterates kept the delay is R1 - 1
    int parity = 0;

    // element e of this thread is column col0[e / VEC] + e % VEC; columns from d on do not exist
    uint32_t off[Frag::kChunks];
#pragma unroll
    for (int c = 0; c < Frag::kChunks; ++c) off[c] = (uint32_t)((c * NT + tid) * VEC) * (uint32_t)sizeof(TX);
    auto column = [&](int e) { return (uint32_t)(((e / VEC) * NT + tid) * VEC + e % VEC); };

    auto block_sums = [&](auto &v, auto count_tag) {
        constexpr int COUNT = decltype(count_tag)::value;
        wave_sums_to_lds<COUNT, 1>(v, &red[parity][wave][0], lane);
        __syncthreads();
#pragma unroll
        for (int t = 0; t < COUNT; ++t) {
            double sum = red[parity][0][t];
#pragma unroll
            for (int w = 1; w < NW; ++w) sum += red[parity][w][t];
            v[t] = sum;
        }
        parity ^= 1;
    };

    double r[R1][EPT], n2[CHECK ? R1 : 1];
    {
        double v[1] = {0.0};
#pragma unroll
        for (int e = 0; e < EPT; ++e) {
            const uint32_t col = column(e);
            const double w = (a.w_start && col < d) ? (double)a.w_start[col] : 0.0;
#pragma unroll
            for (int i = 0; i < R1; ++i) r[i][e] = w;
            v[0] += w * w;
        }
        if constexpr (CHECK) {                       // (the squared lengths are the tests' business)
            block_sums(v, std::integral_constant<int, 1>{});
#pragma unroll
            for (int i = 0; i < R1; ++i) n2[i] = v[0];
        }
    }

    // Rows and labels of the next PF samples are on their way at any time; beyond the end the last sample's again, so that no request
    // sits under a branch, where each would be waited for on the spot, and labels travel with the rows (a scalar load would be
    // drained by the exchange of sums; through a resource of their own they need no address registers).  128 servers of up to 400 samples, fp32, d = 4096, tau = 0,
    // without Check: 470 -> 301 us.
    RowWindow win;
    win.init(a.seed_lo, a.seed_hi, (uint32_t)chain, (uint32_t)a.m);
    Frag x[PF];
    float ys[PF];
    auto request = [&](int u, int64_t s) {
        const uint32_t row = win.get(s < n ? s : n - 1);
        ys[u] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(make_rsrc(a.y + row, 4u), 0, 0, 0));
        const __amdgpu_buffer_rsrc_t rx = make_rsrc(X + (int64_t)row * row_stride, row_bytes);
#pragma unroll
        for (int c = 0; c < Frag::kChunks; ++c) x[u].load_chunk(c, rx, off[c]);
    };
    if (n > 0) {
#pragma unroll
        for (int u = 0; u < PF; ++u) request(u, u);
    }

    // What a sample costs here is issue and the exchange, so more servers than compute units want two or three workgroups on each.  The
    // sample's code therefore stands once per place in a round, and calls under Check have a kernel of their own: with the last round
    // written out a second time, and one kernel for both, it took up to 115 registers more and half the waves per SIMD (us, 600
    // servers of up to 400 samples, fp32: d = 2047, tau = 4, under Check 1141 -> 726; d = 4096, tau = 0, without it 780 -> 540).
    int64_t J = 0;
    for (int64_t s0 = 0; s0 < n; s0 += PF) {
#pragma unroll
        for (int u = 0; u < PF; ++u) {
            const int64_t s = s0 + u;
            if (s >= n) break;
            double xe[EPT];
#pragma unroll
            for (int e = 0; e < EPT; ++e) xe[e] = (double)x[u].at(e);
            const double y = (double)ys[u];
            request(u, s + PF);

            double v[R1 + 1];                        // v[i] = w_{J-i}.x, v[R1] = x.x
#pragma unroll
            for (int i = 0; i <= R1; ++i) v[i] = 0.0;
            if constexpr (CHECK) {
#pragma unroll
                for (int e = 0; e < EPT; ++e) {
                    v[R1] += xe[e] * xe[e];
#pragma unroll
                    for (int i = 0; i < R1; ++i) v[i] += r[i][e] * xe[e];
                }
                block_sums(v, std::integral_constant<int, R1 + 1>{});
            } else {                                 // only the projection the gradient needs
#pragma unroll
                for (int e = 0; e < EPT; ++e) v[0] += (no_delay ? r[0][e] : r[R1 - 1][e]) * xe[e];
                block_sums(v, std::integral_constant<int, 1>{});
                v[R1 - 1] = v[0];
            }
            const double beta2 = v[R1];
            const double yhat = no_delay ? v[0] : v[R1 - 1];           // the gradient is taken at w_{J-tau}

            // The cheapest tests come first and a failed one ends the sample: the parts across x (no root,
            // no slope), then the intervals of the first call (the root), then the candidate's (the slope).
            bool keep = true;
            double g = 0.0;
            if constexpr (CHECK) {
                if (beta2 > 0.0) {
#pragma unroll
                    for (int i = 0; i + 1 < R1; ++i)      // pairs (w_{J-i-1}, w_{J-i}) that some triple holds
                        if (J >= i + 1) keep = keep && across_does_not_grow(v[i + 1], v[i], n2[i + 1], n2[i], beta2);
                } else {
#pragma unroll
                    for (int i = 0; i + 1 < R1; ++i)
                        if (J >= i + 1) keep = keep && !(n2[i] > n2[i + 1]);
                }
                if (keep) {
                    const double rate = delay_root<R1 - 1>(eta_lambda + eta * beta2);
                    keep = rate < 1.0 || J == 0;          // with no triple to test nothing is rejected
#pragma unroll
                    for (int i = 0; i + 2 < R1; ++i)
                        if (J >= i + 2) keep = keep && inside_interval(v[i + 2], v[i + 1], v[i], rate);
                    if (keep && J >= 1) {
                        g = a.loss == kLossHinge ? loss_slope<kLossHinge>(y, yhat) : loss_slope<kLossLogistic>(y, yhat);
                        const double L_cand = v[0] - eta_lambda * yhat - eta * g * beta2;
                        keep = inside_interval(v[1], v[0], L_cand, rate);
                    } else if (keep) {
                        g = a.loss == kLossHinge ? loss_slope<kLossHinge>(y, yhat) : loss_slope<kLossLogistic>(y, yhat);
                    }
                }
            } else {
                g = a.loss == kLossHinge ? loss_slope<kLossHinge>(y, yhat) : loss_slope<kLossLogistic>(y, yhat);
            }
            if (keep) {
                const double eg = eta * g;
                double u2[1] = {0.0};
#pragma unroll
                for (int e = 0; e < EPT; ++e) {
                    const double old = no_delay ? r[0][e] : r[R1 - 1][e];
                    const double w = r[0][e] - eta_lambda * old - eg * xe[e];
#pragma unroll
                    for (int i = R1 - 1; i >= 1; --i) r[i][e] = r[i - 1][e];
                    r[0][e] = w;
                    u2[0] += w * w;
                }
                if constexpr (CHECK) {
                    block_sums(u2, std::integral_constant<int, 1>{});
#pragma unroll
                    for (int i = R1 - 1; i >= 1; --i) n2[i] = n2[i - 1];
                    n2[0] = u2[0];
                }
                ++J;
            }
        }
    }

    float *out = a.W + (int64_t)chain * a.d;
#pragma unroll
    for (int e = 0; e < EPT; ++e) {
        const uint32_t col = column(e);
        if (col < d) out[col] = (float)r[0][e];
    }
    if (tid == 0) a.accepted[chain] = J;
}

// Rows on their way from HBM into LDS.  A ring of S row slots (sample s in slot s mod S), filled by loads
// that land in LDS directly and need no registers while in flight; in front of each wave's part of a slot, a pad that
// receives, the same way, a small record per sample: SIDE dwords from an array indexed by the sample's
// row (SIDE = 1: its label; SIDE = 8: its entry of the row table, see DelayRowEntry).  Every wave requests, and later reads back, only its own
// part of a row (the columns its lanes own), so the slots need no barrier.  The compiler does not see
// these loads; a wave's loads complete in issue order, so waiting until at most (S - B) samples' worth of
// them are outstanding means the B oldest samples have landed.  Samples past the end of the stream are
// requested all the same (the last valid row again), which keeps that count a constant.  The record goes
// out before its row, so it has landed when the row has; fetched by an ordinary load inside the loop it
// would queue behind the rows on their way and wait for all of them.
template <typename TX, int EPT, int VEC, int S, int SIDE>
struct LdsRows {
    static_assert(SIDE >= 1 && SIDE <= kWave && (SIDE & (SIDE - 1)) == 0, "a power of two of dwords");
    static constexpr int NT = kDelayThreads, NW = kDelayWaves;
    using Frag = RowFrag<TX, NT, EPT, VEC>;
    static_assert(VEC * sizeof(TX) == 16, "16-byte loads only");
    static constexpr int CHUNKS = EPT / VEC;
    static_assert(Frag::kWords == 4 * CHUNKS, "four words per chunk");
    static constexpr uint32_t kPadBytes = kWave * 4;                     // a wave's copy of one record (64 / SIDE times)
    static constexpr uint32_t kWaveBytes = kPadBytes + CHUNKS * kWave * 16;      // and what it holds of one row, behind it
    static constexpr uint32_t kSlotBytes = NW * kWaveBytes;
    static constexpr int kLoadsPerSample = CHUNKS + 1;                   // the row's chunks and its record
    static constexpr size_t kBytes = (size_t)S * kSlotBytes;
    typedef __attribute__((address_space(3))) uint32_t *lds_words;

    lds_words stage;            // S slots
    uint32_t slot0;             // LDS byte address of this wave's part of slot 0
    uint32_t voff, lane, wave, side_lane;
    u32x4 ry;                   // the records as a buffer
    const char *X;              // kPadBytes in front of the rows
    int64_t row_stride, n;
    uint32_t row_bytes;
    RowWindow ahead;

    // clears the slots (lanes whose columns lie beyond the row are out of the buffer's range: whether such
    // a load writes zeros or nothing, the slots read as zero there afterwards); ends with a barrier
    __device__ void init(lds_words lds, const DelayArgs &a, int chain, int64_t samples, const void *records)
    {
        const int tid = threadIdx.x;
        stage = lds;
        lane = (uint32_t)(tid & (kWave - 1));
        wave = (uint32_t)__builtin_amdgcn_readfirstlane(tid / kWave);
        slot0 = (uint32_t)__builtin_amdgcn_readfirstlane((int)((uint32_t)(size_t)lds + wave * kWaveBytes));
        voff = (uint32_t)(tid * 16);                 // this lane's bytes of chunk 0; chunk c adds c*NT*16
        const uint64_t ybase = (uint64_t)(uintptr_t)records;
        ry[0] = (uint32_t)ybase;
        ry[1] = (uint32_t)(ybase >> 32) & 0xffffu;
        ry[2] = (uint32_t)(SIDE > 1 && a.visits ? a.visits : a.m) * (uint32_t)(SIDE * 4);
        ry[3] = 0x00020000u;
        side_lane = (lane & (uint32_t)(SIDE - 1)) * 4u;
        X = static_cast<const char *>(a.dense) - kPadBytes;
        row_stride = a.ld * (int64_t)sizeof(TX);
        row_bytes = (uint32_t)a.d * (uint32_t)sizeof(TX);
        n = samples;
        ahead.init(a.seed_lo, a.seed_hi, (uint32_t)chain, (uint32_t)a.m);
        for (uint32_t i = (uint32_t)tid; i < (uint32_t)S * (kSlotBytes / 4); i += NT) stage[i] = 0u;
        __syncthreads();
    }
    // the record and the row of sample s (of the last sample, beyond the end) into slot s mod S
    __device__ void request(int64_t s)
    {
        const uint32_t row = ahead.get_stream(s < n ? s : n - 1);
        request_row(s, row, row);
    }
    // One statement that writes M0 once: an instruction's offset moves the place in LDS and the place in memory alike, so the row's first chunk
    // takes kPadBytes of it, which its descriptor starts early (X does), and chunk c another c KiB, with the rest of its way through memory from a scalar.
    // (s_nop: the wait state that a load to LDS wants behind the write of M0.  A scalar that a vector instruction wrote, as a descriptor that the compiler
    // has spilled is, wants five; none comes that late, which a test reads from the built library.)  us, 128 servers of up to 8000 samples, tau = 2, without
    // Check, a write of M0 and four wait states for each load -> this: d = 4096 fp32 3420 -> 3250, bf16 3480 -> 3230; d = 2048 2675 -> 2470 and
    // 2440 -> 2365; under Check 2490 -> 2480, 1930 -> 1840, 1645 -> 1525 and 1500 -> 1405.
    __device__ void request_row(int64_t s, uint32_t row, uint32_t record)
    {
        const uint64_t base = (uint64_t)(uintptr_t)(X + (int64_t)row * row_stride);
        u32x4 rx;
        rx[0] = (uint32_t)base;
        rx[1] = (uint32_t)(base >> 32) & 0xffffu;
        rx[2] = row_bytes + kPadBytes;
        rx[3] = 0x00020000u;
        constexpr uint32_t kRest = NT * 16 - kWave * 16;
        static_assert(kPadBytes == 256 && kWave * 16 == 1024 && (CHUNKS == 1 || CHUNKS == 2 || CHUNKS == 4), "the offsets below");
        const uint32_t slot = slot0 + (uint32_t)(s % S) * kSlotBytes, at = record * (uint32_t)(SIDE * 4) + side_lane;
#define WPSGD_RECORD_AND_CHUNK                                                                                                    \
    "s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dword %1, %2, 0 offen lds\n\tbuffer_load_dwordx4 %3, %4, 0 offen offset:256 lds"
        if constexpr (CHUNKS == 1)
            asm volatile(WPSGD_RECORD_AND_CHUNK : : "s"(slot), "v"(at), "s"(ry), "v"(voff), "s"(rx) : "memory", "m0");
        else if constexpr (CHUNKS == 2)
            asm volatile(WPSGD_RECORD_AND_CHUNK "\n\tbuffer_load_dwordx4 %3, %4, %5 offen offset:1280 lds"
                         :
                         : "s"(slot), "v"(at), "s"(ry), "v"(voff), "s"(rx), "s"(kRest)
                         : "memory", "m0");
        else
            asm volatile(WPSGD_RECORD_AND_CHUNK "\n\tbuffer_load_dwordx4 %3, %4, %5 offen offset:1280 lds\n\t"
                                                "buffer_load_dwordx4 %3, %4, %6 offen offset:2304 lds\n\tbuffer_load_dwordx4 %3, %4, %7 offen offset:3328 lds"
                         :
                         : "s"(slot), "v"(at), "s"(ry), "v"(voff), "s"(rx), "s"(kRest), "s"(2 * kRest), "s"(3 * kRest)
                         : "memory", "m0");
#undef WPSGD_RECORD_AND_CHUNK
    }
    // waits until the B oldest of the S samples requested last have landed
    // (gfx9 encoding: vmcnt split over bits 3:0 and 15:14; expcnt and lgkmcnt left open)
    template <int B>
    __device__ static void wait_for_oldest()
    {
        constexpr int kLater = (S - B) * kLoadsPerSample;
        static_assert(kLater >= 0 && kLater < 64, "the counter holds 63");
        __builtin_amdgcn_s_waitcnt(((kLater & 0xF) | ((kLater >> 4) << 14)) | 0x0F70);
        __builtin_amdgcn_sched_barrier(0);
    }
    // this thread's elements of the row of sample s
    __device__ void take(int64_t s, Frag &x) const
    {
        const lds_words src = stage + (size_t)(s % S) * (kSlotBytes / 4) + (size_t)wave * (kWaveBytes / 4) + kPadBytes / 4 + lane * 4;
        typedef __attribute__((address_space(3))) const u32x4 *lds_quads;
#pragma unroll
        for (int c = 0; c < CHUNKS; ++c) {
            const u32x4 q = *(lds_quads)(src + c * (kWave * 4));
            x.w[4 * c + 0] = q[0];
            x.w[4 * c + 1] = q[1];
            x.w[4 * c + 2] = q[2];
            x.w[4 * c + 3] = q[3];
        }
    }
    // dword j of sample s's record (the same address in every lane)
    __device__ uint32_t side(int64_t s, int j) const
    {
        return stage[(size_t)(s % S) * (kSlotBytes / 4) + (size_t)wave * (kWaveBytes / 4) + j];
    }
    __device__ double side_f64(int64_t s, int j) const
    {
        return __longlong_as_double((long long)(((uint64_t)side(s, j + 1) << 32) | side(s, j)));
    }
    // every LDS read of a slot must have returned before the slot is requested again
    __device__ static void reads_done() { __builtin_amdgcn_s_waitcnt(0xC07F); }
    // nothing may still be landing when the wave ends
    __device__ static void drain() { asm volatile("s_waitcnt vmcnt(0)" : : : "memory"); }
};

// What the Check function needs of a row and not of the model, formed ahead of the servers by workgroups that wait for nobody: once per
// row of the data set instead of once per visit, or per visit where the servers together visit less than a quarter as many
// (one server of 8000 samples, m = 65536, d = 4096: 9150 us with the per-sample kernel, 195 with the table and a team).  32 bytes, read as eight dwords.
struct DelayRowEntry {
    double beta2;       // x.x
    double rate;        // (eta*lambda + eta*beta2)^(1/reach)
    float y;            // the label
    float pad[3];
};
static_assert(sizeof(DelayRowEntry) == 32, "eight dwords");

// For a whole wave: the server i with before(i) <= at < before(i + 1), where before(i) = count(0) + .. + count(i - 1) in list order;
// -1 if the counts end before `at`.  The counts together are below 2^31.
template <typename F>
__device__ inline int server_of_item(int k, int at, int &before, F &&count)
{
    const int lane = (int)(threadIdx.x & (kWave - 1));
    before = 0;
    for (int c = 0; c < k; c += kWave) {
        const int mine = c + lane < k ? count(c + lane) : 0;
        int upto = mine;
        for (int o = 1; o < kWave; o <<= 1) {
            const int t = __shfl_up(upto, o);
            if (lane >= o) upto += t;
        }
        const uint64_t hit = __builtin_amdgcn_ballot_w64(at < before + upto);
        if (hit) {
            const int j = __builtin_ctzll(hit);
            before += __builtin_amdgcn_readlane(upto, j) - __builtin_amdgcn_readlane(mine, j);
            return c + j;
        }
        before += __builtin_amdgcn_readlane(upto, kWave - 1);
    }
    return -1;
}

// The same from the sums themselves, which begin with 0 and do not fall (`at` is below the sum of all counts): every round
// leaves a 64th of the servers.  (us a call, d = 64, 20000 servers of up to 100 samples: 14476 with the counts
// added up for every visit, 1938 now, 1998 with the per-sample kernel and no table; 4000 servers 893, 396, 467.)
__device__ inline int server_of_visit(int k, int64_t at, const int64_t *before)
{
    const int lane = (int)(threadIdx.x & (kWave - 1));
    int first = 0;
    for (int left = k; left > 1;) {
        const int step = (left + kWave - 1) / kWave;
        const bool reached = lane * step < left && before[first + lane * step] <= at;
        const int whole = __builtin_popcountll(__builtin_amdgcn_ballot_w64(reached)) - 1;
        first += whole * step;
        left = left - whole * step < step ? left - whole * step : step;
    }
    return first;
}

template <typename TX, int VEC>
__global__ __launch_bounds__(kDelayThreads) void delay_row_table_kernel(DelayArgs a, DelayRowEntry *table, int reach)
{
    const int lane = threadIdx.x & (kWave - 1);
    const int64_t entry = (int64_t)blockIdx.x * kDelayWaves + threadIdx.x / kWave;       // one wave per entry
    if (a.team)                                         // (the teams' tables start out zero)
        for (int64_t i = (int64_t)blockIdx.x * kDelayThreads + threadIdx.x; i < (int64_t)a.k * kDelayTeamWords;
             i += (int64_t)gridDim.x * kDelayThreads)
            a.team[i] = 0;
    int64_t row = entry;
    if (a.visits) {
        if (entry >= a.visits) return;
        int64_t first;
        int server;
        if (a.visits_before) {
            server = server_of_visit(a.k, entry, a.visits_before);
            first = a.visits_before[server];
        } else {
            int sum;
            server = server_of_item(a.k, (int)entry, sum, [&](int i) { return (int)a.n_samples[i]; });
            if (server < 0) return;
            first = sum;
        }
        row = sample_row(a.seed_lo, a.seed_hi, (uint32_t)server, (uint64_t)(entry - first), (uint32_t)a.m);
    }
    if (row >= a.m) return;
    const TX *xr = static_cast<const TX *>(a.dense) + row * a.ld;
    double acc = 0.0;
    for (int64_t col = (int64_t)lane * VEC; col < a.d; col += (int64_t)kWave * VEC) {
        DelayRow<TX, VEC> c;
        c.load(xr + col);
#pragma unroll
        for (int j = 0; j < VEC; ++j) acc += c.x[j] * c.x[j];
    }
    const double beta2 = wave_sum(acc);
    if (lane == 0) {
        const double base = a.eta * a.lambda + a.eta * beta2;
        DelayRowEntry e;
        e.beta2 = beta2;
        e.rate = reach == 1 ? base : reach == 2 ? delay_root<2>(base) : reach == 3 ? delay_root<3>(base) : delay_root<4>(base);
        e.y = a.y[row];
        e.pad[0] = e.pad[1] = e.pad[2] = 0.0f;
        table[entry] = e;
    }
}

// All tests of the Check function for one sample, from its scalars alone and without branches on the
// data: L[i] = w_{J-i}.x; n2[i] = |w_{J-i}|^2; beta2 = x.x and rate from the row table; yhat and g
// belong to w_{J-tau}.
template <int R1>
__device__ inline bool window_passes(const double *L, const double (&n2)[R1], double beta2, double rate, int64_t J,
                                     double eta, double eta_lambda, double yhat, double g)
{
    // (bitwise and/or on purpose: nothing here is worth a branch, and without branches the tests of
    // several samples can be interleaved)
    bool ok = true;
#pragma unroll
    for (int i = 0; i + 1 < R1; ++i) {          // pairs (w_{J-i-1}, w_{J-i}) that some triple holds
        const bool along = across_does_not_grow(L[i + 1], L[i], n2[i + 1], n2[i], beta2);
        const bool plain = !(n2[i] > n2[i + 1]);
        ok = ok & ((J < i + 1) | (beta2 > 0.0 ? along : plain));
    }
    ok = ok & ((rate < 1.0) | (J == 0));        // with no triple to test nothing is rejected
#pragma unroll
    for (int i = 0; i + 2 < R1; ++i) ok = ok & ((J < i + 2) | inside_interval(L[i + 2], L[i + 1], L[i], rate));
    const double L_cand = L[0] - eta_lambda * yhat - eta * g * beta2;
    ok = ok & ((J < 1) | inside_interval(L[1], L[0], L_cand, rate));
    return ok;
}

// Under the Check function nearly every sample is thrown away, and a sample that is thrown away leaves
// the ring as it was.  This kernel therefore looks at B samples at once: it projects the ring on all B
// rows, exchanges the B x R1 sums in one round and takes the B decisions at once, each in a row of 16 lanes
// of its own, as if the samples before it had been rejected.  The decisions up to and including the first acceptance are then the sequential ones;
// that sample's candidate is written and the samples behind it are looked at again, against the new ring,
// as the next batch.
//
// Rows come through LdsRows: the rows of samples pos .. pos+S-1 are always in LDS or on their way, so a
// batch's rows were asked for at least S-B samples earlier, and the row of an accepted sample is still in
// its slot when the candidate is formed.
//
// TEAM: several workgroups per server (128 servers use half of the compute units, and a few servers next to none).  All members of
// a team hold the same ring.  Between two acceptances the decisions depend on the ring alone, so the batches of that stretch, an epoch,
// are dealt out in turn: batch t of the member with rank r of W is samples base + 4*(t*W + r) .. +3.  A member that finds an
// acceptance, or has nothing left below the first one it knows of, puts a record into the team's table and waits; the first
// workgroup, the owner, collects the records, takes the earliest acceptance and orders all members to write that candidate
// and to begin the next epoch behind it.  Every member forms the candidate itself, from the row and the finder's slope: the same
// bits everywhere, the same decisions and results as a server alone.
//  * Records and orders are 64-bit words, each with the epoch they belong to in the upper half, stored and read at device
//    scope: a word is taken whole or not at all, and no order between stores is needed.  A member's record of an epoch follows
//    the order that began it, and the owner gives the next order only when it has all records, so no word is overwritten
//    while anyone may still want it.
//  * A member learns of the others' acceptances from their records, one load per batch that lands in LDS behind the rows
//    (an ordinary load would wait for them).
//  * Nobody waits for a workgroup that is not running: a team is made of those that have reported within some 0.1 ms of the
//    owner's start (owners are launched first), the others leave when they see that an order has been given without them.  All
//    waits are bounded: an owner whose members do not answer goes on alone from the base of the epoch, members without orders leave.
//  * An epoch costs some 8 us of exchange, row fetch and new requests; when acceptances come closer than kTeamGap samples for good
//    the owner sends its members away and goes on alone, as without a team.  (The first updates of a server come thick: 9 to 17 of the
//    first 32 samples and 20 to 40 in all on rows along one direction, which kTeamSlack lets pass.)
// fp32, d = 4096, m = 65536, tau = 2, up to 8000 samples a server, ms per call: 128 servers 4.16 -> 2.16 (two thirds of it HBM: 10.8 GB of
// rows at 6.8 TB/s are 1.6), 64: 4.10 -> 1.06, 8: 3.63 -> 0.29.  Streams of which one sample in ten and more is accepted pay for the
// epochs up to the dissolution, 0.26 ms, and 0.2 us per update for the team's code: 8 servers of 1000 samples, d = 1024, us: 100 accepted 392 -> 628,
// all 1279 -> 1597; 27 accepted 334 -> 256, 9 318 -> 122.
constexpr int kTeamMax = kDelayTeamMax;         // members: one lane each
static_assert(kTeamMax == kWave, "a member is a lane");
constexpr int kTeamPresent = 2 * kTeamMax, kTeamOrder = kTeamPresent + kTeamMax / 2;     // 64-bit words: records, presence (32 bits each), orders
constexpr int kTeamWords = kTeamOrder + 16;     // per server: 1408 bytes
static_assert(kTeamWords == kDelayTeamWords, "as the planner has it");
constexpr uint32_t kTeamFound = 1u << 23;       // upper half of a record: epoch mod 256, found or not, position behind the base
constexpr int kTeamEpoch = 1 << 22;             // samples of an epoch at most: positions have 22 bits
constexpr uint32_t kTeamOver = ~0u;             // an order's epoch: the team is sent away
constexpr uint32_t kTeamNone = ~0u;             // an order's position: nothing was accepted
constexpr int kTeamGather = 128, kTeamPolls = 1 << 22;
constexpr int kTeamGap = 24, kTeamSlack = 32;

__device__ inline void team_store(uint64_t *p, uint32_t hi, uint32_t lo)
{
    __hip_atomic_store(p, ((uint64_t)hi << 32) | lo, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ inline uint64_t team_load(const uint64_t *p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ inline void team_order(uint64_t *team, uint32_t epoch, uint32_t pos, uint64_t payload)
{
    team_store(team + kTeamOrder, epoch, pos);
    team_store(team + kTeamOrder + 1, epoch, (uint32_t)(payload >> 32));
    team_store(team + kTeamOrder + 2, epoch, (uint32_t)payload);
}
// the order that begins `epoch` (or ends the team), for one whole wave; kTeamOver if none comes.  An order of a later epoch is for
// those who were there in time: the owner gives none before a member has answered the one before.
__device__ inline uint32_t team_await_order(const uint64_t *team, uint32_t epoch, uint32_t &pos, uint64_t &payload)
{
    const int lane = (int)(threadIdx.x & (kWave - 1));
    for (int tries = 0; tries < kTeamPolls; ++tries) {
        const uint64_t w = team_load(team + kTeamOrder + (lane < 2 ? lane : 2));
        const uint32_t stamp = (uint32_t)(w >> 32);
        if (__builtin_amdgcn_ballot_w64(stamp > epoch)) return kTeamOver;       // (kTeamOver itself among them)
        if (__builtin_amdgcn_ballot_w64(stamp == epoch) == ~0ull) {
            pos = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)w, 0);
            payload = ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)w, 1) << 32) |
                      (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)w, 2);
            return epoch;
        }
        __builtin_amdgcn_s_sleep(2);
    }
    return kTeamOver;
}
// the smallest position among the records that say "found" in this epoch, and whose it is; kTeamNone if there is none
__device__ inline uint32_t team_first_found(uint32_t record, bool mine, uint32_t epoch, int &whose)
{
    const bool found = mine && (record >> 24) == (epoch & 255u) && (record & kTeamFound);
    uint32_t first = kTeamNone;
    whose = 0;
    for (uint64_t left = __builtin_amdgcn_ballot_w64(found); left; left &= left - 1) {
        const int w = __builtin_ctzll(left);
        const uint32_t pos = (uint32_t)__builtin_amdgcn_readlane((int)record, w) & (kTeamFound - 1u);
        if (pos < first) {
            first = pos;
            whose = w;
        }
    }
    return first;
}

// What a workgroup is: the server, its place in the server's team, the members launched for it.  Workgroups 0 .. k-1 are
// the owners; the others take the servers' further seats in order.
__device__ inline void team_seat(const DelayArgs &a, int &chain, int &member, int &size)
{
    member = 0;
    chain = (int)blockIdx.x;
    if (chain < a.k) {
        size = delay_team_size(a.n_samples[chain], a.team_share);
        return;
    }
    int before;
    const int seat = chain - a.k, i = server_of_item(a.k, seat, before, [&](int j) { return delay_team_size(a.n_samples[j], a.team_share) - 1; });
    size = i < 0 ? 0 : delay_team_size(a.n_samples[i], a.team_share);       // (0: no such seat, the workgroup leaves)
    chain = i < 0 ? 0 : i;
    member = seat - before + 1;
}

template <typename TX, int EPT, int VEC, int R1, int B, int S, bool TEAM>
__global__ __launch_bounds__(kDelayThreads) void delay_server_batch_kernel(DelayArgs a)
{
    constexpr int NT = kDelayThreads, NW = kDelayWaves, NV = B * R1;
    static_assert(B == 4, "one row of 16 lanes per sample");
    using Rows = LdsRows<TX, EPT, VEC, S, 8>;       // with each row its entry of the row table
    using Frag = typename Rows::Frag;
    extern __shared__ __attribute__((aligned(16))) uint32_t stage[];     // Rows::kBytes
    __shared__ __attribute__((aligned(16))) double red[2][NV][NW];       // [sample * R1 + iterate][wave]
    __shared__ uint32_t others[TEAM ? kWave : 1];   // the members' records, as last seen
    __shared__ uint32_t known[2], verdict[4];       // the first acceptance known of; what wave 0 has learnt

    const int tid = threadIdx.x;
    const int lane = tid & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    int chain = blockIdx.x, member = 0, size = 1;
    if constexpr (TEAM) {
        team_seat(a, chain, member, size);
        chain = __builtin_amdgcn_readfirstlane(chain);
        member = __builtin_amdgcn_readfirstlane(member);
        size = __builtin_amdgcn_readfirstlane(size);
        if (size == 0) return;
    }
    const int64_t n = a.n_samples[chain];
    const uint32_t d = (uint32_t)a.d;
    const double eta = a.eta, eta_lambda = a.eta * a.lambda;
    const bool no_delay = R1 == 2 && a.tau == 0;
    int parity = 0;

    auto column = [&](int e) { return (uint32_t)(((e / VEC) * NT + tid) * VEC + e % VEC); };

    auto block_sum = [&](double &v) {
        const double t = wave_sum_lane63(v);
        if (lane == kWave - 1) red[parity][0][wave] = t;
        __syncthreads();
        v = ((red[parity][0][0] + red[parity][0][1]) + red[parity][0][2]) + red[parity][0][3];
        parity ^= 1;
    };

    // A member reports itself at once; the owner looks who is there when its own ring is filled.
    uint64_t *team = TEAM ? a.team + (size_t)chain * kTeamWords : nullptr;
    uint64_t members = 1;
    if constexpr (TEAM) {
        if (member > 0 && tid == 0)
            __hip_atomic_store(reinterpret_cast<uint32_t *>(team + kTeamPresent) + member, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }

    double r[R1][EPT], n2[R1];
    {
        double v = 0.0;
#pragma unroll
        for (int e = 0; e < EPT; ++e) {
            const uint32_t col = column(e);
            const double w = (a.w_start && col < d) ? (double)a.w_start[col] : 0.0;
#pragma unroll
            for (int i = 0; i < R1; ++i) r[i][e] = w;
            v += w * w;
        }
        block_sum(v);
#pragma unroll
        for (int i = 0; i < R1; ++i) n2[i] = v;
    }
    if (n <= 0) {
        float *out0 = a.W + (int64_t)chain * a.d;
#pragma unroll
        for (int e = 0; e < EPT; ++e) {
            const uint32_t col = column(e);
            if (col < d) out0[col] = (float)r[0][e];
        }
        if (tid == 0) a.accepted[chain] = 0;
        return;
    }

    int W = 1, rank = 0;                            // members at work on this server, and this one's place among them
    uint32_t epoch = 1;
    if constexpr (TEAM) {
        if (size > 1) {
            if (wave == 0) {
                uint32_t pos = 0;
                uint64_t there = 0;
                if (member == 0) {
                    for (int tries = 0; tries < kTeamGather; ++tries) {
                        const uint32_t x = lane > 0 && lane < size ? __hip_atomic_load(reinterpret_cast<uint32_t *>(team + kTeamPresent) + lane,
                                                                                       __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 1u;
                        there = __builtin_amdgcn_ballot_w64(lane < size && x != 0u);
                        if (__builtin_popcountll(there) == size) break;
                        __builtin_amdgcn_s_sleep(8);
                    }
                    if (lane == 0) team_order(team, epoch, 0, there);
                } else if (team_await_order(team, epoch, pos, there) == kTeamOver) {
                    there = 0;
                }
                if (lane == 0) {
                    verdict[0] = (uint32_t)there;
                    verdict[1] = (uint32_t)(there >> 32);
                }
            }
            __syncthreads();
            members = ((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)verdict[1]) << 32) |
                      (uint32_t)__builtin_amdgcn_readfirstlane((int)verdict[0]);
            if (!(members >> member & 1)) return;
            W = __builtin_popcountll(members);
            rank = __builtin_popcountll(members & ((1ull << member) - 1));
        }
    }

    Rows rows;
    rows.init((typename Rows::lds_words)&stage[0], a, chain, n, a.row_table);
    // Samples are counted from the base of an epoch, in the order in which this workgroup looks at them (alone: the stream's).
    // (In a team's kernel they are fewer than 2^30.)
    using Index = std::conditional_t<TEAM, int32_t, int64_t>;
    const Index end = (Index)n;
    uint32_t first_visit = 0;                       // this server's first entry in a table of visits
    if (a.visits_before) {
        first_visit = (uint32_t)a.visits_before[chain];
    } else if (a.visits) {                          // (at most 64 servers: a lane each)
        int sum = lane < chain ? (int)a.n_samples[lane] : 0;
        for (int o = 1; o < kWave; o <<= 1) sum += __shfl_xor(sum, o);
        first_visit = (uint32_t)__builtin_amdgcn_readfirstlane(sum);
    }
    Index base = 0, limit = end, window = -1;
    uint32_t window_rows = 0;
    auto sample_of = [&](Index l) {
        if constexpr (TEAM) return base + (((l >> 2) * W + rank) << 2) + (l & 3);
        else return l;
    };
    // (a team's kernel finds a sample's slot in 32 bits: 128 servers as above 2.48 -> 2.33 ms)
    auto slot_of = [&](Index l) {
        if constexpr (TEAM) return (int64_t)((uint32_t)l % (uint32_t)S);
        else return l;
    };
    auto request = [&](Index l) {
        const Index w = l & ~(Index)(kWave - 1);
        if (w != window) {
            window = w;
            const Index s = sample_of(w + lane);
            window_rows = sample_row(a.seed_lo, a.seed_hi, (uint32_t)chain, (uint64_t)(s < end ? s : end - 1), (uint32_t)a.m);
        }
        const uint32_t row = (uint32_t)__builtin_amdgcn_readlane((int)window_rows, (int)(l & (kWave - 1)));
        const Index s = sample_of(l);
        rows.request_row(slot_of(l), row, a.visits ? first_visit + (uint32_t)(s < end ? s : end - 1) : row);
    };
    // the members' records into LDS, behind the row requests made before
    u32x4 rteam;
    if constexpr (TEAM) {
        const uint64_t at = (uint64_t)(uintptr_t)team;
        rteam[0] = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)at);
        rteam[1] = (uint32_t)__builtin_amdgcn_readfirstlane((int)((uint32_t)(at >> 32) & 0xffffu));
        rteam[2] = 2 * kTeamMax * 8;
        rteam[3] = 0x00020000u;
    }
    typedef __attribute__((address_space(3))) uint32_t *lds_words;
    auto request_records = [&]() {
        const uint32_t pad = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(size_t)(lds_words)&others[0]);
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 3\n\tbuffer_load_dword %1, %2, 0 offen sc1 lds"
                     :
                     : "s"(pad), "v"((uint32_t)lane * 16u + 4u), "s"(rteam)
                     : "memory", "m0");
    };
    if constexpr (TEAM) {
        if (wave == 0) others[lane] = 0;
        limit = W > 1 && kTeamEpoch < end ? kTeamEpoch : end;
    }
    for (Index l = 0; l < S; ++l) request(l);
    int64_t J = 0;
    Index pos = 0;                                  // this workgroup's next sample, counted from the base
    while (TEAM || pos < end) {
        // Batches in which nothing is accepted: the ring does not change in this loop and stays in its registers (with
        // the update as a branch of the same loop the compiler moved the whole ring, 115 registers' worth, every batch).
        double slope = 0.0;
        int taken = B;
        Index stop = limit, at = sample_of(pos);
        while (at < stop) {
            Rows::template wait_for_oldest<B>();        // samples pos .. pos+B-1 have landed
            // Row b of 16 lanes decides sample b: the sums are merged so that w_{J-i}.x_b ends up there, and the
            // decision is straight-line code that all four samples share: a quarter of the decisions' instructions and
            // a third of the sums' (128 servers of up to 8000 samples, rows of 16 KiB: 6.77 -> 4.52 ms; with the ring
            // left in place and the sampler in line 4.19 ms).
            const int mine = lane / 16;
            double v[NV];                               // v[4*i + merged_row(b)] = w_{J-i}.x_b
#pragma unroll
            for (int t = 0; t < NV; ++t) v[t] = 0.0;
#pragma unroll
            for (int b = 0; b < B; ++b) {
                Frag x;
                rows.take(slot_of(pos + b), x);
#pragma unroll
                for (int e = 0; e < EPT; ++e) {
                    const double xe = (double)x.at(e);
#pragma unroll
                    for (int i = 0; i < R1; ++i) v[4 * i + merged_row(b)] += r[i][e] * xe;
                }
            }
            double L[R1];                               // first this wave's sums for sample `mine`, then the workgroup's
            wave_sums_merged(v, L);
            if (lane % 16 == 0) {
#pragma unroll
                for (int i = 0; i < R1; ++i) red[parity][mine * R1 + i][wave] = L[i];
            }
            if constexpr (TEAM) {
                // (Records are those that the batch before asked for: an epoch's first batch has none.  What LDS still holds may be 256
                // epochs old and carry this one's stamp.)
                if (W > 1 && wave == 0) {
                    int whose;
                    const uint32_t first = pos == 0 ? kTeamNone : team_first_found(*(volatile uint32_t *)&others[lane], members >> lane & 1, epoch, whose);
                    if (lane == 0) known[parity] = first;
                }
            }
            const double beta2 = rows.side_f64(slot_of(pos + mine), 0), rate = rows.side_f64(slot_of(pos + mine), 2);     // the row's entry of the table
            const double y = (double)__uint_as_float(rows.side(slot_of(pos + mine), 4));
            __syncthreads();
#pragma unroll
            for (int i = 0; i < R1; ++i) {
                const double *part = red[parity][mine * R1 + i];
                L[i] = ((part[0] + part[1]) + part[2]) + part[3];
            }
            if constexpr (TEAM) {
                if (W > 1) {
                    const uint32_t first = (uint32_t)__builtin_amdgcn_readfirstlane((int)known[parity]);
                    if (first != kTeamNone && base + (Index)first < stop) stop = base + (Index)first;
                }
            }
            parity ^= 1;

            const double yhat = no_delay ? L[0] : L[R1 - 1];
            slope = a.loss == kLossHinge ? loss_slope<kLossHinge>(y, yhat) : loss_slope<kLossLogistic>(y, yhat);
            const bool keep = (at + mine < limit) & window_passes<R1>(L, n2, beta2, rate, J, eta, eta_lambda, yhat, slope);
            // (every lane of a row, and every wave, holds the same sums, hence the same verdict)
            const uint64_t kept = __builtin_amdgcn_ballot_w64(keep);
            taken = kept ? __builtin_ctzll(kept) / 16 : B;          // the first sample of the batch that is accepted
            if (taken < B) break;
            // the slots of the samples left behind take the rows that follow the ones on their way
            Rows::reads_done();
            if constexpr (TEAM) {
                if (W > 1 && wave == 0) request_records();
            }
#pragma unroll
            for (int i = 0; i < B; ++i) request(pos + S + i);
            pos += B;
            at = sample_of(pos);
        }
        const bool alone = !TEAM || W == 1;
        if (alone && taken == B) break;                 // the end of the stream
        Frag x;
        double eg = 0.0;
        if (alone) {
            // w_{J+1} = w_J - eta*lambda*w_{J-tau} - eta*u*x; the row is still in its slot
            eg = eta * lane_read(slope, 16 * taken);
            rows.take(slot_of(pos + taken), x);
        } else if constexpr (TEAM) {
            // The end of an epoch for this member.  verdict[0]: 0 nothing accepted, 1 write the candidate, 2 the same and go on alone,
            // 3 leave, 4 go on alone from the base.
            if (wave == 0) {
                uint64_t bits = (uint64_t)__double_as_longlong(lane_read(slope, 16 * (taken < B ? taken : 0)));
                const uint32_t record = (epoch << 24) | (taken < B ? kTeamFound | (uint32_t)(at + taken - base) : 0u);
                if (lane == 0) {
                    team_store(team + 2 * member, record, (uint32_t)(bits >> 32));
                    team_store(team + 2 * member + 1, record, (uint32_t)bits);
                }
                uint32_t what = 3, first = kTeamNone;
                if (member == 0) {
                    what = 4;
                    for (int tries = 0; tries < kTeamPolls; ++tries) {
                        const uint64_t hi = team_load(team + 2 * lane), lo = team_load(team + 2 * lane + 1);
                        const bool in = members >> lane & 1;
                        const bool ready = (hi >> 56) == (epoch & 255u) && (hi >> 32) == (lo >> 32);
                        if (__builtin_amdgcn_ballot_w64(in && !ready)) {
                            __builtin_amdgcn_s_sleep(1);
                            continue;
                        }
                        int whose;
                        first = team_first_found((uint32_t)(hi >> 32), in, epoch, whose);
                        bits = ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)hi, whose) << 32) |
                               (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)lo, whose);
                        what = first != kTeamNone ? 1 : limit < end ? 0 : 3;
                        if (what == 1 && J + 1 > kTeamSlack + (base + first) / kTeamGap) what = 2;
                        break;
                    }
                    if (lane == 0) team_order(team, what <= 1 ? epoch + 1 : kTeamOver, first, bits);
                } else if (team_await_order(team, epoch + 1, first, bits) != kTeamOver) {
                    what = first != kTeamNone ? 1 : 0;
                }
                if (lane == 0) {
                    verdict[0] = what;
                    verdict[1] = first;
                    verdict[2] = (uint32_t)(bits >> 32);
                    verdict[3] = (uint32_t)bits;
                }
            }
            __syncthreads();
            const uint32_t what = (uint32_t)__builtin_amdgcn_readfirstlane((int)verdict[0]);
            const uint32_t first = (uint32_t)__builtin_amdgcn_readfirstlane((int)verdict[1]);
            const uint64_t bits = ((uint64_t)verdict[2] << 32) | verdict[3];
            __syncthreads();                            // (the verdict may be overwritten from here on)
            if (what == 3) break;
            eg = eta * __longlong_as_double((long long)bits);
            const bool write = what == 1 || what == 2;
            if (write) {
                const uint32_t row = sample_row(a.seed_lo, a.seed_hi, (uint32_t)chain, (uint64_t)(base + first), (uint32_t)a.m);
                const char *at_row = static_cast<const char *>(a.dense) + (int64_t)__builtin_amdgcn_readfirstlane((int)row) * (a.ld * (int64_t)sizeof(TX));
                const __amdgpu_buffer_rsrc_t rx = make_rsrc(at_row, d * (uint32_t)sizeof(TX));
#pragma unroll
                for (int c = 0; c < Frag::kChunks; ++c) x.load_chunk(c, rx, (uint32_t)((c * NT + tid) * VEC) * (uint32_t)sizeof(TX));
                base += (Index)first + 1;
            } else if (what == 0) {
                base = limit;
            }
            if (what == 2 || what == 4) {
                W = 1;
                rank = 0;
            }
            ++epoch;
            pos = 0;
            limit = W > 1 && base + kTeamEpoch < end ? base + kTeamEpoch : end;
            window = -1;
            Rows::reads_done();
            for (Index l = 0; l < S; ++l) request(l);
            if (!write) continue;
        }
        double u2 = 0.0;
#pragma unroll
        for (int e = 0; e < EPT; ++e) {
            const double old = no_delay ? r[0][e] : r[R1 - 1][e];
            const double w = r[0][e] - eta_lambda * old - eg * (double)x.at(e);
#pragma unroll
            for (int i = R1 - 1; i >= 1; --i) r[i][e] = r[i - 1][e];
            r[0][e] = w;
            u2 += w * w;
        }
        block_sum(u2);
#pragma unroll
        for (int i = R1 - 1; i >= 1; --i) n2[i] = n2[i - 1];
        n2[0] = u2;
        ++J;
        if (alone) {
            Rows::reads_done();
            for (int i = 0; i <= taken; ++i) request(pos + S + i);
            pos += taken + 1;
        }
    }
    Rows::drain();
    if (member > 0) return;

    float *out = a.W + (int64_t)chain * a.d;
#pragma unroll
    for (int e = 0; e < EPT; ++e) {
        const uint32_t col = column(e);
        if (col < d) out[col] = (float)r[0][e];
    }
    if (tid == 0) a.accepted[chain] = J;
}

// f(integral_constant<int, 0>) .. f(integral_constant<int, N-1>): a loop whose index is a constant
// expression in its body (register arrays indexed through it are never indexed at run time).
template <int N, typename F, int I = 0>
__device__ inline void static_for(F &&f)
{
    if constexpr (I < N) {
        f(std::integral_constant<int, I>{});
        static_for<N, F, I + 1>(static_cast<F &&>(f));
    }
}

// Without the Check function every sample is an update, and the delay itself gives the parallelism: the
// gradients of the next tau + 1 samples are taken at w_{J-tau} .. w_J, which all exist already.  One
// batch is R1 = tau + 1 samples: R1 projections (sample i on the iterate tau - i back) cross the workgroup
// in one exchange, then R1 updates follow, element by element, with no further exchange.  The ring holds
// exactly R1 iterates, so an update overwrites the oldest one - the very iterate its gradient was taken
// at - and after a whole batch every iterate is back in the registers it started in: slot (i + 1) mod R1
// is both where sample i's gradient is taken and where w_{J+i+1} goes; no register is ever moved.  (Slots
// start as w_0, which is what an iterate before the start means.)  Rows come through LdsRows.
template <typename TX, int EPT, int VEC, int R1, int S>
__global__ __launch_bounds__(kDelayThreads) void delay_server_plain_kernel(DelayArgs a)
{
    constexpr int NT = kDelayThreads, NW = kDelayWaves, B = R1;
    static_assert(R1 >= 2, "a delay of at least one");
    using Rows = LdsRows<TX, EPT, VEC, S, 1>;       // with each row its label
    using Frag = typename Rows::Frag;
    extern __shared__ __attribute__((aligned(16))) uint32_t stage[];     // Rows::kBytes
    __shared__ __attribute__((aligned(16))) double red[2][B][NW];

    const int tid = threadIdx.x;
    const int lane = tid & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int chain = blockIdx.x;
    const int64_t n = a.n_samples[chain];
    const uint32_t d = (uint32_t)a.d;
    const double eta = a.eta, eta_lambda = a.eta * a.lambda;
    int parity = 0;
    auto column = [&](int e) { return (uint32_t)(((e / VEC) * NT + tid) * VEC + e % VEC); };

    double r[R1][EPT];                              // r[p]: the iterate w_t with t mod R1 = p (w_0 before that)
#pragma unroll
    for (int e = 0; e < EPT; ++e) {
        const uint32_t col = column(e);
        const double w = (a.w_start && col < d) ? (double)a.w_start[col] : 0.0;
#pragma unroll
        for (int p = 0; p < R1; ++p) r[p][e] = w;
    }
    int newest = 0;                                 // slot of w_J when the loop ends
    if (n > 0) {
        Rows rows;
        rows.init((typename Rows::lds_words)&stage[0], a, chain, n, a.y);
        for (int64_t s = 0; s < S; ++s) rows.request(s);
        // One batch: J = pos is a multiple of R1, so w_J sits in slot 0.  Only the last batch can be short; the others
        // carry no branch on it (with one, the compiler moved a third of the ring every batch).
        auto batch = [&](int64_t pos, auto last_tag) {
            constexpr bool kLast = decltype(last_tag)::value;
            Rows::template wait_for_oldest<B>();
            double v[B];
            Frag x[B];
            static_for<B>([&](auto ic) {
                constexpr int i = decltype(ic)::value;
                rows.take(pos + i, x[i]);
                v[i] = 0.0;
#pragma unroll
                for (int e = 0; e < EPT; ++e) v[i] += r[(i + 1) % R1][e] * (double)x[i].at(e);
            });
            // Four sums share a register; row merged_row(i mod 4) of 16 lanes takes sample i's slope, all rows at once
            // (128 servers of up to 8000 samples, tau = 2: 4.45 -> 3.63 ms; without the moves of the ring 3.20)
            wave_sums_to_lds<B, NW>(v, &red[parity][0][wave], lane);
            constexpr int Q = (B + 3) / 4;
            double eg[B];
            auto sum_of = [&](int i) {
                const double *part = red[parity][i];
                return ((part[0] + part[1]) + part[2]) + part[3];
            };
            if (B == 2 && a.loss == kLossHinge) {   // (two comparisons: every lane makes both, 128 servers of 600 samples, d = 16: 245 -> 225 us)
                double y[B];
#pragma unroll
                for (int i = 0; i < B; ++i) y[i] = (double)__uint_as_float(rows.side(pos + i, 0));
                __syncthreads();
#pragma unroll
                for (int i = 0; i < B; ++i) eg[i] = eta * loss_slope<kLossHinge>(y[i], sum_of(i));
            } else {
                double y[Q], eg_row[Q];
#pragma unroll
                for (int q = 0; q < Q; ++q) {
                    const int i = 4 * q + merged_row(lane / 16);
                    y[q] = (double)__uint_as_float(rows.side(pos + (i < B ? i : B - 1), 0));
                }
                __syncthreads();
#pragma unroll
                for (int q = 0; q < Q; ++q) {
                    const int i = 4 * q + merged_row(lane / 16);
                    const double sum = sum_of(i < B ? i : B - 1);
                    eg_row[q] = eta * (a.loss == kLossHinge ? loss_slope<kLossHinge>(y[q], sum) : loss_slope<kLossLogistic>(y[q], sum));
                }
#pragma unroll
                for (int i = 0; i < B; ++i) eg[i] = lane_read(eg_row[i / 4], 16 * merged_row(i % 4));
            }
            parity ^= 1;
            // w_{J+i+1} = w_{J+i} - eta*lambda*w_{J+i-tau} - eta*u*x_i, for the samples that exist
            static_for<B>([&](auto ic) {
                constexpr int i = decltype(ic)::value;
                if (!kLast || pos + i < n) {
#pragma unroll
                    for (int e = 0; e < EPT; ++e)
                        r[(i + 1) % R1][e] = r[i % R1][e] - eta_lambda * r[(i + 1) % R1][e] - eg[i] * (double)x[i].at(e);
                    if (kLast) newest = (i + 1) % R1;
                }
            });
            if constexpr (!kLast) {
                Rows::reads_done();
#pragma unroll
                for (int i = 0; i < B; ++i) rows.request(pos + S + i);
            }
        };
        int64_t pos = 0;
        for (; pos + B < n; pos += B) batch(pos, std::false_type{});
        batch(pos, std::true_type{});               // 1 .. B samples
        Rows::drain();
    }

    float *out = a.W + (int64_t)chain * a.d;
    static_for<R1>([&](auto pc) {                   // (a branch per slot: the ring is never indexed at run time)
        constexpr int p = decltype(pc)::value;
        if (newest == p) {
#pragma unroll
            for (int e = 0; e < EPT; ++e) {
                const uint32_t col = column(e);
                if (col < d) out[col] = (float)r[p][e];
            }
        }
    });
    if (tid == 0) a.accepted[chain] = n > 0 ? n : 0;
}

constexpr int kDelayRegMaxTau = 4;
constexpr int kDelayAhead = 4;          // samples whose rows are in flight
constexpr int kDelayBatch = 4;          // samples looked at side by side under Check
constexpr int kDelaySlots = 8;          // rows in LDS or on their way there

template <typename TX, int EPT, int VEC, int R1>
void launch_sample(const DelayArgs &a, hipStream_t s)
{
    if (a.check)
        hipLaunchKernelGGL((delay_server_reg_kernel<TX, EPT, VEC, R1, kDelayAhead, true>), dim3(a.k), dim3(kDelayThreads), 0, s, a);
    else
        hipLaunchKernelGGL((delay_server_reg_kernel<TX, EPT, VEC, R1, kDelayAhead, false>), dim3(a.k), dim3(kDelayThreads), 0, s, a);
}

// A call with teams wants its members seated together: an owner whose members start late goes on alone.  So launches with teams
// that do not fit on the device side by side run in turn, on whatever streams this process queues them: what went before is waited
// for, from the newest launch that leaves no room on.  (us, two calls on two streams, fp32, up to 8000 samples a server: without teams | with
// teams, as they come | in turn: d = 4096, 128 servers 4587 | 6013 | 4374, 64 servers 4302 | 5184 | 2100; d = 1024, up to 4000, 128 servers 1939 | 1968 |
// 1371.  One call: 4162 | 2207 | 2160, 4098 | 1073 | 1060, 1480 | 708 | 700.)  The rule for which launches it is worth stands with the teams' sizes.
// An order for the sake of time only: where an event fails, and under stream capture, launches go without.
struct TeamLaunches {
    static constexpr int kMaxDevices = 64, kKept = 8;
    struct Launch {
        hipEvent_t done;
        hipStream_t stream;
        int workgroups;                             // 0: none
    };
    std::mutex lock;
    Launch kept[kMaxDevices][kKept] = {};           // the latest launches, the next one goes to kept[next]
    int next[kMaxDevices] = {};
};
TeamLaunches g_team_launches;

template <typename F>
hipError_t launch_in_turn(const DelayArgs &a, hipStream_t s, F &&launch)
{
    int dev = 0;
    hipStreamCaptureStatus capturing = hipStreamCaptureStatusNone;
    if (!a.in_turn) {
        launch(nullptr);
        return hipGetLastError();
    }
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= TeamLaunches::kMaxDevices ||
        hipStreamIsCapturing(s, &capturing) != hipSuccess || capturing != hipStreamCaptureStatusNone) {
        (void)hipGetLastError();
        launch(nullptr);
        return hipGetLastError();
    }
    using Turns = TeamLaunches;
    std::lock_guard<std::mutex> guard(g_team_launches.lock);
    Turns::Launch(&kept)[Turns::kKept] = g_team_launches.kept[dev];
    int &next = g_team_launches.next[dev];
    bool ok = true;
    int beside = a.k + a.helpers;                   // workgroups that may run at once
    for (int i = 1; i <= Turns::kKept; ++i) {       // newest first; the oldest makes room for this one
        Turns::Launch &l = kept[(next + Turns::kKept - i) % Turns::kKept];
        if (l.workgroups == 0 || l.stream == s) continue;
        beside += l.workgroups;
        if (beside > a.units || i == Turns::kKept) ok = ok && hipStreamWaitEvent(s, l.done, 0) == hipSuccess;
    }
    Turns::Launch &mine = kept[next];
    mine.workgroups = 0;
    if (!mine.done) ok = ok && hipEventCreateWithFlags(&mine.done, hipEventDisableTiming | hipEventDisableSystemFence) == hipSuccess;
    if (!ok) (void)hipGetLastError();
    launch(ok ? mine.done : nullptr);               // (an event of the kernel's own: recorded behind it, it cost a call 1.5 us more)
    const hipError_t launched = hipGetLastError();
    if (ok && launched == hipSuccess) {
        mine.stream = s;
        mine.workgroups = a.k + a.helpers;
        next = (next + 1) % Turns::kKept;
    }
    return launched;
}

// The batch kernel claims S row slots of LDS, which is more than a kernel may have without asking.
template <typename TX, int EPT, int VEC, int R1, bool TEAM>
bool launch_batch(const DelayArgs &a, hipStream_t s, hipError_t *launched)
{
    auto kernel = delay_server_batch_kernel<TX, EPT, VEC, R1, kDelayBatch, kDelaySlots, TEAM>;
    // (members of teams get a compute unit each: more than half of its LDS)
    constexpr size_t rows = LdsRows<TX, EPT, VEC, kDelaySlots, 8>::kBytes, bytes = TEAM && rows < 84 * 1024 ? 84 * 1024 : rows;
    static std::atomic<int> allowed{0};             // 0 not asked yet, 1 granted, -1 refused (asking twice is harmless)
    int may = allowed.load(std::memory_order_relaxed);
    if (may == 0) {
        may = hipFuncSetAttribute(reinterpret_cast<const void *>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize,
                                  (int)bytes) == hipSuccess ? 1 : -1;
        if (may < 0) (void)hipGetLastError();
        allowed.store(may, std::memory_order_relaxed);
    }
    if (may < 0) return false;                      // the per-sample kernel serves instead
    // what depends on a row alone, once per row or visit
    const int64_t entries = a.visits ? a.visits : a.m;
    hipLaunchKernelGGL((delay_row_table_kernel<TX, VEC>), dim3((unsigned)((entries + kDelayWaves - 1) / kDelayWaves)), dim3(kDelayThreads),
                       0, s, a, static_cast<DelayRowEntry *>(a.row_table), R1 - 1);
    *launched = hipGetLastError();
    if (*launched != hipSuccess) return true;
    if constexpr (TEAM) {
        *launched = launch_in_turn(a, s, [&](hipEvent_t done) {
            hipExtLaunchKernelGGL(kernel, dim3(a.k + a.helpers), dim3(kDelayThreads), bytes, s, nullptr, done, 0, a);
        });
    } else {
        hipLaunchKernelGGL(kernel, dim3(a.k), dim3(kDelayThreads), bytes, s, a);
        *launched = hipGetLastError();
    }
    return true;
}

template <typename TX, int EPT, int VEC, int R1>
bool launch_plain(const DelayArgs &a, hipStream_t s)
{
    auto kernel = delay_server_plain_kernel<TX, EPT, VEC, R1, kDelaySlots>;
    constexpr size_t bytes = LdsRows<TX, EPT, VEC, kDelaySlots, 1>::kBytes;
    static std::atomic<int> allowed{0};
    int may = allowed.load(std::memory_order_relaxed);
    if (may == 0) {
        may = hipFuncSetAttribute(reinterpret_cast<const void *>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize,
                                  (int)bytes) == hipSuccess ? 1 : -1;
        if (may < 0) (void)hipGetLastError();
        allowed.store(may, std::memory_order_relaxed);
    }
    if (may < 0) return false;
    hipLaunchKernelGGL(kernel, dim3(a.k), dim3(kDelayThreads), bytes, s, a);
    return true;
}

// Launches the register kernel if one is built for this shape; *done tells.  staged: rows are whole 16-byte
// pieces, which the kernels that stage them in LDS want; the per-sample kernel only needs dwords.
template <typename TX, int VEC>
hipError_t launch_reg(const DelayArgs &a, bool staged, hipStream_t s, bool *done)
{
    hipError_t e = hipSuccess;
    const int r1 = (a.tau > 1 ? a.tau : 1) + 1;
    *done = true;
#define WPSGD_DELAY_REG(EPT, R1)                                                                                 \
    if (a.d <= (int64_t)kDelayThreads * EPT && r1 == R1) {                                                       \
        if (a.check && staged && a.row_table && a.m < (1 << 27) &&                                               \
            (a.team ? launch_batch<TX, EPT, VEC, R1, true>(a, s, &e) : launch_batch<TX, EPT, VEC, R1, false>(a, s, &e))) \
            return e;                                                                                            \
        else if (!a.check && staged && a.tau >= 1 && a.m < (1 << 30) && launch_plain<TX, EPT, VEC, R1>(a, s))    \
            return hipGetLastError();                                                                            \
        else                                                                                                     \
            launch_sample<TX, EPT, VEC, R1>(a, s);                                                               \
        return hipGetLastError();                                                                                \
    }
    WPSGD_DELAY_REG(8, 2) WPSGD_DELAY_REG(8, 3) WPSGD_DELAY_REG(8, 4) WPSGD_DELAY_REG(8, 5)
    WPSGD_DELAY_REG(16, 2) WPSGD_DELAY_REG(16, 3) WPSGD_DELAY_REG(16, 4) WPSGD_DELAY_REG(16, 5)
#undef WPSGD_DELAY_REG
    *done = false;
    return hipSuccess;
}

// bfloat16 rows that are no whole 16-byte pieces: the per-sample kernel with a load per element (81 servers of 400 samples, d = 301,
// tau = 0, without Check: 216 us, 1024 with the ring in memory; 30 of up to 1000, d = 4001, tau = 4, under it: 1.62 ms, 15.2).
hipError_t launch_reg_elements(const DelayArgs &a, hipStream_t s, bool *done)
{
    const int r1 = (a.tau > 1 ? a.tau : 1) + 1;
    *done = true;
#define WPSGD_DELAY_REG(EPT, R1)                                                                                 \
    if (a.d <= (int64_t)kDelayThreads * EPT && r1 == R1) {                                                       \
        launch_sample<uint16_t, EPT, 1, R1>(a, s);                                                               \
        return hipGetLastError();                                                                                \
    }
    WPSGD_DELAY_REG(2, 2) WPSGD_DELAY_REG(2, 3) WPSGD_DELAY_REG(2, 4) WPSGD_DELAY_REG(2, 5)
    WPSGD_DELAY_REG(8, 2) WPSGD_DELAY_REG(8, 3) WPSGD_DELAY_REG(8, 4) WPSGD_DELAY_REG(8, 5)
    WPSGD_DELAY_REG(16, 2) WPSGD_DELAY_REG(16, 3) WPSGD_DELAY_REG(16, 4) WPSGD_DELAY_REG(16, 5)
#undef WPSGD_DELAY_REG
    *done = false;
    return hipSuccess;
}

template <typename TX, int VEC>
hipError_t launch_reach(const DelayArgs &a, hipStream_t s)
{
    const int need = (a.tau > 1 ? a.tau : 1) + 1;
#define WPSGD_DELAY_TRY(MAXW)                                                                                   \
    if (need <= MAXW) {                                                                                         \
        hipLaunchKernelGGL((delay_server_kernel<TX, VEC, MAXW>), dim3(a.k), dim3(kDelayThreads), 0, s, a);      \
        return hipGetLastError();                                                                               \
    }
    WPSGD_DELAY_TRY(3)
    WPSGD_DELAY_TRY(5)
    WPSGD_DELAY_TRY(kDelayMaxTau + 1)
#undef WPSGD_DELAY_TRY
    return hipErrorInvalidValue;
}

}  // namespace

hipError_t launch_delay_servers(const DelayArgs &a, int dtype, int vec, int buffer_vec, hipStream_t s)
{
    if (a.tau <= kDelayRegMaxTau && (buffer_vec > 1 || dtype == WPSGD_BF16) && a.d * (dtype == WPSGD_BF16 ? 2 : 4) < (int64_t)1 << 31) {
        bool done = false;
        const hipError_t e = buffer_vec == 1 ? launch_reg_elements(a, s, &done)
                             : dtype == WPSGD_BF16 ? launch_reg<uint16_t, 8>(a, vec > 1, s, &done)
                                                 : launch_reg<float, 4>(a, vec > 1, s, &done);
        if (done) return e;
    }
    if (dtype == WPSGD_BF16) return vec > 1 ? launch_reach<uint16_t, 8>(a, s) : launch_reach<uint16_t, 1>(a, s);
    return vec > 1 ? launch_reach<float, 4>(a, s) : launch_reach<float, 1>(a, s);
}

}  // namespace wpsgd
