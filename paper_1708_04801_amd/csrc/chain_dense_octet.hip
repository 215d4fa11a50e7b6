// Dense logistic chains with compute units to spare, eight steps at a time; the products between rows come from other workgroups.
//
// For the eight rows x_0..x_7 of a block and the vector v at its start,
//     yhat_j = s_j * (v.x_j + sum_{a<j} c_a x_a.x_j),   c_a = -eta*g_a / s_{a+1}:
// eight dot products, one exchange between the waves, eight slopes that wait for each other (one multiply-add across eight lanes each)
// and one update of v, instead of an exchange every step or two.  The 28 products between the rows of a block do not depend on v: helper
// workgroups on compute units no chain occupies form them some blocks ahead (which also brings the rows into the cache all compute units of
// an XCD share) and leave them in a ring in memory, each number with its block's stamp in one 64-bit word.  The chain asks for a
// block's record a block ahead.  It never waits for one: where a record is not there yet it forms the same products from the rows it
// holds, with the same code and in the same order, so results do not depend on who was faster.
//
// A chain's workgroup: NT threads hold v and two blocks of rows in registers (element e of a thread is column ((e/VEC)*NT + tid)*VEC + e%VEC), and
// one more wave, the clerk, fetches records and prepares blocks.  The clerk is a wave of its own because loads return in order: a wave that waits
// for a record waits for every row it requested before.
//
// What bounds it: instruction issue of one wave per SIMD (some 300 instructions a block) and eight dependent slopes of some 60 cycles.  us per step,
// sixteen chains, two-step rounds (chain_dense_reg.hip) -> this: fp32 d = 1024 0.1445 -> 0.1115; bf16 d = 1024 0.167 -> 0.128,
// d = 2048 0.175 -> 0.128.  Longer fp32 rows gain little or lose (d = 2048 0.170 -> 0.154 with sixteen chains, 0.173 -> 0.179 with 64; d = 4096 takes
// 0.213 from cached rows alone, what the two-step rounds take with everything).  The eight steps' sum is added to v at once: error against fp64 0.35 of
// what it was (d = 1024, 4000 steps: 1.03e-6 -> 3.5e-7).
#include "device_utils.h"
#include "dense_rows.h"
#include "internal.h"
#include "step_rows.h"

namespace wpsgd {
namespace {

constexpr int kOctet = 8;                             // steps per block
constexpr int kPairs = kOctet * (kOctet - 1) / 2;     // products between its rows: of rows j > t at j(j-1)/2 + t
constexpr int kOctetsPerWindow = kWave / kOctet;
constexpr int kHelperLooks = 1 << 15;                 // (0.4 us each: a sleep of 256 cycles, a load from memory and a barrier)
constexpr uint32_t kLdsClaim = 84 * 1024;             // more than half a compute unit's: helpers stay off the chains' compute units

template <typename TX, int NT, int EPT>
struct OctetRows {
    static constexpr int VEC = 16 / (int)sizeof(TX), CH = EPT / VEC;
    static_assert(EPT % VEC == 0, "whole 16-byte loads");
    u32x4 q[kOctet][CH];

    // base: per lane, the address of the row of a window's step
    __device__ void request(uint64_t base, uint32_t row_bytes, int first)
    {
#pragma unroll
        for (int t = 0; t < kOctet; ++t) {
            const __amdgpu_buffer_rsrc_t rx = make_rsrc(reinterpret_cast<const void *>(lane_read_i64((int64_t)base, first + t)), row_bytes);
#pragma unroll
            for (int c = 0; c < CH; ++c) q[t][c] = __builtin_amdgcn_raw_buffer_load_b128(rx, (uint32_t)((c * NT + (int)threadIdx.x) * 16), 0, 0);
        }
    }
    __device__ float at(int t, int e) const
    {
        const uint32_t w = q[t][e / VEC][(e % VEC) * (int)sizeof(TX) / 4];
        if constexpr (sizeof(TX) == 4) return __uint_as_float(w);
        else return (e & 1) ? bf16_hi(w) : bf16_lo(w);
    }
};

enum : uint32_t { kMissing = 0, kThere = 1, kOdd = 2 };

template <int NW>
struct OctetLds {
    float dots[2][kOctet][NW];                // the waves' shares of v.x_j
    float own[2][kOctet][kOctet];             // [j][t], t < j: what a unit of slope of step t adds to q_j; zero elsewhere
    float zs[2][kOctet], cs[2][kOctet];       // y_j s_j log2 e, y_j eta / s_{j+1} (0 past the chain's end)
    uint32_t state[2];                        // are the block's products there, and all finite?
    float part[2][NW][32];                    // the waves' shares of the products between rows
    float sums[2][NW];                        // one step at a time: the waves' shares of v.x
    uint32_t seen[2];                         // helpers: blocks the chain has done
};

// one ring of records per chain
__device__ inline unsigned long long *record_of(const ChainArgs &a, int cb, int64_t b)
{
    return static_cast<unsigned long long *>(a.xchg) + ((size_t)cb * kOctetRingRecords + (size_t)(b % kOctetRingRecords)) * 32;
}

// How many blocks a chain has done, in a line of its own among the helpers' (the last words of its ring, which no record fills: with all
// chains' counters side by side their helpers' looks at them queue up, 0.26 us per step instead of 0.12 with sixteen chains).
__device__ inline uint32_t *progress_of(const ChainArgs &a, int cb) { return reinterpret_cast<uint32_t *>(record_of(a, cb, kOctetRingRecords - 1) + 31); }

// this wave's shares of the products between a block's rows
template <typename TX, int NT, int EPT>
__device__ inline void wave_products(const OctetRows<TX, NT, EPT> &x, float *part, int lane)
{
    float acc[kPairs], t[kPairs / 4];
#pragma unroll
    for (int p = 0; p < kPairs; ++p) acc[p] = 0.0f;
#pragma unroll
    for (int e = 0; e < EPT; ++e)
#pragma unroll
        for (int j = 1; j < kOctet; ++j)
#pragma unroll
            for (int i = 0; i < j; ++i) acc[j * (j - 1) / 2 + i] = __builtin_fmaf(x.at(j, e), x.at(i, e), acc[j * (j - 1) / 2 + i]);
    wave_sums_merged<float, kPairs>(acc, t);
    if (lane % 16 == 0) {
#pragma unroll
        for (int q = 0; q < kPairs / 4; ++q) part[4 * q + merged_row(lane / 16)] = t[q];
    }
}
template <int NW>
__device__ inline float product_of(const float (&part)[NW][32], int pair)
{
    float s = part[0][pair];
#pragma unroll
    for (int w = 1; w < NW; ++w) s += part[w][pair];
    return s;
}

__device__ inline void beat_barrier()         // everything this wave wrote to LDS is there before it arrives
{
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

// Helper q of a chain's Q forms the products of blocks q+1, q+1+Q, ...; it leaves out those the chain is about to form itself, stays
// `lead` blocks ahead at most (so that the rows are still cached when the chain asks for them), and ends when the chain has ended, or has
// not moved for kHelperLooks looks (13 ms; a block takes the chain a microsecond).  Its last wave watches the chain, adds up the others' shares and writes the records.
template <typename TX, int NT, int EPT>
__device__ inline void help(const ChainArgs &a, OctetLds<NT / kWave> &lds, int cb, int q, int Q)
{
    constexpr int NW = NT / kWave;
    const int tid = (int)threadIdx.x, lane = tid & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int64_t n = a.nsteps[cb], nblk = (n + kOctet - 1) / kOctet;
    const uint32_t base = (uint32_t)(a.span * (nblk + 1));
    const int lead = min(Q + 4, kOctetRingRecords - 1);
    int64_t cur = 1 + q;
    if (cur >= nblk) return;
    int polls = kHelperLooks;                 // every look while too far ahead draws on this, until the chain moves
    int64_t seen = 0, nxt = cur + Q;
    int parity = 0;
    // All waves of the workgroup take the same decisions from what the last wave has seen.
    auto look = [&]() {
        beat_barrier();
        const int64_t now = max((int)((uint32_t)__builtin_amdgcn_readfirstlane((int)lds.seen[parity]) - base), 0);
        if (now > seen) polls = kHelperLooks;
        seen = now;
        parity ^= 1;
    };
    auto far_ahead = [&]() { return nxt < nblk && nxt > seen + lead; };
    auto go_on = [&]() {
        if (nxt >= nblk) return false;
        cur = nxt;
        nxt += Q;
        if (nxt < seen + 3) nxt += (seen + 3 - nxt + Q - 1) / Q * Q;
        return true;
    };
    if (wave == NW) {
        uint32_t *progress = progress_of(a, cb);
        auto report = [&]() {
            const uint32_t now = __hip_atomic_load(progress, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (lane == 0) lds.seen[parity] = now;
        };
        for (;;) {
            while (far_ahead()) {
                if (--polls < 0) return;
                __builtin_amdgcn_s_sleep(4);
                report();
                look();
            }
            report();
            const int mine = parity;
            look();
            if (lane < kPairs) {
                const unsigned long long word = ((unsigned long long)(base + (uint32_t)cur + 1u) << 32) | __float_as_uint(product_of(lds.part[mine], lane));
                __hip_atomic_store(record_of(a, cb, cur) + lane, word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
            if (!go_on()) return;
        }
    }
    StepRows steps;
    steps.init(a, cb, lane);
    const int64_t row_stride = a.ld * (int64_t)sizeof(TX);
    const uint32_t row_bytes = (uint32_t)(a.d * (int64_t)sizeof(TX));
    int64_t window = -1;
    uint64_t rows = 0;
    auto request = [&](OctetRows<TX, NT, EPT> &x, int64_t b) {
        if (b / kOctetsPerWindow != window) {
            window = b / kOctetsPerWindow;
            rows = (uint64_t)(uintptr_t)a.dense + (uint64_t)steps.at(min(window * kWave + lane, n - 1)) * (uint64_t)row_stride;
        }
        x.request(rows, row_bytes, (int)(b % kOctetsPerWindow) * kOctet);
    };
    // false: nothing is left to do
    auto beat = [&](OctetRows<TX, NT, EPT> &now, OctetRows<TX, NT, EPT> &then) {
        while (far_ahead()) {
            if (--polls < 0) return false;
            look();
        }
        request(then, min(nxt, nblk - 1));
        wave_products(now, lds.part[parity][wave], lane);
        look();
        return go_on();
    };
    OctetRows<TX, NT, EPT> one, two;
    request(one, cur);
    while (beat(one, two) && beat(two, one)) {}
}

// The last wave of a chain's workgroup prepares a block while the others are at the one before: fetches its record, multiplies the products with
// everything known beforehand, and says how far the chain has come.  (Its waits are its own: the others' wait for their rows only.)
template <int NW>
__device__ inline void clerk(const ChainArgs &a, OctetLds<NW> &lds, int cb, int64_t n, int64_t nblk, uint32_t base, int lane)
{
    StepRows steps;
    steps.init(a, cb, lane);
    const double rho64 = a.pow_tab[kWave - 1] * a.rho, inv_rho64 = a.pow_tab[2 * kWave - 1];
    const double up = a.pow_tab[lane], down = a.pow_tab[kWave + lane];
    int pj = 1;                               // this lane's pair of rows
#pragma unroll
    for (int r = 2; r < kOctet; ++r) pj += lane >= r * (r - 1) / 2 ? 1 : 0;
    const int pt = lane < kPairs ? lane - pj * (pj - 1) / 2 : 0;
    double s_w = 1.0, eos_w = a.eta;
    float zs = 0.0f, cs = 0.0f;               // of the window's step in this lane
    float y_next = a.y[steps.at(min((int64_t)lane, n - 1))];
    auto fetch = [&](int64_t b) { return __hip_atomic_load(record_of(a, cb, b) + (lane < kPairs ? lane : 0), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); };
    auto complete = [&](unsigned long long r, int64_t b) {
        return __builtin_amdgcn_ballot_w64(lane >= kPairs || (uint32_t)(r >> 32) == base + (uint32_t)b + 1u) == ~0ull;
    };
    // leaves the block's products in LDS, given what they are before scaling
    auto hand_out = [&](int64_t b, float p) {
        const int first = (int)(b % kOctetsPerWindow) * kOctet, buf = (int)(b & 1);
        const float own = p * (__shfl(zs, first + pj) * __shfl(cs, first + pt));
        if (lane < kPairs) lds.own[buf][pj][pt] = own;
        const bool odd = __builtin_amdgcn_ballot_w64(lane < kPairs && !(__builtin_fabsf(own) < __builtin_inff())) != 0;
        if (lane == 0) lds.state[buf] = odd ? kOdd : kThere;
    };
    unsigned long long record = fetch(0);
    for (int64_t b = 0;; ++b) {
        // block b is prepared (behind the last: nobody looks)
        const int first = (int)(b % kOctetsPerWindow) * kOctet, buf = (int)(b & 1);
        if (first == 0) {                     // a new window
            if (b > 0) {
                s_w *= rho64;
                eos_w *= inv_rho64;
                if (s_w < 0x1p-30) {          // (the waves that hold v fold it there)
                    s_w = 1.0;
                    eos_w = a.eta;
                }
            }
            const double y = (double)y_next;
            zs = (float)(s_w * up * y * 1.4426950408889634);
            cs = b * kOctet + lane < n ? (float)(eos_w * down * y) : 0.0f;
            y_next = a.y[steps.at(min((b + kOctetsPerWindow) * kOctet + lane, n - 1))];
        }
        const float z = __shfl(zs, first + lane % kOctet), c = __shfl(cs, first + lane % kOctet);
        if (lane < kOctet) {
            lds.zs[buf][lane] = z;
            lds.cs[buf][lane] = c;
        }
        if (!complete(record, b)) record = fetch(b);
        if (complete(record, b)) hand_out(b, __uint_as_float((uint32_t)record));
        else if (lane == 0) lds.state[buf] = kMissing;
        record = fetch(b + 1);
        if (lane == 0 && b > 0) __hip_atomic_store(progress_of(a, cb), base + (uint32_t)b - 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        beat_barrier();
        if (b >= nblk) return;
        uint32_t state = (uint32_t)__builtin_amdgcn_readfirstlane((int)lds.state[buf]);
        if (state == kMissing) {              // the others form them
            beat_barrier();
            hand_out(b, product_of(lds.part[buf], lane < kPairs ? lane : 0));
            beat_barrier();
            state = (uint32_t)__builtin_amdgcn_readfirstlane((int)lds.state[buf]);
        }
        if (state == kOdd) return;
    }
}

template <typename TX, int NT, int EPT>
__global__ __launch_bounds__(NT + kWave) void chain_dense_octet_kernel(ChainArgs a)
{
    constexpr int NW = NT / kWave;
    constexpr int VEC = OctetRows<TX, NT, EPT>::VEC;
    extern __shared__ __attribute__((aligned(16))) uint8_t lds_raw[];
    OctetLds<NW> &lds = *reinterpret_cast<OctetLds<NW> *>(lds_raw);
    const int tid = (int)threadIdx.x, lane = tid & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);

    // Workgroups go to the XCDs in turn: a chain's helpers are a multiple of eight behind it, so that they share its XCD's cache.
    const int seats = (a.k + 7) & ~7;
    if ((int)blockIdx.x >= seats) {
        const int h = (int)blockIdx.x - seats, cb = h % seats;
        if (cb < a.k) help<TX, NT, EPT>(a, lds, cb, h / seats, a.helpers / a.k);
        return;
    }
    const int cb = (int)blockIdx.x;
    if (cb >= a.k) return;

    const int64_t n = a.nsteps[cb];
    const int d = (int)a.d;
    float *out = a.W + (int64_t)a.order[cb] * a.d;
    auto column = [&](int e) { return ((e / VEC) * NT + tid) * VEC + e % VEC; };
    if (n == 0) {
        for (int c = tid; c < d; c += NT + kWave) out[c] = a.w_start ? a.w_start[c] : 0.0f;
        return;
    }
    const int64_t nblk = (n + kOctet - 1) / kOctet;
    const uint32_t base = (uint32_t)(a.span * (nblk + 1));
    for (int i = tid; i < 2 * kOctet * kOctet; i += NT + kWave) (&lds.own[0][0][0])[i] = 0.0f;
    beat_barrier();
    if (wave == NW) {
        clerk<NW>(a, lds, cb, n, nblk, base, lane);
        if (lane == 0) __hip_atomic_store(progress_of(a, cb), base + (uint32_t)nblk, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }

    float v[EPT];
#pragma unroll
    for (int e = 0; e < EPT; ++e) v[e] = (a.w_start && column(e) < d) ? a.w_start[column(e)] : 0.0f;
    const double rho64 = a.pow_tab[kWave - 1] * a.rho, inv_rho64 = a.pow_tab[2 * kWave - 1];
    StepRows steps;
    steps.init(a, cb, lane);
    const char *X = static_cast<const char *>(a.dense);
    const int64_t row_stride = a.ld * (int64_t)sizeof(TX);
    const uint32_t row_bytes = (uint32_t)(a.d * (int64_t)sizeof(TX));
    const int j = lane % kOctet;
    double s_w = 1.0, eos_w = a.eta;
    int64_t b = 0;
    if (wave < NW) {
        auto addresses = [&](int64_t window) {
            return (uint64_t)(uintptr_t)X + (uint64_t)steps.at(min(window * kWave + lane, n - 1)) * (uint64_t)row_stride;
        };
        uint64_t rows = addresses(0);         // of the window the requests are in
        OctetRows<TX, NT, EPT> x[2];
        x[0].request(rows, row_bytes, 0);
        __builtin_amdgcn_sched_barrier(0);    // in this order: so the wait for a block is not one for the next
        x[1].request(rows, row_bytes, kOctet);
        beat_barrier();                       // block 0 is prepared
        // Block b's products in LDS, formed here if need be.  False: they are not all finite, or the chain has ended.  (The only way out of the
        // loop, behind a block's requests: on every path the compiler then sees how many loads came after the ones it waits for.)
        auto ready = [&](OctetRows<TX, NT, EPT> &x_b) {
            uint32_t state = (uint32_t)__builtin_amdgcn_readfirstlane((int)lds.state[b & 1]);
            const bool more = b < nblk;
            if (more && state == kMissing) {
                wave_products(x_b, lds.part[b & 1][wave], lane);
                beat_barrier();
                beat_barrier();               // the clerk has handed them out
                state = (uint32_t)__builtin_amdgcn_readfirstlane((int)lds.state[b & 1]);
            }
            return more && state != kOdd;
        };
        auto beat = [&](OctetRows<TX, NT, EPT> &now) {
            const int buf = (int)(b & 1);
            float own[kOctet];
#pragma unroll
            for (int r = 0; r < kOctet; ++r) own[r] = lds.own[buf][j][r];
            const float z = lds.zs[buf][j], mine = lds.cs[buf][j];
            float p[kOctet], t[2];
#pragma unroll
            for (int r = 0; r < kOctet; ++r) p[r] = 0.0f;
#pragma unroll
            for (int e = 0; e < EPT; ++e)
#pragma unroll
                for (int r = 0; r < kOctet; ++r) p[r] = __builtin_fmaf(v[e], now.at(r, e), p[r]);
            wave_sums_merged<float, kOctet>(p, t);
            if (lane % 16 < 2) lds.dots[buf][4 * (lane % 16) + merged_row(lane / 16)][wave] = lane % 16 == 0 ? t[0] : t[1];
            beat_barrier();                   // (and block b+1 is prepared)
            float dot[NW], c[kOctet];
#pragma unroll
            for (int w = 0; w < NW; ++w) dot[w] = lds.dots[buf][j][w];
#pragma unroll
            for (int w = 1; w < NW; w *= 2)
#pragma unroll
                for (int i = 0; i + w < NW; i += 2 * w) dot[i] += dot[i + w];
            float q = z * dot[0];
            const float slope = mine * take_block_steps<kLossLogistic>(q, own);
#pragma unroll
            for (int r = 0; r < kOctet; ++r) c[r] = lane_read(slope, r);
            // (the eight steps' sum first, then one addition to v: one rounding at v's size instead of eight)
#pragma unroll
            for (int e = 0; e < EPT; ++e) {
                float sum = c[0] * now.at(0, e);
#pragma unroll
                for (int r = 1; r < kOctet; ++r) sum = __builtin_fmaf(c[r], now.at(r, e), sum);
                v[e] += sum;
            }
            const int ahead = (int)((b + 2) % kOctetsPerWindow);
            if (ahead == 0) rows = addresses((b + 2) / kOctetsPerWindow);
            now.request(rows, row_bytes, ahead * kOctet);
            ++b;
            if (b % kOctetsPerWindow == 0 && b < nblk) {      // a new window
                s_w *= rho64;
                eos_w *= inv_rho64;
                if (s_w < 0x1p-30) {
#pragma unroll
                    for (int e = 0; e < EPT; ++e) v[e] *= (float)s_w;
                    s_w = 1.0;
                    eos_w = a.eta;
                }
            }
        };
        bool on = ready(x[0]);
        while (on) {
            beat(x[0]);
            if (!ready(x[1])) break;
            beat(x[1]);
            on = ready(x[0]);
        }
    }
    if (wave == NW) {                         // the clerk leaves when the others have done the last block, or meet an odd one
        return;
    }
    if (b < nblk) {
        // The block has a row that is not finite (or so large that a product, with its coefficient, is not).  Two terms of an infinite product
        // may have different signs, so products must not be split: from here on, on data no model is learnt from, one step is taken after the other.
        for (int64_t t = b * kOctet; t < n; ++t) {
            if (t % kWave == 0 && t > b * kOctet) {
                s_w *= rho64;
                eos_w *= inv_rho64;
                if (s_w < 0x1p-30) {
#pragma unroll
                    for (int e = 0; e < EPT; ++e) v[e] *= (float)s_w;
                    s_w = 1.0;
                    eos_w = a.eta;
                }
            }
            const uint32_t row = steps.at(t);
            const TX *at = reinterpret_cast<const TX *>(X + (int64_t)row * row_stride);
            float p = 0.0f;
#pragma unroll
            for (int e = 0; e < EPT; ++e) {
                float xe = 0.0f;
                if (column(e) < d) {
                    if constexpr (sizeof(TX) == 2) xe = bf16_one(at[column(e)]);
                    else xe = at[column(e)];
                }
                p += v[e] * xe;
            }
            p = wave_sum(p);
            if (lane == 0) lds.sums[t & 1][wave] = p;
            beat_barrier();
            p = lds.sums[t & 1][0];
#pragma unroll
            for (int w = 1; w < NW; ++w) p += lds.sums[t & 1][w];
            const int l = (int)(t % kWave);
            const double y = (double)a.y[row];
            const float ct = (float)(eos_w * a.pow_tab[kWave + l] * y) * unit_slope<kLossLogistic>((float)(s_w * a.pow_tab[l] * y * 1.4426950408889634) * p);
#pragma unroll
            for (int e = 0; e < EPT; ++e) {
                float xe = 0.0f;
                if (column(e) < d) {
                    if constexpr (sizeof(TX) == 2) xe = bf16_one(at[column(e)]);
                    else xe = at[column(e)];
                }
                v[e] += ct * xe;
            }
        }
    }
    const double s_end = s_w * a.pow_tab[(n - 1) % kWave] * a.rho;
#pragma unroll
    for (int e = 0; e < EPT; ++e)
        if (column(e) < d) out[column(e)] = (float)(s_end * (double)v[e]);
}

template <typename TX, int NT, int EPT>
hipError_t launch(const ChainArgs &a, hipStream_t s)
{
    auto kernel = chain_dense_octet_kernel<TX, NT, EPT>;
    static_assert(sizeof(OctetLds<NT / kWave>) <= kLdsClaim, "the tables fit the claim");
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, (int)kLdsClaim);
    if (e != hipSuccess) return e;
    const int seats = (a.k + 7) & ~7;
    hipLaunchKernelGGL(kernel, dim3(seats * (1 + a.helpers / a.k)), dim3(NT + kWave), kLdsClaim, s, a);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_dense_octet(const Plan &p, const ChainArgs &a, hipStream_t s)
{
    if (p.loss != WPSGD_LOGISTIC || a.d < kOctetMinColumns || a.d > octet_max_columns(p.dtype)) return hipErrorInvalidValue;
    if (p.dtype == WPSGD_BF16) return launch<uint16_t, 256, 8>(a, s);
    return launch<float, 256, 4>(a, s);
}

}  // namespace wpsgd
