// Regularised objective and prediction error of a model on a data set (Eq. 3 with Eq. 4):
//     c(w) = lambda/2 |w|^2 + (1/m) sum_j L(x_j, y_j, w.x_j),   error = #{ j : y_j (w.x_j) <= 0 } / m.
//
// A pure stream over the data.  w.x is accumulated in fp64 (the products of two fp32 numbers are exact
// in fp64, so the only rounding is in the order of the sum) by as many lanes as a row keeps busy: the
// whole wave for long dense rows, 4 to 32 lanes for dense rows of up to 128 elements, 16 for sparse
// rows.  Losses are taken 64 at a time: a wave collects the results of 64 rows, one per lane, and every lane
// evaluates its own (one row at a time the fp64 logarithm and exponential were most of a short row's
// instructions).  Which rows a wave takes, and the order in which lanes' and waves' totals are
// added, are fixed by the launch shape, so the result does not depend on timing.  The model vector is read through
// the cache hierarchy (it is at most a few MiB).
#include <algorithm>
#include <atomic>
#include <type_traits>

#include "dense_rows.h"
#include "internal.h"

namespace wpsgd {
namespace {

constexpr int kObjThreads = 256;
constexpr int kObjWaves = kObjThreads / kWave;
typedef uint32_t ou32x4 __attribute__((ext_vector_type(4)));

// loss and "wrong side" indicator of one row from z = y * yhat, both in fp64
__device__ inline void row_loss(int loss, double z, double &l, double &wrong)
{
    if (loss == kLossHinge) {
        l = (z < 1.0) ? 1.0 - z : 0.0;
    } else {
        l = (z > 0.0) ? log1p(exp(-z)) : -z + log1p(exp(z));     // log(1 + exp(-z)) without overflow
    }
    wrong = (z <= 0.0) ? 1.0 : 0.0;
}

// Every wave also adds up the squares of its share of the model vector (for the regulariser): one
// workgroup doing that alone took 0.27 ms at d = 2^20, two thirds as long as the rows themselves.
__device__ inline double squares_of_my_share(const float *w, int64_t d, int64_t wave_id, int64_t nwaves, int lane)
{
    const int64_t per = (d + nwaves - 1) / nwaves;
    const int64_t c0 = wave_id * per, c1 = c0 + per < d ? c0 + per : d;
    double sq = 0.0;
    for (int64_t c = c0 + lane; c < c1; c += kWave) sq += (double)w[c] * (double)w[c];
    return wave_sum(sq);
}

// One lane's totals, and the row it holds the result of until the wave has 64 of them.
struct LossTotals {
    double loss = 0.0, wrong = 0.0;
    __device__ void add(int kind, const float *y, int64_t row, int64_t m, double yhat)
    {
        if (row < m) {
            double l, wr;
            row_loss(kind, (double)y[row] * yhat, l, wr);
            loss += l;
            wrong += wr;
        }
    }
    __device__ void store(double *partials, int64_t wave_id, int lane, double sq) const
    {
        const double l = wave_sum(loss), wr = wave_sum(wrong);
        if (lane == 0) {
            partials[3 * wave_id] = l;
            partials[3 * wave_id + 1] = wr;
            partials[3 * wave_id + 2] = sq;
        }
    }
};

// Rows are read once and the model vector over and over: the rows' loads carry the non-temporal
// hint (cache-policy bit 1 of a buffer load), which keeps them from displacing it (+4 % at 16 KiB rows).
constexpr int kReadOnce = 2;

// VEC elements per lane and load (16 bytes when VEC > 1); RB rows in flight per wave.
// (One row: seven waves per SIMD, which the results held back would else make six: unaligned bf16 rows of 3001 elements
// 327 -> 368 us per 512 MiB.)
template <typename TX, int VEC, int RB>
__global__ __launch_bounds__(kObjThreads) __attribute__((amdgpu_waves_per_eu(RB == 1 ? 7 : 1))) void objective_dense_kernel(const char *X, int64_t row_stride, int64_t m,
                                                                     int64_t d, const float *y, const float *w, int loss,
                                                                     double *partials)
{
    const int lane = threadIdx.x & (kWave - 1);
    const int64_t wave_id = (int64_t)blockIdx.x * kObjWaves + threadIdx.x / kWave;
    const int64_t nwaves = (int64_t)gridDim.x * kObjWaves;
    const uint32_t row_bytes = (uint32_t)(d * (int64_t)sizeof(TX));
    const __amdgpu_buffer_rsrc_t wres =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(w), 0, (int)(uint32_t)(d * 4), 0x00020000);
    const int64_t span = (int64_t)kWave * VEC;                 // columns one wave covers per load
    LossTotals totals;
    constexpr int kTurns = kWave / RB;        // turns of RB rows until every lane holds a row's result
    double held = 0.0;
    int64_t held_row = m;                     // (m: none)
    int turn = 0;

    for (int64_t row0 = wave_id * RB; row0 < m; row0 += nwaves * RB) {
        double acc[RB];
        __amdgpu_buffer_rsrc_t xres[RB];
#pragma unroll
        for (int r = 0; r < RB; ++r) {
            acc[r] = 0.0;
            const int64_t row = row0 + r < m ? row0 + r : m - 1;          // past the end: a row that is ignored below
            xres[r] = __builtin_amdgcn_make_buffer_rsrc(const_cast<char *>(X + row * row_stride), 0, (int)row_bytes, 0x00020000);
        }
#pragma unroll 2
        for (int64_t c0 = 0; c0 < d; c0 += span) {
            const uint32_t col = (uint32_t)(c0 + (int64_t)lane * VEC);
            float wv[VEC];
            if constexpr (VEC == 1) {
                wv[0] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(wres, col * 4u, 0, 0));
            } else {
#pragma unroll
                for (int q = 0; q < VEC / 4; ++q) {
                    const ou32x4 t = __builtin_amdgcn_raw_buffer_load_b128(wres, col * 4u + q * 16u, 0, 0);
#pragma unroll
                    for (int i = 0; i < 4; ++i) wv[q * 4 + i] = __uint_as_float(t[i]);
                }
            }
#pragma unroll
            for (int r = 0; r < RB; ++r) {
                float xv[VEC];
                if constexpr (VEC == 1) {
                    if constexpr (sizeof(TX) == 2)
                        xv[0] = bf16_one((uint16_t)__builtin_amdgcn_raw_buffer_load_b16(xres[r], col * 2u, 0, kReadOnce));
                    else
                        xv[0] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(xres[r], col * 4u, 0, kReadOnce));
                } else {
                    const ou32x4 t = __builtin_amdgcn_raw_buffer_load_b128(xres[r], col * (uint32_t)sizeof(TX), 0, kReadOnce);
                    if constexpr (sizeof(TX) == 2) {
#pragma unroll
                        for (int i = 0; i < 4; ++i) {
                            xv[2 * i] = bf16_lo(t[i]);
                            xv[2 * i + 1] = bf16_hi(t[i]);
                        }
                    } else {
#pragma unroll
                        for (int i = 0; i < 4; ++i) xv[i] = __uint_as_float(t[i]);
                    }
                }
#pragma unroll
                for (int i = 0; i < VEC; ++i) acc[r] += (double)wv[i] * (double)xv[i];
            }
        }
        double yhat;
        int64_t row;
        if constexpr (RB == 4) {              // four sums share a register: row r's ends up in row merged_row(r) of 16 lanes
            double t[1];
            wave_sums_merged(acc, t);
            yhat = t[0];
            row = row0 + merged_row(lane / 16);
        } else {
            yhat = wave_sum(acc[0]);
            row = row0;
        }
        if (lane % kTurns == turn) {
            held = yhat;
            held_row = row;
        }
        if (++turn == kTurns) {
            totals.add(loss, y, held_row, m, held);
            held_row = m;
            turn = 0;
        }
    }
    totals.add(loss, y, held_row, m, held);
    totals.store(partials, wave_id, lane, squares_of_my_share(w, d, wave_id, nwaves, lane));
}

// Dense rows of at most 128 elements: LPR lanes per row, four elements each, 64/LPR rows per load instruction, LPR
// instructions for 64 consecutive rows.  A piece that reaches past the row's end is read from d-4 on, and what the
// piece before has counted already is dropped.  A million rows of 16 elements: 215 -> 20 us
// (hinge), 450 -> 27 us (logistic), of 100: 249 -> 86 and 463 -> 92 us (4.6 TB/s).
template <typename TX, int LPR>
__global__ __launch_bounds__(kObjThreads) void objective_short_rows_kernel(const TX *X, int64_t ld, int64_t m, int d, const float *y,
                                                                          const float *w, int loss, double *partials)
{
    constexpr int ROWS = kWave / LPR;
    constexpr int kAtOnce = LPR < 8 ? LPR : 8;      // loads in flight per lane
    typedef TX four __attribute__((ext_vector_type(4), aligned(sizeof(TX))));
    const int lane = threadIdx.x & (kWave - 1);
    const int64_t wave_id = (int64_t)blockIdx.x * kObjWaves + threadIdx.x / kWave;
    const int64_t nwaves = (int64_t)gridDim.x * kObjWaves;
    const int c = lane % LPR, col = c * 4 < d - 4 ? c * 4 : d - 4;
    double wv[4];
    bool mine[4];                             // (an element that is not this lane's is dropped, not weighted with zero: it may be infinite)
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        mine[e] = col + e >= c * 4;
        wv[e] = (double)w[col + e];
    }
    LossTotals totals;
    for (int64_t row0 = wave_id * kWave; row0 < m; row0 += nwaves * kWave) {
        double held = 0.0;
#pragma unroll
        for (int it0 = 0; it0 < LPR; it0 += kAtOnce) {
            four q[kAtOnce];
#pragma unroll
            for (int i = 0; i < kAtOnce; ++i) {
                const int64_t row = row0 + (it0 + i) * ROWS + lane / LPR;
                q[i] = *reinterpret_cast<const four *>(X + (row < m ? row : m - 1) * ld + col);
            }
#pragma unroll
            for (int i = 0; i < kAtOnce; ++i) {
                double acc = 0.0;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    float x;
                    if constexpr (sizeof(TX) == 2) x = bf16_one(q[i][e]);
                    else x = q[i][e];
                    acc += mine[e] ? wv[e] * (double)x : 0.0;
                }
                acc += dpp_move<0xB1, 0xF>(acc);
                acc += dpp_move<0x4E, 0xF>(acc);
                if constexpr (LPR >= 8) acc += dpp_move<0x141, 0xF>(acc);
                if constexpr (LPR >= 16) acc += dpp_move<0x140, 0xF>(acc);
                if constexpr (LPR >= 32) acc = merge_values<true>(acc, acc);
                held = c == it0 + i ? acc : held;
            }
        }
        totals.add(loss, y, row0 + c * ROWS + lane / LPR, m, held);
    }
    totals.store(partials, wave_id, lane, squares_of_my_share(w, d, wave_id, nwaves, lane));
}

// Sparse rows: 16 lanes per row, four rows at a time; 4*turns <= 64 consecutive rows make a batch, whose offsets are
// loaded at once.  Bound by the gathers of the model: from the caches a compute unit serves a third to half a lane per
// cycle, from LDS many.  HEAD > 0: the model's first HEAD columns are copied to LDS and only the others are gathered from
// memory (lanes that need none ask for an offset past the end, which is no access), if at least a quarter of the sampled
// entries, one per thread, lie there.  A million rows of 80 entries, 2^20 columns (Zipf): 0.41 -> 0.31 ms (2.1 TB/s), the
// same without the copy 0.41, with four entries a load 0.27, of which the gathers from memory take 0.11: a line of L2 each; half a million rows of 40, logistic: 225 -> 70 us.
// Long rows take the whole wave, since with 16 lanes a row keeps a quarter as much on its way: one by one inside a batch
// (one row of 100000 entries among 200000 of 20: 1530 us with 16 lanes, 322 with 64), and one row per wave throughout where
// the average row is long, where rows are so few that each may have a wave, or where no head is used (1000 rows of
// 3000: 63 -> 29 us; 1000000 rows of 80 uniform columns: 632 -> 605).
constexpr int kLongRow = 256;                 // entries
constexpr int kBriefRow = 32;                 // entries of the average row
// E dwords that follow each other, each zero from the resource's end on
template <int E> struct EntryLoad {
    typedef uint32_t words __attribute__((ext_vector_type(E)));
    words q;
    __device__ EntryLoad(__amdgpu_buffer_rsrc_t from, uint32_t off)
    {
        if constexpr (E == 4) q = __builtin_bit_cast(words, __builtin_amdgcn_raw_buffer_load_b128(from, off, 0, 0));
        else if constexpr (E == 2) q = __builtin_bit_cast(words, __builtin_amdgcn_raw_buffer_load_b64(from, off, 0, 0));
        else q[0] = __builtin_amdgcn_raw_buffer_load_b32(from, off, 0, 0);
    }
    __device__ uint32_t at(int i) const { return q[i]; }
};
template <int THREADS, int HEAD>
__global__ __launch_bounds__(THREADS) __attribute__((amdgpu_waves_per_eu(HEAD > 0 ? THREADS / 128 : 1)))
void objective_csr_kernel(const int64_t *row_ptr, const int32_t *col_idx,
                                                                   const float *vals, int64_t m, int64_t d, const float *y,
                                                                   const float *w, int loss, int turns, double *partials)
{
    constexpr int LPR = 16, ROWS = kWave / LPR, WAVES = THREADS / kWave;
    constexpr int kAtOnce = 4;                // entries in flight per lane
    __shared__ float head[HEAD > 0 ? HEAD : 1];
    const int lane = threadIdx.x & (kWave - 1), c = lane % LPR, r = lane / LPR;
    const int64_t wave_id = (int64_t)blockIdx.x * WAVES + __builtin_amdgcn_readfirstlane((int)threadIdx.x / kWave);
    const int64_t nwaves = (int64_t)gridDim.x * WAVES;
    const int batch = ROWS * turns;
    // (The first offsets of either form are asked for beside the ones that choose it, each later batch's beside the batch
    // before; many batches of a copied head have other waves to wait on, and no registers to spare.)
    constexpr bool AHEAD = HEAD == 0;
    auto row_at = [&](int64_t row) { return row < m ? row : m - 1; };
    int64_t lo_wave = 0, hi_wave = 0, lo_lane = 0, hi_lane = 0;
    auto ask_wave = [&](int64_t row) {
        lo_wave = row_ptr[row_at(row)];
        hi_wave = row_ptr[row_at(row) + 1];
    };
    auto ask_lane = [&](int64_t row0) {
        lo_lane = row_ptr[row_at(row0 + lane)];
        hi_lane = row_ptr[row_at(row0 + lane) + 1];
    };
    if constexpr (AHEAD) {
        ask_wave(wave_id);
        ask_lane(wave_id * batch);
    }
    const int64_t first = row_ptr[0], entries = row_ptr[m] - first;
    const __amdgpu_buffer_rsrc_t wres =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(w), 0, (int)(uint32_t)(d * 4), 0x00020000);
    LossTotals totals;

    // a whole row by the whole wave (n > 0)
    auto whole_row = [&](int64_t p0, int n) {
        double acc = 0.0;
        int e0 = 0;
        for (; AHEAD && e0 + kAtOnce * kWave <= n; e0 += kAtOnce * kWave) {
            uint32_t col[kAtOnce];
            float val[kAtOnce], wv[kAtOnce];
#pragma unroll
            for (int i = 0; i < kAtOnce; ++i) {
                col[i] = (uint32_t)col_idx[p0 + e0 + i * kWave + lane];
                val[i] = vals[p0 + e0 + i * kWave + lane];
            }
#pragma unroll
            for (int i = 0; i < kAtOnce; ++i) wv[i] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(wres, col[i] * 4u, 0, 0));
#pragma unroll
            for (int i = 0; i < kAtOnce; ++i) acc += (double)wv[i] * (double)val[i];
        }
        for (int e = e0 + lane; e < n; e += kWave) acc += (double)w[col_idx[p0 + e]] * (double)vals[p0 + e];
        return wave_sum(acc);
    };
    bool whole_waves = entries > m * (m <= 2 * 8192 ? 24 : kLongRow / 2), copied = false;
    if constexpr (HEAD > 0) {                 // (copied whether it is used or not: meanwhile the sampled entry arrives)
        if (!whole_waves) {
            const uint32_t sampled = entries > 0 ? (uint32_t)col_idx[first + (int64_t)((uint64_t)threadIdx.x * (uint64_t)entries / THREADS)] : ~0u;
            for (int i = (int)threadIdx.x; i < HEAD; i += THREADS) head[i] = i < d ? w[i] : 0.0f;
            copied = __syncthreads_count(sampled < (uint32_t)HEAD) >= THREADS / 4;
            whole_waves = !copied && entries > m * (kLongRow / 4);
        }
    }
    if (whole_waves) {
        double held = 0.0;
        int64_t held_row = m;                 // (m: none)
        int turn = 0;
        for (int64_t row = wave_id; row < m; row += nwaves) {
            if constexpr (!AHEAD) ask_wave(row);
            const int64_t lo = lo_wave;
            const int n = (int)(hi_wave - lo);
            if constexpr (AHEAD) ask_wave(row + nwaves);
            const double yhat = n > 0 ? whole_row(lo, n) : 0.0;
            if (lane == turn) {
                held = yhat;
                held_row = row;
            }
            if (++turn == kWave) {
                totals.add(loss, y, held_row, m, held);
                held_row = m;
                turn = 0;
            }
        }
        totals.add(loss, y, held_row, m, held);
        totals.store(partials, wave_id, lane, squares_of_my_share(w, d, wave_id, nwaves, lane));
        return;
    }

    const bool brief = entries <= m * kBriefRow || !copied;
    auto rows_in_batches = [&](auto copied_tag) {
        constexpr bool COPIED = decltype(copied_tag)::value;
        auto near = [](uint32_t col) { return COPIED && col < (uint32_t)HEAD; };
        for (int64_t row0 = wave_id * batch; row0 < m; row0 += nwaves * batch) {
            if constexpr (!AHEAD) ask_lane(row0);
            const int64_t lo = lo_lane;
            const int len = (int)(hi_lane - lo);
            if constexpr (AHEAD) ask_lane(row0 + nwaves * batch);
            double held = 0.0;
            if (entries > 0) {
                // A lane takes four entries that follow each other with one load for the columns and one for the values, a quarter of
                // the instructions of single entries (a million rows of 80, Zipf: 313 -> 272 us; of 110, 433 -> 369).  A lane's entries wait for each other's
                // loads of the model, so the last 16 or 32 of brief rows go one or two to a lane (us, a million rows, half of the columns behind the head,
                // single entries | four to a lane | this: mean 2 69 | 73 | 49, 10 72 | 80 | 59, 16 75 | 82 | 63, 40 190 | 172 | 170; all columns in it, mean 10
                // 77 | 76 | 55).  Not where longer rows meet a copied head: 260 us for the rows of 80 with every rest to a lane's four, 267 this way.  The loads
                // are checked against the arrays' end, dword by dword, and count from the batch's first entry; a batch too long
                // for their 32-bit offsets goes row by row.
                const int64_t base = lane_read_i64(lo, 0);
                const bool near_rows = lane_read_i64(lo, kWave - 1) + __builtin_amdgcn_readlane(len, kWave - 1) - base < (1 << 28);
                const uint32_t room = (uint32_t)min(first + entries - base, (int64_t)(1 << 29)) * 4u;
                const __amdgpu_buffer_rsrc_t cres = make_rsrc(col_idx + base, room), vres = make_rsrc(vals + base, room);
                const uint32_t mine = (uint32_t)(lo - base);
                for (int it = 0; it < turns; ++it) {
                    const int from = it * ROWS + r;
                    const uint32_t p0 = (uint32_t)__shfl((int)mine, from);
                    const int whole = __shfl(len, from), n = whole > kLongRow || !near_rows ? 0 : whole;
                    double acc = 0.0;
                    auto take = [&](auto entries_tag, int e0) {
                        constexpr int E = decltype(entries_tag)::value;      // a lane's entries from e0 on
                        const int e = e0 + E * c;
                        const uint32_t off = e < n ? (p0 + (uint32_t)e) * 4u : 0xFFFFFFF0u;
                        const EntryLoad<E> col(cres, off), val(vres, off);
                        float wv[E];
#pragma unroll
                        for (int i = 0; i < E; ++i) {
                            const float far = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(wres, e + i < n && !near(col.at(i)) ? col.at(i) * 4u : 0xFFFFFFF0u, 0, 0));
                            wv[i] = near(col.at(i)) ? head[near(col.at(i)) ? col.at(i) : 0u] : far;
                        }
#pragma unroll
                        for (int i = 0; i < E; ++i) acc += e + i < n ? (double)wv[i] * (double)__uint_as_float(val.at(i)) : 0.0;
                    };
                    for (int e0 = 0; __any(e0 < n); e0 += kAtOnce * LPR) {
                        if (brief && !__any(e0 + 2 * LPR < n)) {       // the rest of the four rows
                            if (__any(e0 + LPR < n)) take(std::integral_constant<int, 2>{}, e0);
                            else take(std::integral_constant<int, 1>{}, e0);
                            break;
                        }
                        take(std::integral_constant<int, kAtOnce>{}, e0);
                    }
                    acc += dpp_move<0xB1, 0xF>(acc);
                    acc += dpp_move<0x4E, 0xF>(acc);
                    acc += dpp_move<0x141, 0xF>(acc);
                    acc += dpp_move<0x140, 0xF>(acc);
                    held = c == it ? acc : held;
                    uint64_t longer = __builtin_amdgcn_ballot_w64((whole > kLongRow || (!near_rows && whole > 0)) && c == 0);
                    while (__builtin_expect(longer != 0, 0)) {                // (one bit per such row, at its first lane)
                        const int at = __builtin_ctzll(longer);
                        longer &= longer - 1;
                        const double yhat = whole_row(lane_read_i64(lo, it * ROWS + at / LPR), __builtin_amdgcn_readlane(whole, at));
                        held = c == it && r == at / LPR ? yhat : held;
                    }
                }
            }
            if (c < turns) totals.add(loss, y, row0 + c * ROWS + r, m, held);
        }
    };
    if constexpr (HEAD > 0) {
        if (copied) rows_in_batches(std::true_type{});
        else rows_in_batches(std::false_type{});
    } else {
        rows_in_batches(std::false_type{});
    }
    totals.store(partials, wave_id, lane, squares_of_my_share(w, d, wave_id, nwaves, lane));
}

// One workgroup: adds the waves' totals (losses, wrong predictions, squares) in wave order and writes the two results.
constexpr int kFinishThreads = 1024;
__global__ __launch_bounds__(kFinishThreads) void objective_finish_kernel(const double *partials, int64_t nwaves,
                                                                         int64_t m, double lambda, double *out)
{
    __shared__ double red[3][kFinishThreads];
    const int t = threadIdx.x;
    double a = 0.0, b = 0.0, sq = 0.0;
    for (int64_t i = t; i < nwaves; i += kFinishThreads) {
        a += partials[3 * i];
        b += partials[3 * i + 1];
        sq += partials[3 * i + 2];
    }
    red[0][t] = a;
    red[1][t] = b;
    red[2][t] = sq;
    __syncthreads();
    for (int s = kFinishThreads / 2; s > 0; s >>= 1) {
        if (t < s) {
            red[0][t] += red[0][t + s];
            red[1][t] += red[1][t + s];
            red[2][t] += red[2][t + s];
        }
        __syncthreads();
    }
    if (t == 0) {
        out[0] = 0.5 * lambda * red[2][0] + red[0][0] / (double)m;
        out[1] = red[1][0] / (double)m;
    }
}

// The workgroups walk the rows with a stride of the whole grid, so the grid should be exactly what the
// device holds at once: with more, the surplus runs as a second, thinly occupied round (2048
// workgroups where 1536 fit cost 14 % at 16 KiB rows, 2048 where 1280 fit 11 % at 1 KiB rows).
// Asked once per kernel.
template <auto kernel>
unsigned resident_grid(unsigned most)
{
    static std::atomic<unsigned> cached{0};        // (one instance per kernel; working it out twice is harmless)
    unsigned resident = cached.load(std::memory_order_relaxed);
    if (resident == 0) {
        // a workgroup is one wave on each of a compute unit's four SIMDs; a SIMD has 512 registers
        // per lane, handed out in blocks of eight, and room for eight waves
        hipFuncAttributes attr;
        int dev = 0, cus = 0;
        if (hipFuncGetAttributes(&attr, reinterpret_cast<const void *>(kernel)) != hipSuccess || hipGetDevice(&dev) != hipSuccess ||
            hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || attr.numRegs < 1 || cus < 1) {
            (void)hipGetLastError();
            return most;
        }
        const int blocks = (attr.numRegs + 7) / 8 * 8;
        const int per_cu = blocks >= 512 ? 1 : (512 / blocks < 8 ? 512 / blocks : 8);
        resident = (unsigned)per_cu * (unsigned)cus;
        cached.store(resident, std::memory_order_relaxed);
    }
    return resident < most ? resident : most;
}

template <typename TX, int LPR>
unsigned launch_short_rows(unsigned most, hipStream_t s, const ChainArgs &a, int loss, const float *w, double *partials)
{
    // one batch of 64 rows per wave at least
    const unsigned rows = (unsigned)std::min<int64_t>((a.m + kWave * kObjWaves - 1) / (kWave * kObjWaves), most);
    const unsigned grid = resident_grid<objective_short_rows_kernel<TX, LPR>>(rows);
    hipLaunchKernelGGL((objective_short_rows_kernel<TX, LPR>), dim3(grid), dim3(kObjThreads), 0, s, static_cast<const TX *>(a.dense), a.ld,
                       a.m, (int)a.d, a.y, w, loss, partials);
    return grid;
}

template <typename TX>
unsigned launch_short_rows(unsigned most, hipStream_t s, const ChainArgs &a, int loss, const float *w, double *partials)
{
    if (a.d <= 16) return launch_short_rows<TX, 4>(most, s, a, loss, w, partials);
    if (a.d <= 32) return launch_short_rows<TX, 8>(most, s, a, loss, w, partials);
    if (a.d <= 64) return launch_short_rows<TX, 16>(most, s, a, loss, w, partials);
    return launch_short_rows<TX, 32>(most, s, a, loss, w, partials);
}

template <typename TX, int VEC>
unsigned launch_dense_rows(int rb, unsigned most, hipStream_t s, const char *X, int64_t stride, int64_t m, int64_t d,
                           const float *y, const float *w, int loss, double *partials)
{
    unsigned grid;
    if (rb == 4) {
        grid = resident_grid<objective_dense_kernel<TX, VEC, 4>>(most);
        hipLaunchKernelGGL((objective_dense_kernel<TX, VEC, 4>), dim3(grid), dim3(kObjThreads), 0, s, X, stride, m, d, y, w, loss, partials);
    } else {
        grid = resident_grid<objective_dense_kernel<TX, VEC, 1>>(most);
        hipLaunchKernelGGL((objective_dense_kernel<TX, VEC, 1>), dim3(grid), dim3(kObjThreads), 0, s, X, stride, m, d, y, w, loss, partials);
    }
    return grid;
}

}  // namespace

int64_t objective_grid(int64_t m)
{
    const int64_t want = (m + kObjWaves - 1) / kObjWaves;
    return want < 2048 ? want : 2048;          // at most eight workgroups per compute unit (the launch takes what fits)
}

size_t objective_partials_bytes(int64_t m) { return (size_t)objective_grid(m) * kObjWaves * 3 * sizeof(double); }

// Partial sums for callers that cannot allocate (wpsgd_objective_static): room for the largest launch,
// 2048 workgroups of four waves with three sums each - 192 KiB that every device the library runs
// on holds until the process ends.  Host code never uses the array's name as an address: it asks for
// the device address once per device and passes that to the kernels, as it passes a workspace.
constexpr size_t kStaticPartials = (size_t)2048 * kObjWaves * 3;
static __device__ __align__(256) double scratch[kStaticPartials];

hipError_t objective_static_partials(double **partials, size_t *bytes)
{
    constexpr int kMaxDevices = 64;
    static std::atomic<double *> address[kMaxDevices];      // (two threads asking at once get the same answer)
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    double *p = address[dev].load(std::memory_order_acquire);
    if (p == nullptr) {
        e = hipGetSymbolAddress(reinterpret_cast<void **>(&p), HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        if (p == nullptr) return hipErrorInvalidSymbol;
        address[dev].store(p, std::memory_order_release);
    }
    *partials = p;
    *bytes = kStaticPartials * sizeof(double);
    return hipSuccess;
}

hipError_t launch_objective(const ChainArgs &a, int dtype, int vec, int loss, const float *w, double lambda,
                            double *partials, double *out, hipStream_t s)
{
    const unsigned most = (unsigned)objective_grid(a.m);      // what the partial sums have room for
    unsigned grid = most;
    if (a.dense) {
        const char *X = static_cast<const char *>(a.dense);
        const int elem = dtype == WPSGD_BF16 ? 2 : 4;
        const int64_t stride = a.ld * elem;
        const bool elements = (uintptr_t)a.dense % (unsigned)elem == 0;
        const int rb = a.d <= (int64_t)kWave * vec * 2 ? 4 : 1;     // short rows: several in flight per wave
        if (a.d >= 4 && a.d <= 128 && elements) {
            grid = dtype == WPSGD_BF16 ? launch_short_rows<uint16_t>(most, s, a, loss, w, partials) : launch_short_rows<float>(most, s, a, loss, w, partials);
        } else if (dtype == WPSGD_BF16) {
            if (vec > 1) grid = launch_dense_rows<uint16_t, 8>(rb, most, s, X, stride, a.m, a.d, a.y, w, loss, partials);
            else grid = launch_dense_rows<uint16_t, 1>(rb, most, s, X, stride, a.m, a.d, a.y, w, loss, partials);
        } else {
            if (vec > 1) grid = launch_dense_rows<float, 4>(rb, most, s, X, stride, a.m, a.d, a.y, w, loss, partials);
            else grid = launch_dense_rows<float, 1>(rb, most, s, X, stride, a.m, a.d, a.y, w, loss, partials);
        }
    } else {
        // Batches that fill whole rounds of the waves that run at once, as long as 64 rows allow (300000 rows of 80, Zipf: one
        // batch for most waves and two for some 90 us, one round 70).  A copy of the model's head per workgroup pays when a
        // wave has some fifty rows to use it on (half a million rows of 80 uniform columns, which do not use it, lose 6 %); two
        // workgroups of 1024 threads fill a compute unit's waves, with 64 KiB of LDS each.
        constexpr int kHeadThreads = 1024, kHeadWaves = kHeadThreads / kWave, kHead = 16384;
        const bool head = a.m >= 400000;
        if (!head) grid = resident_grid<objective_csr_kernel<kObjThreads, 0>>(most);
        const int64_t at_once = head ? 512 * kHeadWaves : std::max<int64_t>((int64_t)grid * kObjWaves, 1);
        const int64_t rounds = (a.m + 64 * at_once - 1) / (64 * at_once);
        const int turns = (int)((a.m + 4 * at_once * rounds - 1) / (4 * at_once * rounds));
        if (head) {
            const int64_t batches = (a.m + 4 * turns - 1) / (4 * turns);
            grid = (unsigned)std::min<int64_t>((batches + kHeadWaves - 1) / kHeadWaves, 512);
            hipLaunchKernelGGL((objective_csr_kernel<kHeadThreads, kHead>), dim3(grid), dim3(kHeadThreads), 0, s, a.row_ptr, a.col_idx, a.vals,
                               a.m, a.d, a.y, w, loss, turns, partials);
            grid *= kHeadWaves / kObjWaves;              // (what the finish kernel counts in)
        } else {                                         // (waves without rows still add up their share of the model's squares)
            hipLaunchKernelGGL((objective_csr_kernel<kObjThreads, 0>), dim3(grid), dim3(kObjThreads), 0, s, a.row_ptr, a.col_idx, a.vals,
                               a.m, a.d, a.y, w, loss, turns, partials);
        }
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    const int64_t nwaves = (int64_t)grid * kObjWaves;
    hipLaunchKernelGGL(objective_finish_kernel, dim3(1), dim3(kFinishThreads), 0, s, partials, nwaves, a.m, lambda, out);
    return hipGetLastError();
}

}  // namespace wpsgd
