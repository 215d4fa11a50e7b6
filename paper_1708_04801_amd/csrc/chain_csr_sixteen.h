// Sparse chains of short rows that hardly ever share a column: sixteen steps at a time, the model in HBM.
//
// Four rows of at most 16 entries lie side by side in a wave, and where rows share no column their steps are independent of each other
// but for the shrink, which the steps' scalars carry.  chain_csr_short.h takes four such steps at once and holds two things against itself: a value that an
// earlier group has written must be read again, so the worker waits for memory, and a group whose rows share a column runs step by
// step.  Here sixteen are taken at once, and the few that share a column wait for a read of their own:
//
//   A value is requested kXAhead blocks before its block's turn, behind all stores of the block whose turn it is.  So it is old only where the
//   block before or an earlier row of its own block has the column, which follows from the rows alone:
//     a block that shares a column with the one before reads its values again, all at once, when that has stored;
//     a step that shares one with an earlier step of its block is taken in turn, behind the block's other steps: it reads its values when they have
//     stored theirs.  So is a step whose row has an element that is not finite (a slope of 0 times it is one too: it stores in any case) or more than 16
//     entries, and with the latter all steps behind it in the block, and the block behind reads again: those entries leave no stamps.
//   Every update is a multiply-add on the model as the steps before left it, and no two lanes of one store have a column in common.
//
//   Two stamp tables (two hashes of the column) hold the block and the entry that wrote last, two blocks ahead of the chain.  An entry that finds the
//   block before in one of them and nothing older in the other may share its column with that block, one that finds its own block in both with an earlier
//   row of it; of the four rows taken together, an entry that does not read its own number back is compared with the one that took its place.  What
//   this says too often costs a read: in one or two blocks of a hundred, where at d = 100000 sixteen have a reason.
//
// Five waves, one barrier per block of sixteen steps:
//   worker  products, slopes and stores of block b; requests the values of block b + kXAhead
//   scout   fetches the rows' entries kXLead blocks ahead and writes records: value, place of the column; finds the long rows
//   stamps  the tables
//   pairs   what the stamps mean
//   sampler the rows of the steps to come, 64 at a time, and the scalars of the recursion
//
// What bounds it: the worker's chain through a block.  With cycle counters in all waves (they cost a tenth), d = 100000: 1520 cycles between two barriers, of
// which the worker takes 1350 (to the slopes 590, updates 200, reading again 120 and steps in turn 90 on the average, requests 70; the rest is
// LDS reads and the counters), pairs 1100, scout 970, stamps 620, sampler 290.  A block that reads again takes some 850 cycles more, a step in turn
// some 1300.  us, ten chains of 10000 steps, hinge, 5 to 10 entries, groups of four | this way: d = 100000 620 | 400, a million 638 | 374;
// d = 300000 with 1000 rows 636 | 441, with 300 rows 727 | 546; d = 100000 with one row in a thousand of 20 entries 666 | 458, of 130 entries 723 | 507.
// Ten chains of up to 100000 steps, d = 100000: 5.70 ms in groups of four, 3.62 this way (0.057 and 0.036 us per step).  Tried, at d = 100000 with 400 us this way:
// updates as additions at the L2, with the product of two entries for every pair that an early value lacks (478: 0.44 us a pair, and each update
// rounded twice), pairs found by comparing a candidate with all entries of two blocks (394, and 1440 instead of 546 with 300 rows), stamps that
// judge for themselves (430), blocks of 32 steps (twice the pairs and the stamps), sums unit by unit in four registers instead of folded into
// one, scalars read in the block's own turn.
// Precision: products, sums and slopes' arguments in fp64 for either loss, updates one rounding to the state's type.  Error of a logistic chain of
// 10000 steps against fp64, groups of four | this way: d = 60000 6.97e-8 | 6.48e-8, 100000 6.83e-8 | 6.29e-8, a million 4.99e-8 | 4.75e-8; hinge the same.
#pragma once

namespace wpsgd {
namespace {

constexpr int kXUnits = 4, kXSteps = 4 * kXUnits;     // steps per block; waves' widths of 64 entries: unit u, lane 16*r + e: entry e of step 4*u + r
constexpr int kXLead = 4;                    // scout: blocks between the request of a row's entries and their records
constexpr int kXAhead = 2;                   // worker: blocks between the request of a value and its block's turn: it misses what the block before and its own write
constexpr int kXTurn = 3;                    // in interval i records of block i are written, stamps of block i-1 left, pairs of block i-2 found, block i-3 taken
constexpr int kXStamps = 16384;              // entries of either table
constexpr int kXRing = 256;                  // steps whose rows and scalars are kept
constexpr int kXWorker = 0, kXScout = 1, kXStampWave = 2, kXPairWave = 3, kXSampler = 4, kXWaves = 5;
constexpr int kXThreads = kXWaves * kWave;
constexpr uint32_t kNowhere = 0xFFFFFFF0u;   // past the end of any buffer: no access

struct __attribute__((aligned(16))) XStep {
    int64_t lo;           // first entry of the row
    int32_t len, pad;
    double zs, cs;        // y*s_l (times log2 e for the logistic loss) and y*eta/s_{l+1}; len = 0 and cs = 0 past the chain's end
};
struct __attribute__((aligned(8))) XTold {  // what scout and pairs have found out about a block
    uint32_t rows;        // scout: a bit per step whose row is long or not finite; 16 bits up, per long row
    uint32_t pairs;       // pairs: a bit per step that shares a column with an earlier one of the block; kXBefore: some entry does with the block before
};
constexpr uint32_t kXBefore = 0x10000u;
struct XLds {
    static constexpr uint32_t section = kXUnits * kWave * 8;                         // records of a block: {value, byte offset}
    static constexpr uint32_t stamp_a = 0;                                           // 16 bits: entry of the block, block modulo 256
    static constexpr uint32_t stamp_b = stamp_a + kXStamps * 2;
    static constexpr uint32_t steps = stamp_b + kXStamps * 2;
    static constexpr uint32_t rec = steps + kXRing * 32;                             // four sections
    static constexpr uint32_t found = rec + 4 * section;                             // two blocks: what the entries found in the tables, as the records
    static constexpr uint32_t told = found + 2 * section;                            // eight blocks: XTold
    static constexpr uint32_t bytes = told + 8 * 8;
    static_assert(kXUnits * kWave == 256 && steps % 16 == 0 && rec % 16 == 0 && told % 16 == 0, "alignment");
};

template <typename T> __device__ inline T &at_lds(char *lds, uint32_t off) { return *reinterpret_cast<T *>(lds + off); }

// a block's values once more, and two words per lane, each a statement of its own that waits (see drained_buffer_load)
#define WPSGD_FOUR_LOADS(OP)                                                                                          \
    asm volatile("s_nop 3\n\ts_waitcnt vmcnt(0)\n\t" OP " %0, %4, %8, 0 offen\n\t" OP " %1, %5, %8, 0 offen\n\t"       \
                 OP " %2, %6, %8, 0 offen\n\t" OP " %3, %7, %8, 0 offen\n\ts_waitcnt vmcnt(0)"                        \
                 : "=&v"(x[0]), "=&v"(x[1]), "=&v"(x[2]), "=&v"(x[3])                                                 \
                 : "v"(off[0]), "v"(off[1]), "v"(off[2]), "v"(off[3]), "s"(rsrc)                                      \
                 : "memory")
__device__ inline void drained_values(pu32x4 rsrc, const uint32_t (&off)[4], double (&x)[4]) { WPSGD_FOUR_LOADS("buffer_load_dwordx2"); }
__device__ inline void drained_values(pu32x4 rsrc, const uint32_t (&off)[4], float (&x)[4]) { WPSGD_FOUR_LOADS("buffer_load_dword"); }
#undef WPSGD_FOUR_LOADS
__device__ inline void drained_global_load_2(const void *p, const void *q, uint32_t &x, uint32_t &y)
{
    asm volatile("s_waitcnt vmcnt(0)\n\tglobal_load_dword %0, %2, off\n\tglobal_load_dword %1, %3, off\n\ts_waitcnt vmcnt(0)"
                 : "=&v"(x), "=&v"(y) : "v"(p), "v"(q) : "memory");
}

template <int LOSS>
struct SixteenSteps {
    using TV = typename StateType<LOSS>::type;
    using L = XLds;
    const ChainArgs &a;
    char *const lds;
    TV *const v;
    const int lane;
    const int64_t n, nblocks;

    __device__ SixteenSteps(const ChainArgs &args, char *l, TV *vec, int64_t steps)
        : a(args), lds(l), v(vec), lane((int)(threadIdx.x & (kWave - 1))), n(steps), nblocks((steps + kXSteps - 1) / kXSteps) {}

    __device__ static constexpr uint32_t step_at(int64_t t) { return L::steps + (uint32_t)(t & (kXRing - 1)) * 32u; }
    __device__ static constexpr uint32_t told_at(int64_t r) { return L::told + (uint32_t)(r & 7) * 8u; }
    __device__ static uint32_t next_section(uint32_t s) { return s == L::rec + 3 * L::section ? L::rec : s + L::section; }
    __device__ int64_t intervals() const { return nblocks + kXTurn; }
    // what a wave does between two barriers
    template <typename F>
    __device__ void interval(F &&work) const
    {
        work();
        wait_lds_then_barrier();
    }

    // ---------------------------------------------------------------- worker
    __device__ static double step_coefficient(double zs, double cs, double sum)
    {
        if constexpr (LOSS == kLossHinge) return zs * sum < 1.0 ? cs : 0.0;
        else return (double)unit_slope<LOSS>((TV)(zs * sum)) * cs;
    }

    // Sums over the sixteen lanes of each step, all sixteen steps in one register: the four units' registers become two, then one, while their sums
    // cross lanes.  Step 4*u + r ends up in the four lanes of row r whose place in the row is 4 * merged_row(u) and behind.
    template <int CTRL, int LOWER, int UPPER>
    __device__ static int halves(int a, int b)
    {
        return __builtin_amdgcn_update_dpp(__builtin_amdgcn_update_dpp(0, a, CTRL, 0xF, LOWER, false), b, CTRL, 0xF, UPPER, false);
    }
    template <int CTRL, int LOWER, int UPPER>      // a in the lanes of the banks LOWER, b in those of UPPER, each with what CTRL brings there added
    __device__ static double fold(double a, double b)
    {
        const long long p = __double_as_longlong(a), q = __double_as_longlong(b);
        const int pl = (int)(p & 0xFFFFFFFFLL), ph = (int)(p >> 32), ql = (int)(q & 0xFFFFFFFFLL), qh = (int)(q >> 32);
        const int ml = halves<CTRL, LOWER, UPPER>(pl, ql), mh = halves<CTRL, LOWER, UPPER>(ph, qh);
        const int kl = __builtin_amdgcn_update_dpp(pl, ql, 0xE4, 0xF, UPPER, false), kh = __builtin_amdgcn_update_dpp(ph, qh, 0xE4, 0xF, UPPER, false);
        return __longlong_as_double(((long long)kh << 32) | (long long)(unsigned int)kl) + __longlong_as_double(((long long)mh << 32) | (long long)(unsigned int)ml);
    }
    __device__ static double sum_steps(const double (&t)[kXUnits])
    {
        const double p = fold<0x128, 0x3, 0xC>(t[0], t[1]), q = fold<0x128, 0x3, 0xC>(t[2], t[3]);      // row_ror:8
        double s = fold<0x141, 0x5, 0xA>(p, q);                                                         // row_half_mirror
        s += dpp_move<0xB1, 0xF>(s);
        s += dpp_move<0x4E, 0xF>(s);
        return s;
    }
    // this lane's step of a block, after sum_steps
    __device__ int my_step() const { return 4 * merged_row((lane >> 2) & 3) + (lane >> 4); }
    // step 4*U + r of a block, one value per step where sum_steps leaves it, in all lanes of row r
    template <int U>
    __device__ static double of_unit(double c)
    {
        constexpr int CTRL = 0x150 + 4 * merged_row(U);                   // row_newbcast
        const long long bits = __double_as_longlong(c);
        const int lo = __builtin_amdgcn_update_dpp(0, (int)(bits & 0xFFFFFFFFLL), CTRL, 0xF, 0xF, false), hi = __builtin_amdgcn_update_dpp(0, (int)(bits >> 32), CTRL, 0xF, 0xF, false);
        return __longlong_as_double(((long long)hi << 32) | (long long)(unsigned int)lo);
    }

    // Steps of a block that are taken in turn, behind the others: each reads its values when all earlier steps have stored theirs.
    __device__ void in_turn(int64_t b, uint32_t steps, uint32_t longs, const uint32_t (&off)[kXUnits], const float (&val)[kXUnits], pu32x4 vdesc) const
    {
#pragma unroll 1
        while (steps != 0) {
            const int j = (int)__builtin_ctz(steps);
            steps &= steps - 1;
            const XStep st = at_lds<XStep>(lds, step_at(b * kXSteps + j));
            if ((longs >> j & 1u) != 0) {
                long_row(st, vdesc);
                continue;
            }
            uint32_t o = off[0];
            float w = val[0];
#pragma unroll
            for (int u = 1; u < kXUnits; ++u) {
                o = u == j / 4 ? off[u] : o;
                w = u == j / 4 ? val[u] : w;
            }
            o = lane >> 4 == (j & 3) ? o : kNowhere;
            const double cur = (double)drained_buffer_load(vdesc, o, TV{}), x = (double)w;
            const double c = step_coefficient(st.zs, st.cs, row_sum(cur * x));
            drained_buffer_store(vdesc, o, (TV)__builtin_fma(c, x, cur));           // (also without a slope: 0 times an element that is not finite is none)
        }
    }
    __device__ void long_row(const XStep &st, pu32x4 vdesc) const
    {
        const int len = __builtin_amdgcn_readfirstlane(st.len);
        uint32_t o = kNowhere;
        double x = 0.0, cur = 0.0, acc = 0.0;
        auto fetch = [&](int e0) __attribute__((always_inline)) {
            const bool in = e0 + lane < len;
            const int64_t at = in ? st.lo + e0 + lane : st.lo;
            uint32_t col, bits;
            drained_global_load_2(a.col_idx + at, a.vals + at, col, bits);
            o = in ? col * (uint32_t)sizeof(TV) : kNowhere;
            x = in ? (double)__uint_as_float(bits) : 0.0;
            cur = (double)drained_buffer_load(vdesc, o, TV{});
        };
#pragma unroll 1
        for (int e0 = 0; e0 < len; e0 += kWave) {
            fetch(e0);
            acc += cur * x;
        }
        const double c = step_coefficient(st.zs, st.cs, wave_sum(acc));
#pragma unroll 1
        for (int e0 = 0; e0 < len; e0 += kWave) {
            if (len > kWave) fetch(e0);
            drained_buffer_store(vdesc, o, (TV)__builtin_fma(c, x, cur));
        }
    }

    __device__ void read_records(uint32_t (&off)[kXUnits], float (&val)[kXUnits], uint32_t section) const
    {
#pragma unroll
        for (int u = 0; u < kXUnits; ++u) {
            val[u] = at_lds<float>(lds, section + (uint32_t)(u * kWave + lane) * 8u);
            off[u] = at_lds<uint32_t>(lds, section + (uint32_t)(u * kWave + lane) * 8u + 4u);
        }
    }
    __device__ static void request_values(__amdgpu_buffer_rsrc_t vres, const uint32_t (&off)[kXUnits], TV (&x)[kXUnits])
    {
#pragma unroll
        for (int u = 0; u < kXUnits; ++u) x[u] = load_state(vres, off[u], TV{});
    }

    __device__ void worker() const
    {
        const uint32_t bytes = (uint32_t)(a.d * (int64_t)sizeof(TV));
        const __amdgpu_buffer_rsrc_t vres = __builtin_amdgcn_make_buffer_rsrc(v, 0, (int)bytes, 0x00020000);
        const pu32x4 vdesc = descriptor(v, bytes);
        uint32_t off[3][kXUnits];            // blocks b, b+1, b+2
        float val[3][kXUnits];
        TV x[3][kXUnits];
        uint32_t section = L::rec;
        wait_lds_then_barrier();             // interval 0
        read_records(off[0], val[0], section);
        request_values(vres, off[0], x[0]);
        wait_lds_then_barrier();             // interval 1
        section = next_section(section);
        read_records(off[1], val[1], section);
        request_values(vres, off[1], x[1]);
        wait_lds_then_barrier();             // interval 2
        bool long_before = false;
        double zs = 0.0, cs = 0.0;           // of this lane's step (my_step) of the block to come: read a turn before they are needed
        const uint32_t mine = (uint32_t)my_step();
        auto read_scalars = [&](int64_t b) __attribute__((always_inline)) {
            const uint32_t at = step_at(b * kXSteps) + mine * 32u;
            zs = at_lds<double>(lds, at + 16u);
            cs = at_lds<double>(lds, at + 24u);
        };
        read_scalars(0);
        auto turn = [&](int64_t b, auto place) {
            constexpr int P = decltype(place)::value, NEXT = (P + 2) % 3;
            const XTold told = at_lds<XTold>(lds, told_at(b));
            section = next_section(section);
            read_records(off[NEXT], val[NEXT], section);
            double c;
            auto take = [&]() __attribute__((always_inline)) {
                double t[kXUnits];
#pragma unroll
                for (int u = 0; u < kXUnits; ++u) t[u] = (double)x[P][u] * (double)val[P][u];
                c = step_coefficient(zs, cs, sum_steps(t));
            };
            // (formed here on every path: under a branch, the compiler would wait for all loads where the paths meet)
            take();
            asm volatile("" : "+v"(c));
            uint32_t turns = 0, longs = 0;
            if (__builtin_expect(__builtin_amdgcn_readfirstlane((int)(told.rows | told.pairs)) != 0 || long_before, 0)) {
                const uint32_t rows = (uint32_t)__builtin_amdgcn_readfirstlane((int)told.rows), pairs = (uint32_t)__builtin_amdgcn_readfirstlane((int)told.pairs);
                if (long_before || (pairs & kXBefore) != 0) {              // requested before the block before stored
                    drained_values(vdesc, off[P], x[P]);
                    take();
                }
                // what a long row shares with those behind it is not known
                longs = rows >> kXSteps;
                turns = (rows | pairs | (longs != 0 ? 0u - (longs & (0u - longs)) : 0u)) & 0xFFFFu;
                if ((b + 1) * kXSteps > n) turns &= (1u << (n - b * kXSteps)) - 1u;
                if ((turns >> mine & 1u) != 0) c = 0.0;
            }
            const double cu[kXUnits] = {of_unit<0>(c), of_unit<1>(c), of_unit<2>(c), of_unit<3>(c)};
#pragma unroll
            for (int u = 0; u < kXUnits; ++u)                              // (a step without a slope leaves the vector alone)
                store_state(vres, cu[u] != 0.0 ? off[P][u] : kNowhere, (TV)__builtin_fma(cu[u], (double)val[P][u], (double)x[P][u]));
            if (__builtin_expect(turns != 0, 0)) in_turn(b, turns, longs, off[P], val[P], vdesc);
            long_before = longs != 0;
            request_values(vres, off[NEXT], x[NEXT]);
            read_scalars(b + 1);
            wait_lds_then_barrier();
        };
        for (int64_t b = 0;; b += 3) {
            turn(b, std::integral_constant<int, 0>{});
            if (b + 1 >= nblocks) break;
            turn(b + 1, std::integral_constant<int, 1>{});
            if (b + 2 >= nblocks) break;
            turn(b + 2, std::integral_constant<int, 2>{});
            if (b + 3 >= nblocks) break;
        }
        __builtin_amdgcn_s_waitcnt(0x0F70);      // all stores done before the vector is read back
    }

    // ---------------------------------------------------------------- scout
    __device__ void scout() const
    {
        uint32_t col[kXLead][kXUnits];
        float val[kXLead][kXUnits];
        int len[kXLead][kXUnits];
        const int e = lane & 15;
        pu32x4 ask[kXUnits];
        auto look = [&](int64_t r) {
#pragma unroll
            for (int u = 0; u < kXUnits; ++u) ask[u] = at_lds<pu32x4>(lds, step_at(r * kXSteps + 4 * u) + (uint32_t)(lane >> 4) * 32u);
        };
        auto request = [&](auto slot) {
            constexpr int S = decltype(slot)::value;
#pragma unroll
            for (int u = 0; u < kXUnits; ++u) {
                // (lanes behind the row's end ask for its last entry once more, those of an empty row for the matrix's first)
                const int ln = (int)ask[u][2];
                const int64_t lo = (int64_t)(((uint64_t)ask[u][1] << 32) | ask[u][0]);
                const int64_t at = ln > 0 ? lo + (e < ln ? e : ln - 1) : 0;
                len[S][u] = ln;
                col[S][u] = (uint32_t)a.col_idx[at];
                val[S][u] = a.vals[at];
            }
        };
        look(0);
        request(std::integral_constant<int, 0>{});
        look(1);
        request(std::integral_constant<int, 1>{});
        look(2);
        request(std::integral_constant<int, 2>{});
        look(3);
        request(std::integral_constant<int, 3>{});
        static_assert(kXLead == 4, "four blocks on their way");
        __builtin_amdgcn_s_waitcnt(0x0F70);  // enter the loop with an empty queue
        uint32_t section = L::rec;
        auto write = [&](int64_t r, auto slot) {
            constexpr int S = decltype(slot)::value;
            look(r + kXLead);
            bool odd = false;
#pragma unroll
            for (int u = 0; u < kXUnits; ++u) {
                const bool in = e < len[S][u];
                const float x = in ? val[S][u] : 0.0f;
                odd |= (len[S][u] > 16) | !(__builtin_fabsf(x) <= 3.4028234663852886e38f);
                pu32x2 rec;
                rec[0] = __float_as_uint(x);
                rec[1] = in ? col[S][u] * (uint32_t)sizeof(TV) : kNowhere;
                at_lds<pu32x2>(lds, section + (uint32_t)(u * kWave + lane) * 8u) = rec;
            }
            uint32_t rows = 0;
            if (__builtin_amdgcn_ballot_w64(odd) != 0) {
#pragma unroll
                for (int u = 0; u < kXUnits; ++u) {
                    const uint64_t apart = __builtin_amdgcn_ballot_w64(len[S][u] > 16);
                    const uint64_t found = apart | __builtin_amdgcn_ballot_w64(e < len[S][u] && !(__builtin_fabsf(val[S][u]) <= 3.4028234663852886e38f));
#pragma unroll
                    for (int r4 = 0; r4 < 4; ++r4)
                        rows |= ((found >> (16 * r4) & 0xFFFFu) != 0 ? 1u << (4 * u + r4) : 0u) | ((apart >> (16 * r4) & 1u) != 0 ? 0x10000u << (4 * u + r4) : 0u);
                }
            }
            if (lane == 0) at_lds<uint32_t>(lds, told_at(r)) = rows;
            section = next_section(section);
            request(slot);
        };
        const int64_t ni = intervals();
        for (int64_t i = 0;; i += 4) {
            interval([&] { write(i, std::integral_constant<int, 0>{}); });
            if (i + 1 >= ni) break;
            interval([&] { write(i + 1, std::integral_constant<int, 1>{}); });
            if (i + 2 >= ni) break;
            interval([&] { write(i + 2, std::integral_constant<int, 2>{}); });
            if (i + 3 >= ni) break;
            interval([&] { write(i + 3, std::integral_constant<int, 3>{}); });
            if (i + 4 >= ni) break;
        }
    }

    // ---------------------------------------------------------------- stamps
    __device__ void stamps() const
    {
        uint32_t section = L::rec;
        auto find = [&](int64_t r) {
            const uint32_t now = ((uint32_t)r & 255u) << 8;
            uint32_t off[kXUnits], sa[kXUnits], sb[kXUnits], back[kXUnits];
#pragma unroll
            for (int u = 0; u < kXUnits; ++u) off[u] = at_lds<uint32_t>(lds, section + (uint32_t)(u * kWave + lane) * 8u + 4u);
            section = next_section(section);
            // What is written does not depend on what is read: all units' reads and writes go out in order, and are judged afterwards.  (Lanes without
            // an entry all fall on one pair of stamps, and are not asked.)
#pragma unroll
            for (int u = 0; u < kXUnits; ++u) {
                const uint32_t c = off[u] / (uint32_t)sizeof(TV);
                const uint32_t pa = L::stamp_a + (c & (kXStamps - 1)) * 2u, pb = L::stamp_b + ((c + (c >> 14) * 2731u) & (kXStamps - 1)) * 2u;
                const uint16_t me = (uint16_t)(now | (uint32_t)(u * kWave + lane));
                sa[u] = at_lds<uint16_t>(lds, pa);
                sb[u] = at_lds<uint16_t>(lds, pb);
                at_lds<uint16_t>(lds, pa) = me;
                at_lds<uint16_t>(lds, pb) = me;
                asm volatile("" ::: "memory");          // the stamp is read back after all lanes have written (one wave's LDS accesses keep their order)
                back[u] = at_lds<uint8_t>(lds, pa);
            }
#pragma unroll
            for (int u = 0; u < kXUnits; ++u) {
                pu32x2 q;
                q[0] = sa[u] | sb[u] << 16;
                q[1] = back[u];
                at_lds<pu32x2>(lds, L::found + (uint32_t)(r & 1) * L::section + (uint32_t)(u * kWave + lane) * 8u) = q;
            }
        };
        const int64_t ni = intervals();
        for (int64_t i = 0; i < ni; ++i) interval([&] { if (i > 0) find(i - 1); });
    }

    // ---------------------------------------------------------------- pairs
    __device__ void pairs() const
    {
        uint32_t section = L::rec;
        auto find = [&](int64_t r) {
            typedef uint16_t u16x2 __attribute__((ext_vector_type(2)));
            const uint32_t now = ((uint32_t)r & 255u) << 8 | 255u;
            uint32_t off[kXUnits], ages[kXUnits];
            uint64_t seen[kXUnits], lost[kXUnits], all = 0;
#pragma unroll
            for (int u = 0; u < kXUnits; ++u) {
                const pu32x2 q = at_lds<pu32x2>(lds, L::found + (uint32_t)(r & 1) * L::section + (uint32_t)(u * kWave + lane) * 8u);
                off[u] = at_lds<uint32_t>(lds, section + (uint32_t)(u * kWave + lane) * 8u + 4u);
                // both blocks at once, in the upper bytes of the halves: how many blocks ago
                ages[u] = __builtin_bit_cast(uint32_t, (u16x2)(u16x2{(uint16_t)now, (uint16_t)now} - __builtin_bit_cast(u16x2, q[0])));
                static_assert(kXAhead == 2, "this block and the one before");
                seen[u] = __builtin_amdgcn_ballot_w64(off[u] != kNowhere && (ages[u] & 0xFE00FE00u) == 0);
                lost[u] = __builtin_amdgcn_ballot_w64(off[u] != kNowhere && q[1] != (uint32_t)(u * kWave + lane));
                all |= seen[u] | lost[u];
            }
            section = next_section(section);
            uint32_t found = 0;
            if (all != 0) {
#pragma unroll
                for (int u = 0; u < kXUnits; ++u) {
                    // Both stamps of this block: written by earlier rows of it, most likely one of them with this column.
                    uint64_t later = __builtin_amdgcn_ballot_w64(off[u] != kNowhere && (ages[u] & 0xFF00FF00u) == 0);
                    // A column that the block before and an earlier row of this one have is of the first kind, and its row is read again in its turn.
                    found |= (seen[u] & ~later) != 0 ? kXBefore : 0u;
                    uint64_t left = lost[u];
                    while (left != 0) {      // entries that lost their place to another of the four rows: to one with the same column?
                        const uint32_t place = (uint32_t)__builtin_amdgcn_readlane((int)off[u], (int)__builtin_ctzll(left));
                        const uint64_t beside = __builtin_amdgcn_ballot_w64(off[u] == place);
                        left &= ~beside;
                        later |= beside & ~(0xFFFFull << ((int)__builtin_ctzll(beside) & 48));       // all rows but the first
                    }
#pragma unroll
                    for (int r4 = 0; r4 < 4; ++r4) found |= (later >> (16 * r4) & 0xFFFFu) != 0 ? 1u << (4 * u + r4) : 0u;
                }
            }
            if (lane == 0) at_lds<uint32_t>(lds, told_at(r) + 4u) = found;
        };
        const int64_t ni = intervals();
        for (int64_t i = 0; i < ni; ++i) interval([&] { if (i > 1) find(i - 2); });
    }

    // ---------------------------------------------------------------- rows and scalars of the steps to come
    __device__ void sampler(int chain, int64_t step0) const
    {
        const double rho64 = a.pow_tab[kWave - 1] * a.rho, inv_rho64 = a.pow_tab[2 * kWave - 1];
        const double rho_pow = a.pow_tab[lane], inv_rho_pow1 = a.pow_tab[kWave + lane];
        double s_w = 1.0, eos_w = a.eta;
        int64_t lo = 0, end = 0;
        float y = 0.0f;
        auto load = [&](int64_t w) {
            const int64_t at = w * kWave + lane;
            const uint64_t step = (uint64_t)(step0 + (at < n ? at : n - 1));
            const uint32_t row = a.perm ? a.perm[shard_position((uint32_t)chain, (uint32_t)a.k, step, (uint32_t)a.m)]
                                        : sample_row(a.seed_lo, a.seed_hi, (uint32_t)chain, step, (uint32_t)a.m);
            lo = a.row_ptr[row];
            end = a.row_ptr[(int64_t)row + 1];
            y = a.y[row];
        };
        auto write = [&](int64_t w) {
            const bool live = w * kWave + lane < n;
            XStep s;
            s.lo = live ? lo : 0;
            s.len = live ? (int32_t)(end - lo) : 0;
            s.pad = 0;
            s.zs = (double)y * s_w * rho_pow * (LOSS == kLossHinge ? 1.0 : 1.4426950408889634);
            s.cs = live ? (double)y * eos_w * inv_rho_pow1 : 0.0;
            at_lds<XStep>(lds, step_at(w * kWave + lane)) = s;
            s_w *= rho64;
            eos_w *= inv_rho64;
        };
        load(0);
        write(0);
        load(1);
        write(1);
        load(2);
        __syncthreads();                     // (the others wait for the first two windows)
        const int64_t ni = intervals();
        for (int64_t i = 0; i < ni; ++i) {
            // A window is four intervals.  In interval i the scout asks for the steps up to 16 * (i + 5), and the steps from 16 * (i - 4) on are still read.
            static_assert(kXSteps * 4 == kWave && kXSteps * (kXLead + 1 + 4) + kWave <= kXRing, "the ring holds what is read and what is written");
            if ((i & 3) == 2) {
                write(i / 4 + 2);
                load(i / 4 + 3);
            }
            wait_lds_then_barrier();
        }
    }
};

template <int LOSS>
__device__ inline void run_sixteen(const ChainArgs &a, char *lds, typename StateType<LOSS>::type *v, int wave, int chain, int64_t n, int64_t step0)
{
    // Everything that is read before it is written starts at zero, and the stamps 64 blocks and more away from the first ones: when their block comes
    // they look recent, so they are of 128 different blocks, and a column finds two that differ.
    for (uint32_t o = threadIdx.x * 4u; o < XLds::bytes; o += kXThreads * 4u) {
        const uint32_t slot = o / 2u, block = o < XLds::stamp_b ? slot & 127u : slot >> 7 & 127u;
        at_lds<uint32_t>(lds, o) = o < XLds::steps ? (block + 64u) * 0x1000100u : 0u;
    }
    __syncthreads();
    const SixteenSteps<LOSS> waves(a, lds, v, n);
    if (wave == kXSampler) {
        waves.sampler(chain, step0);
        return;
    }
    __syncthreads();                         // the first two windows are there
    if (wave == kXWorker) waves.worker();
    else if (wave == kXScout) waves.scout();
    else if (wave == kXStampWave) waves.stamps();
    else waves.pairs();
}

// (A kernel of its own, and not a branch of chain_csr_pair_kernel: there it cost the other chains 0.8 %.)
template <int LOSS>
__global__ __launch_bounds__(kXThreads) void chain_csr_sixteen_kernel(ChainArgs a)
{
    using TV = typename StateType<LOSS>::type;
    __shared__ __attribute__((aligned(16))) char lds[XLds::bytes];
    const int64_t n = a.nsteps[blockIdx.x];
    // (the vector in the workspace: as in chain_csr_pair_kernel, which takes the other chains)
    if (a.status[1] != kShortApart || n < kShortWorth) return;
    const int chain = a.order[blockIdx.x];
    run_sixteen<LOSS>(a, lds, static_cast<TV *>(a.state) + (int64_t)chain * a.d, __builtin_amdgcn_readfirstlane((int)threadIdx.x / kWave), chain, n,
                      first_step(a, (int)blockIdx.x));
}

}  // namespace
}  // namespace wpsgd
