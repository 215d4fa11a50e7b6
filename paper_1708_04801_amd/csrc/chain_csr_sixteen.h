// Sparse chains of short rows that hardly ever share a column: sixteen steps at a time, the model in HBM.
//
// Four rows of at most 16 entries lie side by side in a wave, and where rows share no column their steps are independent of each other
// but for the shrink, which the steps' scalars carry.  chain_csr_short.h takes four such steps at once and holds two things against itself: a value that an
// earlier group has written must be read again, so the worker waits for memory, and a group whose rows share a column runs step by
// step.  Here a shared column is an addition instead:
//
//   Updates are additions made at the L2 (buffer atomics without a result), which need no current value.  So a value, requested kXAhead
//   blocks before its block's turn, can be old in a product only, and what it lacks is known: the earlier step's coefficient times
//   the product of the two entries.  Such a pair is an item, and an item costs the chain a multiply-add.
//
//   Pairs are found from the rows alone, two blocks ahead of the chain.  Two stamp tables (two hashes of the column) hold the block and the entry
//   that wrote last: an entry that finds recent blocks in both is a candidate, and so is one that, of the four rows taken together, did not find
//   its own number again.  Candidates are compared with the entries of the rows before them; there are few.
//
// Five waves, one barrier per block of sixteen steps:
//   worker  products, slopes and additions of block b; requests the values of block b + kXAhead
//   scout   fetches the rows' entries kXLead blocks ahead and writes records: value, place of the column
//   stamps  the tables and the candidates
//   items   the candidates' pairs
//   sampler the rows of the steps to come, 64 at a time, and the scalars of the recursion
// A block with a row of more than 16 entries, with an element that is not finite (a slope of 0 times it is one too), or with more pairs than the lists
// hold runs step by step on the sampler's wave while the others wait; values requested before it are requested again.
//
// What bounds it: the worker's chain through a block, some 1150 cycles of the 1480 between two barriers at d = a million (products and sums 670, the
// branch for items 200, additions and requests 140), and the stamps beside it (1160); the rest is what the slowest of five waves has over the worker
// from block to block.  An item costs some hundred cycles.  Ten chains of up to 100000 steps, 5 to 10 of 100000 columns: 5.70 ms four
// steps at a time, 4.04 this way (0.057 and 0.040 us per step).  Tried: blocks of 32 steps (0.057: twice the pairs and the stamps), sums unit by
// unit in four registers instead of folded into one (0.0449), scalars read in the block's own turn (0.0477).
// Precision: products, sums and slopes' arguments in fp64 for either loss; the fp32 state of the logistic loss takes a rounded product where it took a
// fused multiply-add: error against fp64 after 10000 steps 5.89e-8 before, 5.85e-8 now (d = 100000; the output's own rounding is most of it).
#pragma once

namespace wpsgd {
namespace {

constexpr int kXUnits = 4, kXSteps = 4 * kXUnits;     // steps per block; waves' widths of 64 entries: unit u, lane 16*r + e: entry e of step 4*u + r
constexpr int kXLead = 4;                    // scout: blocks between the request of a row's entries and their records
constexpr int kXAhead = 2;                   // worker: blocks between the request of a value and its block's turn: it misses what the block before and its own write
constexpr int kXTurn = 3;                    // in interval i records of block i are written, candidates of block i-1 and items of block i-2 found, block i-3 taken
constexpr int kXStamps = 16384;              // entries of either table
constexpr int kXRing = 256;                  // steps whose rows and scalars are kept
constexpr int kXLists = 64;                  // items and candidates per block
constexpr int kXWorker = 0, kXScout = 1, kXStampWave = 2, kXItemWave = 3, kXSampler = 4, kXWaves = 5;
constexpr int kXThreads = kXWaves * kWave;
constexpr uint32_t kNowhere = 0xFFFFFFF0u;   // past the end of any buffer: no access

struct __attribute__((aligned(16))) XStep {
    int64_t lo;           // first entry of the row
    int32_t len, pad;
    double zs, cs;        // y*s_l (times log2 e for the logistic loss) and y*eta/s_{l+1}; len = 0 and cs = 0 past the chain's end
};
struct __attribute__((aligned(16))) XItem {  // product of two entries, of step a (modulo 64) and of the later step j (of the block)
    double product;
    int32_t a, j;
};
struct __attribute__((aligned(16))) XTold {  // what the other waves have found out about a block
    uint32_t odd;         // a byte per wave that can tell that it runs step by step
    int32_t across, inside;       // items with the block before, between steps of the block
    int32_t cands;
};
struct XLds {
    static constexpr uint32_t section = kXUnits * kWave * 8;                         // records of a block: {value, byte offset}
    static constexpr uint32_t stamp_a = 0;                                           // 16 bits: entry of the block, block modulo 256
    static constexpr uint32_t stamp_b = stamp_a + kXStamps * 2;
    static constexpr uint32_t steps = stamp_b + kXStamps * 2;
    static constexpr uint32_t rec = steps + kXRing * 32;                             // four sections
    static constexpr uint32_t coef = rec + 4 * section;                              // coefficients of the last 64 steps
    static constexpr uint32_t sums = coef + 64 * 8;                                  // the block's sums, where steps of it share a column
    static constexpr uint32_t items = sums + kXSteps * 8;                            // two lists of items with earlier blocks
    static constexpr uint32_t within = items + 2 * kXLists * 16;                     // two lists of items between steps of the block
    static constexpr uint32_t cands = within + 2 * kXLists * 16;                     // two lists: 16 bits, entry of the block
    static constexpr uint32_t losers = cands + 2 * kXLists * 2;                      // two blocks: per unit, the lanes that lost their place in table a
    static constexpr uint32_t told = losers + 2 * kXUnits * 8;                       // eight blocks: XTold
    static constexpr uint32_t bytes = told + 8 * 16;
    static_assert(kXUnits * kWave == 256 && steps % 16 == 0 && rec % 16 == 0 && items % 16 == 0 && within % 16 == 0 && losers % 16 == 0 && told % 16 == 0, "alignment");
};

template <typename T> __device__ inline T &at_lds(char *lds, uint32_t off) { return *reinterpret_cast<T *>(lds + off); }
__device__ inline void lds_add(char *lds, uint32_t off, double x)
{
    unsafeAtomicAdd(reinterpret_cast<double *>(lds + off), x);                       // ds_add_f64, no result
}

// raw buffer atomics (no result: the intrinsic's is unused); dropped past the buffer's end like any raw access
extern "C" __device__ double wpsgd_buffer_add_f64(double, __amdgpu_buffer_rsrc_t, int, int, int) __asm("llvm.amdgcn.raw.ptr.buffer.atomic.fadd.f64");
extern "C" __device__ float wpsgd_buffer_add_f32(float, __amdgpu_buffer_rsrc_t, int, int, int) __asm("llvm.amdgcn.raw.ptr.buffer.atomic.fadd.f32");
__device__ inline void state_add(__amdgpu_buffer_rsrc_t r, uint32_t off, double x) { (void)wpsgd_buffer_add_f64(x, r, (int)off, 0, 0); }
__device__ inline void state_add(__amdgpu_buffer_rsrc_t r, uint32_t off, float x) { (void)wpsgd_buffer_add_f32(x, r, (int)off, 0, 0); }
// device scope: what the additions left at the L2, whatever a first-level line may hold
constexpr int kDeviceScope = 16;
__device__ inline double state_load(__amdgpu_buffer_rsrc_t r, uint32_t off, double)
{
    const pu32x2 q = __builtin_amdgcn_raw_buffer_load_b64(r, off, 0, kDeviceScope);
    return __longlong_as_double(((long long)q[1] << 32) | (long long)q[0]);
}
__device__ inline float state_load(__amdgpu_buffer_rsrc_t r, uint32_t off, float)
{
    return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(r, off, 0, kDeviceScope));
}
// the same in a statement of its own that waits, for the paths off the common one (see drained_buffer_load)
__device__ inline double drained_state_load(pu32x4 rsrc, uint32_t off, double)
{
    double r;
    asm volatile("s_nop 3\n\ts_waitcnt vmcnt(0)\n\tbuffer_load_dwordx2 %0, %1, %2, 0 offen sc1\n\ts_waitcnt vmcnt(0)" : "=v"(r) : "v"(off), "s"(rsrc) : "memory");
    return r;
}
__device__ inline float drained_state_load(pu32x4 rsrc, uint32_t off, float)
{
    float r;
    asm volatile("s_nop 3\n\ts_waitcnt vmcnt(0)\n\tbuffer_load_dword %0, %1, %2, 0 offen sc1\n\ts_waitcnt vmcnt(0)" : "=v"(r) : "v"(off), "s"(rsrc) : "memory");
    return r;
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
    __device__ static constexpr uint32_t told_at(int64_t r) { return L::told + (uint32_t)(r & 7) * 16u; }
    __device__ static uint32_t next_section(uint32_t s) { return s == L::rec + 3 * L::section ? L::rec : s + L::section; }
    __device__ int64_t intervals() const { return nblocks + kXTurn; }
    __device__ uint32_t flag_word(int64_t b) const { return at_lds<uint32_t>(lds, told_at(b)); }
    __device__ static bool is_odd(uint32_t word) { return __builtin_amdgcn_readfirstlane((int)word) != 0; }

    // interval i of a wave that has no part in a block that runs step by step
    template <typename F>
    __device__ void interval(int64_t i, F &&work) const
    {
        const uint32_t word = flag_word(i - kXTurn);
        work();
        const bool odd = i >= kXTurn && is_odd(word);
        wait_lds_then_barrier();
        if (__builtin_expect(odd, 0)) wait_lds_then_barrier();
    }

    // ---------------------------------------------------------------- worker
    __device__ static double step_coefficient(double zs, double cs, double sum) { return (double)unit_slope<LOSS>((TV)(zs * sum)) * cs; }

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

    // A block's steps where some share a column.  Lane i: the i-th item with the block before (`it`) and its earlier step's coefficient.
    __device__ double with_items(int64_t b, int across, int inside, const XItem &it, double earlier, double sum, double c, double zs, double cs) const
    {
        const uint32_t mine = (uint32_t)my_step();
        if (across > 0) {
            const double add = it.product * earlier;
#pragma unroll 1
            for (int q = 0; q < across; ++q) sum += __builtin_amdgcn_readlane(it.j, q) == (int)mine ? lane_read(add, q) : 0.0;
            c = step_coefficient(zs, cs, sum);
        }
        if (inside > 0) {
            // In the order of their later steps: a step's coefficient is final when its turn comes.
            const uint32_t coef = L::coef + (uint32_t)((b * kXSteps) & 63) * 8u + mine * 8u;
            at_lds<double>(lds, L::sums + mine * 8u) = sum;
            at_lds<double>(lds, coef) = c;
            asm volatile("" ::: "memory");   // (one wave's LDS accesses keep their order)
            const XItem within = at_lds<XItem>(lds, L::within + (uint32_t)(b & 1) * (kXLists * 16) + (uint32_t)lane * 16u);
            uint64_t all = __builtin_amdgcn_ballot_w64(lane < inside);
#pragma unroll 1
            while (all != 0) {
                uint64_t left = all;         // those of the first later step, bit by bit
#pragma unroll
                for (int bit = 3; bit >= 0; --bit) {
                    const uint64_t zero = left & __builtin_amdgcn_ballot_w64((within.j >> bit & 1) == 0);
                    left = zero != 0 ? zero : left;
                }
                all &= ~left;
                const int j = __builtin_amdgcn_readlane(within.j, (int)__builtin_ctzll(left));
                const uint32_t st = step_at(b * kXSteps + j);
                double p = at_lds<double>(lds, L::sums + (uint32_t)j * 8u);
                while (left != 0) {
                    const int l = (int)__builtin_ctzll(left);
                    left &= left - 1;
                    p += lane_read(within.product, l) * at_lds<double>(lds, L::coef + (uint32_t)(__builtin_amdgcn_readlane(within.a, l) & 63) * 8u);
                }
                at_lds<double>(lds, L::coef + (uint32_t)((b * kXSteps + j) & 63) * 8u) =
                    step_coefficient(at_lds<double>(lds, st + 16u), at_lds<double>(lds, st + 24u), p);
                asm volatile("" ::: "memory");
            }
            c = at_lds<double>(lds, coef);
        }
        return c;
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
        for (int u = 0; u < kXUnits; ++u) x[u] = state_load(vres, off[u], TV{});
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
        bool odd_before = false, odd_before2 = false;
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
            const XItem it = at_lds<XItem>(lds, L::items + (uint32_t)(b & 1) * (kXLists * 16) + (uint32_t)lane * 16u);       // (whatever is there)
            section = next_section(section);
            read_records(off[NEXT], val[NEXT], section);
            const double earlier = at_lds<double>(lds, L::coef + (uint32_t)(it.a & 63) * 8u);
            double sum, c;
            auto take = [&](const TV (&value)[kXUnits]) __attribute__((always_inline)) {
                double t[kXUnits];
#pragma unroll
                for (int u = 0; u < kXUnits; ++u) t[u] = (double)value[u] * (double)val[P][u];
                sum = sum_steps(t);
                c = step_coefficient(zs, cs, sum);
            };
            // (formed here on every path: under a branch, the compiler would wait for all loads where the paths meet)
            take(x[P]);
            asm volatile("" : "+v"(c), "+v"(sum));
            bool odd = false;
            const bool again = odd_before || odd_before2;      // requested before a block that ran step by step
            if (__builtin_amdgcn_readfirstlane((int)told.odd | told.across | told.inside) != 0 || again) {
                odd = is_odd(told.odd);
                if (!odd && again) {
                    TV fresh[kXUnits];
#pragma unroll
                    for (int u = 0; u < kXUnits; ++u) fresh[u] = drained_state_load(vdesc, off[P][u], TV{});
                    take(fresh);
                }
                const int across = again ? 0 : __builtin_amdgcn_readfirstlane(told.across), inside = __builtin_amdgcn_readfirstlane(told.inside);
                if (!odd && (across | inside) != 0) c = with_items(b, across, inside, it, earlier, sum, c, zs, cs);
                if (odd) c = 0.0;
            }
            const double cu[kXUnits] = {of_unit<0>(c), of_unit<1>(c), of_unit<2>(c), of_unit<3>(c)};
#pragma unroll
            for (int u = 0; u < kXUnits; ++u)                              // (a step without a slope leaves the vector alone)
                state_add(vres, cu[u] != 0.0 ? off[P][u] : kNowhere, (TV)(cu[u] * (double)val[P][u]));
            request_values(vres, off[NEXT], x[NEXT]);
            at_lds<double>(lds, L::coef + (uint32_t)((b * kXSteps) & 63) * 8u + mine * 8u) = c;
            read_scalars(b + 1);
            odd_before2 = odd_before;
            odd_before = odd;
            if (__builtin_expect(odd, 0)) {
                asm volatile("s_waitcnt vmcnt(0)" ::: "memory");           // the additions are made before the block's steps
                wait_lds_then_barrier();
            }
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
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");                   // all additions made
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
            const bool any = __builtin_amdgcn_ballot_w64(odd) != 0;
            if (lane == 0) at_lds<uint8_t>(lds, told_at(r)) = any ? 1 : 0;
            section = next_section(section);
            request(slot);
        };
        const int64_t ni = intervals();
        for (int64_t i = 0;; i += 4) {
            interval(i, [&] { write(i, std::integral_constant<int, 0>{}); });
            if (i + 1 >= ni) break;
            interval(i + 1, [&] { write(i + 1, std::integral_constant<int, 1>{}); });
            if (i + 2 >= ni) break;
            interval(i + 2, [&] { write(i + 2, std::integral_constant<int, 2>{}); });
            if (i + 3 >= ni) break;
            interval(i + 3, [&] { write(i + 3, std::integral_constant<int, 3>{}); });
            if (i + 4 >= ni) break;
        }
    }

    // ---------------------------------------------------------------- candidates
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
            uint64_t seen[kXUnits], lost[kXUnits], all = 0;
            typedef uint16_t u16x2 __attribute__((ext_vector_type(2)));
#pragma unroll
            for (int u = 0; u < kXUnits; ++u) {
                const bool real = off[u] != kNowhere;
                // both blocks at once, in the upper bytes of the halves: how many blocks ago
                const u16x2 latest = {(uint16_t)(now | 255u), (uint16_t)(now | 255u)};
                const uint32_t ages = __builtin_bit_cast(uint32_t, (u16x2)(latest - __builtin_bit_cast(u16x2, sa[u] | sb[u] << 16)));
                static_assert(kXAhead == 2, "this block and the one before");
                seen[u] = __builtin_amdgcn_ballot_w64(real & ((ages & 0xFE00FE00u) == 0));
                lost[u] = __builtin_amdgcn_ballot_w64(real & (back[u] != (uint32_t)(u * kWave + lane)));
                all |= seen[u] | lost[u];
            }
            int count = 0;
            if (all != 0) {
#pragma unroll
                for (int u = 0; u < kXUnits; ++u) {
                    const uint64_t any = seen[u] | lost[u];
                    const int place = count + (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(any >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)any, 0u));
                    if ((any >> lane & 1u) != 0 && place < kXLists)
                        at_lds<uint16_t>(lds, L::cands + (uint32_t)(r & 1) * (kXLists * 2) + (uint32_t)place * 2u) = (uint16_t)(u * kWave + lane);
                    if (lane == 0) at_lds<uint64_t>(lds, L::losers + (uint32_t)(r & 1) * (kXUnits * 8) + u * 8u) = lost[u];
                    count += (int)__builtin_popcountll(any);
                }
            }
            if (lane == 0) at_lds<int>(lds, told_at(r) + 12u) = count;
        };
        const int64_t ni = intervals();
        for (int64_t i = 0; i < ni; ++i) interval(i, [&] { if (i > 0) find(i - 1); });
    }

    // ---------------------------------------------------------------- items
    __device__ void items() const
    {
        static_assert(kXAhead == 2, "the entries of one block before are compared");
        uint32_t off[2][kXUnits], val[2][kXUnits];             // places and values of the entries of this block and the one before, in turn
#pragma unroll
        for (int q = 0; q < 2; ++q)
#pragma unroll
            for (int u = 0; u < kXUnits; ++u) {
                off[q][u] = kNowhere;
                val[q][u] = 0u;
            }
        uint32_t section = L::rec;
        auto find = [&](int64_t r, auto turn) {
            constexpr int NOW = decltype(turn)::value, BEFORE = 1 - NOW;
#pragma unroll
            for (int u = 0; u < kXUnits; ++u) {
                const pu32x2 q = at_lds<pu32x2>(lds, section + (uint32_t)(u * kWave + lane) * 8u);
                val[NOW][u] = q[0];
                off[NOW][u] = q[1];
            }
            section = next_section(section);
            const int count = __builtin_amdgcn_readfirstlane(at_lds<int>(lds, told_at(r) + 12u));
            int across = 0, inside = 0;
            if (count > kXLists) across = kXLists + 1;                     // (as many would take longer than the block's steps)
            if (count > 0 && count <= kXLists) {
                const int mine = at_lds<uint16_t>(lds, L::cands + (uint32_t)(r & 1) * (kXLists * 2) + (uint32_t)lane * 2u);
#pragma unroll 1
                for (int q = 0; q < count; ++q) {
                    const int entry = __builtin_amdgcn_readlane(mine, q), unit = entry / kWave, who = entry & (kWave - 1), row = who >> 4;
                    uint32_t o = off[NOW][0], w = val[NOW][0];
#pragma unroll
                    for (int u = 1; u < kXUnits; ++u) {
                        o = u == unit ? off[NOW][u] : o;
                        w = u == unit ? val[NOW][u] : w;
                    }
                    const uint32_t place = (uint32_t)__builtin_amdgcn_readlane((int)o, who);
                    const double x = (double)__uint_as_float((uint32_t)__builtin_amdgcn_readlane((int)w, who));
                    uint32_t bits = 0;       // bit 7 - R: this lane's entry of unit R of the two blocks has the column
#pragma unroll
                    for (int R = 0; R < 2 * kXUnits; ++R) bits = 2u * bits + (off[R < kXUnits ? BEFORE : NOW][R % kXUnits] == place ? 1u : 0u);
                    const uint64_t losers = at_lds<uint64_t>(lds, L::losers + (uint32_t)(r & 1) * (kXUnits * 8) + (uint32_t)unit * 8u);
                    const uint32_t here = 1u << (kXUnits - 1 - unit);
                    const uint64_t beside = __builtin_amdgcn_ballot_w64((bits & here) != 0);        // the unit's lanes with this column
                    // entry l of unit R, with the entry of step j of the block
                    auto item_of = [&](int R, int l, double xa, double xj, int j) __attribute__((always_inline)) {
                        XItem it;
                        it.product = xa * xj;
                        it.a = (int32_t)((r * kXSteps + R * 4 - kXSteps + (l >> 4)) & 63);
                        it.j = j;
                        return it;
                    };
                    auto value_of = [&](int R, int l) __attribute__((always_inline)) {
                        uint32_t t = 0;
#pragma unroll
                        for (int s = 0; s < 2 * kXUnits; ++s) t = s == R ? val[s < kXUnits ? BEFORE : NOW][s % kXUnits] : t;
                        return (double)__uint_as_float((uint32_t)__builtin_amdgcn_readlane((int)t, l));
                    };
                    // with the rows of earlier units
                    const uint32_t earlier = bits & ~(2u * here - 1u);
                    uint64_t lanes = __builtin_amdgcn_ballot_w64(earlier != 0);
                    while (lanes != 0) {
                        const int l = (int)__builtin_ctzll(lanes);
                        lanes &= lanes - 1;
                        uint32_t found = (uint32_t)__builtin_amdgcn_readlane((int)earlier, l);
                        while (found != 0) {
                            const int R = 2 * kXUnits - 1 - (int)__builtin_ctz(found);
                            found &= found - 1;
                            const XItem it = item_of(R, l, value_of(R, l), x, 4 * unit + row);
                            const bool before = R < kXUnits;
                            const int place_of = before ? across : inside;
                            if (lane == 0 && place_of < kXLists)
                                at_lds<XItem>(lds, (before ? L::items : L::within) + (uint32_t)(r & 1) * (kXLists * 16) + (uint32_t)place_of * 16u) = it;
                            across += before ? 1 : 0;
                            inside += before ? 0 : 1;
                        }
                    }
                    // Rows of its own unit: an entry that lost its place to one of them.  All pairs of the column at once, when its first loser is looked at.
                    const uint64_t self = 1ull << who;
                    if ((losers & self) != 0 && (losers & beside & (self - 1ull)) == 0) {
                        uint64_t later = beside;
                        while (later != 0) {
                            const int lj = (int)__builtin_ctzll(later);
                            later &= later - 1;
                            uint64_t before = beside & ((1ull << lj) - 1ull);
                            const double xj = value_of(kXUnits + unit, lj);
                            while (before != 0) {
                                const int la = (int)__builtin_ctzll(before);
                                before &= before - 1;
                                const XItem it = item_of(kXUnits + unit, la, value_of(kXUnits + unit, la), xj, 4 * unit + (lj >> 4));
                                if (lane == 0 && inside < kXLists) at_lds<XItem>(lds, L::within + (uint32_t)(r & 1) * (kXLists * 16) + (uint32_t)inside * 16u) = it;
                                ++inside;
                            }
                        }
                    }
                }
            }
            if (lane == 0) {
                at_lds<int>(lds, told_at(r) + 4u) = across < kXLists ? across : kXLists;
                at_lds<int>(lds, told_at(r) + 8u) = inside < kXLists ? inside : kXLists;
                at_lds<uint8_t>(lds, told_at(r) + 1u) = across > kXLists || inside > kXLists ? 1 : 0;
            }
        };
        const int64_t ni = intervals();
        for (int64_t i = 0;; i += 2) {
            interval(i, [&] { if (i > 1) find(i - 2, std::integral_constant<int, 0>{}); });
            if (i + 1 >= ni) break;
            interval(i + 1, [&] { if (i > 0) find(i - 1, std::integral_constant<int, 1>{}); });
            if (i + 2 >= ni) break;
        }
    }

    // ---------------------------------------------------------------- rows and scalars of the steps to come; steps one by one
    __device__ void step_by_step(int64_t b) const
    {
        const pu32x4 vdesc = descriptor(v, (uint32_t)(a.d * (int64_t)sizeof(TV)));
#pragma unroll 1
        for (int64_t t = b * kXSteps; t < (b + 1) * kXSteps && t < n; ++t) {
            const XStep st = at_lds<XStep>(lds, step_at(t));
            const int len = __builtin_amdgcn_readfirstlane(st.len);
            double acc = 0.0;
#pragma unroll 1
            for (int e0 = 0; e0 < len; e0 += kWave) {
                const bool in = e0 + lane < len;
                const uint32_t c = drained_global_load_u32(a.col_idx + (in ? st.lo + e0 + lane : st.lo));
                const float x = __uint_as_float(drained_global_load_u32(a.vals + (in ? st.lo + e0 + lane : st.lo)));
                const double cur = (double)drained_state_load(vdesc, in ? c * (uint32_t)sizeof(TV) : kNowhere, TV{});
                if (in) acc += cur * (double)x;
            }
            const double coef = step_coefficient(st.zs, st.cs, wave_sum(acc));
#pragma unroll 1
            for (int e0 = 0; e0 < len; e0 += kWave) {
                const bool in = e0 + lane < len;
                const uint32_t c = drained_global_load_u32(a.col_idx + (in ? st.lo + e0 + lane : st.lo));
                const float x = __uint_as_float(drained_global_load_u32(a.vals + (in ? st.lo + e0 + lane : st.lo)));
                const uint32_t off = in ? c * (uint32_t)sizeof(TV) : kNowhere;
                const double cur = (double)drained_state_load(vdesc, off, TV{});
                drained_buffer_store(vdesc, off, (TV)(cur + coef * (double)x));
            }
        }
    }

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
            const int64_t b = i - kXTurn;
            const bool odd = b >= 0 && is_odd(flag_word(b));
            wait_lds_then_barrier();
            if (__builtin_expect(odd, 0)) {
                step_by_step(b);
                wait_lds_then_barrier();
            }
        }
    }
};

template <int LOSS>
__device__ inline void run_sixteen(const ChainArgs &a, char *lds, typename StateType<LOSS>::type *v, int wave, int chain, int64_t n, int64_t step0)
{
    // stamps: half the range of block numbers away from the first blocks; everything else that is read before it is written starts at zero
    for (uint32_t o = threadIdx.x * 4u; o < XLds::bytes; o += kXThreads * 4u) at_lds<uint32_t>(lds, o) = o < XLds::steps ? 0x80008000u : 0u;
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
    else waves.items();
}

// (waves_per_eu: with the default, which aims at the most waves the workgroup's size allows, the same code is scheduled for fewer registers and takes
// 4.64 ms instead of 4.06.  A kernel of its own, and not a branch of chain_csr_pair_kernel: there it cost the other chains 0.8 %.)
template <int LOSS>
__global__ __launch_bounds__(kXThreads) __attribute__((amdgpu_waves_per_eu(1, 2))) void chain_csr_sixteen_kernel(ChainArgs a)
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
