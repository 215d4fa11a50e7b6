// Sparse chains whose rows are short (at most 16 entries, nearly all of them) and seldom share columns: four steps at a
// time, one row of 16 lanes each.
//
// A short row leaves most of a wave idle, and two short rows of a wide matrix seldom share a column.  Steps
// whose rows share none are independent of each other but for the shrink, which the per-step scalars carry:
// their products, slopes and updates can be taken side by side with the results of one step after the
// other.  A group is four consecutive steps; lane 16*r + e holds entry e of the row of its step r.
//
// The waves and the ring are those of chain_csr_pair_kernel with a group in the place of a step: the record scout
// writes 64 records and four steps' scalars per group, the stamp scout marks
//   stale      groups whose HBM-resident values were fetched before one of the last 2*kShortAhead groups wrote them,
//   in turn    groups in which two rows share a column (or a slot of the table that finds them: every lane
//              writes its number to the slot of its column and reads the slot back; of two lanes with one
//              column at most one finds its own number), or in which a row is longer than 16 entries.
// The worker takes a group in turn step by step, reading every value when its step comes; so it takes the group in which
// the chain ends, and leaves out the steps behind the end.  The steps after a long
// row re-read their values, since its columns leave no stamps.
//
// What bounds it: some 480 cycles a group, much the same with fp64 and with fp32 state: the stamp scout's tables beside
// the worker's dependent chain (LDS read, product, four levels of a sum over 16 lanes, slope, LDS write): without the
// tables, for timing only, 0.033 us per step; a fourth wave for the shared columns gained 2 % here and lost half a per
// cent on long rows; groups that re-read or run in turn cost an eighth.  Ten chains of up to 100000 steps, rows of 5 to 10
// entries, d = 100000: 0.213 us per step one at a time, 0.057 this way (21.3 -> 5.7 ms).  Requests three or six groups
// ahead instead of four: the same within 2 %.
#pragma once

namespace wpsgd {
namespace {

constexpr int kShortLen = 16;                // entries per row of lanes
constexpr int kShortRows = 4;                // steps per group
constexpr int kShortLead = 2 * kG;           // scouts: groups between a row's request and its records: one window of 64 steps
static_assert(kShortLead * kShortRows == kWave, "one window ahead: requests read the next window's tables");
constexpr uint32_t kShortScalars = 32;       // bytes per step: StepScalars, StepRow
constexpr uint32_t kGroupBytes = kWave * 16 + kShortRows * kShortScalars;
constexpr uint32_t kShortSectionBytes = kG * kGroupBytes;
constexpr int kShortAhead = 4;               // worker: HBM-resident values are requested this many groups ahead
constexpr uint16_t kShortRecent = 2 * kShortAhead;
static_assert(kShortAhead + 1 < kG, "record and value rings are indexed modulo kG");
constexpr int kStale = 1, kInTurn = 2;       // marks of a group, in the pad of its first StepRow

constexpr int kOwners = 16384;               // slots of the table that finds shared columns
struct __attribute__((aligned(16))) RowToRequest {
    int64_t lo;           // first entry (1 for a row without entries: its lanes request entry 0 and drop it)
    int32_t len, pad;
};

template <typename TV>
struct ShortLds {
    static constexpr uint32_t head = 0;                                           // kPHead model values, then one scratch slot per lane
    static constexpr uint32_t head_scratch = head + kPHead * sizeof(TV);
    static constexpr uint32_t stamp_a = head_scratch + kWave * sizeof(TV);        // kPStamps + scratch slots
    static constexpr uint32_t stamp_b = stamp_a + (kPStamps + kWave) * 2;
    static constexpr uint32_t owner = stamp_b + (kPStamps + kWave) * 2;           // which lane of a group holds a column
    static constexpr uint32_t rows = (owner + (kOwners + kWave) + 15u) & ~15u;    // per scout, 64 rows to request: RowToRequest
    static constexpr uint32_t ring = rows + 2 * kWave * 16;
    static constexpr uint32_t bytes = ring + kSections * kShortSectionBytes;
};

// Do a matrix's chains run faster four steps at a time?  One workgroup of the launch in front of the chains looks at 768
// rows spread over the matrix and leaves the answer in the workspace; either answer gives correct results.
//   Rows: hardly any may be longer than 16 entries.
//   Shared columns: 192 of the rows, also spread over all of it, are put into 48 groups of four, and the groups that share a
//   column counted.  us per step (ten chains, 5 to 10 entries, fp64), one at a time | a group in turn | side by side:
//   0.22 | 0.45 | 0.06 if the group has HBM-resident columns, which it then reads and writes four times over, and
//   0.22 | 0.20 | 0.06 if all its columns are in LDS.  The first costs more than it gains from two groups in five on (a
//   column that all rows share, such as a constant term, at d = 100000: 0.22 one at a time, 0.46 in groups).  The second
//   has to earn back the start of the scouts' deeper pipeline.
//   Rows far apart: among the 48 rows that a wave looks at, entries that find their column with one looked at before are counted.  Sixteen steps
//   at a time (chain_csr_sixteen.h) read some values again for each such pair, where groups of four hardly notice one.  us, four at a time | sixteen, ten
//   chains of 10000 steps, hinge, uniform columns (the count expected): 5 to 10 entries, d = 10000 (20) 641 | 657, 15000 (13) 633 | 597, 30000 (7)
//   632 | 493, 100000 (2) 620 | 400; 12 to 16 entries, d = 15000 (45) 1014 | 953, 60000 (14) 938 | 615; 2 or 3 entries, d = 2000 (11) 523 | 536, 5000 (5)
//   514 | 436.  Rows that come back are not counted: with 1000 rows of 5 to 10 entries 636 | 441, with 200 802 | 605; fewer show as pairs.
constexpr uint32_t kShortAlways = 1, kShortLongChains = 2, kShortApart = 3;       // answers, in the word behind the status word
constexpr int kLookPairs = 16;
// Calls with fewer columns do without the count and the launch, 2 us of a call whose matrix is refused (200 steps, 5 to 10 entries, d = 100000: 49 one way,
// 37 the other).  Rows of 5 to 10 entries are near the line there; ones of two or three would gain down to d = 3000.
constexpr int64_t kApartColumns = 24576;
constexpr int kLookThreads = 256, kLookEach = 3, kLookGroups = 48, kLookMost = 19, kLookSlots = 4096;
// Chains of less than 128 steps do not earn back that start (8 steps of rows without a shared column: 24 us one at a
// time, 30 in groups; 100 steps, d = 100000: 52.6 and 52.5), nor ones of less than 512 if most groups run in turn.
constexpr int64_t kShortWorth = 128, kShortWorthInTurn = 512;

// owner: this wave's table.  (All loads of the look go out at once, a quarter of the groups per wave: two trips to memory.)
__device__ inline void look_for_short_rows(const int64_t *row_ptr, const int32_t *col_idx, int64_t m, int64_t d, uint8_t *owner, uint32_t *answer)
{
    constexpr int kRows = kLookThreads * kLookEach, kMine = kLookGroups / (kLookThreads / kWave);        // groups of a wave
    static_assert(kMine <= kShortLen, "lane 16*r + g holds row r of the wave's group g");
    const int lane = (int)(threadIdx.x & (kWave - 1)), wave = (int)threadIdx.x / kWave, r = lane / kShortLen, e = lane % kShortLen;
    auto row_of = [&](int i) { return (int64_t)((uint64_t)i * (uint64_t)m / kRows); };
    const int64_t entries = row_ptr[m];
    int too_long = 0;
#pragma unroll
    for (int q = 0; q < kLookEach; ++q) {
        const int64_t row = row_of((int)threadIdx.x * kLookEach + q);
        too_long |= row_ptr[row + 1] - row_ptr[row] > kShortLen;
    }
    // (the four rows of a group lie a quarter of the matrix apart)
    const int64_t row = row_of((r * kLookGroups + wave * kMine + (e < kMine ? e : 0)) * (kRows / (kShortRows * kLookGroups)));
    const int64_t lo = row_ptr[row], len = row_ptr[row + 1] - lo;
    uint32_t col[kMine], real = 0;
#pragma unroll
    for (int g = 0; g < kMine; ++g) {
        const int from = r * kShortLen + g;
        const int64_t p = (int64_t)(((uint64_t)(uint32_t)__shfl((int)(lo >> 32), from) << 32) | (uint32_t)__shfl((int)(uint32_t)lo, from));
        const bool in = e < __shfl((int)len, from);
        real |= in ? 1u << g : 0u;
        col[g] = 0;
        if (entries > 0) col[g] = (uint32_t)col_idx[in ? p + e : 0];         // (the matrix has an entry 0)
    }
    // (the columns are on their way: other matrices need not wait for them)
    if (__syncthreads_count(too_long) > 1 || entries == 0) {
        if (threadIdx.x == 0) *answer = 0u;
        return;
    }
    int npairs = kLookPairs + 1;
    if (d >= kApartColumns) {
        // the wave's rows against those it has looked at before: a table of columns (one that another column has replaced is not found again)
        uint32_t *const seen = reinterpret_cast<uint32_t *>(owner);
        constexpr int kSeen = kLookSlots / 4;
#pragma unroll
        for (int q = 0; q < kSeen / kWave; ++q) seen[q * kWave + lane] = 0;
        uint32_t before[kMine];
#pragma unroll
        for (int g = 0; g < kMine; ++g) {
            uint32_t *const slot = seen + ((real >> g) & 1u ? col[g] & (kSeen - 1) : (uint32_t)(kSeen + e));
            asm volatile("" ::: "memory");      // (one wave's LDS accesses keep their order)
            before[g] = *slot;
            *slot = col[g] + 1u;
        }
        asm volatile("" ::: "memory");
        npairs = 0;
#pragma unroll
        for (int g = 0; g < kMine; ++g) npairs += (int)__builtin_popcountll(__builtin_amdgcn_ballot_w64(((real >> g) & 1u) != 0 && before[g] == col[g] + 1u));
    }
    uint32_t in_turn = 0, far = 0;            // a bit per group
    int who[kMine];
#pragma unroll
    for (int g = 0; g < kMine; ++g) {
        uint8_t *const slot = owner + ((real >> g) & 1u ? col[g] & (kLookSlots - 1) : (uint32_t)(kLookSlots + lane));
        *slot = (uint8_t)lane;
        asm volatile("" ::: "memory");          // the slot is read back after all lanes have written (one wave's LDS accesses keep their order)
        who[g] = *slot;
        asm volatile("" ::: "memory");
    }
#pragma unroll
    for (int g = 0; g < kMine; ++g) {
        const bool in = (real >> g) & 1u;
        // (the table is small: its owner's column is compared)
        const bool shared = in & (who[g] / kShortLen != r) & ((uint32_t)__shfl((int)col[g], who[g]) == col[g]);
        if (__builtin_amdgcn_ballot_w64(shared) != 0) in_turn |= 1u << g;
        if (__builtin_amdgcn_ballot_w64(in & (col[g] >= (uint32_t)kPHead)) != 0) far |= 1u << g;
    }
    __shared__ int found[kLookThreads / kWave][4];
    if (lane == 0) {
        found[wave][0] = npairs;
        found[wave][1] = __builtin_popcount(in_turn);
        found[wave][2] = __builtin_popcount(in_turn & far);
    }
    __syncthreads();
    if (threadIdx.x != 0) return;
    int pairs = 0, nturn = 0, nfar = 0;
#pragma unroll
    for (int w = 0; w < kLookThreads / kWave; ++w) {
        pairs += found[w][0];
        nturn += found[w][1];
        nfar += found[w][2];
    }
    *answer = nfar > kLookMost ? 0u : pairs <= kLookPairs ? kShortApart : (nturn > kLookMost ? kShortLongChains : kShortAlways);
}

template <int LOSS, typename TV>
__device__ inline void short_scout(const ChainArgs &a, char *lds, int chain, int64_t n, int64_t step0, int64_t nsections, bool marks)
{
    using L = ShortLds<TV>;
    const int lane = (int)(threadIdx.x & (kWave - 1)), r = lane / kShortLen, e = lane % kShortLen;
    const double rho = a.rho, inv_rho = 1.0 / rho;
    const double rho64 = a.pow_tab[kWave - 1] * rho, inv_rho64 = a.pow_tab[2 * kWave - 1];
    const double rho_pow = a.pow_tab[lane], inv_rho_pow1 = a.pow_tab[kWave + lane];
    double s_w = 1.0, eos_w = a.eta;
    // per lane: the row of step (window start + lane), for the window being written (A), the next (B) and the one after (C)
    // (as loaded: a difference taken here would wait for the loads, and with them for every row on its way)
    struct Window { int64_t lo, end; float y; };
    auto load_window = [&](int64_t w) {
        const uint64_t step = (uint64_t)(step0 + w * kWave + lane);
        const uint32_t row = a.perm ? a.perm[shard_position((uint32_t)chain, (uint32_t)a.k, step, (uint32_t)a.m)]
                                    : sample_row(a.seed_lo, a.seed_hi, (uint32_t)chain, step, (uint32_t)a.m);
        Window t;
        t.lo = a.row_ptr[row];
        t.end = a.row_ptr[(int64_t)row + 1];
        t.y = a.y[row];
        return t;
    };
    Window A = load_window(0), B = load_window(1), C = load_window(2);

    auto run = [&](auto role_tag) {
        constexpr bool MARKS = decltype(role_tag)::value;
        uint32_t er_col[kShortLead];
        float er_val[kShortLead];
        int er_len[kShortLead];
        // The rows to request pass through LDS once per window, so that a group costs one 16-byte read at a fixed place
        // (three exchanges between lanes per group had made the scouts the slowest waves: 0.076 us per step against 0.066).
        RowToRequest *const rows = reinterpret_cast<RowToRequest *>(lds + L::rows) + (MARKS ? kWave : 0);
        auto announce = [&](const Window &t) {
            RowToRequest q;
            q.len = (int)(t.end - t.lo);
            q.lo = q.len > 0 ? t.lo : 1;
            q.pad = 0;
            rows[lane] = q;
        };
        // entry e of the row of step 4*u + r of the window announced last
        auto request = [&](int u, const RowToRequest &q) {
            const int64_t at = q.lo + (e < q.len ? e : q.len - 1);
            er_len[u] = q.len;
            er_col[u] = (uint32_t)a.col_idx[at];
            if constexpr (!MARKS) er_val[u] = a.vals[at];
        };
        announce(A);
#pragma unroll
        for (int u = 0; u < kShortLead; ++u) request(u, rows[kShortRows * u + r]);
        __builtin_amdgcn_s_waitcnt(0x0F70);      // enter the loop with an empty queue
        StepScalars<TV> sc_tab;
        int redo = 0;                            // (marks) groups still to re-read their values because they follow a long row
        struct { bool tail, real; uint16_t now, sa, sb; uint8_t who; } prev;
        uint32_t stale_bits = 0, turn_bits = 0;  // (marks) the verdicts on this section's groups
        auto settle = [&](int u) {               // the verdict on group u, when its table reads have arrived
            const bool recent = ((uint16_t)(prev.now - prev.sa) < kShortRecent) & ((uint16_t)(prev.now - prev.sb) < kShortRecent);
            if (__builtin_amdgcn_ballot_w64(prev.tail & recent) != 0) stale_bits |= 1u << u;
            if (__builtin_amdgcn_ballot_w64(prev.real & ((int)prev.who / kShortLen != r)) != 0) turn_bits |= 1u << u;
        };

        // one section: groups kG*i .. kG*i + kG-1, HALF = i & 1 of the window
        auto write_section = [&](int64_t i, auto half_tag) {
            constexpr int HALF = decltype(half_tag)::value;
            const int64_t w = i / 2;
            if constexpr (HALF == 0) {
                if (w > 0) {
                    s_w *= rho64;
                    eos_w *= inv_rho64;
                    A = B;
                    B = C;
                    C = load_window(w + 2);
                }
                announce(B);
                if constexpr (!MARKS) {
                    const double yd = (double)A.y;
                    const double sl = yd * s_w * rho_pow, el = yd * eos_w * inv_rho_pow1;
                    const bool live = w * kWave + lane < n;
                    if constexpr (LOSS == kLossHinge) {
                        sc_tab.zs = sl;
                        sc_tab.cs = live ? el : 0.0;
                    } else {
                        sc_tab.zs = (float)(sl * 1.4426950408889634);
                        sc_tab.cs = live ? (float)el : 0.0f;
                    }
                }
            }
            RowToRequest ask[kG];                // the rows this section requests, read at once
#pragma unroll
            for (int u = 0; u < kG; ++u) ask[u] = rows[kShortRows * (HALF * kG + u) + r];
            char *sec = lds + L::ring + (uint32_t)(i % kSections) * kShortSectionBytes;
            if constexpr (!MARKS) {              // the lanes that hold this section's 32 steps publish their scalars
                if (lane / 32 == HALF) {
                    const int t = lane % 32;
                    char *h = sec + (t / kShortRows) * kGroupBytes + kWave * 16 + (t % kShortRows) * kShortScalars;
                    *reinterpret_cast<StepScalars<TV> *>(h) = sc_tab;
                    reinterpret_cast<StepRow *>(h + 16)->lo = A.lo;
                    reinterpret_cast<StepRow *>(h + 16)->len = (int)(A.end - A.lo);
                }
            }
#pragma unroll
            for (int u = 0; u < kG; ++u) {
                const int slot = HALF * kG + u;
                const int len = er_len[slot];
                const uint32_t col = er_col[slot];
                const bool in = e < len, tail = in && col >= (uint32_t)kPHead;
                if constexpr (MARKS) {
                    const uint16_t now = (uint16_t)(i * kG + u);
                    uint16_t *const pa = reinterpret_cast<uint16_t *>(lds + L::stamp_a) + (tail ? stamp_slot_a(col) : (uint32_t)(kPStamps + lane));
                    uint16_t *const pb = reinterpret_cast<uint16_t *>(lds + L::stamp_b) + (tail ? stamp_slot_b(col) : (uint32_t)(kPStamps + lane));
                    uint8_t *const po = reinterpret_cast<uint8_t *>(lds + L::owner) + (in ? col & (kOwners - 1) : (uint32_t)(kOwners + lane));
                    const uint16_t sa = *pa, sb = *pb;
                    *pa = now;
                    *pb = now;
                    *po = (uint8_t)lane;
                    asm volatile("" ::: "memory");          // the slot is read back after all lanes have written (one wave's LDS accesses keep their order)
                    const uint8_t who = *po;
                    if (u > 0) settle(u - 1);
                    else stale_bits = turn_bits = 0;
                    if (__builtin_amdgcn_ballot_w64(len > kShortLen) != 0) {
                        redo = kShortRecent;
                        turn_bits |= 1u << u;
                    }
                    if (redo > 0) {
                        stale_bits |= 1u << u;
                        --redo;
                    }
                    prev.tail = tail; prev.real = in; prev.now = now; prev.sa = sa; prev.sb = sb; prev.who = who;
                    if (u == kG - 1) {           // the section's marks go out together, before its barrier
                        settle(u);
                        // The chain ends in this section: its last group and those behind it go step by step, and a step behind the
                        // end is left out, whatever its row holds (0 times a NaN is one).
                        if (i == nsections - 1) turn_bits |= ~0u << (int)((a.nsteps[blockIdx.x] - i * (kG * kShortRows)) / kShortRows);
                        if (lane < kG)
                            reinterpret_cast<StepRow *>(sec + lane * kGroupBytes + kWave * 16 + 16)->pad =
                                (int32_t)(((stale_bits >> lane) & 1u) * kStale + ((turn_bits >> lane) & 1u) * kInTurn);
                    }
                } else {
                    pu32x4 rec;
                    rec[0] = in ? __float_as_uint(er_val[slot]) : 0u;
                    rec[1] = in && !tail ? L::head + col * (uint32_t)sizeof(TV) : L::head_scratch + lane * (uint32_t)sizeof(TV);
                    rec[2] = tail ? col * (uint32_t)sizeof(TV) : 0xFFFFFFF0u;        // (past the end of the vector: no access)
                    rec[3] = tail ? 0x80000000u : 0u;
                    *reinterpret_cast<pu32x4 *>(sec + u * kGroupBytes + lane * 16) = rec;
                }
                request(slot, ask[u]);
            }
        };
        for (int64_t i = 0; i <= nsections; i += 2) {
            write_section(i, std::integral_constant<int, 0>{});
            wait_lds_then_barrier();
            if (i + 1 <= nsections) {
                write_section(i + 1, std::integral_constant<int, 1>{});
                wait_lds_then_barrier();
            }
        }
    };
    if (marks) run(std::true_type{});
    else run(std::false_type{});
}

template <int LOSS, typename TV>
__device__ inline TV short_coefficient(const StepScalars<TV> &sc, TV dot)
{
    if constexpr (LOSS == kLossHinge) return sc.zs * dot < 1.0 ? sc.cs : 0.0;
    else return sc.cs * __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(sc.zs * dot));
}

// sum over a row of 16 lanes, in every lane of it
template <typename TV>
__device__ inline TV row_sum(TV v)
{
    v += dpp_move<0xB1, 0xF>(v);
    v += dpp_move<0x4E, 0xF>(v);
    v += dpp_move<0x141, 0xF>(v);
    v += dpp_move<0x140, 0xF>(v);
    return v;
}

template <int LOSS, typename TV>
__device__ inline void short_worker(const ChainArgs &a, char *lds, TV *v, int64_t nsections)
{
    using L = ShortLds<TV>;
    const int lane = (int)(threadIdx.x & (kWave - 1)), r = lane / kShortLen;
    const uint32_t v_bytes = (uint32_t)(a.d * (int64_t)sizeof(TV));
    const __amdgpu_buffer_rsrc_t vres = __builtin_amdgcn_make_buffer_rsrc(v, 0, (int)v_bytes, 0x00020000);
    const pu32x4 vdesc = descriptor(v, v_bytes);
    TV *head = reinterpret_cast<TV *>(lds + L::head);
    pu32x4 rec[kG];
    TV vr[kG];
    StepScalars<TV> scr[kG];
    int markr[kG];
    const char *ring = lds + L::ring;
    auto fetch = [&](int q, const char *group) {
        rec[q] = *reinterpret_cast<const pu32x4 *>(group + lane * 16);
        scr[q] = *reinterpret_cast<const StepScalars<TV> *>(group + kWave * 16 + r * kShortScalars);
        markr[q] = reinterpret_cast<const StepRow *>(group + kWave * 16 + 16)->pad;
    };
    wait_lds_then_barrier();          // section 0 written
    wait_lds_then_barrier();          // section 1 written
#pragma unroll
    for (int q = 0; q <= kShortAhead; ++q) fetch(q, ring + q * kGroupBytes);
#pragma unroll
    for (int q = 0; q < kShortAhead; ++q) vr[q] = load_state(vres, rec[q][2], TV{});
    __builtin_amdgcn_s_waitcnt(0x0F70);      // enter the loop with an empty queue

    for (int64_t g = 0; g < nsections; ++g) {
        if (g > 0) wait_lds_then_barrier();  // section g+1 written
        const char *cur = ring + (uint32_t)(g % kSections) * kShortSectionBytes;
        const char *nxt = ring + (uint32_t)((g + 1) % kSections) * kShortSectionBytes;
#pragma unroll
        for (int u = 0; u < kG; ++u) {
            const TV hv = *reinterpret_cast<const TV *>(lds + rec[u][1]);
            fetch((u + kShortAhead + 1) % kG, (u + kShortAhead + 1 < kG ? cur : nxt) + ((u + kShortAhead + 1) % kG) * kGroupBytes);
            const bool tail = (int32_t)rec[u][3] < 0;
            const TV val = (TV)__uint_as_float(rec[u][0]);
            TV vv = tail ? vr[u] : hv;
            const int marks = __builtin_amdgcn_readfirstlane(markr[u]);
            if (__builtin_expect((marks & kInTurn) == 0, 1)) {
                if (__builtin_expect(marks != 0, 0)) {
                    const TV fresh = drained_buffer_load(vdesc, rec[u][2], TV{});
                    if (tail) vv = fresh;
                }
                const TV coef = short_coefficient<LOSS, TV>(scr[u], row_sum(vv * val));
                const TV nv = vv + coef * val;
                *reinterpret_cast<TV *>(lds + rec[u][1]) = nv;
                store_state(vres, rec[u][2], nv);
            } else {
                const bool far = __any(tail);    // (no HBM-resident column in the group: its short rows leave the queue alone)
#pragma unroll 1
                for (int t = 0; t < kShortRows; ++t) {          // step by step, each value read when its step comes
                    const StepRow row = *reinterpret_cast<const StepRow *>(cur + u * kGroupBytes + kWave * 16 + t * kShortScalars + 16);
                    const StepScalars<TV> sc = *reinterpret_cast<const StepScalars<TV> *>(cur + u * kGroupBytes + kWave * 16 + t * kShortScalars);
                    const int len = __builtin_amdgcn_readfirstlane(row.len);
                    if (__builtin_amdgcn_ballot_w64(sc.cs != (TV)0) == 0) continue;      // behind the chain's end
                    if (len <= kShortLen) {
                        const uint32_t off = r == t ? rec[u][2] : 0xFFFFFFF0u;
                        TV now = *reinterpret_cast<const TV *>(lds + rec[u][1]);
                        if (far) {
                            const TV fresh = drained_buffer_load(vdesc, off, TV{});
                            if (tail) now = fresh;
                        }
                        const TV nv = now + short_coefficient<LOSS, TV>(sc, row_sum(now * val)) * val;
                        if (r == t) *reinterpret_cast<TV *>(lds + rec[u][1]) = nv;
                        if (far) drained_buffer_store(vdesc, off, nv);
                    } else {
                        TV acc = (TV)0;
                        for (int e0 = 0; e0 < len; e0 += kWave) {
                            const bool in = e0 + lane < len;
                            const uint32_t xc = drained_global_load_u32(a.col_idx + (in ? row.lo + e0 + lane : row.lo));
                            const float xv = __uint_as_float(drained_global_load_u32(a.vals + (in ? row.lo + e0 + lane : row.lo)));
                            const bool hd = xc < (uint32_t)kPHead;
                            const TV old = drained_buffer_load(vdesc, in && !hd ? xc * (uint32_t)sizeof(TV) : 0xFFFFFFF0u, TV{});
                            if (in) acc += (hd ? head[xc] : old) * (TV)xv;
                        }
                        const TV coef = short_coefficient<LOSS, TV>(sc, wave_sum(acc));
                        for (int e0 = 0; e0 < len; e0 += kWave) {
                            const bool in = e0 + lane < len;
                            const uint32_t xc = drained_global_load_u32(a.col_idx + (in ? row.lo + e0 + lane : row.lo));
                            const float xv = __uint_as_float(drained_global_load_u32(a.vals + (in ? row.lo + e0 + lane : row.lo)));
                            const bool hd = xc < (uint32_t)kPHead;
                            const uint32_t off = in && !hd ? xc * (uint32_t)sizeof(TV) : 0xFFFFFFF0u;
                            const TV old = drained_buffer_load(vdesc, off, TV{});
                            if (in && hd) head[xc] += coef * (TV)xv;
                            drained_buffer_store(vdesc, off, old + coef * (TV)xv);
                        }
                    }
                }
            }
            // HBM-resident values of group u + kShortAhead (its records arrived one group ago)
            vr[(u + kShortAhead) % kG] = load_state(vres, rec[(u + kShortAhead) % kG][2], TV{});
        }
    }
    __builtin_amdgcn_s_waitcnt(0x0F70);      // all stores done before the vector is read back
}

}  // namespace
}  // namespace wpsgd
