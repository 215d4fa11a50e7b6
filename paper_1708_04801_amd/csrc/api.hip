// The C ABI of libwpsgd (see wpsgd.h): argument checks, the kernel planner, the host-side
// weights of Eq. 6 / Eq. 8, and the small host->device hand-overs the kernels need.
#include <algorithm>
#include <atomic>
#include <climits>
#include <cmath>
#include <cstdio>
#include <cstring>
#include <mutex>
#include <numeric>
#include <vector>

#include "device_utils.h"
#include "internal.h"

namespace wpsgd {

hipError_t dense_reg_dispatch_f32_loss0(Plan &, const ChainArgs *, hipStream_t);
hipError_t dense_reg_dispatch_f32_loss1(Plan &, const ChainArgs *, hipStream_t);
hipError_t dense_reg_dispatch_bf16_loss0(Plan &, const ChainArgs *, hipStream_t);
hipError_t dense_reg_dispatch_bf16_loss1(Plan &, const ChainArgs *, hipStream_t);
bool dense_reg_shape_f32_loss0(int, int, int);
bool dense_reg_shape_f32_loss1(int, int, int);
bool dense_reg_shape_bf16_loss0(int, int, int);
bool dense_reg_shape_bf16_loss1(int, int, int);

static thread_local int g_last_hip_error = 0;

static int hip_fail(hipError_t e)
{
    g_last_hip_error = (int)e;
    return WPSGD_HIP_ERROR;
}

static hipError_t dense_reg_dispatch(Plan &p, const ChainArgs *a, hipStream_t s)
{
    if (p.dtype == WPSGD_BF16)
        return p.loss == WPSGD_HINGE ? dense_reg_dispatch_bf16_loss0(p, a, s)
                                     : dense_reg_dispatch_bf16_loss1(p, a, s);
    return p.loss == WPSGD_HINGE ? dense_reg_dispatch_f32_loss0(p, a, s)
                                 : dense_reg_dispatch_f32_loss1(p, a, s);
}

static bool dense_reg_shape(int dtype, int loss, int threads, int ept, int vec)
{
    if (dtype == WPSGD_BF16)
        return loss == WPSGD_HINGE ? dense_reg_shape_bf16_loss0(threads, ept, vec)
                                   : dense_reg_shape_bf16_loss1(threads, ept, vec);
    return loss == WPSGD_HINGE ? dense_reg_shape_f32_loss0(threads, ept, vec)
                               : dense_reg_shape_f32_loss1(threads, ept, vec);
}

static size_t align256(size_t b) { return (b + 255) & ~(size_t)255; }

static int check_matrix(const wpsgd_matrix *X)
{
    if (!X) return WPSGD_INVALID_ARG;
    if (X->m < 1 || X->m > 0xFFFFFFFFLL || X->d < 1) return WPSGD_INVALID_ARG;
    const bool has_csr = X->row_ptr || X->col_idx || X->vals;
    if (X->dense) {
        if (has_csr) return WPSGD_INVALID_ARG;
        if (X->ld < X->d) return WPSGD_INVALID_ARG;
        if (X->dtype != WPSGD_F32 && X->dtype != WPSGD_BF16) return WPSGD_INVALID_ARG;
    } else {
        if (!(X->row_ptr && X->col_idx && X->vals)) return WPSGD_INVALID_ARG;
    }
    return WPSGD_OK;
}

// Elements a row is aligned to in units of 16 bytes: every row start and every fragment whole, or single elements.
static int dense_vec(const wpsgd_matrix *X)
{
    const int wide = X->dtype == WPSGD_BF16 ? 8 : 4;
    const bool ok = ((uintptr_t)X->dense % 16 == 0) && (X->ld % wide == 0) && (X->d % wide == 0);
    return ok ? wide : 1;
}

// Widest load of the kernels that fetch rows with raw buffer loads into registers.  Such a load of four
// dwords needs dword alignment only and is checked against the row's end dword by dword, so every fp32
// row takes it, whatever its length and stride (d = 3001, fp64 state: 0.383 -> 0.289 us per step with a
// quarter of the load instructions).  bfloat16 rows of odd length start in the middle of a dword.
static int buffer_vec(const wpsgd_matrix *X)
{
    if (X->dtype == WPSGD_F32 && (uintptr_t)X->dense % 4 == 0) return 4;
    return dense_vec(X);
}

// Chooses the kernel family and its parameters.  Dense rows go to the register kernel when
// some instantiated shape holds d elements, else to the HBM-state kernel.
static int compute_units()
{
    static std::atomic<int> cached{0};          // (asking twice is harmless)
    int cus = cached.load(std::memory_order_relaxed);
    if (cus == 0) {
        int dev = 0, n = 0;
        if (hipGetDevice(&dev) != hipSuccess || hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) {
            (void)hipGetLastError();
            return 256;                 // no device to ask (planning on a host without one): the target's count
        }
        cus = n;
        cached.store(cus, std::memory_order_relaxed);
    }
    return cus;
}

// Helper workgroups per chain of blocks of eight steps: a multiple of eight behind the chains, on compute units of the chain's XCD that no chain
// occupies (one that has to wait for a compute unit is worse than none: d = 767, 84 chains, two helpers each: 33 workgroups for the 32 units of an XCD,
// 0.147 us per step, as without).  A workgroup has its compute unit to itself, so helpers leave as many units as the chains take for a call on another
// stream: its chains start at once, without helpers until the first call's have ended (us, one call of 4000 steps | two on two streams, 64 chains: d = 1024
// three helpers each 456 | 885, two 464 | 685, rounds of two steps 582 | 775; bf16 d = 2048 524 | 1022, 528 | 790, 712 | 1000).
static int octet_helpers(int k) { return std::min(compute_units() / ((k + 7) / 8 * 8) - 2, 3); }

static int resolve_plan(const wpsgd_matrix *X, int k, wpsgd_loss loss, const wpsgd_plan *force, Plan *out,
                        double rho = 1.0, int64_t max_steps = 0)
{
    Plan p{};
    p.loss = (int)loss;
    p.dtype = X->dense ? (int)X->dtype : WPSGD_F32;
    const size_t state_elem = (loss == WPSGD_HINGE) ? sizeof(double) : sizeof(float);
    const wpsgd_plan f = force ? *force : wpsgd_plan{0, 0, 0, 0, 0, 0, 0, 0};
    if (f.threads < 0 || f.block_steps < 0 || f.prefetch < 0 || f.rows < 0 || f.rows > 3 || f.helpers < -1 || f.helpers > 3 || f.slices < 0 || f.slices > 8) return WPSGD_INVALID_ARG;
    if (f.slice_wait_us < -1 || f.slice_wait_us > 60 * 1000 * 1000) return WPSGD_INVALID_ARG;

    if (!X->dense) {
        if (f.threads && f.threads != kWave && f.threads != 3 * kWave) return WPSGD_UNSUPPORTED;
        if (f.block_steps > 1 || (f.prefetch > 1 && f.prefetch != 4 && f.prefetch != 8) || f.rows || f.slices > 1) return WPSGD_UNSUPPORTED;
        p.family = Family::Csr;
        p.threads = kWave;
        p.vec = p.align = 1;
        p.block_steps = 1;
        // The LDS-cached kernels (prefetch 4: one wave per chain, 8: three) never fold their lazy scale
        // back into the vector, so they need (1-eta*lambda)^steps to stay well inside fp32 range.
        // They park unused lanes on scratch columns at the start of the vector, and the kernels of more waves
        // address the vector with 32-bit byte offsets, of which 0xFFFFFFF0 stands for no access: it may not lie inside the vector.
        const bool no_fold = (double)max_steps * std::log(rho) > -55.0;       // scale > 2^-80
        const bool cached_ok = X->d >= 64 && no_fold;
        const bool pair_ok = X->d >= 128 && no_fold && (uint64_t)X->d * state_elem <= 0xFFFFFFF0ull;
        if (f.prefetch == 4 && !cached_ok) return WPSGD_UNSUPPORTED;
        if (f.prefetch == 8 && !pair_ok) return WPSGD_UNSUPPORTED;
        p.prefetch = f.prefetch ? f.prefetch : (pair_ok ? 8 : (cached_ok ? 4 : 1));
        if (p.prefetch == 8) p.threads = 3 * kWave;
        p.state_bytes_per_elem = state_elem;
        *out = p;
        return WPSGD_OK;
    }

    const int aligned = dense_vec(X), wide = buffer_vec(X);
    p.vec = p.align = aligned;
    // Chains of at most sixteen steps (unknown: long) are bound by their start: kernels that fill a deeper pipeline of rows, or
    // round the steps up to more, do not pay there.
    const bool brief = max_steps > 0 && max_steps <= 16;
    // Four dwords at a time from rows that are not aligned: a chain that waits for its own rows is up to a third faster
    // that way, but where enough chains share a compute unit to keep its memory pipe full a load that touches nine
    // 128-byte lines instead of eight costs 2 to 8 % (us, single dwords | four: d = 767, 768 chains of 1541 steps 609 | 644;
    // d = 3001, 256 chains 667 | 723; d = 4093, 5000 chains 1389 | 1465; against 576 | 418 for one chain at d = 1501).  Rows of
    // 129 to 512 elements have fewer waves or loads that way and gain throughout; shorter ones have twice the elements per lane
    // (d = 65, 512 chains of 200 steps 48 | 51).
    const bool wide_pays = wide == aligned || (X->d > 128 && X->d <= 512) || (!brief && X->d > 512 && k <= 2 * compute_units() && (X->d <= 2048 || k < compute_units()));
    // The register kernel folds its lazy scale once per 64 steps, which needs
    // (1-eta*lambda)^64 to stay far inside fp32 range; a harsher shrink takes the HBM kernel,
    // which checks every step.
    const bool mild_shrink = rho >= 0.55;
    if (!f.state_in_hbm && mild_shrink) {
        static const int kThreads[] = {64, 128, 256, 512, 1024};
        static const int kEpt[] = {1, 2, 4, 8, 16, 32, 64, 128};
        // smallest workgroup first, then the smallest fragment that covers d; fragments much
        // narrower than one wide load use scalar loads so that all lanes carry data
        auto search_loads = [&](int slices, int wide, Plan *found) -> bool {
        for (int nt : kThreads) {
            if (f.threads && f.threads != nt) continue;
            if (slices > 1 && nt != 256 && nt != 512) continue;
            for (int ept : kEpt) {
                // the shape covers d, or one slice of it with no slice left empty
                if ((int64_t)nt * ept * slices < X->d) continue;
                if (slices > 1 && (int64_t)nt * ept * (slices - 1) >= X->d) break;
                // bf16 rows of 513 to 1024 elements: with a compute unit to itself a chain is faster on two
                // waves (0.204 us per step, fp64 state; one wave 0.222), beyond that on one (0.237 against 0.244)
                if (nt == 64 && ept == 16 && !f.threads && k <= compute_units()) continue;
                // fp32 column slices of more than 4096 elements: two waves per SIMD with half the columns each keep four
                // rounds of rows on their way where one wave has registers for two (us per step, 8 slices of 8192
                // columns, four chains, one wave | two: logistic 1.24 | 0.92, hinge 1.43 | 1.11; calls of four steps 25 | 32 us).
                // Slices of up to 4096 have the registers (logistic 0.69 | 0.73, hinge 0.80 | 0.93).
                if (slices > 1 && !f.threads && p.dtype == WPSGD_F32 && nt == 256 && ept == 32 && !f.block_steps && !f.prefetch && !brief) continue;
                int vec = wide;
                if (wide > 1 && ept * 4 <= wide) vec = 1;
                if (ept % vec != 0) continue;
                if (!dense_reg_shape(p.dtype, p.loss, nt, ept, vec)) continue;
                Plan q = p;
                q.vec = vec;
                q.family = Family::DenseReg;
                q.threads = nt;
                q.ept = ept;
                q.block_steps = f.block_steps;
                q.prefetch = f.prefetch;
                q.rows = f.rows;
                q.slices = slices;
                q.state_bytes_per_elem = 0;
                if (vec > aligned) {                // the kernels that stage rows in LDS or stream them twice want whole fragments
                    if (f.rows > 1) continue;
                    q.rows = 1;
                }
                if (slices > 1) {
                    // the slices' exchange carries twelve words: ten fp32 sums (4 steps per round) or three fp64 sums (2 steps)
                    q.rows = 1;
                    if (f.rows > 1 || vec == 1 || k * slices > compute_units()) continue;
                    if ((size_t)X->d * state_elem < 2304) continue;       // the exchange table borrows the HBM-state area: 2080 bytes a chain
                    if (!q.block_steps) q.block_steps = 2;             // one exchange per two steps
                    if (q.block_steps > (p.loss == WPSGD_LOGISTIC ? 4 : 2)) continue;
                }
                // A workgroup of two or more waves with a compute unit (nearly) to itself is bound by the
                // latency of a step: two steps per reduction round (three sums instead of two, one exchange
                // instead of two) shorten it by 8 to 17 % (us per step, one -> two: fp32 hinge d = 1024
                // 0.219 -> 0.183, d = 2048 0.246 -> 0.216, d = 4096 0.296 -> 0.267; logistic 0.179 -> 0.148,
                // 0.199 -> 0.176, 0.238 -> 0.213; bf16 d = 2048 0.253 -> 0.223).  At two chains per compute unit the
                // two are within 2 %; with more the extra Gram products only cost throughput.  Rows of
                // 8192 elements (32 per thread) gained nothing.
                const bool few = k <= 2 * compute_units() && slices == 1 && nt <= 256;
                // (sliced hinge: four rounds on their way 0.80, two 1.09; calls of four steps 40 us and 30)
                const bool few_sliced = slices > 1 && p.dtype == WPSGD_F32 && ept == 16 && !(brief && p.loss == WPSGD_HINGE);
                if (!f.block_steps && !f.prefetch && !f.rows && nt >= 128 && ept <= 16 && (few || few_sliced)) {
                    Plan two = q;
                    two.block_steps = 2;
                    two.prefetch = 4;
                    if (dense_reg_dispatch(two, nullptr, nullptr) == hipSuccess) {
                        *found = two;
                        return true;
                    }
                }
                if (dense_reg_dispatch(q, nullptr, nullptr) == hipSuccess) {
                    *found = q;
                    return true;
                }
            }
        }
        return false;
        };
        auto search = [&](int slices, Plan *found) -> bool {
            if (wide == aligned) return search_loads(slices, wide, found);
            if (wide_pays) return search_loads(slices, wide, found) || search_loads(slices, aligned, found);
            return search_loads(slices, aligned, found) || ((slices == 1 || f.slices > 1) && search_loads(slices, wide, found));
        };
        Plan found;
        bool have = search(f.slices > 1 ? f.slices : 1, &found);
        // Rows too long for 256 threads (or for any one workgroup), few chains: rather than one chain
        // per 1024-thread workgroup, cut each chain into as many column slices as there are compute
        // units for (the widest workload: 8 slices of 8192 columns run 3 times as fast as one
        // workgroup of 1024; with fp64 state that row length has no one-workgroup shape at all).
        // bf16 rows of 8193 to 16384 elements fit 256 threads, but with 64 elements each: eight chains at d = 16384 take 0.58 us
        // per step in slices instead of 1.73 (hinge) and 0.35 instead of 0.63 (logistic, which two slices would slow down, and
        // which has to earn back the start of the slices: d = 8200, 50 steps 47 us in one piece, 53 in six).
        const bool crowded = have && found.threads == 256 && found.ept >= 64 && !(loss == WPSGD_LOGISTIC && max_steps > 0 && max_steps < 128);
        if (f.slices == 0 && !f.threads && !f.block_steps && !f.prefetch && !f.rows && (!have || found.threads == 1024 || crowded)) {
            for (int c = 8; c >= (crowded && loss == WPSGD_LOGISTIC ? 3 : 2); --c) {
                Plan cut;
                if (k * c <= compute_units() && search(c, &cut)) {
                    found = cut;
                    have = true;
                    break;
                }
            }
        }
        // Short rows, chains few enough: sixteen steps per block, three more waves per chain.  The lines are where the
        // one-wave kernel catches up, which runs more chains on a compute unit (us per step, one wave | blocks): d = 64
        // hinge, 1024 chains 0.130 | 0.099, 2048 chains 0.145 | 0.164; d = 128, 1024 chains, hinge 0.157 | 0.161, logistic 0.123 |
        // 0.107; d = 256 logistic, 256 chains 0.108 | 0.097, 512 chains 0.119 | 0.123.  fp32 hinge rows of more than 128
        // elements gain nothing (0.135 | 0.132 with eight chains, 0.148 | 0.189 with 512).
        const int64_t block_chains = X->d <= 64 ? 4 * compute_units()
                                     : X->d <= 128 ? (loss == WPSGD_LOGISTIC ? 4 : 2) * compute_units()
                                     : (loss == WPSGD_LOGISTIC || X->dtype == WPSGD_BF16) ? compute_units() : 0;
        // A block kernel starts later (three beats of its scouts, more code to fetch) and rounds up to sixteen steps, so chains
        // have to be long enough (us, one wave | blocks: d = 64, 1024 chains of 100 steps 35 | 40, of 300 57 | 57; d = 128, 64
        // chains of 50 steps 15.6 | 16.7; d = 128 logistic, 1024 chains of 300 56 | 61; bf16 d = 256 hinge, 64 chains of 50 17.7 | 24).
        const int64_t block_worth = X->d <= 64 ? (k <= compute_units() ? 1 : k <= 2 * compute_units() ? 64 : 256)
                                    : X->d <= 128 ? (k <= compute_units() ? 100 : k <= 2 * compute_units() ? 256 : 768)
                                    : 512;
        const bool block_shape = X->d >= kBlockMinColumns && X->d <= kBlockMaxColumns && (uintptr_t)X->dense % (X->dtype == WPSGD_BF16 ? 2 : 4) == 0;
        // A forced plan names one kernel, whatever the chains' lengths: the blocks, or with the pipeline's lead the pipeline.
        const bool asked = f.block_steps == 16 && (!f.threads || f.threads == kWave) && !f.rows && f.slices <= 1;
        const bool asked_block = asked && !f.prefetch;
        const bool asked_pipe = asked && f.prefetch == kPipeAhead && (loss == WPSGD_LOGISTIC || X->d <= kPipeHingeMaxColumns);
        if (block_shape && (asked_block || asked_pipe || (have && !f.threads && !f.block_steps && !f.prefetch && !f.rows && f.slices <= 1 && k <= block_chains &&
                                            (max_steps == 0 || max_steps >= block_worth)))) {
            if (!have) found = p;
            found.family = Family::DenseReg;
            found.threads = kWave;
            found.ept = X->d <= 64 ? 1 : (X->d <= 128 ? 2 : 4);
            found.block_steps = 16;
            found.prefetch = asked_pipe ? kPipeAhead : 2;
            found.rows = 1;
            found.slices = 1;
            found.scouts = 3;
            found.state_bytes_per_elem = 0;
            have = true;
            // With everything but the slopes off the dependent path a block takes half to two thirds of the time where a chain has a
            // compute unit to itself, but twice the matrix products: fp64 ones (hinge) bind rows of more than 64 elements, and so does a
            // second chain on the unit, which bf16 products and short fp32 rows leave room for.  Lines (us, blocks | pipelined, longest
            // chain of so many steps): d = 64 hinge, one chain, 200 29.8 | 29.0, 1000 68.8 | 63.5, 512 chains of 1000 90 | 103; d = 128 hinge
            // 85.6 | 86.0; logistic d = 64, 32 20.3 | 19.6, 1000 59.1 | 46.8, 512 chains of 200 42.4 | 40.4, of 32 32.0 | 35.0, 1024 chains of
            // 1000 97 | 116; d = 128, 50 22.3 | 22.8, 300 34.6 | 32.4, 512 chains of 300 54.0 | 51.6; d = 256, 50 22.8 | 24.9, 300 48.0 | 41.5, 512 chains of
            // 300 60.6 | 76.0; bf16 logistic d = 256, 50 24.7 | 23.0, 1000 103.5 | 62.4.  (Where block_worth is
            // the later line, that one counts; more than 128 columns come here with a compute unit per chain only.)
            const bool light = loss == WPSGD_LOGISTIC && X->dtype == WPSGD_BF16;
            int64_t pipe_worth = 0;                      // steps of the longest chain from which it pays; 0: it does not
            if (loss == WPSGD_HINGE) pipe_worth = X->d <= kPipeHingeMaxColumns && k <= compute_units() ? 200 : 0;
            else if (k <= compute_units()) pipe_worth = light || X->d <= 64 ? 32 : X->d <= 128 ? 100 : 160;
            else if (k <= 2 * compute_units()) pipe_worth = X->d <= 64 || light ? 200 : 300;
            found.pipelined = asked_pipe || (!asked_block && pipe_worth > 0 && max_steps >= pipe_worth);
        }
        const bool octet_shape = loss == WPSGD_LOGISTIC && X->d >= kOctetMinColumns && X->d <= octet_max_columns((int)X->dtype) &&
                                 wide == (X->dtype == WPSGD_BF16 ? 8 : 4);
        if (octet_shape && f.block_steps == 8 && (!f.threads || f.threads == 256) && !f.prefetch && !f.rows && f.slices <= 1) {
            p.family = Family::DenseReg;                 // asked for: with as many helpers as there is room for, or as the plan says
            p.threads = 256;
            p.ept = X->dtype == WPSGD_BF16 ? 8 : 4;
            p.vec = wide;
            p.block_steps = 8;
            p.prefetch = 2;
            p.rows = p.slices = 1;
            p.octets = true;
            *out = p;
            return WPSGD_OK;
        }
        if (have) {
            // Longer rows, fewer chains: blocks of eight steps whose products between rows two or three helper workgroups per chain form (chain_dense_octet.hip).
            // One helper is too slow (us per step, rounds of two steps | blocks of eight, 128 chains: d = 1024 0.150 | 0.139, bf16 d = 2048 0.176 |
            // 0.168, d = 512 0.120 | 0.132; 64 chains: 0.148 | 0.115, bf16 d = 2048 0.174 | 0.131; us per call of 80 chains of 300 steps, alone | two on two
            // streams: d = 1024 68 | 96, 69 | 102, bf16 77 | 112, 79 | 116).  Up to 512 columns the register kernel has one or two waves
            // and there is little to gain (0.121 | 0.107, bf16 64 chains 0.129 | 0.129).  The start costs some 3 us more (us per call: d = 1024, 16 chains of
            // 64 steps 27.3 | 28.2, of 150 38.8 | 37.3, 64 chains of 200 44.5 | 45.1; bf16 d = 2048, 64 chains of 200 52.6 | 50.6).
            // (found above holds what runs where the workspace has no room for records)
            found.octets = octet_shape && found.family == Family::DenseReg && found.scouts == 0 && found.slices == 1 && octet_helpers(k) >= 2 && max_steps >= (k <= 32 ? 192 : 256) &&
                           !f.threads && !f.block_steps && !f.prefetch && !f.rows && !f.slices && !f.helpers;
            *out = found;
            return WPSGD_OK;
        }
        if (f.threads || f.block_steps || f.prefetch || f.rows || f.slices > 1) return WPSGD_UNSUPPORTED;
    }
    if (f.rows || f.slices > 1) return WPSGD_UNSUPPORTED;
    p.family = Family::DenseMem;
    p.threads = f.threads ? f.threads : (X->d >= 16384 ? 1024 : 256);
    if (p.threads != 256 && p.threads != 1024) return WPSGD_UNSUPPORTED;
    if (f.block_steps > 1 || f.prefetch > 1) return WPSGD_UNSUPPORTED;
    p.block_steps = 1;
    p.prefetch = 1;
    p.state_bytes_per_elem = state_elem;
    *out = p;
    return WPSGD_OK;
}


// shuffled row order of partition-and-shuffle sampling (always reserved: the workspace query does
// not know which sampling a call will ask for)
static size_t perm_bytes(int64_t m) { return align256((size_t)m * sizeof(uint32_t)); }

static size_t state_elem_bytes(wpsgd_loss loss)
{
    return loss == WPSGD_HINGE ? sizeof(double) : sizeof(float);
}

// Workspace header.  First a status block (word 0: bit 0 set by chains that could not finish, see
// wpsgd_chains_status); then the chain order; then, in that order, step counts, stream offsets,
// two 32-bit numbers per chain describing its share under partition-and-shuffle sampling, and a
// progress counter per chain (zero at launch) that helper workgroups watch; last, the powers
// (1-eta*lambda)^l and (1-eta*lambda)^-(l+1), l = 0..63, in fp64.  Every part is 256-byte aligned.
constexpr size_t kStatusBytes = 256;
constexpr int kSliceWaitDefaultUs = 2 * 1000 * 1000;      // two seconds
constexpr size_t kPowTabBytes = 2 * 64 * sizeof(double);
struct HeaderLayout {
    size_t order, steps, offsets, shard, progress, pow_tab, total;
};
static HeaderLayout header_layout(int k)
{
    HeaderLayout h;
    h.order = kStatusBytes;
    h.steps = h.order + align256((size_t)k * sizeof(int32_t));
    h.offsets = h.steps + align256((size_t)k * sizeof(int64_t));
    h.shard = h.offsets + align256((size_t)k * sizeof(int64_t));
    h.progress = h.shard + align256((size_t)k * 2 * sizeof(uint32_t));
    h.pow_tab = h.progress + align256(((size_t)k * 2 + 16) * sizeof(uint32_t));
    h.total = h.pow_tab + kPowTabBytes;
    return h;
}
static size_t header_bytes(int k) { return header_layout(k).total; }

// 32-bit words of the table the column slices of k chains exchange their sums through: per chain
// 8 slices x 2 round parities x 32 words of records, then 8 words (the slices' XCD numbers)
static size_t slice_table_words(int k) { return (size_t)k * (8 * 2 * 32 + 8); }

// Helper workgroups per chain for a resolved plan: only the 256-thread register kernels have
// them, and only on compute units no chain occupies (at most 128 chains).
static int helpers_per_chain(const Plan &p, const wpsgd_matrix *X, int k, const wpsgd_plan *force)
{
    if (p.octets) {
        const int asked = force ? force->helpers : 0, room = compute_units() / ((k + 7) / 8 * 8) - 1;
        return asked < 0 ? 0 : std::max(0, std::min(asked > 0 ? asked : octet_helpers(k), room));
    }
    if (p.family != Family::DenseReg || p.threads != 256 || p.rows != 1 || k > 128 || p.slices > 1) return 0;
    const int asked = force ? force->helpers : 0;
    if (asked < 0) return 0;
    const int room = (compute_units() - k) / k;
    const int64_t row_bytes = X->d * (X->dtype == WPSGD_BF16 ? 2 : 4);
    const int want = asked > 0 ? asked : (row_bytes >= 8192 ? 2 : 0);      // a third helper only adds L2 traffic
    return std::max(0, std::min(want, std::min(room, 3)));
}

// Host arrays (chain order, step counts, weights) reach the device through a small ring of pinned
// staging buffers per host thread.  An event marks the last copy out of a buffer; it is rewritten
// only after that copy has finished, so the caller's arrays can be released as soon as a call returns.
struct StagingSlot {
    void *host = nullptr;
    size_t capacity = 0;
    hipEvent_t last_copy = nullptr;
    bool pending = false;
};
constexpr int kStagingSlots = 4;     // copies that may be queued before a call has to wait
struct StagingRing {
    StagingSlot slot[kStagingSlots];
    int next = 0;
    // A host thread that ends gives its buffers back (once their last copies have finished).  If the
    // runtime is already shutting down the calls fail and the process's exit reclaims everything.
    ~StagingRing()
    {
        int dev = 0;
        if (hipGetDevice(&dev) != hipSuccess) {
            (void)hipGetLastError();
            return;
        }
        for (StagingSlot &st : slot) {
            if (st.pending && st.last_copy) (void)hipEventSynchronize(st.last_copy);
            if (st.last_copy) (void)hipEventDestroy(st.last_copy);
            if (st.host) (void)hipHostFree(st.host);
            st = StagingSlot{};
        }
        (void)hipGetLastError();
    }
};
static thread_local StagingRing g_staging;

// fill(host) writes the bytes into the staging buffer
template <typename F>
static int upload_filled(void *dst, size_t bytes, hipStream_t s, F &&fill)
{
    StagingSlot &st = g_staging.slot[g_staging.next];
    g_staging.next = (g_staging.next + 1) % kStagingSlots;
    hipError_t e;
    if (st.pending) {
        e = hipEventSynchronize(st.last_copy);
        if (e != hipSuccess) return hip_fail(e);
        st.pending = false;
    }
    if (st.capacity < bytes) {
        if (st.host) (void)hipHostFree(st.host);
        st.host = nullptr;
        st.capacity = 0;
        const size_t want = std::max<size_t>(bytes, 1 << 16);
        e = hipHostMalloc(&st.host, want, hipHostMallocDefault);
        if (e != hipSuccess) return hip_fail(e);
        st.capacity = want;
    }
    if (!st.last_copy) {
        e = hipEventCreateWithFlags(&st.last_copy, hipEventDisableTiming);
        if (e != hipSuccess) return hip_fail(e);
    }
    fill(st.host);
    e = hipMemcpyAsync(dst, st.host, bytes, hipMemcpyHostToDevice, s);
    if (e != hipSuccess) return hip_fail(e);
    e = hipEventRecord(st.last_copy, s);
    if (e != hipSuccess) return hip_fail(e);
    st.pending = true;
    return WPSGD_OK;
}

static int upload(void *dst, const void *src, size_t bytes, hipStream_t s)
{
    return upload_filled(dst, bytes, s, [&](void *host) { std::memcpy(host, src, bytes); });
}

static int check_steps(int k, const int64_t *n_steps)
{
    if (k < 1 || !n_steps) return WPSGD_INVALID_ARG;
    for (int i = 0; i < k; ++i)
        if (n_steps[i] < 0) return WPSGD_INVALID_ARG;
    return WPSGD_OK;
}

static const char *family_name(Family f)
{
    switch (f) {
    case Family::DenseReg: return "dense_reg";
    case Family::DenseMem: return "dense_mem";
    default: return "csr";
    }
}

}  // namespace wpsgd

using namespace wpsgd;

extern "C" {

size_t wpsgd_run_chains_workspace(const wpsgd_matrix *X, int k, wpsgd_loss loss, const wpsgd_plan *plan)
{
    if (check_matrix(X) != WPSGD_OK || k < 1) return 0;
    if (loss != WPSGD_HINGE && loss != WPSGD_LOGISTIC) return 0;
    Plan p;
    if (resolve_plan(X, k, loss, plan, &p) != WPSGD_OK) return 0;
    // Always room for the model vectors in HBM: which kernel runs also depends on eta*lambda,
    // which this query does not see.
    return header_bytes(k) + perm_bytes(X->m) + align256((size_t)k * (size_t)X->d * state_elem_bytes(loss));
}

int wpsgd_describe_plan(const wpsgd_matrix *X, int k, wpsgd_loss loss, const wpsgd_plan *plan,
                        char *buf, size_t buf_bytes)
{
    if (!buf || buf_bytes == 0 || k < 1) return WPSGD_INVALID_ARG;
    int rc = check_matrix(X);
    if (rc != WPSGD_OK) return rc;
    if (loss != WPSGD_HINGE && loss != WPSGD_LOGISTIC) return WPSGD_INVALID_ARG;
    Plan p;
    rc = resolve_plan(X, k, loss, plan, &p);
    if (rc != WPSGD_OK) return rc;
    static const char *const kRows[] = {"", " rows=registers", " rows=lds", " rows=twice"};
    char helped[32] = "";
    const int hp = helpers_per_chain(p, X, k, plan);
    if (hp > 0) std::snprintf(helped, sizeof(helped), " helpers=%d", hp);
    if (p.family == Family::DenseReg && p.slices > 1) std::snprintf(helped, sizeof(helped), " slices=%d", p.slices);
    if (p.scouts > 0) std::snprintf(helped, sizeof(helped), " scouts=%d", p.scouts);
    // (the steps of a call are not known here: what long chains run on instead, unless the plan names the kernel)
    char longer[32] = "";
    Plan steady;
    if (p.pipelined) std::snprintf(longer, sizeof(longer), " pipelined");
    else if (p.octets) std::snprintf(longer, sizeof(longer), " octets");
    else if (resolve_plan(X, k, loss, plan, &steady, 1.0, INT32_MAX) == WPSGD_OK && (steady.pipelined || steady.octets))
        std::snprintf(longer, sizeof(longer), steady.pipelined ? " long=pipelined" : " long=octets");
    char load[16] = "";                  // rows of single elements that are fetched several at a time all the same
    if (p.vec > p.align && p.scouts == 0) std::snprintf(load, sizeof(load), " load=%d", p.vec);
    std::snprintf(buf, buf_bytes, "%s %s %s nt=%d ept=%d vec=%d%s B=%d P=%d state=%s%s%s%s",
                  family_name(p.family), p.dtype == WPSGD_BF16 ? "bf16" : "f32",
                  p.loss == WPSGD_HINGE ? "hinge" : "logistic", p.threads, p.ept, std::min(p.vec, p.align), load,
                  p.block_steps, p.prefetch,
                  p.state_bytes_per_elem == 0 ? "registers" : (p.state_bytes_per_elem == 8 ? "hbm-f64" : "hbm-f32"),
                  p.family == Family::DenseReg ? kRows[p.rows] : "", helped, longer);
    return WPSGD_OK;
}

int wpsgd_run_chains(const wpsgd_matrix *X, const float *y, int k, const int64_t *n_steps,
                     double eta, double lambda, wpsgd_loss loss, uint64_t seed, float *W,
                     void *workspace, size_t workspace_bytes, const wpsgd_plan *plan, void *stream)
{
    return wpsgd_run_chains_from(X, y, k, n_steps, eta, lambda, loss, seed, WPSGD_SAMPLE_STREAM, nullptr, nullptr, W,
                                 workspace, workspace_bytes, plan, stream);
}

// Chains cut into column slices wait for each other's workgroups.  Two such launches seated half and
// half on the device would each wait for workgroups that cannot start before the other launch's have
// ended, so within this process they run one after the other: a launch first makes its stream wait
// for the previous sliced launch on the device (on whatever stream that was queued).
struct SlicedLaunchOrder {
    static constexpr int kMaxDevices = 64;
    std::mutex lock;
    hipEvent_t last[kMaxDevices] = {};
    bool queued[kMaxDevices] = {};
};
static SlicedLaunchOrder g_sliced;

static hipError_t launch_whole(Plan p, const ChainArgs &a, hipStream_t s)
{
    switch (p.family) {
    case Family::DenseReg:
        if (p.octets) return launch_dense_octet(p, a, s);
        if (p.pipelined) return launch_dense_pipe(p, a, s);
        return p.scouts > 0 ? launch_dense_block(p, a, s) : dense_reg_dispatch(p, &a, s);
    case Family::DenseMem: return launch_dense_mem(p, a, s);
    default: return launch_csr(p, a, s);
    }
}

static hipError_t launch_sliced(Plan p, const ChainArgs &a, hipStream_t s)
{
    hipError_t e = launch_zero_words(static_cast<uint32_t *>(a.xchg), slice_table_words(a.k), s);
    if (e != hipSuccess) return e;
    int dev = 0;
    e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= SlicedLaunchOrder::kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> guard(g_sliced.lock);
    if (!g_sliced.last[dev]) {
        e = hipEventCreateWithFlags(&g_sliced.last[dev], hipEventDisableTiming);
        if (e != hipSuccess) return e;
    }
    if (g_sliced.queued[dev]) {
        e = hipStreamWaitEvent(s, g_sliced.last[dev], 0);
        if (e != hipSuccess) return e;
    }
    e = dense_reg_dispatch(p, &a, s);
    if (e != hipSuccess) return e;
    e = hipEventRecord(g_sliced.last[dev], s);
    g_sliced.queued[dev] = e == hipSuccess;
    return e;
}

// Periodic averaging: after each of `count` spans the models are averaged into `average`, from which the next span
// starts.  Everything the spans share - header, shuffled order, weights - is prepared once per call, so that a span
// is its launches and nothing else (25 spans of 200 steps, 16 chains, d = 1024: 1.03 ms with a header copied per span, 0.92 without).
constexpr int kStartModelsMost = 63;       // chains whose models each chain averages for itself
struct Spans {
    int64_t count;
    const double *weights;         // HOST, k entries
    double *weights_dev;
    float *average;
};

static int run_chains_from(const wpsgd_matrix *X, const float *y, int k, const int64_t *n_steps,
                           double eta, double lambda, wpsgd_loss loss, uint64_t seed, wpsgd_sampling sampling,
                           const float *w_start, const int64_t *step_offsets, float *W,
                           void *workspace, size_t workspace_bytes, const wpsgd_plan *plan, void *stream, const Spans *spans)
{
    int rc = check_matrix(X);
    if (rc != WPSGD_OK) return rc;
    if (!y || !W) return WPSGD_INVALID_ARG;
    if (sampling != WPSGD_SAMPLE_STREAM && sampling != WPSGD_SAMPLE_SHARDS) return WPSGD_INVALID_ARG;
    if (sampling == WPSGD_SAMPLE_SHARDS && (int64_t)k > X->m) return WPSGD_INVALID_ARG;     // a node without examples
    rc = check_steps(k, n_steps);
    if (rc != WPSGD_OK) return rc;
    if (step_offsets)
        for (int i = 0; i < k; ++i)
            if (step_offsets[i] < 0 || step_offsets[i] > INT64_MAX - n_steps[i]) return WPSGD_INVALID_ARG;
    if (!(eta > 0.0) || !(lambda >= 0.0) || !(eta * lambda < 1.0)) return WPSGD_INVALID_ARG;
    if (loss != WPSGD_HINGE && loss != WPSGD_LOGISTIC) return WPSGD_INVALID_ARG;
    Plan p;
    int64_t max_steps = 0;
    for (int i = 0; i < k; ++i) max_steps = std::max(max_steps, n_steps[i]);
    rc = resolve_plan(X, k, loss, plan, &p, 1.0 - eta * lambda, max_steps);
    if (rc != WPSGD_OK) return rc;
    // behind the header and the shuffled order: the model vectors of the HBM-state kernels, or the
    // table the column slices of a chain exchange their sums through
    const bool sliced = p.family == Family::DenseReg && p.slices > 1;
    const size_t behind = sliced ? slice_table_words(k) * sizeof(uint32_t) : (size_t)k * (size_t)X->d * p.state_bytes_per_elem;
    const HeaderLayout h = header_layout(k);
    const size_t need = h.total + perm_bytes(X->m) + align256(behind);
    if (!workspace || ((uintptr_t)workspace % 256) != 0) return WPSGD_INVALID_ARG;
    if (workspace_bytes < need) return WPSGD_WORKSPACE_TOO_SMALL;
    // (a caller that brings less than the query asks for, which the register kernels do not need, gets those)
    const size_t ring = (size_t)k * kOctetRingRecords * 256;
    if (p.octets && workspace_bytes < h.total + perm_bytes(X->m) + ring) {
        if (p.block_steps == 8) return WPSGD_WORKSPACE_TOO_SMALL;         // (asked for)
        p.octets = false;
    }
    hipStream_t s = static_cast<hipStream_t>(stream);

    // longest chain first (stable, so equal lengths keep their order); order and step counts
    // travel in one copy, laid out exactly as the workspace header
    std::vector<int32_t> order(k);
    std::iota(order.begin(), order.end(), 0);
    std::stable_sort(order.begin(), order.end(),
                     [&](int32_t x, int32_t z) { return n_steps[x] > n_steps[z]; });
    std::vector<char> header(h.total, 0);
    std::memcpy(header.data() + h.order, order.data(), (size_t)k * sizeof(int32_t));
    int64_t *sorted_steps = reinterpret_cast<int64_t *>(header.data() + h.steps);
    int64_t *sorted_offsets = reinterpret_cast<int64_t *>(header.data() + h.offsets);
    uint32_t *shard = reinterpret_cast<uint32_t *>(header.data() + h.shard);
    for (int b = 0; b < k; ++b) {
        sorted_steps[b] = n_steps[order[b]];
        sorted_offsets[b] = step_offsets ? step_offsets[order[b]] : 0;
        if (sampling == WPSGD_SAMPLE_SHARDS) {
            const uint64_t lo = (uint64_t)order[b] * (uint64_t)X->m / (uint64_t)k;
            const uint64_t hi = ((uint64_t)order[b] + 1) * (uint64_t)X->m / (uint64_t)k;
            shard[b] = (uint32_t)lo;
            shard[k + b] = (uint32_t)(hi - lo);
        }
    }

    double *pow_tab = reinterpret_cast<double *>(header.data() + h.pow_tab);
    {
        const double rho = 1.0 - eta * lambda, inv_rho = 1.0 / rho;
        double up = 1.0, down = inv_rho;
        for (int l = 0; l < 64; ++l) {
            pow_tab[l] = up;
            pow_tab[64 + l] = down;
            up *= rho;
            down *= inv_rho;
        }
    }
    char *ws = static_cast<char *>(workspace);
    uint32_t *perm_dev = reinterpret_cast<uint32_t *>(ws + h.total);
    void *state_dev = ws + h.total + perm_bytes(X->m);
    rc = upload(ws, header.data(), header.size(), s);             // (clears the status block, once per call: a span that fails stays reported)
    if (rc != WPSGD_OK) return rc;

    if (spans) {
        rc = upload(spans->weights_dev, spans->weights, (size_t)k * sizeof(double), s);
        if (rc != WPSGD_OK) return rc;
    }

    ChainArgs a{};
    a.dense = X->dense;
    a.ld = X->ld;
    a.row_ptr = X->row_ptr;
    a.col_idx = X->col_idx;
    a.vals = X->vals;
    a.y = y;
    a.m = X->m;
    a.d = X->d;
    a.k = k;
    a.status = reinterpret_cast<uint32_t *>(ws);
    a.order = reinterpret_cast<const int32_t *>(ws + h.order);
    a.nsteps = reinterpret_cast<const int64_t *>(ws + h.steps);
    a.longest = max_steps;
    a.step0 = reinterpret_cast<const int64_t *>(ws + h.offsets);
    a.w_start = w_start;
    a.pow_tab = reinterpret_cast<const double *>(ws + h.pow_tab);
    a.progress = reinterpret_cast<uint32_t *>(ws + h.progress);
    a.helpers = helpers_per_chain(p, X, k, plan) * k;
    a.slices = sliced ? p.slices : 1;
    a.xchg = state_dev;
    // how long a slice waits for the others before it gives up, as a number of polls: a poll takes 600 to
    // 1200 cycles of a 2.4 GHz clock, so four polls per microsecond are at least the time asked for and
    // at most twice that; 0: no poll at all (the plan's test hook)
    const int wait_us = plan ? plan->slice_wait_us : 0;
    a.slice_max_polls = wait_us < 0 ? 0u : (uint32_t)std::min<int64_t>((int64_t)(wait_us > 0 ? wait_us : kSliceWaitDefaultUs) * 4, INT32_MAX);
    a.eta = eta;
    a.rho = 1.0 - eta * lambda;
    a.seed_lo = (uint32_t)(seed & 0xFFFFFFFFu);
    a.seed_hi = (uint32_t)(seed >> 32);
    a.perm = nullptr;
    if (sampling == WPSGD_SAMPLE_SHARDS) {
        hipError_t pe = launch_permute_rows(a.seed_lo, a.seed_hi, (uint32_t)X->m, perm_dev, s);
        if (pe != hipSuccess) return hip_fail(pe);
        a.perm = perm_dev;
        a.shard = reinterpret_cast<const uint32_t *>(ws + h.shard);
    }
    a.W = W;
    a.state = state_dev;

    hipError_t e = hipSuccess;
    if (p.octets) {
        e = launch_zero_words(static_cast<uint32_t *>(state_dev), ring / sizeof(uint32_t), s);
        if (e != hipSuccess) return hip_fail(e);
    }
    // Between two spans the chains of short rows form the average themselves (start_values), one launch instead of two: the models then
    // lie in two places in turn, W and the part of the workspace that holds the vectors of the HBM-state kernels, which these plans leave
    // idle.  Every chain reads all models, 16 rows at once, in the order in which combine_kernel adds fewer than
    // 64.  us a span, two launches -> one: d = 64 hinge, spans of up to 200 steps, 16 chains 19.6 -> 16.3, 63 chains 28.9 -> 18.4, of up to 20
    // 11.3 -> 7.8, 20.0 -> 10.0; d = 128 logistic, up to 120, 4 chains 15.1 -> 13.0, 63 chains 25.8 -> 17.1; d = 256 logistic, up to 520, 4 chains 47.0 -> 45.9,
    // 63 chains 57.8 -> 49.7, bf16 hinge 74.8 -> 73.1, 85.0 -> 79.8.  Longer rows gain nothing
    // or lose (blocks of eight steps: d = 1024, 16 chains 29.4 -> 30.2, bf16 d = 2048 34.8 -> 45.8: a workgroup alone draws k rows more
    // slowly than the average's own launch does).
    float *other = nullptr;
    if (spans && spans->count > 1 && p.family == Family::DenseReg && p.scouts > 0 && !p.octets && k <= kStartModelsMost) {
        const size_t models = (size_t)k * (size_t)X->d * sizeof(float), used = h.total + perm_bytes(X->m);
        if (workspace_bytes >= used + models) other = reinterpret_cast<float *>(ws + used);
    }
    for (int64_t span = 0; span < (spans ? spans->count : 1); ++span) {
        a.span = span;
        if (span > 0 && other) {
            a.models = a.W;
            a.model_weights = spans->weights_dev;
            a.W = a.W == W ? other : W;
        } else if (span > 0) {
            a.w_start = spans->average;
            // the helpers' counters start at zero (the first time they come zeroed with the header; blocks of eight steps count on)
            if (a.helpers > 0 && !p.octets) e = launch_zero_words(a.progress, (size_t)k * 2 + 16, s);
            if (e != hipSuccess) return hip_fail(e);
        }
        e = a.slices > 1 ? launch_sliced(p, a, s) : launch_whole(p, a, s);
        if (e == hipErrorInvalidValue) return WPSGD_UNSUPPORTED;
        if (e != hipSuccess) return hip_fail(e);
        if (spans && (!other || span + 1 == spans->count)) {
            e = launch_combine(a.W, spans->weights_dev, k, X->d, spans->average, s);
            if (e != hipSuccess) return hip_fail(e);
        }
    }
    return WPSGD_OK;
}

int wpsgd_run_chains_from(const wpsgd_matrix *X, const float *y, int k, const int64_t *n_steps,
                          double eta, double lambda, wpsgd_loss loss, uint64_t seed, wpsgd_sampling sampling,
                          const float *w_start, const int64_t *step_offsets, float *W,
                          void *workspace, size_t workspace_bytes, const wpsgd_plan *plan, void *stream)
{
    return run_chains_from(X, y, k, n_steps, eta, lambda, loss, seed, sampling, w_start, step_offsets, W, workspace,
                           workspace_bytes, plan, stream, nullptr);
}

static size_t delay_ring_bytes(const wpsgd_matrix *X, int k, int tau)
{
    return (size_t)k * (size_t)(std::max(tau, 1) + 2) * (size_t)X->d * sizeof(double);
}

// a table of 32 bytes per row: what the Check function needs of a row and not of the model
static size_t delay_table_bytes(const wpsgd_matrix *X) { return align256((size_t)X->m * 32); }

// Teams of workgroups for the servers of a call under the Check function: the smallest number of samples per member at which all members
// find a compute unit.  What a team costs are some ten exchanges of 8 us, one per acceptance, mostly at the start, so short servers
// stay alone (fp32, d = 1024, m = 4000, 16 servers of 200 samples: 114 us alone, 146 in teams; 4 of up to 600: 247 and 113), and so does
// every server where the longest would gain little.
constexpr int64_t kDelayTeamShare = 32, kDelayTeamWorth = 384, kDelayVisitsWorth = 96;
// Launches with teams run in turn (chain_delay.hip) where their members look at this many samples each and teams gain a third and
// more.  The event costs a call 1.5 to 2 us (29 servers of up to 2300 samples, bf16, d = 1912: 116 | 117), and a launch as short as that is over before
// an owner gives up waiting for members (two calls of them on two streams 109 us as they come, 122 in turn).  Where teams
// gain less, calls side by side are the better for sharing units (200 servers of up to 4000, d = 256, four calls on each of two streams: 6986 us without
// teams, 7977 as they come, 9289 in turn; one call 1458 | 1190).
constexpr int64_t kDelayTurnShare = 128;
static int64_t delay_team_share(int k, const int64_t *n_samples, int *helpers)
{
    *helpers = 0;
    int64_t most = 0;
    for (int i = 0; i < k; ++i) most = std::max(most, n_samples[i]);
    const int units = compute_units();
    if (k >= units || most < kDelayTeamWorth || most > ((int64_t)1 << 30)) return 0;
    auto members = [&](int64_t share) {
        int64_t sum = 0;
        for (int i = 0; i < k; ++i) sum += delay_team_size(n_samples[i], share);
        return sum;
    };
    int64_t lo = kDelayTeamShare, hi = most;       // hi: one workgroup per server
    while (lo < hi) {
        const int64_t mid = lo + (hi - lo) / 2;
        if (members(mid) <= units) hi = mid;
        else lo = mid + 1;
    }
    *helpers = (int)(members(lo) - k);
    return *helpers > 0 && lo <= most - most / 8 ? lo : 0;
}

size_t wpsgd_run_delay_chains_workspace(const wpsgd_matrix *X, int k, int tau)
{
    if (check_matrix(X) != WPSGD_OK || !X->dense || k < 1 || tau < 0 || tau > kDelayMaxTau) return 0;
    return align256((size_t)k * sizeof(int64_t)) + align256(delay_ring_bytes(X, k, tau)) + delay_table_bytes(X);
}

int wpsgd_run_delay_chains(const wpsgd_matrix *X, const float *y, int k, const int64_t *n_samples,
                           double eta, double lambda, wpsgd_loss loss, uint64_t seed, int tau, int check,
                           const float *w_start, float *W, int64_t *accepted,
                           void *workspace, size_t workspace_bytes, void *stream)
{
    int rc = check_matrix(X);
    if (rc != WPSGD_OK) return rc;
    if (!y || !W || !accepted || tau < 0) return WPSGD_INVALID_ARG;
    rc = check_steps(k, n_samples);
    if (rc != WPSGD_OK) return rc;
    if (!(eta > 0.0) || !(lambda >= 0.0) || !(eta * lambda < 1.0)) return WPSGD_INVALID_ARG;
    if (loss != WPSGD_HINGE && loss != WPSGD_LOGISTIC) return WPSGD_INVALID_ARG;
    if (!X->dense || tau > kDelayMaxTau) return WPSGD_UNSUPPORTED;
    if (!workspace || ((uintptr_t)workspace % 256) != 0) return WPSGD_INVALID_ARG;
    if (workspace_bytes < wpsgd_run_delay_chains_workspace(X, k, tau)) return WPSGD_WORKSPACE_TOO_SMALL;
    hipStream_t s = static_cast<hipStream_t>(stream);
    char *base = static_cast<char *>(workspace);
    const size_t head = align256((size_t)k * sizeof(int64_t)), ring = align256(delay_ring_bytes(X, k, tau));
    // The table of what the Check function needs of a row costs a pass over the data set: one entry per row where the servers
    // together visit a good part of the rows, else one per visit.  Servers of a few dozen samples do without (fp32, d = 4096,
    // m = 65536: 200 servers of 50 samples 98 us without, 112 with; one of 200 samples 242 and 125).
    int64_t visits = 0, most = 0;
    for (int i = 0; i < k; ++i) {
        visits += std::min<int64_t>(n_samples[i], INT64_MAX / 2 / k);
        most = std::max(most, n_samples[i]);
    }
    const bool per_visit = visits < X->m / 4, table = check != 0 && (!per_visit || most >= kDelayVisitsWorth);
    // With an entry per visit go the servers' first entries, where the ring begins (no kernel that has a table keeps its iterates there);
    // up to 64 servers a wave adds them up as fast as it reads them, and short rings keep their room for teams.
    size_t used = 0;
    if (table && per_visit && k > kWave) {
        rc = upload_filled(base, head + (size_t)k * sizeof(int64_t), s, [&](void *host) {
            int64_t *counts = static_cast<int64_t *>(host), *first = counts + head / sizeof(int64_t);
            int64_t before = 0;
            for (int i = 0; i < k; ++i) {
                counts[i] = n_samples[i];
                first[i] = before;
                before += n_samples[i];
            }
        });
        used = head;
    } else {
        rc = upload(base, n_samples, (size_t)k * sizeof(int64_t), s);
    }
    if (rc != WPSGD_OK) return rc;
    DelayArgs a{};
    a.dense = X->dense;
    a.ld = X->ld;
    a.y = y;
    a.m = X->m;
    a.d = X->d;
    a.k = k;
    a.n_samples = reinterpret_cast<const int64_t *>(base);
    a.w_start = w_start;
    a.eta = eta;
    a.lambda = lambda;
    a.loss = (int)loss;
    a.tau = tau;
    a.check = check != 0;
    a.seed_lo = (uint32_t)seed;
    a.seed_hi = (uint32_t)(seed >> 32);
    a.ring = reinterpret_cast<double *>(base + head);
    a.W = W;
    a.accepted = accepted;
    a.row_table = table ? base + head + ring : nullptr;
    a.visits = table && per_visit ? visits : 0;
    a.visits_before = used ? reinterpret_cast<const int64_t *>(base + head) : nullptr;
    if (a.row_table && used + (size_t)k * kDelayTeamWords * sizeof(uint64_t) <= ring) {
        a.team_share = delay_team_share(k, n_samples, &a.helpers);
        a.units = compute_units();
        a.in_turn = a.team_share >= kDelayTurnShare && 3 * a.team_share <= 2 * most;
        a.team = a.team_share ? reinterpret_cast<uint64_t *>(base + head + used) : nullptr;
    }
    const bool start_ok = !w_start || (uintptr_t)w_start % 4 == 0;
    if (!start_ok) return WPSGD_INVALID_ARG;
    hipError_t e = launch_delay_servers(a, (int)X->dtype, dense_vec(X), buffer_vec(X), s);
    return e == hipSuccess ? WPSGD_OK : hip_fail(e);
}

int wpsgd_chains_status(const void *workspace, void *stream)
{
    if (!workspace) return WPSGD_INVALID_ARG;
    hipStream_t s = static_cast<hipStream_t>(stream);
    uint32_t word = 0;
    hipError_t e = hipMemcpyAsync(&word, workspace, sizeof(word), hipMemcpyDeviceToHost, s);
    if (e == hipSuccess) e = hipStreamSynchronize(s);
    if (e != hipSuccess) return hip_fail(e);
    return (word & 1u) ? WPSGD_INCOMPLETE : WPSGD_OK;
}

int wpsgd_weights_rate(int k, const int64_t *n_steps, double rate, double *a)
{
    int rc = check_steps(k, n_steps);
    if (rc != WPSGD_OK) return rc;
    if (!a || !(rate > 0.0) || !(rate <= 1.0)) return WPSGD_INVALID_ARG;
    int64_t t = 0;
    for (int i = 0; i < k; ++i) t = std::max(t, n_steps[i]);
    // rate^T = exp(T * log(rate)); the fastest chain has T = 0, so the sum is at least 1
    const double log_rate = std::log(rate);
    double total = 0.0;
    for (int i = 0; i < k; ++i) {
        a[i] = std::exp((double)(t - n_steps[i]) * log_rate);
        total += a[i];
    }
    for (int i = 0; i < k; ++i) a[i] /= total;
    return WPSGD_OK;
}

int wpsgd_weights(int k, const int64_t *n_steps, double eta, double lambda, double *a)
{
    if (!(eta > 0.0) || !(lambda >= 0.0) || !(eta * lambda < 1.0)) return WPSGD_INVALID_ARG;
    int rc = check_steps(k, n_steps);
    if (rc != WPSGD_OK) return rc;
    if (!a) return WPSGD_INVALID_ARG;
    int64_t t = 0;
    for (int i = 0; i < k; ++i) t = std::max(t, n_steps[i]);
    const double log_rate = std::log1p(-eta * lambda);    // log(1 - eta*lambda) without cancellation
    double total = 0.0;
    for (int i = 0; i < k; ++i) {
        a[i] = std::exp((double)(t - n_steps[i]) * log_rate);
        total += a[i];
    }
    for (int i = 0; i < k; ++i) a[i] /= total;
    return WPSGD_OK;
}

int wpsgd_benefit_margin(int k, const int64_t *n_steps, double rate, double *margin)
{
    int rc = check_steps(k, n_steps);
    if (rc != WPSGD_OK) return rc;
    if (!margin || !(rate > 0.0) || !(rate <= 1.0)) return WPSGD_INVALID_ARG;
    int64_t t = 0;
    for (int i = 0; i < k; ++i) t = std::max(t, n_steps[i]);
    const double log_rate = std::log(rate);
    double total = 0.0;
    for (int i = 0; i < k; ++i) total += std::exp((double)(t - n_steps[i]) * log_rate);
    *margin = 2.0 * total - (std::sqrt((double)k) + (double)k);
    return WPSGD_OK;
}

size_t wpsgd_combine_workspace(int k, int64_t d)
{
    (void)d;
    return k < 1 ? 0 : align256((size_t)k * sizeof(double));
}

int wpsgd_combine(const float *W, const double *a, int k, int64_t d, float *w_out, void *workspace,
                  size_t workspace_bytes, void *stream)
{
    if (!W || !a || !w_out || k < 1 || d < 1) return WPSGD_INVALID_ARG;
    if (!workspace || ((uintptr_t)workspace % 256) != 0) return WPSGD_INVALID_ARG;
    if (workspace_bytes < wpsgd_combine_workspace(k, d)) return WPSGD_WORKSPACE_TOO_SMALL;
    for (int i = 0; i < k; ++i)
        if (!std::isfinite(a[i])) return WPSGD_INVALID_ARG;
    hipStream_t s = static_cast<hipStream_t>(stream);
    int rc = upload(workspace, a, (size_t)k * sizeof(double), s);
    if (rc != WPSGD_OK) return rc;
    hipError_t e = launch_combine(W, static_cast<const double *>(workspace), k, d, w_out, s);
    return e == hipSuccess ? WPSGD_OK : hip_fail(e);
}

size_t wpsgd_run_spans_workspace(const wpsgd_matrix *X, int k, wpsgd_loss loss, const wpsgd_plan *plan)
{
    const size_t chains = wpsgd_run_chains_workspace(X, k, loss, plan);
    if (chains == 0) return 0;
    return chains + align256((size_t)k * (size_t)X->d * sizeof(float)) + wpsgd_combine_workspace(k, X->d);
}

int wpsgd_run_spans(const wpsgd_matrix *X, const float *y, int k, const int64_t *steps_per_span, int64_t n_spans,
                    double eta, double lambda, wpsgd_loss loss, uint64_t seed, wpsgd_sampling sampling,
                    const float *w_start, float *w_out, void *workspace, size_t workspace_bytes,
                    const wpsgd_plan *plan, void *stream)
{
    int rc = check_matrix(X);
    if (rc != WPSGD_OK) return rc;
    rc = check_steps(k, steps_per_span);
    if (rc != WPSGD_OK) return rc;
    if (!w_out || n_spans < 1) return WPSGD_INVALID_ARG;
    int64_t span = 0;
    for (int i = 0; i < k; ++i) span = std::max(span, steps_per_span[i]);
    if (span < 1 || span > ((int64_t)1 << 62) / n_spans) return WPSGD_INVALID_ARG;
    if (!workspace || ((uintptr_t)workspace % 256) != 0) return WPSGD_INVALID_ARG;
    // the chains' workspace comes first, so that its status word is the first word of this one too
    const size_t chains = wpsgd_run_chains_workspace(X, k, loss, plan);
    const size_t models = align256((size_t)k * (size_t)X->d * sizeof(float));
    const size_t average = wpsgd_combine_workspace(k, X->d);
    if (chains == 0) return WPSGD_UNSUPPORTED;
    if (workspace_bytes < chains + models + average) return WPSGD_WORKSPACE_TOO_SMALL;
    char *ws = static_cast<char *>(workspace);
    float *W = reinterpret_cast<float *>(ws + chains);
    std::vector<double> a(k);
    rc = wpsgd_weights(k, steps_per_span, eta, lambda, a.data());
    if (rc != WPSGD_OK) return rc;
    for (int i = 0; i < k; ++i)
        if (!std::isfinite(a[i])) return WPSGD_INVALID_ARG;
    const Spans spans{n_spans, a.data(), reinterpret_cast<double *>(ws + chains + models), w_out};
    return run_chains_from(X, y, k, steps_per_span, eta, lambda, loss, seed, sampling, w_start, nullptr, W, ws, chains, plan, stream,
                           &spans);
}

int wpsgd_span_condition(int k, const int64_t *steps_per_span, double rate, double *value)
{
    int rc = check_steps(k, steps_per_span);
    if (rc != WPSGD_OK) return rc;
    if (!value || !(rate > 0.0) || !(rate <= 1.0)) return WPSGD_INVALID_ARG;
    int64_t span = 0;
    for (int i = 0; i < k; ++i) span = std::max(span, steps_per_span[i]);
    const double log_rate = std::log(rate);
    double total = 0.0;
    for (int i = 0; i < k; ++i) total += std::exp((double)(span - steps_per_span[i]) * log_rate);
    *value = (double)k / total * std::exp((double)span * log_rate);
    return WPSGD_OK;
}

size_t wpsgd_objective_workspace(const wpsgd_matrix *X)
{
    if (check_matrix(X) != WPSGD_OK) return 0;
    return align256(objective_partials_bytes(X->m));
}

static int objective_check(const wpsgd_matrix *X, const float *y, const float *w, double lambda, wpsgd_loss loss,
                           const double *out)
{
    int rc = check_matrix(X);
    if (rc != WPSGD_OK) return rc;
    if (!y || !w || !out || !(lambda >= 0.0)) return WPSGD_INVALID_ARG;
    if (loss != WPSGD_HINGE && loss != WPSGD_LOGISTIC) return WPSGD_INVALID_ARG;
    if ((uintptr_t)out % sizeof(double) != 0) return WPSGD_INVALID_ARG;
    if (X->d >= (1ll << 29)) return WPSGD_UNSUPPORTED;           // 32-bit byte offsets into a row and into w
    return WPSGD_OK;
}

static int objective_launch(const wpsgd_matrix *X, const float *y, const float *w, double lambda, wpsgd_loss loss,
                            double *out, double *partials, hipStream_t s)
{
    ChainArgs a{};
    a.dense = X->dense;
    a.ld = X->ld;
    a.row_ptr = X->row_ptr;
    a.col_idx = X->col_idx;
    a.vals = X->vals;
    a.y = y;
    a.m = X->m;
    a.d = X->d;
    int vec = 1;
    if (X->dense && (uintptr_t)w % 4 == 0) vec = buffer_vec(X);         // (w is read with the same kind of load)
    hipError_t e = launch_objective(a, X->dense ? (int)X->dtype : WPSGD_F32, vec, (int)loss, w, lambda, partials, out, s);
    return e == hipSuccess ? WPSGD_OK : hip_fail(e);
}

int wpsgd_objective(const wpsgd_matrix *X, const float *y, const float *w, double lambda, wpsgd_loss loss,
                    double *out, void *workspace, size_t workspace_bytes, void *stream)
{
    int rc = objective_check(X, y, w, lambda, loss, out);
    if (rc != WPSGD_OK) return rc;
    if (!workspace || ((uintptr_t)workspace % 256) != 0) return WPSGD_INVALID_ARG;
    if (workspace_bytes < wpsgd_objective_workspace(X)) return WPSGD_WORKSPACE_TOO_SMALL;
    return objective_launch(X, y, w, lambda, loss, out, static_cast<double *>(workspace), static_cast<hipStream_t>(stream));
}

int wpsgd_objective_static(const wpsgd_matrix *X, const float *y, const float *w, double lambda, wpsgd_loss loss,
                           double *out, void *stream)
{
    int rc = objective_check(X, y, w, lambda, loss, out);
    if (rc != WPSGD_OK) return rc;
    double *partials = nullptr;          // the library's own area on this device, in place of a workspace
    size_t room = 0;
    hipError_t e = objective_static_partials(&partials, &room);
    if (e != hipSuccess) return hip_fail(e);
    if (objective_partials_bytes(X->m) > room) return WPSGD_UNSUPPORTED;     // more partial sums than that area holds
    return objective_launch(X, y, w, lambda, loss, out, partials, static_cast<hipStream_t>(stream));
}

int wpsgd_sample_indices(uint64_t seed, int chain, int64_t n0, int64_t count, int64_t m,
                         int64_t *out_host)
{
    if (chain < 0 || n0 < 0 || count < 0 || m < 1 || m > 0xFFFFFFFFLL) return WPSGD_INVALID_ARG;
    if (count > 0 && !out_host) return WPSGD_INVALID_ARG;
    for (int64_t t = 0; t < count; ++t)
        out_host[t] = (int64_t)sample_row((uint32_t)(seed & 0xFFFFFFFFu), (uint32_t)(seed >> 32),
                                          (uint32_t)chain, (uint64_t)(n0 + t), (uint32_t)m);
    return WPSGD_OK;
}

int wpsgd_sample_indices_device(uint64_t seed, int chain, int64_t n0, int64_t count, int64_t m,
                                int64_t *out_device, void *stream)
{
    if (chain < 0 || n0 < 0 || count < 0 || m < 1 || m > 0xFFFFFFFFLL) return WPSGD_INVALID_ARG;
    if (count > 0 && !out_device) return WPSGD_INVALID_ARG;
    hipError_t e = launch_sample_rows((uint32_t)(seed & 0xFFFFFFFFu), (uint32_t)(seed >> 32),
                                      (uint32_t)chain, n0, count, (uint32_t)m, 0u, out_device,
                                      static_cast<hipStream_t>(stream));
    return e == hipSuccess ? WPSGD_OK : hip_fail(e);
}

int wpsgd_shard_indices(uint64_t seed, int chain, int k, int64_t n0, int64_t count, int64_t m,
                        int64_t *out_host)
{
    if (chain < 0 || k < 1 || chain >= k || n0 < 0 || count < 0 || m < 1 || m > 0xFFFFFFFFLL || (int64_t)k > m)
        return WPSGD_INVALID_ARG;
    if (count > 0 && !out_host) return WPSGD_INVALID_ARG;
    for (int64_t t = 0; t < count; ++t)
        out_host[t] = (int64_t)shard_row((uint32_t)(seed & 0xFFFFFFFFu), (uint32_t)(seed >> 32), (uint32_t)chain,
                                         (uint32_t)k, (uint64_t)(n0 + t), (uint32_t)m);
    return WPSGD_OK;
}

int wpsgd_shard_indices_device(uint64_t seed, int chain, int k, int64_t n0, int64_t count, int64_t m,
                               int64_t *out_device, void *stream)
{
    if (chain < 0 || k < 1 || chain >= k || n0 < 0 || count < 0 || m < 1 || m > 0xFFFFFFFFLL || (int64_t)k > m)
        return WPSGD_INVALID_ARG;
    if (count > 0 && !out_device) return WPSGD_INVALID_ARG;
    hipError_t e = launch_sample_rows((uint32_t)(seed & 0xFFFFFFFFu), (uint32_t)(seed >> 32),
                                      (uint32_t)chain, n0, count, (uint32_t)m, (uint32_t)k, out_device,
                                      static_cast<hipStream_t>(stream));
    return e == hipSuccess ? WPSGD_OK : hip_fail(e);
}

int wpsgd_stream_rows(const wpsgd_matrix *X, int groups, int64_t rows_per_group, uint64_t seed,
                      float *sink, void *stream)
{
    int rc = check_matrix(X);
    if (rc != WPSGD_OK) return rc;
    if (!X->dense || !sink || groups < 1 || rows_per_group < 1) return WPSGD_INVALID_ARG;
    const int64_t elem = X->dtype == WPSGD_BF16 ? 2 : 4;
    const int64_t row_bytes = X->d * elem;
    // 16-byte loads: rows must start on 16-byte boundaries and be a whole number of them
    if ((uintptr_t)X->dense % 16 != 0 || (X->ld * elem) % 16 != 0 || row_bytes % 16 != 0 ||
        row_bytes > 0x7FFFFFFF)
        return WPSGD_UNSUPPORTED;
    hipError_t e = launch_stream_rows(X->dense, X->ld * elem, (uint32_t)row_bytes, (uint32_t)X->m, groups,
                                      rows_per_group, (uint32_t)(seed & 0xFFFFFFFFu), (uint32_t)(seed >> 32),
                                      sink, static_cast<hipStream_t>(stream));
    return e == hipSuccess ? WPSGD_OK : hip_fail(e);
}

const char *wpsgd_strerror(int status)
{
    switch (status) {
    case WPSGD_OK: return "ok";
    case WPSGD_INVALID_ARG: return "invalid argument";
    case WPSGD_HIP_ERROR: return "HIP call failed (see wpsgd_last_hip_error)";
    case WPSGD_WORKSPACE_TOO_SMALL: return "workspace too small";
    case WPSGD_UNSUPPORTED: return "no kernel implements the forced plan";
    case WPSGD_INCOMPLETE: return "chains cut into column slices gave up waiting for each other; their rows of W are NaN";
    default: return "unknown status";
    }
}

int wpsgd_last_hip_error(void) { return g_last_hip_error; }

}  // extern "C"
