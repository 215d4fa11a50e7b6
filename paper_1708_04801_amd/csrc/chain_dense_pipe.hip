// Dense-row SGD chains of short rows, sixteen steps at a time, with everything but the slopes off the dependent path.
//
// For the sixteen rows x_0..x_15 of block b, the rows x'_0..x'_15 of the block before and the vector v' at THAT block's start,
//     yhat_j = s_j * (v'.x_j + sum_t c'_t x'_t.x_j + sum_{a<j} c_a x_a.x_j),   c_a = -eta*g_a / s_{a+1}.
// The products between rows do not depend on v, and v'.x_j does not depend on the steps of the block before: while one wave takes
// the sixteen slopes of a block, others update v with the block before and multiply it with the rows of the block behind.  What is
// left on the dependent path of a step is one slope and one multiply-add across sixteen lanes; the second sum grows in
// its shadow, one term per step of the block before.  It is the same arithmetic as single steps up to the order of sums, in the same
// precision (fp64 for the hinge, fp32 for the logistic loss).
//
// A workgroup runs one chain, one barrier per beat; beat b is the time of block b:
//     slopes (wave 0)     block b: q_j = the first two sums, then sixteen slopes; collects block b+1's second sum; leaves c in LDS
//     model  (1 or 2)     v += sum c x of block b-1 (lane owns a column), then v.x_j for block b+1 (lane (j, g): columns of quarter g)
//     scouts (2 or 3)     each a part of the columns: rows of block b+7 requested, rows of block b+4 to LDS, their products
//                         with each other and with those of block b+3 on the matrix cores; a beat later these are added up, multiplied with
//                         everything known beforehand and left in LDS
//
// What bounds it: fp32 rows of up to 64 elements and bf16 ones the slopes (a beat of some 1250 cycles, of which the sixteen slopes
// take 900: exponential, addition, reciprocal, multiply-add, each waiting for the one before); hinge rows and longer fp32 rows the scouts:
// fp64 and fp32 matrix products (64 and 32 cycles) keep a SIMD's vector unit to themselves, 2 * C / 4 of them a block.
// us per step, eight chains, blocks without the pipeline -> with: logistic d = 64 0.0445 -> 0.0323, d = 128 0.0538 -> 0.047, d = 256 0.090 ->
// 0.075; bf16 d = 64 0.045 -> 0.033, d = 128 0.055 -> 0.039, d = 256 0.098 -> 0.048; hinge d = 64 0.0542 -> 0.0476 (d = 128 0.0703 | 0.0715,
// d = 256 on one wave 0.130 | 0.125: not taken).  The sums of four steps are added to v at a time: its error against fp64 is
// 0.6 of what it was (d = 64, 4000 steps: 6.9e-7 -> 4.1e-7).
#include <type_traits>

#include "device_utils.h"
#include "internal.h"
#include "step_rows.h"

namespace wpsgd {
namespace {

constexpr int kBlock = 16;                    // steps per block
constexpr int kLead = 4;                      // beats between a block's rows reaching LDS and its slopes
constexpr int kTiles = kLead + 1;             // blocks whose rows are in LDS: from kLead beats before the slopes to the slopes' own
constexpr int kBlocksPerWindow = kWave / kBlock;
static_assert(kPipeAhead == kLead + 3, "rows are requested three beats before they reach LDS");
static_assert(kBlocksPerWindow == kWindowParts && kWindowParts == 4, "the scouts' requests run three blocks ahead of their rows, in one window of 64 steps or the next");

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef double f64x4 __attribute__((ext_vector_type(4)));
typedef short s16x4 __attribute__((ext_vector_type(4)));

// PE elements of a row from any element boundary
template <typename TX, int PE> struct Elements;
template <int PE> struct Elements<float, PE> {
    typedef float packed __attribute__((ext_vector_type(PE), aligned(4)));
    packed q;
    __device__ void load(const float *p) { q = *reinterpret_cast<const packed *>(p); }
    __device__ float at(int e) const { return q[e]; }
};
template <int PE> struct Elements<uint16_t, PE> {
    typedef uint16_t packed __attribute__((ext_vector_type(PE), aligned(2)));
    packed q;
    __device__ void load(const uint16_t *p) { q = *reinterpret_cast<const packed *>(p); }
    __device__ float at(int e) const { return bf16_one(q[e]); }
};

// the matrix cores' 16x16x4 product in the state's precision: D[i][j] += sum_k A[i][k] B[k][j], A's row and
// B's column in lane mod 16, k in lane / 16
template <typename TV> struct Product;
template <> struct Product<double> {
    f64x4 d = {0.0, 0.0, 0.0, 0.0};
    __device__ void add(double a, double b) { d = __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, d, 0, 0, 0); }
    static __device__ int row(int r, int lane) { return 4 * r + lane / 16; }       // D's register r holds row .. of column lane mod 16
};
template <> struct Product<float> {
    f32x4 d = {0.0f, 0.0f, 0.0f, 0.0f};
    __device__ void add(float a, float b) { d = __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, d, 0, 0, 0); }
    static __device__ int row(int r, int lane) { return 4 * (lane / 16) + r; }
};

__device__ inline void beat_barrier()         // everything this wave wrote to LDS is there before it arrives
{
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

// Who does what.  Waves sit on the four SIMDs in turn.  fp64 and fp32 matrix products keep a SIMD's vector unit to themselves, so scouts
// share theirs with as little as possible: up to 128 columns two scouts have two SIMDs alone, beyond that there are three.
template <typename TX, int LOSS, int C>
struct Team {
    static constexpr bool kLight = sizeof(TX) == 2 && LOSS == kLossLogistic;       // bf16 products: four times as fast, and beside the vector unit
    static constexpr int S = C <= 64 || kLight ? 2 : 3;          // scouts
    static constexpr int M = C > 128 ? 2 : 1;                    // waves that hold the model
    static constexpr int kWaves = 1 + S + M + 2;
    static constexpr int kSlopes = 0, kModel = 16, kClerk = 32;  // roles: scout h is 1 + h, model wave w kModel + w, clerk i kClerk + i
    static __device__ int role(int wave)
    {
        if constexpr (S == 2 && M == 1) {
            constexpr uint64_t r = 0x20210201'1000ull;           // wave 0 in the lowest byte
            return (int)((r >> (8 * wave)) & 0xff);
        } else if constexpr (S == 2) {
            constexpr uint64_t r = 0x2120110201'1000ull;
            return (int)((r >> (8 * wave)) & 0xff);
        } else {
            constexpr uint64_t r = M == 1 ? 0x21201001'020300ull : 0x21201110'01020300ull;
            return (int)((r >> (8 * wave)) & 0xff);
        }
    }
};

template <typename TX, int LOSS, int C>
struct PipeLds {
    using TV = typename StateType<LOSS>::type;
    using Acc = decltype(Product<TV>::d);
    float tile[kTiles][kBlock][C + 4];        // (rows four banks apart: sixteen lanes' 16-byte accesses spread over all banks)
    Acc part[2][Team<TX, LOSS, C>::S][2][kWave];           // the scouts' shares of a block's products: with each other, with the block before
    TV own[4][kBlock][kBlock + 4];            // [j][a], a < j: what a unit of slope of step a adds to q_j
    TV cross[2][kBlock][kBlock + 4];          // [j][t]: what a unit of slope of step t of the block before adds to q_j
    TV zs[4][kBlock], cs[4][kBlock];          // y_j s_j (times log2 e for the logistic loss), y_j eta / s_{j+1} (0 past the chain's end)
    TV model[C];
    uint32_t rows[2][kWave];                  // rows of a window's steps
    TV dots[2][Team<TX, LOSS, C>::M][kBlock];       // the model waves' shares of v.x_j
    TV c[2][kBlock];                          // the steps' coefficients
    uint32_t odd[4][2];                       // are the block's products with itself, or with the block before, not all finite?
    TV sums[2][Team<TX, LOSS, C>::M];               // one step at a time: the waves' shares of v.x
};

// a lane's four products into its column's line
__device__ inline void store_products(float *line, const f32x4 &q, int g) { *reinterpret_cast<f32x4 *>(line + 4 * g) = q; }
__device__ inline void store_products(double *line, const f64x4 &q, int g)
{
#pragma unroll
    for (int r = 0; r < 4; ++r) line[4 * r + g] = q[r];
}

// acc[t % 4] += (c of lane t of the row of sixteen lanes) * x[t], t = 0..15.  (One statement, so that nothing can come between the
// wait states a DPP operand needs and its uses.)
#define WPSGD_ADD(OP, A, T, X) OP " %" #A ", %4, %" #X " row_newbcast:" #T " row_mask:0xf bank_mask:0xf\n\t"
#define WPSGD_ADD_BLOCK(OP)                                                                                                  \
    "s_nop 1\n\t" WPSGD_ADD(OP, 0, 0, 5) WPSGD_ADD(OP, 1, 1, 6) WPSGD_ADD(OP, 2, 2, 7) WPSGD_ADD(OP, 3, 3, 8)                  \
    WPSGD_ADD(OP, 0, 4, 9) WPSGD_ADD(OP, 1, 5, 10) WPSGD_ADD(OP, 2, 6, 11) WPSGD_ADD(OP, 3, 7, 12)                              \
    WPSGD_ADD(OP, 0, 8, 13) WPSGD_ADD(OP, 1, 9, 14) WPSGD_ADD(OP, 2, 10, 15) WPSGD_ADD(OP, 3, 11, 16)                           \
    WPSGD_ADD(OP, 0, 12, 17) WPSGD_ADD(OP, 1, 13, 18) WPSGD_ADD(OP, 2, 14, 19) WPSGD_ADD(OP, 3, 15, 20)
#define WPSGD_OPERANDS                                                                                                       \
    : "+v"(acc[0]), "+v"(acc[1]), "+v"(acc[2]), "+v"(acc[3]) : "v"(c), "v"(x[0]), "v"(x[1]), "v"(x[2]), "v"(x[3]), "v"(x[4]), "v"(x[5]), \
      "v"(x[6]), "v"(x[7]), "v"(x[8]), "v"(x[9]), "v"(x[10]), "v"(x[11]), "v"(x[12]), "v"(x[13]), "v"(x[14]), "v"(x[15])
__device__ inline void add_block(float (&acc)[4], float c, const float (&x)[kBlock]) { asm volatile(WPSGD_ADD_BLOCK("v_fmac_f32_dpp") WPSGD_OPERANDS); }
__device__ inline void add_block(double (&acc)[4], double c, const double (&x)[kBlock]) { asm volatile(WPSGD_ADD_BLOCK("v_fmac_f64_dpp") WPSGD_OPERANDS); }
#undef WPSGD_ADD
#undef WPSGD_ADD_BLOCK
#undef WPSGD_OPERANDS

template <typename TX, int LOSS, int C>
__global__ __launch_bounds__((Team<TX, LOSS, C>::kWaves) * kWave) void chain_dense_pipe_kernel(ChainArgs a)
{
    using TV = typename StateType<LOSS>::type;
    using Lds = PipeLds<TX, LOSS, C>;
    using Us = Team<TX, LOSS, C>;
    constexpr int kScouts = Us::S, M = Us::M, CE = C / (M * kWave);      // waves that hold the model, columns a lane of them owns
    extern __shared__ __attribute__((aligned(16))) uint8_t lds_raw[];
    Lds &lds = *reinterpret_cast<Lds *>(lds_raw);

    const int lane = (int)(threadIdx.x & (kWave - 1));
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x / kWave);
    const int role = Us::role(wave);
    const int j = lane % 16, g = lane / 16;
    const int cb = (int)blockIdx.x;
    const int64_t n = a.nsteps[cb];
    const int d = (int)a.d;
    float *out = a.W + (int64_t)a.order[cb] * a.d;
    if (n == 0) {
        for (int c = (int)threadIdx.x; c < d; c += Us::kWaves * kWave) out[c] = start_value(a, c);
        return;
    }
    const int64_t nblk = (n + kBlock - 1) / kBlock;
    const double rho64 = a.pow_tab[kWave - 1] * a.rho, inv_rho64 = a.pow_tab[2 * kWave - 1];

    if (role == Us::kSlopes) {
        // ------------------------------------------------------------------------- slopes
        __builtin_amdgcn_s_setprio(3);
        struct Known { TV own[kBlock], cross[kBlock], zs, cs; uint2 odd; } first, second;
        auto fetch = [&](Known &f, int64_t b) {           // what block b's slopes need beside the dots
#pragma unroll
            for (int t = 0; t < kBlock; ++t) {
                f.own[t] = lds.own[b & 3][j][t];
                f.cross[t] = lds.cross[(b + 1) & 1][j][t];
            }
            f.zs = lds.zs[b & 3][j];
            f.cs = lds.cs[b & 3][j];
            f.odd = *reinterpret_cast<const uint2 *>(lds.odd[b & 3]);
        };
        TV next = (TV)0;
        // false: the block is odd, or was the last
        auto beat = [&](Known &now, Known &then, int64_t b) {
            if (b >= nblk || __builtin_amdgcn_readfirstlane((int)(now.odd.x | now.odd.y)) != 0) return false;
            TV p = lds.dots[b & 1][0][j];
#pragma unroll
            for (int w = 1; w < M; ++w) p += lds.dots[b & 1][w][j];
            TV q = next + now.zs * p;
            next = (TV)0;
            fetch(then, b + 1);
            const TV c = now.cs * take_block_steps<LOSS>(q, now.own, next, now.cross);
            if (lane < kBlock) lds.c[b & 1][lane] = c;
            beat_barrier();
            return true;
        };
#pragma unroll 1
        for (int q = 0; q < 2 + kLead - 1; ++q) beat_barrier();
        fetch(first, 0);
        beat_barrier();
        for (int64_t b = 0;; b += 2)
            if (!beat(first, second, b) || !beat(second, first, b + 1)) return;
    }

    if (role >= Us::kModel && role < Us::kClerk) {
        // ------------------------------------------------------------------------- model
        __builtin_amdgcn_s_setprio(2);
        const int w0 = role - Us::kModel, first = w0 * CE * kWave, col = first + lane * CE;      // (of the wave, of the lane)
        TV v[CE];
        start_values(a, v, [&](int e) { return col + e; });
        double s_w = 1.0, eos_w = a.eta;
        TV xu[CE][kBlock];                    // rows of the block to update with: this lane's columns
        f32x4 xd[4 * CE];                     // rows of the block to multiply with: row j, columns 16*i + 4*g ..
        auto fetch_update = [&](int tile) {
#pragma unroll
            for (int t = 0; t < kBlock; ++t)
#pragma unroll
                for (int e = 0; e < CE; ++e) xu[e][t] = (TV)lds.tile[tile][t][col + e];
        };
        auto fetch_dot = [&](int tile) {
#pragma unroll
            for (int i = 0; i < 4 * CE; ++i) xd[i] = *reinterpret_cast<const f32x4 *>(&lds.tile[tile][j][first + 16 * i + 4 * g]);
        };
        auto multiply = [&](int64_t b) {      // v.x_j of block b
#pragma unroll
            for (int e = 0; e < CE; ++e) lds.model[col + e] = v[e];
            TV acc[4] = {(TV)0, (TV)0, (TV)0, (TV)0};
#pragma unroll
            for (int i = 0; i < 4 * CE; ++i)
#pragma unroll
                for (int e = 0; e < 4; ++e) acc[e] += lds.model[first + 16 * i + 4 * g + e] * (TV)xd[i][e];
            TV p = (acc[0] + acc[1]) + (acc[2] + acc[3]);
            p = merge_values<false>(p, p);    // the four quarters of the columns: every lane ends with the whole sum
            p = merge_values<true>(p, p);
            if (lane < kBlock) lds.dots[b & 1][w0][lane] = p;
        };
#pragma unroll 1
        for (int q = 0; q < 2 + kLead - 1; ++q) beat_barrier();
        fetch_dot(0);
        multiply(0);
        fetch_dot(1);
        beat_barrier();
        uint2 odd = *reinterpret_cast<const uint2 *>(lds.odd[0]);
        int64_t b = 0;
        int tile = 0, tile_dot = 2;           // of blocks b and b+2
        for (;; ++b) {
            if (b > 0) {
                const TV c = lds.c[(b - 1) & 1][j];
#pragma unroll
                for (int e = 0; e < CE; ++e) {
                    TV acc[4] = {v[e], (TV)0, (TV)0, (TV)0};
                    add_block(acc, c, xu[e]);
                    v[e] = (acc[0] + acc[1]) + (acc[2] + acc[3]);
                }
                if (b % kBlocksPerWindow == 0 && b < nblk) {
                    s_w *= rho64;
                    eos_w *= inv_rho64;
                    if (s_w < 0x1p-30) {      // fold the scale into v; the clerk does the same to its own
#pragma unroll
                        for (int e = 0; e < CE; ++e) v[e] *= (TV)s_w;
                        s_w = 1.0;
                        eos_w = a.eta;
                    }
                }
            }
            if (b == nblk || __builtin_amdgcn_readfirstlane((int)(odd.x | odd.y)) != 0) break;
            multiply(b + 1);                  // (behind the last block: of rows nobody asks for)
            odd = *reinterpret_cast<const uint2 *>(lds.odd[(b + 1) & 3]);
            fetch_update(tile);
            fetch_dot(tile_dot);
            tile = tile == kTiles - 1 ? 0 : tile + 1;
            tile_dot = tile_dot == kTiles - 1 ? 0 : tile_dot + 1;
            beat_barrier();
        }
        if (b < nblk) {
            // The block has a row that is not finite (or so large that a product, with its coefficient, is not).  Two terms of an infinite product may
            // have different signs, and a step that is not taken still adds 0 times its row, so products must not be split: from
            // here on, on data no model is learnt from, one step is taken after the other.
            StepRows rows;
            rows.init(a, cb, lane);
            for (int64_t t = b * kBlock; t < n; ++t) {
                if (t % kWave == 0 && t > b * kBlock) {
                    s_w *= rho64;
                    eos_w *= inv_rho64;
                    if (s_w < 0x1p-30) {
#pragma unroll
                        for (int e = 0; e < CE; ++e) v[e] *= (TV)s_w;
                        s_w = 1.0;
                        eos_w = a.eta;
                    }
                }
                const uint32_t row = rows.at(t);
                const TX *at = static_cast<const TX *>(a.dense) + (int64_t)row * a.ld + col;
                TV x[CE], p = (TV)0;
#pragma unroll
                for (int e = 0; e < CE; ++e) {
                    float xf = 0.0f;
                    if (col + e < d) {
                        if constexpr (sizeof(TX) == 2) xf = bf16_one(at[e]);
                        else xf = at[e];
                    }
                    x[e] = (TV)xf;
                    p += v[e] * x[e];
                }
                p = wave_sum(p);
                if constexpr (M > 1) {
                    if (lane == 0) lds.sums[t & 1][w0] = p;
                    beat_barrier();
                    p = lds.sums[t & 1][0];
#pragma unroll
                    for (int w = 1; w < M; ++w) p += lds.sums[t & 1][w];
                }
                const int l = (int)(t % kWave);
                const double y = (double)a.y[row], sl = s_w * a.pow_tab[l] * y, el = eos_w * a.pow_tab[kWave + l] * y;
                TV ct;
                if constexpr (LOSS == kLossHinge) ct = sl * p < 1.0 ? el : 0.0;
                else ct = (float)el * unit_slope<LOSS>((float)(sl * 1.4426950408889634) * p);
#pragma unroll
                for (int e = 0; e < CE; ++e) v[e] += ct * x[e];
            }
        }
        const int64_t last_w = (n - 1) / kWave;
        const int rem = (int)(n - last_w * kWave);                          // 1..64 steps in the last window
        const double s_end = s_w * a.pow_tab[rem - 1] * a.rho;
#pragma unroll
        for (int e = 0; e < CE; ++e)
            if (col + e < d) out[col + e] = (float)(s_end * (double)v[e]);
        return;
    }

    if (role >= Us::kClerk) {
        // ------------------------------------------------------------------------- clerks
        __builtin_amdgcn_s_setprio(1);
        const int kind = role - Us::kClerk;               // 0: products within a block, 1: with the block before (and rows)
        StepRows rows;
        rows.init(a, cb, lane);
        const double up = a.pow_tab[lane], down = a.pow_tab[kWave + lane];
        const uint32_t row = rows.window(0, lane), row_next = rows.window(1, lane);
        float y_next = a.y[row];
        if (kind == 0) {
            lds.rows[0][lane] = row;
            lds.rows[1][lane] = row_next;
        }
        beat_barrier();
        beat_barrier();                       // the scouts have taken the rows of window 0
        double s_w = 1.0, eos_w = a.eta;      // scale and eta/scale at the start of the window
        // per lane, for the steps of a window: y s (times log2 e) and y eta / s; and those of the window before
        TV zs = (TV)0, cs = (TV)0, zs_before = (TV)0, cs_before = (TV)0;
        for (int64_t w = 0;; ++w) {
            zs_before = zs;
            cs_before = cs;
            {
                const double y = (double)y_next;
                double s_unfolded = s_w;
                if (w > 0) {
                    s_w *= rho64;
                    eos_w *= inv_rho64;
                    s_unfolded = s_w;
                    if (s_w < 0x1p-30) {
                        s_w = 1.0;
                        eos_w = a.eta;
                    }
                }
                // (products with what came before a folding need the scale as it was)
                const double sl = (kind == 1 && lane < kBlock ? s_unfolded : s_w) * up * y, el = w * kWave + lane < n ? eos_w * down * y : 0.0;
                if constexpr (LOSS == kLossHinge) {
                    zs = sl;
                    cs = el;
                } else {
                    zs = (float)(sl * 1.4426950408889634);
                    cs = (float)el;
                }
            }
#pragma unroll
            for (int u = 0; u < kBlocksPerWindow; ++u) {
                const int64_t m = w * kBlocksPerWindow + u;          // the block whose rows have arrived; block m-1 is finished
                if (u == 0) y_next = a.y[lds.rows[(w + 1) & 1][lane]];
                if (m > 0) {
                    typename Lds::Acc sum = lds.part[(m - 1) & 1][0][kind][lane];
#pragma unroll
                    for (int s = 1; s < kScouts; ++s) sum += lds.part[(m - 1) & 1][s][kind][lane];
                    const int lu = kBlock * ((u + 3) % 4);           // block m-1 in its window
                    const int lv = kBlock * ((u + 2) % 4);           // block m-2 in its window
                    const TV z = __shfl(u == 0 ? zs_before : zs, lu + j);
                    // the steps the products are with: the block's own, or those of the block before
                    const TV with = kind == 0 ? (u == 0 ? cs_before : cs) : (u <= 1 ? cs_before : cs);
                    const int l0 = kind == 0 ? lu : lv;
                    TV cc[4];
#pragma unroll
                    for (int r = 0; r < 4; ++r) cc[r] = z * __shfl(with, l0 + Product<TV>::row(r, lane));
                    bool odd = false;
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        sum[r] *= cc[r];
                        odd = odd || !((sum[r] < (TV)0 ? -sum[r] : sum[r]) < (TV)__builtin_inf());
                    }
                    const bool any = __builtin_amdgcn_ballot_w64(odd) != 0;
                    if (lane == 0) lds.odd[(m - 1) & 3][kind] = any ? 1u : 0u;
                    if (kind == 0) {
                        const TV mine = __shfl(with, lu + j);
#pragma unroll
                        for (int r = 0; r < 4; ++r) sum[r] = Product<TV>::row(r, lane) < j ? sum[r] : (TV)0;
                        store_products(lds.own[(m - 1) & 3][j], sum, g);
                        if (g == 0) lds.cs[(m - 1) & 3][j] = mine;
                    } else {
                        store_products(lds.cross[(m - 1) & 1][j], sum, g);
                        if (g == 0) lds.zs[(m - 1) & 3][j] = z;
                    }
                }
                if (m > nblk) return;
                if (kind == 1) {
                    const uint32_t row = rows.window_part(u, w + 2, lane);
                    if (u == kBlocksPerWindow - 1) lds.rows[w & 1][lane] = row;
                }
                beat_barrier();
            }
        }
    }

    // ----------------------------------------------------------------------------- scouts
    constexpr int PE = 4;                     // elements per lane of a load
    constexpr int K = C / (4 * PE);           // loads a row takes, 4 * PE columns each
    constexpr int KS = (K + kScouts - 1) / kScouts;       // .. of a scout: loads h, h + 3, ..
    using Load = Elements<TX, PE>;
    // rows are multiplied as they are loaded, but for fp64 products
    constexpr bool kAsLoaded = std::is_same_v<TV, float>;
    const int h = role - 1;
    const TX *X = static_cast<const TX *>(a.dense);
    Load raw[kBlocksPerWindow][KS];           // of block m in slot m mod 4
    TV wide[kAsLoaded ? 1 : 2][KS][PE];       // of blocks m and m-1
#pragma unroll
    for (int i = 0; i < KS; ++i)
#pragma unroll
        for (int e = 0; e < PE; ++e) {
            raw[3][i].q[e] = 0;
            if constexpr (!kAsLoaded) wide[1][i][e] = (TV)0;
        }
    int off[KS];                              // this lane's columns of a load; one that reaches past the row's end is made from d-PE on
#pragma unroll
    for (int i = 0; i < KS; ++i) off[i] = min(4 * PE * (h + kScouts * i) + PE * g, d - PE);
    auto request = [&](Load (&slot)[KS], uint32_t row) {
        const TX *x = X + (int64_t)row * a.ld;
#pragma unroll
        for (int i = 0; i < KS; ++i) slot[i].load(x + off[i]);
    };
    // .. and shifted; columns from d on are zero.
    const int edge = d / (4 * PE), shift = 4 * PE * edge + PE * g - (d - PE);      // the load the row ends in (edge >= K: none)
    auto trim = [&](Load &l, int kk) {
        if (kk < edge) return;                // (uniform)
        const Load q = l;
#pragma unroll
        for (int e = 0; e < PE; ++e) {
            TX r = 0;
#pragma unroll
            for (int s = 0; e + s < PE; ++s) r = (s == 0 ? shift <= 0 : shift == s) ? (TX)q.q[e + s] : r;
            l.q[e] = kk == edge ? r : (TX)0;
        }
    };
    beat_barrier();
#pragma unroll
    for (int u = 0; u + 1 < kBlocksPerWindow; ++u) request(raw[u], lds.rows[0][kBlock * u + j]);
    beat_barrier();
    int tile = 0;                             // of the block whose rows have arrived
    for (int64_t w = 0;; ++w) {
#pragma unroll
        for (int u = 0; u < kBlocksPerWindow; ++u) {
            const int64_t m = w * kBlocksPerWindow + u;              // the block whose rows have arrived
            if (m > nblk) return;
            const uint32_t row = lds.rows[(u == 0 ? w : w + 1) & 1][kBlock * ((u + 3) % 4) + j];       // of block m+3
            Load(&now)[KS] = raw[u];
            Load(&before)[KS] = raw[(u + 3) % 4];
            Product<TV> own, cross;
#pragma unroll
            for (int i = 0; i < KS; ++i) {
                if (K % kScouts != 0 && i == KS - 1 && h >= K % kScouts) continue;      // (uniform)
                trim(now[i], h + kScouts * i);
                f32x4 q;
#pragma unroll
                for (int e = 0; e < PE; ++e) q[e] = now[i].at(e);
                float *at = &lds.tile[tile][j][4 * PE * (h + kScouts * i) + PE * g];
                *reinterpret_cast<f32x4 *>(at) = q;
                if constexpr (kAsLoaded && std::is_same_v<TX, uint16_t>) {
                    const s16x4 b = __builtin_bit_cast(s16x4, now[i].q), c = __builtin_bit_cast(s16x4, before[i].q);
                    own.d = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(b, b, own.d, 0, 0, 0);
                    cross.d = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(c, b, cross.d, 0, 0, 0);
                } else if constexpr (kAsLoaded) {
#pragma unroll
                    for (int e = 0; e < PE; ++e) {
                        own.add(now[i].q[e], now[i].q[e]);
                        cross.add(before[i].q[e], now[i].q[e]);
                    }
                } else {
#pragma unroll
                    for (int e = 0; e < PE; ++e) {
                        const TV x = (TV)q[e];
                        own.add(x, x);
                        cross.add(wide[(u + 1) & 1][i][e], x);
                        wide[u & 1][i][e] = x;
                    }
                }
            }
            request(before, row);
            lds.part[m & 1][h][0][lane] = own.d;
            lds.part[m & 1][h][1][lane] = cross.d;
            tile = tile == kTiles - 1 ? 0 : tile + 1;
            beat_barrier();
        }
    }
}

template <typename TX, int LOSS, int C>
hipError_t launch(const ChainArgs &a, hipStream_t s)
{
    auto kernel = chain_dense_pipe_kernel<TX, LOSS, C>;
    constexpr size_t bytes = sizeof(PipeLds<TX, LOSS, C>);
    static_assert(bytes <= 160 * 1024, "a compute unit's LDS");
    if constexpr (bytes > 64 * 1024) {
        const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(kernel, dim3(a.k), dim3(Team<TX, LOSS, C>::kWaves * kWave), bytes, s, a);
    return hipGetLastError();
}

template <typename TX, int LOSS>
hipError_t launch_width(const ChainArgs &a, hipStream_t s)
{
    if (a.d <= 64) return launch<TX, LOSS, 64>(a, s);
    static_assert(kPipeHingeMaxColumns == 64, "what is built for the hinge");
    if constexpr (LOSS == kLossLogistic) {
        if (a.d <= 128) return launch<TX, LOSS, 128>(a, s);
        return launch<TX, LOSS, 256>(a, s);
    }
    return hipErrorInvalidValue;
}

}  // namespace

hipError_t launch_dense_pipe(const Plan &p, const ChainArgs &a, hipStream_t s)
{
    if (a.d < kBlockMinColumns || a.d > kBlockMaxColumns) return hipErrorInvalidValue;
    if (p.dtype == WPSGD_BF16)
        return p.loss == WPSGD_HINGE ? launch_width<uint16_t, kLossHinge>(a, s) : launch_width<uint16_t, kLossLogistic>(a, s);
    return p.loss == WPSGD_HINGE ? launch_width<float, kLossHinge>(a, s) : launch_width<float, kLossLogistic>(a, s);
}

}  // namespace wpsgd
