// Dense-row SGD chains of short rows (at most 256 elements), sixteen steps at a time.
//
// With rows this short a step of the register kernel is one wave's chain of dependent instructions: two
// multiplications, six levels of a wave-wide sum, the slope, the update.  Only the slopes have to be taken
// one after the other.  For the sixteen rows x_0..x_15 of a block and the vector v at its start,
//     yhat_j = s_j * (v.x_j + sum_{a<j} c_a x_a.x_j),   c_a = -eta*g_a / s_{a+1},
// so with the sixteen products v.x_j and the Gram matrix x_a.x_j in hand a step is one comparison (or one
// sigmoid) and one multiply-add across sixteen lanes, lane j holding yhat_j.  It is the same arithmetic as
// sixteen single steps up to the order of sums, in the same precision (fp64 for the hinge, fp32 for the logistic loss).
//
// The Gram matrix does not depend on v and is a contraction: three scout waves form it on the matrix cores
// (16x16x4 products in the state's precision; row j in lane j mod 16 is the layout of either operand, so a
// row's registers serve as both).  Wave 0 runs the chain:
//     v.x_j         lane (j, g) multiplies the columns of its quarter g, then two exchanges between rows of lanes
//     16 slopes     as above, the Gram rows premultiplied by the scouts with everything known beforehand
//     v += sum c_a x_a    lane owns columns
// Rows pass through LDS as fp32 (a tile of 16 rows per section), because wave 0 reads them in both layouts.
//
// Scout h of S takes blocks h, h+S, ..: S block times for one block, one barrier per block time.  It requests a block's
// rows one block (of its own) ahead and fills section (block mod 2) in its last block time, while wave 0 is
// at the block before; wave 0 is S blocks behind the first scout.  All waves pass the same number of barriers.
//
// What bounds it: wave 0's dependent instructions (a step is its slope and one multiply-add that fetches the slope from its
// lane, some 40 cycles; reading the slope into a scalar register, testing it there and selecting cost 50 to 60: us per step, eight
// chains, hinge d = 64 0.062 -> 0.054, d = 128 0.078 -> 0.070, logistic d = 64 0.050 -> 0.0445); with fp64 rows of more than 128
// elements the matrix products (a quarter of them, for timing only: 0.129 -> 0.103 at d = 256; a fourth scout, which shares
// wave 0's vector unit, gave nothing: fp64 and fp32 matrix products keep it to themselves).
// us per step, eight chains, one step at a time -> blocks: hinge d = 64 0.110 -> 0.054, d = 128 0.133 -> 0.070; logistic 0.090 ->
// 0.0445, d = 256 0.104 -> 0.090; bf16 d = 256 0.162 -> 0.110, logistic (64 chains) 0.132 -> 0.098.
#include <type_traits>

#include "device_utils.h"
#include "internal.h"
#include "step_rows.h"

namespace wpsgd {
namespace {

constexpr int kBlock = 16;                    // steps per block
constexpr int kScouts = 3;
constexpr int kBlockThreads = (1 + kScouts) * kWave;
constexpr int kBlocksPerWindow = kWave / kBlock;

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef double f64x4 __attribute__((ext_vector_type(4)));

// four elements of a row from any element boundary
template <typename TX> struct FourElements;
template <> struct FourElements<float> {
    typedef float packed __attribute__((ext_vector_type(4), aligned(4)));
    packed q;
    __device__ void load(const float *p) { q = *reinterpret_cast<const packed *>(p); }
    __device__ float at(int e) const { return q[e]; }
};
template <> struct FourElements<uint16_t> {
    typedef uint16_t packed __attribute__((ext_vector_type(4), aligned(2)));
    packed q;
    __device__ void load(const uint16_t *p) { q = *reinterpret_cast<const packed *>(p); }
    __device__ float at(int e) const { return bf16_one(q[e]); }
};

// the matrix cores' 16x16x4 product in the state's precision: D[i][j] += sum_k A[i][k] B[k][j], A's row and
// B's column in lane mod 16, k in lane / 16
template <typename TV> struct Gram;
template <> struct Gram<double> {
    f64x4 d = {0.0, 0.0, 0.0, 0.0};
    __device__ void add(float x) { const double a = (double)x; d = __builtin_amdgcn_mfma_f64_16x16x4f64(a, a, d, 0, 0, 0); }
    static __device__ int row(int r, int lane) { return 4 * r + lane / 16; }       // D's register r holds row .. of column lane mod 16
};
template <> struct Gram<float> {
    f32x4 d = {0.0f, 0.0f, 0.0f, 0.0f};
    __device__ void add(float x) { d = __builtin_amdgcn_mfma_f32_16x16x4f32(x, x, d, 0, 0, 0); }
    static __device__ int row(int r, int lane) { return 4 * (lane / 16) + r; }
};

__device__ inline void section_barrier()      // everything this wave wrote to LDS is there before it arrives
{
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

template <typename TX, int LOSS, int C>
__global__ __launch_bounds__(kBlockThreads) void chain_dense_block_kernel(ChainArgs a)
{
    using TV = typename StateType<LOSS>::type;
    constexpr int CE = C / kWave;             // columns a lane of wave 0 owns
    constexpr int K = C / 16;                 // pieces of 16 columns
    constexpr int kStride = C + 4;            // (rows four banks apart: sixteen lanes' 16-byte accesses spread over all banks)
    struct Section {
        float tile[kBlock][kStride];
        TV gram[kBlock][kBlock];              // [a][j], a < j: what a unit of step a adds to yhat_j
        TV zs[kBlock], cs[kBlock];            // y_j s_j (times log2 e for the logistic loss), y_j eta / s_{j+1} (0 past the chain's end)
    };
    __shared__ __attribute__((aligned(16))) Section section[2];
    __shared__ __attribute__((aligned(16))) TV model[C];
    // does block b (in word b mod 4) hold an element whose products with others may not be finite?
    __shared__ uint32_t excess[4];
    // (fp64 products of fp32 numbers do not overflow; 256 fp32 squares of less than 2^58 do not)
    constexpr float kProbe = LOSS == kLossHinge ? 0.0f : 0x1p70f;

    const int lane = (int)(threadIdx.x & (kWave - 1));
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x / kWave);
    const int j = lane % 16, g = lane / 16;
    const int chain = a.order[blockIdx.x];
    const int64_t n = a.nsteps[blockIdx.x];
    const int d = (int)a.d;
    float *out = a.W + (int64_t)chain * a.d;
    if (n == 0) {
        for (int c = (int)threadIdx.x; c < d; c += kBlockThreads) out[c] = start_value(a, c);
        return;
    }
    const int64_t nblk = (n + kBlock - 1) / kBlock, beats = nblk + kScouts;
    const double rho64 = a.pow_tab[kWave - 1] * a.rho, inv_rho64 = a.pow_tab[2 * kWave - 1];

    if (wave == 0) {
        // ------------------------------------------------------------------------- the chain
        __builtin_amdgcn_s_setprio(2);
        TV v[CE];
        start_values(a, v, [&](int e) { return lane * CE + e; });
#pragma unroll
        for (int e = 0; e < CE; ++e) model[lane * CE + e] = v[e];
        double s_w = 1.0;
#pragma unroll 1
        for (int q = 0; q < kScouts; ++q) section_barrier();
        int64_t b = 0;
        uint32_t odd = excess[0];
#pragma unroll 1
        for (int64_t end = odd ? 0 : nblk; b < end; ++b) {
            if ((b % kBlocksPerWindow) == 0 && b > 0) {
                s_w *= rho64;
                if (s_w < 0x1p-30) {          // fold the scale into v; the scouts do the same to theirs
#pragma unroll
                    for (int e = 0; e < CE; ++e) {
                        v[e] *= (TV)s_w;
                        model[lane * CE + e] = v[e];
                    }
                    s_w = 1.0;
                }
            }
            const Section &sec = section[b & 1];
            TV acc[4] = {(TV)0, (TV)0, (TV)0, (TV)0};
#pragma unroll
            for (int kk = 0; kk < K; ++kk) {
                const f32x4 x = *reinterpret_cast<const f32x4 *>(&sec.tile[j][16 * kk + 4 * g]);
#pragma unroll
                for (int e = 0; e < 4; ++e) acc[e] += model[16 * kk + 4 * g + e] * (TV)x[e];
            }
            TV gram[kBlock];
#pragma unroll
            for (int t = 0; t < kBlock; ++t) gram[t] = sec.gram[t][j];
            const TV zs = sec.zs[j], cs = sec.cs[j];
            odd = excess[(b + 1) & 3];        // (the next block's, there for a block time; read here, it has arrived when the loop asks)
            TV p = (acc[0] + acc[1]) + (acc[2] + acc[3]);
            p = merge_values<false>(p, p);    // the four quarters of the columns: every lane ends with the whole sum
            p = merge_values<true>(p, p);
            TV q = zs * p, c[kBlock];
            const TV mine = cs * take_block_steps<LOSS>(q, gram);
#pragma unroll
            for (int t = 0; t < kBlock; ++t) c[t] = lane_read(mine, t);
#pragma unroll
            for (int t = 0; t < kBlock; ++t)
#pragma unroll
                for (int e = 0; e < CE; ++e) v[e] += c[t] * (TV)sec.tile[t][lane * CE + e];
#pragma unroll
            for (int e = 0; e < CE; ++e) model[lane * CE + e] = v[e];
            if (__builtin_amdgcn_readfirstlane((int)odd) != 0) end = b + 1;
            section_barrier();
        }
        // The block has a row that is not finite (or too large for fp32 products).  Two terms of an infinite product may
        // have different signs, and a step that is not taken still adds 0 times its row, so products must not be split
        // into v.x and Gram terms: from here on, on data no model is learnt from, one step is taken after the other.
        // (The look-out for such rows, at eight chains: hinge d = 64 2 %, logistic d = 256 3 %, none elsewhere.)
        for (; b < nblk; ++b) {
            if ((b % kBlocksPerWindow) == 0 && b > 0) {
                s_w *= rho64;
                if (s_w < 0x1p-30) {
#pragma unroll
                    for (int e = 0; e < CE; ++e) v[e] *= (TV)s_w;
                    s_w = 1.0;
                }
            }
            const Section &sec = section[b & 1];
#pragma unroll 1
            for (int t = 0; t < kBlock; ++t) {
                TV x[CE], dot = (TV)0;
#pragma unroll
                for (int e = 0; e < CE; ++e) {
                    x[e] = (TV)sec.tile[t][lane * CE + e];
                    dot += v[e] * x[e];
                }
                const TV q = sec.zs[t] * wave_sum(dot), cs = sec.cs[t];
                TV ct;
                if constexpr (LOSS == kLossHinge) ct = q < 1.0 ? cs : 0.0;
                else ct = cs * __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(q));
#pragma unroll
                for (int e = 0; e < CE; ++e) v[e] += ct * x[e];
            }
            section_barrier();
        }
        const int rem = (int)(n - (n - 1) / kWave * kWave);                  // 1..64 steps in the last window
        const double s_end = s_w * a.pow_tab[rem - 1] * a.rho;
#pragma unroll
        for (int e = 0; e < CE; ++e) {
            const int col = lane * CE + e;
            if (col < d) out[col] = (float)(s_end * (double)v[e]);
        }
        return;
    }

    // ----------------------------------------------------------------------------- scouts
    const int h = wave - 1;
    const TX *X = static_cast<const TX *>(a.dense);
    const int64_t step0 = first_step(a, (int)blockIdx.x);
    const uint32_t m32 = (uint32_t)a.m;
    uint32_t shard_lo = 0, shard_len = 1, shard_inc = 0, shard_pos = 0;
    if (a.perm) {
        shard_lo = a.shard[blockIdx.x];
        shard_len = a.shard[a.k + blockIdx.x];
        shard_inc = (uint32_t)(kScouts * kBlock) % shard_len;
        shard_pos = (uint32_t)(((uint64_t)step0 + (uint32_t)(kBlock * h + j)) % shard_len);
    }
    // row of step 16*b + j, past the chain's end that of its last step once more (such a step adds 0 times its
    // row, which must be a row the chain has visited: 0 times a NaN is one); asked for b = h, h+3, h+6, .. in turn
    auto sample = [&](int64_t b) {
        uint32_t r;
        if (a.perm) {
            r = a.perm[(uint64_t)shard_lo + shard_pos];
            const uint32_t t = shard_pos + shard_inc;                 // may wrap past 2^32: then it is past the share too
            shard_pos = (t < shard_pos || t >= shard_len) ? t - shard_len : t;
        } else {
            r = sample_row(a.seed_lo, a.seed_hi, (uint32_t)chain, (uint64_t)(step0 + b * kBlock + j), m32);
        }
        if (b == nblk - 1) {                  // (blocks behind the last are asked for, but not run)
            const int last = (int)((n - 1) % kBlock);
            const uint32_t row = (uint32_t)__builtin_amdgcn_readlane((int)r, last);
            r = j < last ? r : row;
        }
        return r;
    };
    // Lane (j, g) takes columns 16*kk + 4*g .. +3 of row j.  A piece that reaches past the row's end is read from
    // d-4 on instead and shifted; columns from d on are zero.
    FourElements<TX> raw[K];
    auto request = [&](uint32_t row) {
        const TX *x = X + (int64_t)row * a.ld;
#pragma unroll
        for (int kk = 0; kk < K; ++kk) {
            const int col = 16 * kk + 4 * g;
            raw[kk].load(x + (col < d - 4 ? col : d - 4));
        }
    };
    const int edge = d / 16, shift = 16 * edge + 4 * g - (d - 4);          // the piece the row ends in (edge = K: none)
    float x[K][4];
    auto take = [&]() {
#pragma unroll
        for (int kk = 0; kk < K; ++kk) {
#pragma unroll
            for (int e = 0; e < 4; ++e) x[kk][e] = kk <= edge ? raw[kk].at(e) : 0.0f;
            if (kk == edge) {                 // (uniform)
                const float q0 = x[kk][0], q1 = x[kk][1], q2 = x[kk][2], q3 = x[kk][3];
                x[kk][0] = shift <= 0 ? q0 : (shift == 1 ? q1 : (shift == 2 ? q2 : (shift == 3 ? q3 : 0.0f)));
                x[kk][1] = shift <= 0 ? q1 : (shift == 1 ? q2 : (shift == 2 ? q3 : 0.0f));
                x[kk][2] = shift <= 0 ? q2 : (shift == 1 ? q3 : 0.0f);
                x[kk][3] = shift <= 0 ? q3 : 0.0f;
            }
        }
    };
    double s_w = 1.0, eos_w = a.eta;          // scale and eta/scale at the start of window w
    int64_t w = 0;

    uint32_t row = sample(h);
    request(row);
    float y_next = a.y[row];
    uint32_t row_next = sample(h + kScouts);
    int64_t beat = 0;
#pragma unroll 1
    for (; beat < h; ++beat) section_barrier();
#pragma unroll 1
    for (int64_t b = h;; b += kScouts) {
        Gram<TV> gram;
        auto add = [&](auto from, auto to) {
#pragma unroll
            for (int kk = decltype(from)::value; kk < decltype(to)::value; ++kk)
#pragma unroll
                for (int e = 0; e < 4; ++e) gram.add(x[kk][e]);
        };
        take();
        const double y = (double)y_next;
        request(row_next);
        y_next = a.y[row_next];
        row_next = sample(b + 2 * kScouts);
        const int l = (int)(b % kBlocksPerWindow) * kBlock + j;
        const double up = a.pow_tab[l], down = a.pow_tab[kWave + l];
        add(std::integral_constant<int, 0>{}, std::integral_constant<int, K / kScouts>{});
        section_barrier();
        if (++beat == beats) break;

        add(std::integral_constant<int, K / kScouts>{}, std::integral_constant<int, 2 * K / kScouts>{});
        // (behind the matrix products: mixed in with them it cost the scouts of bf16 rows of 256 elements 18 % of a block)
        __builtin_amdgcn_sched_barrier(0);
        float probe[4] = {0.0f, 0.0f, 0.0f, 0.0f};       // infinite or NaN once an element is, or is too large for products
#pragma unroll
        for (int kk = 0; kk < K; ++kk)
#pragma unroll
            for (int e = 0; e < 4; ++e) probe[e] = fmaf(x[kk][e], kProbe, probe[e]);
        const float probed = (probe[0] + probe[1]) + (probe[2] + probe[3]);
        const uint64_t odd = __builtin_amdgcn_ballot_w64(!(probed - probed == 0.0f));
        if (lane == 0) excess[b & 3] = odd != 0 ? 1u : 0u;
        section_barrier();
        if (++beat == beats) break;

        add(std::integral_constant<int, (kScouts - 1) * K / kScouts>{}, std::integral_constant<int, K>{});
        for (; w < b / kBlocksPerWindow; ++w) {
            s_w *= rho64;
            eos_w *= inv_rho64;
            if (s_w < 0x1p-30) {
                s_w = 1.0;
                eos_w = a.eta;
            }
        }
        Section &sec = section[b & 1];
#pragma unroll
        for (int kk = 0; kk < K; ++kk) {
            f32x4 q;
#pragma unroll
            for (int e = 0; e < 4; ++e) q[e] = x[kk][e];
            *reinterpret_cast<f32x4 *>(&sec.tile[j][16 * kk + 4 * g]) = q;
        }
        const bool live = b * kBlock + j < n;
        const double sl = s_w * up * y, el = live ? eos_w * down * y : 0.0;
        TV zs, cs;
        if constexpr (LOSS == kLossHinge) {
            zs = sl;
            cs = el;
        } else {
            zs = (float)(sl * 1.4426950408889634);
            cs = (float)el;
        }
        if (g == 0) {
            sec.zs[j] = zs;
            sec.cs[j] = cs;
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int t = Gram<TV>::row(r, lane);
            // zs and cs first: for t < j they are eta log2 e s_j/s_{t+1} at most eta log2 e, whatever the scale has shrunk to; cs alone may be
            // eta 2^85 (a window may start at 2^-30 and end at 2^-85).  (In every lane: a lane that stands aside has nothing to give.)
            TV unit = (zs * __shfl(cs, t)) * gram.d[r];
            // A large eta may take a product of 2^124 past the largest number; a slope of 0 times an infinity would be a NaN where nothing is added.
            if constexpr (LOSS == kLossLogistic) unit = __builtin_amdgcn_fmed3f(unit, -0x1.fffffep127f, 0x1.fffffep127f);
            sec.gram[t][j] = t < j ? unit : (TV)0;
        }
        section_barrier();
        if (++beat == beats) break;
    }
}

template <typename TX, int LOSS>
hipError_t launch(const ChainArgs &a, hipStream_t s)
{
    if (a.d <= 64) hipLaunchKernelGGL((chain_dense_block_kernel<TX, LOSS, 64>), dim3(a.k), dim3(kBlockThreads), 0, s, a);
    else if (a.d <= 128) hipLaunchKernelGGL((chain_dense_block_kernel<TX, LOSS, 128>), dim3(a.k), dim3(kBlockThreads), 0, s, a);
    else hipLaunchKernelGGL((chain_dense_block_kernel<TX, LOSS, 256>), dim3(a.k), dim3(kBlockThreads), 0, s, a);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_dense_block(const Plan &p, const ChainArgs &a, hipStream_t s)
{
    if (a.d < kBlockMinColumns || a.d > kBlockMaxColumns) return hipErrorInvalidValue;
    if (p.dtype == WPSGD_BF16)
        return p.loss == WPSGD_HINGE ? launch<uint16_t, kLossHinge>(a, s) : launch<uint16_t, kLossLogistic>(a, s);
    return p.loss == WPSGD_HINGE ? launch<float, kLossHinge>(a, s) : launch<float, kLossLogistic>(a, s);
}

}  // namespace wpsgd
