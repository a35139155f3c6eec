// zipml_loss: F(x) = 1/(2n) sum_i (a_i^T x - b_i)^2  (Sec. 1 eq. (1) with the square loss; Sec. 2).
//
// Streaming, sync-free kernels: every workgroup reduces a range of samples to one fp64 partial in
// pinned host memory, and the call adds the partials in a fixed order.
#include "zipml_device.h"
#include "zipml_host.h"
#include "zipml_mfma_ops.h"

#include <mutex>

namespace zipml {

constexpr int kLossThreads = 256;
constexpr int kLossMaxBlocks = 2048;

// fp32 rows: `lpr` lanes (a power of two <= 64) share one sample and stride over its features.
__global__ __launch_bounds__(kLossThreads) void k_loss_fp32(
    const float *__restrict__ A, int64_t lda, const float *__restrict__ b,
    const float *__restrict__ x, int64_t n, int64_t d, int lpr, int vec_ok,
    double *__restrict__ partial)
{
    __shared__ double scratch[kLossThreads / kWave + 1];
    const int tid = threadIdx.x;
    const int sub = tid % lpr;
    const int64_t rows_per_block = kLossThreads / lpr;
    double acc = 0.0;
    for (int64_t i = (int64_t)blockIdx.x * rows_per_block + tid / lpr; i < n;
         i += (int64_t)gridDim.x * rows_per_block) {
        const float *row = A + i * lda;
        float z = 0.0f;
        if (vec_ok) {
            for (int64_t j = 4 * sub; j < d; j += 4 * lpr) {
                const float4 av = *reinterpret_cast<const float4 *>(row + j);
                const float4 xv = *reinterpret_cast<const float4 *>(x + j);
                z = fmaf(av.x, xv.x, z);
                z = fmaf(av.y, xv.y, z);
                z = fmaf(av.z, xv.z, z);
                z = fmaf(av.w, xv.w, z);
            }
        } else {
            for (int64_t j = sub; j < d; j += lpr) z = fmaf(row[j], x[j], z);
        }
        for (int off = lpr / 2; off > 0; off >>= 1) z += __shfl_xor(z, off, kWave);
        if (sub == 0) {
            const double r = (double)z - (double)b[i];
            acc += r * r;
        }
    }
    const double tot = block_sum<double>(acc, scratch);
    if (tid == 0) partial[blockIdx.x] = tot;
}

// Launch before the packed copy-2 kernel, kLossPrepBlocks blocks: are the level tables evenly spaced (fp64
// formula, rounded once; the same test as in the preparation of the SGD kernels) -- one flag per block --,
// y_j = delta_j x_j in fp64, and per block the largest and the smallest |y_j| that is not zero (rounded to fp32) and
// the sum of mid_j x_j.  (Every block of the main kernel needs all of y; taking it from the ends of the level rows
// there, a cache line per feature, was a quarter of its time at 4,096 features.)
constexpr int kLossPrepBlocks = 64;
struct LossPrep {
    int even[kLossPrepBlocks];
    float ymax[kLossPrepBlocks], ymin[kLossPrepBlocks];
    double midx[kLossPrepBlocks];
};
__global__ __launch_bounds__(256) void k_loss_prepare(const float *__restrict__ levels, const float *__restrict__ x,
                                                      int64_t d, int K, double off, LossPrep *__restrict__ prep,
                                                      double *__restrict__ y)
{
    __shared__ float fmax_s[4], fmin_s[4];
    __shared__ double fsum_s[4];
    int ok = 1;
    if (K >= 4) {                                          // (two levels are always evenly spaced)
        const int spf = K / 4;
        const int64_t total = d * spf;
        const int64_t per = (total + kLossPrepBlocks - 1) / kLossPrepBlocks;
        const int64_t s_end = (blockIdx.x + 1) * per < total ? (blockIdx.x + 1) * per : total;
        for (int64_t sg = blockIdx.x * per + threadIdx.x; sg < s_end; sg += 256) {
            const int64_t j = sg / spf;
            const int c0 = (int)(sg % spf) * 4;
            const float *row = levels + j * K;
            const double lo = (double)row[0], wdt = (double)row[K - 1] - lo;
            const float4 v = *reinterpret_cast<const float4 *>(row + c0);
            ok &= (v.x == (float)(lo + ((double)(c0 + 0) * wdt) / (double)(K - 1)));
            ok &= (v.y == (float)(lo + ((double)(c0 + 1) * wdt) / (double)(K - 1)));
            ok &= (v.z == (float)(lo + ((double)(c0 + 2) * wdt) / (double)(K - 1)));
            ok &= (v.w == (float)(lo + ((double)(c0 + 3) * wdt) / (double)(K - 1)));
        }
    }
    constexpr float kInf = __builtin_inff();
    float ymax = 0.0f, ymin = kInf;
    double cq = 0.0;
    for (int64_t j = (int64_t)blockIdx.x * 256 + threadIdx.x; j < d; j += (int64_t)kLossPrepBlocks * 256) {
        const double lo = (double)levels[j * K], dl = ((double)levels[j * K + K - 1] - lo) / (double)(K - 1);
        const double xj = (double)x[j], yj = dl * xj;
        const float m = fabsf((float)yj);
        cq += (lo + off * dl) * xj;
        ymax = fmaxf(ymax, m);
        if (yj != 0.0) ymin = fminf(ymin, m);
        ok &= m < kInf;                                    // (no digits for an infinity or a NaN: the tables take it)
        y[j] = yj;
    }
    ymax = wave_reduce_dpp(ymax, [](float u, float v) { return fmaxf(u, v); });
    ymin = wave_reduce_dpp(ymin, [](float u, float v) { return fminf(u, v); });
    cq = wave_sum_dpp(cq);
    const int wave = threadIdx.x >> 6;
    if ((threadIdx.x & (kWave - 1)) == 0) { fmax_s[wave] = ymax; fmin_s[wave] = ymin; fsum_s[wave] = cq; }
    ok = __syncthreads_and(ok);
    if (threadIdx.x == 0) {
        prep->even[blockIdx.x] = ok;
        prep->ymax[blockIdx.x] = fmaxf(fmaxf(fmax_s[0], fmax_s[1]), fmaxf(fmax_s[2], fmax_s[3]));
        prep->ymin[blockIdx.x] = fminf(fminf(fmin_s[0], fmin_s[1]), fminf(fmin_s[2], fmin_s[3]));
        prep->midx[blockIdx.x] = (fsum_s[0] + fsum_s[1]) + (fsum_s[2] + fsum_s[3]);
    }
}

// The level tables of a chunk of features, multiplied by x, in LDS.  One look-up serves kPer features:
// with at most 3 bits the sums T_j[c] + T_j'[c'] of two neighbouring features are tabled, so that a look-up
// in 16 or 64 words -- words apart, so the lanes' gathers meet no bank conflicts -- takes the place of two,
// one multiply-add each.
// 131,072 x 4,096 codes of 3 bits (201 MB): 632 us a call with a look-up per code in the table in memory, 109 us
// with chunks of 512 features, 85 with 480; bound by the LDS gathers and the field extraction (three vector operations
// and a gather per pair).  The 480: at 3 bits the tables of 512 features and what they are built from are 82 KiB, and a
// compute unit holds one block; of 480 it holds two, one looking up while the other builds.  Where no
// compute unit has a second block the larger chunks are the fewer (4,096 x 4,096: 46 and 47 us; 8,192 x 16,384: 118 and 122).
template <int BITS> struct LossTable {
    static constexpr int K = 1 << BITS;
    static constexpr int kPer = BITS <= 3 ? 2 : 1;         // features per look-up
    static constexpr int kRow = 1 << (BITS * kPer);        // entries of a look-up's table
    static constexpr int kFeatures = 16384 / kRow * kPer < 512 ? 16384 / kRow * kPer : 512;   // per chunk
    static constexpr int kFeaturesTwo = BITS == 3 ? 480 : kFeatures;   // where two blocks share a compute unit
    __host__ __device__ static constexpr size_t tab_bytes(int features) { return (size_t)features / kPer * kRow * 4; }
    __host__ __device__ static constexpr size_t bytes(int features)      // (levels and model, on the way, behind the tables)
    {
        return tab_bytes(features) + (kPer == 2 ? (size_t)features * (K + 1) * 4 : 0);
    }
};

// Packed copy 2 (sample-major units) through the tables.  A block takes `spb` samples (64 to 512, a power of
// two) and `chunk` features at a time, a thread one of the samples and every (512 / spb)-th feature group; the parts of a sample meet in LDS.
constexpr int kLossPackedThreads = 512;
template <int BITS>
__device__ __forceinline__ double loss_copy2_table(const uint32_t *__restrict__ p2, const float *__restrict__ levels,
                                                   const float *__restrict__ b, const float *__restrict__ x, int64_t n,
                                                   int64_t d, int64_t n_pad, int spb, int chunk, unsigned char *smem)
{
    using LT = LossTable<BITS>;
    constexpr int K = LT::K, kPer = LT::kPer, kRow = LT::kRow, kT = kLossPackedThreads;
    constexpr int kBatch = BITS <= 4 ? 4 : 2;              // units in use, and as many on the way
    float *const tab = (float *)smem, *const one = (float *)(smem + LT::tab_bytes(chunk));
    double *const zs = (double *)smem;                     // [512 / spb][spb], after the last chunk
    const int tid = threadIdx.x, splits = kT / spb;
    const int smp = tid & (spb - 1), fs = tid / spb;       // (whole waves share fs)
    double acc = 0.0;
    for (int64_t T = blockIdx.x; T * spb < n; T += gridDim.x) {
        const int64_t i = T * spb + smp, row = i < n_pad ? i : n_pad - 1;
        float z[4] = {0.0f, 0.0f, 0.0f, 0.0f};
        for (int64_t c0 = 0; c0 < d; c0 += chunk) {
            const int nf = d - c0 < chunk ? (int)(d - c0) : chunk, nfp = (nf + 31) & ~31;
            // the first units are requested before the tables are built, the next ones before a batch is used
            const uint32_t *src = p2 + ((c0 / 32) * n_pad + row) * BITS;
            const int ng = nfp / 32;
            uint32_t u[kBatch][BITS], un[kBatch][BITS];
            auto request = [&](int g0, uint32_t (&dst)[kBatch][BITS]) __attribute__((always_inline)) {
#pragma unroll
                for (int m = 0; m < kBatch; ++m) {
                    const int g = g0 + m * splits < ng ? g0 + m * splits : ng - 1;
#pragma unroll
                    for (int q = 0; q < BITS; ++q) dst[m][q] = __builtin_nontemporal_load(src + g * n_pad * BITS + q);
                }
            };
            request(fs, u);
            // tables (entries of padding features are zero)
            if constexpr (kPer == 1) {
                for (int e = tid; e < nfp * K; e += kT) {
                    const int j = e / K;
                    tab[e] = j < nf ? levels[(c0 + j) * K + e % K] * x[c0 + j] : 0.0f;
                }
                __syncthreads();
            } else {
                // the levels and the model first, then a pair's sums, with one rounding each
                if constexpr (K >= 4) {
                    const float4 *src = reinterpret_cast<const float4 *>(levels + c0 * K);
                    for (int e = tid; e < nfp * K / 4; e += kT)
                        reinterpret_cast<float4 *>(one)[e] = e < nf * K / 4 ? src[e] : make_float4(0.0f, 0.0f, 0.0f, 0.0f);
                } else {
                    for (int e = tid; e < nfp * K; e += kT) one[e] = e < nf * K ? levels[c0 * K + e] : 0.0f;
                }
                for (int j = tid; j < nfp; j += kT) one[nfp * K + j] = j < nf ? x[c0 + j] : 0.0f;
                __syncthreads();
                for (int r = tid; r < nfp / 2 * K; r += kT) {
                    const int p = r / K, hi = r % K;
                    const float x0 = one[nfp * K + 2 * p], v = one[(2 * p + 1) * K + hi] * one[nfp * K + 2 * p + 1];
                    float *row = tab + p * kRow + hi * K;
                    if constexpr (K >= 4) {
#pragma unroll
                        for (int q = 0; q < K; q += 4) {
                            float4 t = *reinterpret_cast<const float4 *>(one + 2 * p * K + q);
                            t.x = fmaf(t.x, x0, v); t.y = fmaf(t.y, x0, v); t.z = fmaf(t.z, x0, v); t.w = fmaf(t.w, x0, v);
                            *reinterpret_cast<float4 *>(row + q) = t;
                        }
                    } else {
                        row[0] = fmaf(one[2 * p * K], x0, v);
                        row[1] = fmaf(one[2 * p * K + 1], x0, v);
                    }
                }
                __syncthreads();
            }
            for (int g0 = fs; g0 < ng; g0 += kBatch * splits) {
                request(g0 + kBatch * splits, un);
#pragma unroll
                for (int m = 0; m < kBatch; ++m) {
                    const int g = g0 + m * splits;
                    if (g < ng) {
                        const unsigned char *t = (const unsigned char *)(tab + g * (32 / kPer) * kRow);
#pragma unroll
                        for (int k = 0; k < 32 / kPer; ++k) {
                            constexpr int kField = BITS * kPer;
                            const int bit = k * kField, wi = bit >> 5, sh = bit & 31;
                            uint32_t at;                    // byte offset in the look-up's table
                            if (sh + kField > 32) at = (__builtin_amdgcn_alignbit(u[m][wi + 1 < BITS ? wi + 1 : wi], u[m][wi], sh) << 2) & (4u * kRow - 4u);
                            else at = (sh >= 2 ? u[m][wi] >> (sh - 2) : u[m][wi] << (2 - sh)) & (4u * kRow - 4u);
                            z[k & 3] += *reinterpret_cast<const float *>(t + k * kRow * 4 + at);
                        }
                    }
                }
#pragma unroll
                for (int m = 0; m < kBatch; ++m)
#pragma unroll
                    for (int q = 0; q < BITS; ++q) u[m][q] = un[m][q];
            }
            __syncthreads();
        }
        zs[fs * spb + smp] = ((double)z[0] + (double)z[1]) + ((double)z[2] + (double)z[3]);
        __syncthreads();
        if (tid < spb && i < n) {
            double zt = 0.0;
            for (int v = 0; v < splits; ++v) zt += zs[v * spb + tid];
            const double r = zt - (double)b[i];
            acc += r * r;
        }
        __syncthreads();
    }
    return acc;
}

// Packed copy 2.  Evenly spaced levels go to the matrix cores: a value is mid_j + (code - off) delta_j, so
// a_i^T x = sum_j mid_j x_j + sum_j (code_ij - off) y_j  with y_j = delta_j x_j.  y goes to fixed point in eight
// signed base-256 digits kept in LDS (as many as the sixteen rows of v_mfma_i32_16x16x64_i8 hold twice over: they
// cost no instruction more than four, 65,536 x 2,048 codes of 6 bits 44 us a call with either); a workgroup takes
// tiles of 64 samples, its eight waves split the 64-feature blocks (one instruction per 16 samples x 64 features,
// two sample tiles sharing an accumulator), the partial sums meet in LDS and wave 0 squares the residuals.  Exact
// integer sums; the unit of y is 2^-61 of the largest, and a model with an element below 2^-37 of that, which would
// keep fewer bits than fp32 has, goes through loss_copy2_table.  So do other level tables (the flags of
// k_loss_prepare say so; all blocks alike), a model with no digits, and problems whose digits do not fit in LDS
// (NKB == 0: more than 19,904 features).
template <int BITS>
__global__ __launch_bounds__(kLossPackedThreads) void k_loss_copy2(
    const uint32_t *__restrict__ p2, const float *__restrict__ levels, const float *__restrict__ b,
    const float *__restrict__ x, int64_t n, int64_t d, int64_t n_pad, int64_t d32, int NKB, int spb, int chunk,
    const LossPrep *__restrict__ prep, const double *__restrict__ y, double *__restrict__ partial)
{
    constexpr int HW = kOpDwords<BITS>, kW = kLossPackedThreads / kWave;
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ double scratch[kW + 1];
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid >> 6;
    const int n16 = lane & 15, q4 = lane >> 4;
    int ok_all = 0;
    float ymax = 0.0f;
    double cq = 0.0;
    if (NKB > 0) {
        ok_all = prep->even[lane];                         // (kLossPrepBlocks == kWave)
        ymax = wave_reduce_dpp(prep->ymax[lane], [](float u, float v) { return fmaxf(u, v); });
        cq = wave_sum_dpp(prep->midx[lane]);
        ok_all &= prep->ymin[lane] >= ldexpf(ymax, -37);
    }
    if (!__syncthreads_and(ok_all)) {
        const double acc = loss_copy2_table<BITS>(p2, levels, b, x, n, d, n_pad, spb, chunk, smem);
        const double tot = block_sum<double>(acc, scratch);
        if (tid == 0) partial[blockIdx.x] = tot;
        return;
    }
    int8_t *const ydig = (int8_t *)smem;                                  // [NKB][8 digits][4 q][16]
    longlong2 *const zpart = (longlong2 *)(smem + (size_t)NKB * 512);     // [kW][64]
    int8_t *const zeros = (int8_t *)(smem + (size_t)NKB * 512 + kW * 64 * 16);   // [16]
    if (tid < 4) reinterpret_cast<int *>(zeros)[tid] = 0;
    // 2^ky |y| < 2^61, however small the model (the sums are scaled back in fp64)
    int ey = 0;
    (void)frexpf(ymax, &ey);
    const int ky = ymax > 0.0f ? 60 - ey : 0;              // (ymax is rounded: one bit to spare)
    // four features whose codes are the bytes of one dword at a time: their digits are stored as dwords, too
    for (int e = tid; e < NKB * 16; e += kLossPackedThreads) {
        const int unit = e >> 3, half = (e >> 2) & 1, dword = e & 3;      // (unit: a group of 32 features)
        uint32_t lo[4], hi[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int j = 32 * unit + slot_code<BITS>(half, dword, i);
            const uint64_t dg = signed_digits_64<8>(__double2ll_rn(ldexp(j < d ? y[j] : 0.0, ky)));
            lo[i] = (uint32_t)dg;
            hi[i] = (uint32_t)(dg >> 32);
        }
        bytes_transpose(lo);
        bytes_transpose(hi);
        uint32_t *const at = reinterpret_cast<uint32_t *>(ydig + (unit >> 1) * 512 + (2 * (unit & 1) + half) * 16) + dword;
#pragma unroll
        for (int k = 0; k < 4; ++k) { at[16 * k] = lo[k]; at[16 * (k + 4)] = hi[k]; }
    }
    __syncthreads();

    // ---- tiles of 64 samples
    const int dig_off = (n16 & 7) * 64 + q4 * 16, slot_of = n16 >> 3;
    const int zero_off = (int)(zeros - ydig);
    const uint32_t shift = op_shift<BITS>(q4 & 1);
    const int64_t NT = n_pad / 64;
    double acc = 0.0;
    for (int64_t T = blockIdx.x; T < NT; T += gridDim.x) {
        const int64_t row0 = 64 * T;
        v4i c[2] = {{0, 0, 0, 0}, {0, 0, 0, 0}};
        for (int kb = wave; kb < NKB; kb += kW) {
            // lane = sample 16 sl + n16 of the tile, 16 codes (half q4 & 1) of feature group 2 kb + q4 / 2;
            // a padding group (odd number of groups) reads the block's first group: its digits are zero
            int64_t g = 2 * kb + (q4 >> 1);
            g = g < d32 ? g : 2 * kb;
            uint32_t w[4][HW];
#pragma unroll
            for (int sl = 0; sl < 4; ++sl) {
                const uint32_t *q = static_cast<const uint32_t *>(__builtin_assume_aligned(
                    p2 + (g * n_pad + row0 + 16 * sl + n16) * BITS + (q4 & 1) * kOpStride<BITS>, kOpAlign<BITS>));
#pragma unroll
                for (int h = 0; h < HW; ++h) w[sl][h] = __builtin_nontemporal_load(q + h);
            }
#pragma unroll
            for (int sl = 0; sl < 4; ++sl) {
                const v4i ad = *reinterpret_cast<const v4i *>(ydig + (slot_of == (sl & 1) ? kb * 512 + dig_off : zero_off));
                c[sl >> 1] = __builtin_amdgcn_mfma_i32_16x16x64_i8(ad, expand_codes<BITS>(w[sl], shift), c[sl >> 1], 0, 0, 0);
            }
        }
        // this lane: sample tiles q4 / 2 (.x) and 2 + q4 / 2 (.y), the lower (q4 even) or the upper four digits
        zpart[wave * 64 + lane] = make_longlong2(combine_digits(c[0]), combine_digits(c[1]));
        __syncthreads();
        if (wave == 0) {
            // lane = sample 16 q4 + n16 of the tile
            long long lo = 0, hi = 0;
            const int from = 32 * (q4 & 1) + n16;
#pragma unroll
            for (int v = 0; v < kW; ++v) {
                const longlong2 p = zpart[v * 64 + from], q = zpart[v * 64 + from + 16];
                lo += q4 & 2 ? p.y : p.x;
                hi += q4 & 2 ? q.y : q.x;
            }
            if (row0 + lane < n) {
                const double r = ldexp(fma((double)hi, 4294967296.0, (double)lo), -ky) + cq - (double)b[row0 + lane];
                acc += r * r;
            }
        }
        __syncthreads();
    }
    const double tot = block_sum<double>(acc, scratch);
    if (tid == 0) partial[blockIdx.x] = tot;
}

// LDS of k_loss_copy2's matrix-core path; the kernel's static part (scratch of the block-wide sums and the vote) has
// to fit beside it.
constexpr size_t kLossStaticLds = 1024;
constexpr size_t kLossScratchLds = 384;      // (336 bytes are what it takes: where two blocks share the LDS of a compute unit)
inline size_t loss_mfma_lds_bytes(int NKB)
{
    return (size_t)NKB * 512 + (kLossPackedThreads / kWave) * 64 * 16 + 16;
}

// Packed copy 1 (feature-major units: one feature x 32 samples).  A lane takes one feature of a group of 64
// (or of 32, two sample groups to a wave, where the problem has no more) and keeps the 32 partial dot products
// of its sample group in registers through all its features; the level tables of a chunk of features,
// multiplied by x, are in LDS with their rows K + 1 words apart (the lanes look up different rows).  At
// the end the 32 sums of a lane are added over the lanes by halving, in fp64: a lane hands half of its sums to the
// lane it is paired with and takes the other half of that lane's, 31 exchanges instead of 32 for each of
// five or six steps.  Every eighth product the 32 sums go to second ones: one fp32 chain over every 64th
// feature had an error of 3.0e-7 of the dot product (8 bits, 16,384 features), this 1.2e-7 -- chains over every
// 256th would have 1.7e-7 --, and the compiler finds more to overlap (65,536 x 2,048, 3 bits 98 -> 75 us a call).  A block's eight waves take `sgb` (1 to 8) sample groups, and share the features of
// one where there are fewer groups than that.
constexpr int kLoss1Threads = 512;
template <int BITS> constexpr int kLoss1Features = 16384 / ((1 << BITS) + 1) / 64 * 64 < 512 ? 16384 / ((1 << BITS) + 1) / 64 * 64 : 512;
template <int BITS> constexpr int kLoss1Chunk = kLoss1Features<BITS> < 64 ? 64 : kLoss1Features<BITS>;
template <int BITS> constexpr size_t kLoss1Lds = (size_t)kLoss1Chunk<BITS> * ((1 << BITS) + 1) * 4;
template <int BITS>
__global__ __launch_bounds__(kLoss1Threads) void k_loss_copy1(
    const uint32_t *__restrict__ p1, const float *__restrict__ levels, const float *__restrict__ b,
    const float *__restrict__ x, int64_t n, int64_t d, int64_t n32, int d32, int sgb, double *__restrict__ partial)
{
    constexpr int K = 1 << BITS, kW = kLoss1Threads / kWave, FC = kLoss1Chunk<BITS>;
    extern __shared__ __align__(16) unsigned char smem[];
    float *const tab = (float *)smem;
    __shared__ double scratch[kW + 1];
    __shared__ double zs[kW][64];
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid >> 6;
    const int lpg = d32 == 1 ? 32 : 64;                    // lanes per sample group
    const int gpw = kWave / lpg;                           // sample groups per wave
    const int sub = lane / lpg, fl = lane & (lpg - 1);
    const int splits = kW / sgb, slot = wave % sgb, fs = wave / sgb;
    double acc = 0.0;
    for (int64_t T = blockIdx.x; T * sgb * gpw < n32; T += gridDim.x) {
        const int64_t rg = (T * sgb + slot) * gpw + sub, rgc = rg < n32 ? rg : n32 - 1;
        float z[32], zlong[32];
#pragma unroll
        for (int k = 0; k < 32; ++k) z[k] = zlong[k] = 0.0f;
        int terms = 0;
        for (int64_t c0 = 0; c0 < d; c0 += FC) {
            const int nf = d - c0 < FC ? (int)(d - c0) : FC, nfp = (nf + 63) & ~63;
            for (int e = tid; e < nfp * K; e += kLoss1Threads) {
                const int j = e / K;
                tab[e + j] = j < nf ? levels[(c0 + j) * K + e % K] * x[c0 + j] : 0.0f;
            }
            __syncthreads();
            for (int f0 = fs * lpg; f0 < nfp; f0 += splits * lpg) {
                const int f = f0 + fl;
                const int64_t j = c0 + f, g = j / 32 < d32 ? j / 32 : 0;   // (a padding group: its table is zero)
                const uint32_t *src = p1 + ((g * n32 + rgc) * 32 + (int)(j & 31)) * BITS;
                uint32_t u[BITS];
#pragma unroll
                for (int q = 0; q < BITS; ++q) u[q] = __builtin_nontemporal_load(src + q);
                const float *t = tab + f * (K + 1);
#pragma unroll
                for (int k = 0; k < 32; ++k) z[k] += t[unit_code<BITS>(u, k)];
                if ((++terms & 7) == 0) {
#pragma unroll
                    for (int k = 0; k < 32; ++k) { zlong[k] += z[k]; z[k] = 0.0f; }
                }
            }
            __syncthreads();
        }
        {
            double zd[32];
#pragma unroll
            for (int k = 0; k < 32; ++k) zd[k] = (double)zlong[k] + (double)z[k];
            if (lpg == 64) {
#pragma unroll
                for (int k = 0; k < 32; ++k) zd[k] += __shfl_xor(zd[k], 32, kWave);
            }
#pragma unroll
            for (int h = 16; h >= 1; h >>= 1) {
                const bool up = (lane & h) != 0;
#pragma unroll
                for (int k = 0; k < h; ++k) {
                    const double mine = up ? zd[k + h] : zd[k], give = up ? zd[k] : zd[k + h];
                    zd[k] = mine + __shfl_xor(give, h, kWave);
                }
            }
            zs[wave][lane] = zd[0];                        // of sample lane & 31 of the group
        }
        __syncthreads();
        // one thread per sample: slot tid / 64, in it sub group (tid / 32) % gpw
        if (tid < sgb * kWave) {
            const int sl = tid >> 6, ln = tid & (kWave - 1);
            const int64_t g = (T * sgb + sl) * gpw + ln / lpg, i = g * 32 + (ln & 31);
            if (ln % lpg < 32 && g < n32 && i < n) {
                double zt = 0.0;
                for (int v = 0; v < splits; ++v) zt += zs[v * sgb + sl][ln];
                const double r = zt - (double)b[i];
                acc += r * r;
            }
        }
        __syncthreads();
    }
    const double tot = block_sum<double>(acc, scratch);
    if (tid == 0) partial[blockIdx.x] = tot;
}

// Pinned host memory for the blocks' partial sums: the kernels store them there directly and the call adds
// them up after it has waited for the stream, in place of a second kernel and a copy back (a loss over
// 4,096 x 64 values: 31 -> 19 us).  A call takes a buffer for its duration; at most kMax of them (16 KiB
// each) are kept for later calls, of any thread and stream.  A buffer that a kernel may still write to is never
// given back: abandon().
class LossBuffer {
public:
    LossBuffer()
    {
        {
            std::lock_guard<std::mutex> lock(mutex());
            if (count() > 0) p = kept()[--count()];
        }
        if (p) return;
        // (an allocation is no part of a graph that another thread may be recording, and must not end its recording)
        hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
        const bool swapped = hipThreadExchangeStreamCaptureMode(&mode) == hipSuccess;
        if (HIP_FAILED(hipHostMalloc((void **)&p, kLossMaxBlocks * sizeof(double), hipHostMallocPortable | hipHostMallocMapped)))
            p = nullptr;
        if (swapped) (void)hipThreadExchangeStreamCaptureMode(&mode);
    }
    ~LossBuffer()
    {
        if (!p) return;
        {
            std::lock_guard<std::mutex> lock(mutex());
            if (count() < kMax) { kept()[count()++] = p; return; }
        }
        (void)hipHostFree(p);
    }
    void abandon() { p = nullptr; }
    LossBuffer(const LossBuffer &) = delete;
    LossBuffer &operator=(const LossBuffer &) = delete;
    double *p = nullptr;

private:
    static constexpr int kMax = 8;
    static std::mutex &mutex() { static std::mutex m; return m; }
    static double **kept() { static double *k[kMax]; return k; }
    static int &count() { static int c = 0; return c; }
};

template <int BITS>
static int launch_loss_packed(hipStream_t s, const uint32_t *p, int copy, const Layout &lay, const float *levels,
                              const float *b, const float *x, LossPrep *prep, int cus, int lds_limit, double *partial)
{
    if (copy == 1) {
        const int gpw = lay.d32 == 1 ? 2 : 1;
        // as many sample groups per block as leave two blocks per compute unit
        int sgb = 8;
        while (sgb > 1 && (lay.n32 + sgb * gpw - 1) / (sgb * gpw) < 2 * cus) sgb >>= 1;
        const int64_t tiles = (lay.n32 + sgb * gpw - 1) / (sgb * gpw);
        const int blocks = (int)(tiles < kLossMaxBlocks ? tiles : kLossMaxBlocks);
        if (HIP_FAILED(hipFuncSetAttribute((const void *)k_loss_copy1<BITS>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                           (int)kLoss1Lds<BITS>)))
            return ZIPML_ELAUNCH;
        hipLaunchKernelGGL(k_loss_copy1<BITS>, dim3(blocks), dim3(kLoss1Threads), kLoss1Lds<BITS>, s, p, levels, b, x,
                           lay.n, lay.d, lay.n32, (int)lay.d32, sgb, partial);
        return blocks;
    }
    int NKB = (int)((lay.d32 + 1) / 2);
    if (!prep || loss_mfma_lds_bytes(NKB) + kLossStaticLds > (size_t)lds_limit) NKB = 0;   // through the tables, whatever the levels
    // samples per block on the table path: as many as leave two blocks per compute unit
    int spb = kLossPackedThreads;
    while (spb > 64 && (lay.n + spb - 1) / spb < 2 * cus) spb >>= 1;
    // the smaller chunks only where two blocks do share a compute unit: enough of them, and room beside the even levels'
    // digits (at 3 bits none from 9,153 features on: 16,896 x 12,000 163 us with the larger ones, 168 with the smaller)
    const size_t least = std::max<size_t>(4096, NKB > 0 ? loss_mfma_lds_bytes(NKB) : 0);
    const bool two = (lay.n + spb - 1) / spb > cus &&
                     2 * (std::max(LossTable<BITS>::bytes(LossTable<BITS>::kFeaturesTwo), least) + kLossScratchLds) <= (size_t)lds_limit;
    const int chunk = two ? LossTable<BITS>::kFeaturesTwo : LossTable<BITS>::kFeatures;
    const size_t shmem = std::max(LossTable<BITS>::bytes(chunk), least);
    if (HIP_FAILED(hipFuncSetAttribute((const void *)k_loss_copy2<BITS>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)shmem)))
        return ZIPML_ELAUNCH;
    const int64_t NT = lay.n_pad / 64;
    const int blocks = (int)(NT < 1024 ? NT : 1024);
    double *y = (double *)(prep + 1);
    if (NKB > 0)
        hipLaunchKernelGGL(k_loss_prepare, dim3(kLossPrepBlocks), dim3(256), 0, s, levels, x, lay.d, 1 << BITS,
                           BITS == 8 ? 128.0 : 0.0, prep, y);
    hipLaunchKernelGGL(k_loss_copy2<BITS>, dim3(blocks), dim3(kLossPackedThreads), shmem, s, p, levels, b, x, lay.n,
                       lay.d, lay.n_pad, lay.d32, NKB, spb, chunk, prep, y, partial);
    return blocks;
}

// A plain streaming kernel of known size: reads `n16` 16-byte words once (non-temporal loads, four
// in flight per thread), XORs their dwords into *sink, and, with dst, stores them as well.
__global__ __launch_bounds__(256) void k_stream_probe(const uint4 *__restrict__ src, uint4 *__restrict__ dst,
                                                      size_t n16, uint32_t *sink)
{
    typedef unsigned int u4 __attribute__((ext_vector_type(4)));
    const u4 *in = reinterpret_cast<const u4 *>(src);
    u4 *out = reinterpret_cast<u4 *>(dst);
    const size_t stride = (size_t)gridDim.x * 256;
    size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
    uint32_t x = 0;
    for (; i + 3 * stride < n16; i += 4 * stride) {
        u4 v[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) v[k] = __builtin_nontemporal_load(in + i + k * stride);
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            if (out) __builtin_nontemporal_store(v[k], out + i + k * stride);
            x ^= v[k][0] ^ v[k][1] ^ v[k][2] ^ v[k][3];
        }
    }
    for (; i < n16; i += stride) {
        const u4 v = __builtin_nontemporal_load(in + i);
        if (out) __builtin_nontemporal_store(v, out + i);
        x ^= v[0] ^ v[1] ^ v[2] ^ v[3];
    }
    x = wave_reduce_dpp(x, [](uint32_t p, uint32_t q) { return p ^ q; });
    if ((threadIdx.x & (kWave - 1)) == 0) atomicXor(sink, x);
}

}  // namespace zipml

using namespace zipml;

extern "C" int zipml_debug_stream(void *stream, const void *src_dev, void *dst_dev, size_t bytes,
                                  uint32_t *sink_dev)
{
    if (!src_dev || !sink_dev || bytes == 0 || bytes % 16 != 0) return ZIPML_EINVAL;
    if (!aligned16(src_dev) || (dst_dev && !aligned16(dst_dev)) || (reinterpret_cast<uintptr_t>(sink_dev) & 3u))
        return ZIPML_EALIGN;
    hipStream_t s = entry_stream(stream);
    const size_t n16 = bytes / 16;
    const size_t want = (n16 + 256 * 4 - 1) / (256 * 4);
    const unsigned blocks = (unsigned)(want < 1 ? 1 : want > 4096 ? 4096 : want);
    hipLaunchKernelGGL(k_stream_probe, dim3(blocks), dim3(256), 0, s, (const uint4 *)src_dev, (uint4 *)dst_dev,
                       n16, sink_dev);
    if (HIP_FAILED(hipGetLastError())) return ZIPML_ELAUNCH;
    return ZIPML_OK;
}

extern "C" int zipml_loss(void *stream, const float *A_dev, int64_t lda, const void *packed_dev,
                          int copy, const float *levels_dev, int bits, const float *b_dev,
                          const float *x_dev, int64_t n, int64_t d, double *loss_host,
                          void *workspace_dev, size_t workspace_bytes)
{
    if (!b_dev || !x_dev || !loss_host || n <= 0 || d <= 0) return ZIPML_EINVAL;
    if (!workspace_dev || workspace_bytes < (size_t)(kLossMaxBlocks + 1) * sizeof(double))
        return ZIPML_EWORKSPACE;
    if (!aligned16(workspace_dev) || !aligned16(x_dev)) return ZIPML_EALIGN;
    if (A_dev) {
        if (lda < d) return ZIPML_EINVAL;
        if (reinterpret_cast<uintptr_t>(A_dev) & 3u) return ZIPML_EALIGN;
    } else {
        if (!packed_dev || !levels_dev || !valid_bits(bits) || (copy != 1 && copy != 2)) return ZIPML_EINVAL;
        if (!aligned16(packed_dev) || !aligned16(levels_dev)) return ZIPML_EALIGN;
    }
    hipStream_t s = entry_stream(stream);
    // a stream that is being recorded cannot be waited for: refused before anything becomes part of the graph
    hipStreamCaptureStatus capture = hipStreamCaptureStatusNone;
    if (HIP_FAILED(hipStreamIsCapturing(s, &capture)) || capture != hipStreamCaptureStatusNone) return ZIPML_ELAUNCH;
    LossBuffer sums;
    if (!sums.p) return ZIPML_ELAUNCH;
    int blocks = 0;
    if (A_dev) {
        int lpr = 1;
        while (lpr < 64 && lpr * 4 < d) lpr <<= 1;
        const int vec_ok = (lda % 4 == 0) && (d % 4 == 0) && aligned16(A_dev);
        const int64_t rows_per_block = kLossThreads / lpr;
        blocks = (int)((n + rows_per_block - 1) / rows_per_block);
        if (blocks > kLossMaxBlocks) blocks = kLossMaxBlocks;
        hipLaunchKernelGGL(k_loss_fp32, dim3(blocks), dim3(kLossThreads), 0, s, A_dev, lda, b_dev,
                           x_dev, n, d, lpr, vec_ok, sums.p);
    } else {
        const Layout lay = make_layout(n, d, bits);
        const uint32_t *p = (const uint32_t *)packed_dev;
        int dev = 0, cus = 0, lds = 0;
        if (HIP_FAILED(hipGetDevice(&dev)) ||
            HIP_FAILED(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev)) ||
            HIP_FAILED(hipDeviceGetAttribute(&lds, hipDeviceAttributeMaxSharedMemoryPerBlock, dev)))
            return ZIPML_ELAUNCH;
        // (the matrix-core path needs room for the preparation's results)
        LossPrep *prep = workspace_bytes >= sizeof(LossPrep) + (size_t)d * 8 && knob(ZIPML_KNOB_NO_MATRIX_CORES) <= 0
                             ? (LossPrep *)workspace_dev : nullptr;
#define ZIPML_LOSS(B) case B: blocks = launch_loss_packed<B>(s, p, copy, lay, levels_dev, b_dev, x_dev, prep, cus, lds, sums.p); break
        switch (bits) {
            ZIPML_LOSS(1); ZIPML_LOSS(2); ZIPML_LOSS(3); ZIPML_LOSS(4);
            ZIPML_LOSS(5); ZIPML_LOSS(6); ZIPML_LOSS(7); ZIPML_LOSS(8);
        }
#undef ZIPML_LOSS
        if (blocks < 0) return blocks;
    }
    const bool launched = !HIP_FAILED(hipGetLastError());
    if (HIP_FAILED(hipStreamSynchronize(s))) {
        sums.abandon();
        return ZIPML_ELAUNCH;
    }
    if (!launched) return ZIPML_ELAUNCH;
    double tot = 0.0;
    for (int i = 0; i < blocks; ++i) tot += sums.p[i];
    *loss_host = tot / (2.0 * (double)n);
    return ZIPML_OK;
}
