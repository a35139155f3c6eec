// Step loop of the epoch kernel for evenly spaced levels and an fp32 model, every code width, minibatches of up to
// 1,024 samples (included by zipml_sgd.hip).
//
// The arithmetic is that of zipml_sgd_mfma.h: both passes of eq. (5), Sec. 2.2, are integer sums of codes times the
// signed base-256 digits of y = delta x and of the residuals, on v_mfma_i32_16x16x64_i8.  What a step of this size
// costs is no arithmetic but a chain of latencies -- one device-wide exchange and what stands between two of them --, so
// here a WAVE is the unit of work:
//   - a wave owns 64 SB samples of the minibatch and takes both passes over them for all features of the workgroup
//     (64).  A lane looks after one sample of a block of 64 from the dot product to the digits of the residual: it
//     publishes the sum, polls the same word, and its digits go to the matrix cores through LDS that only this wave
//     reads, with a scale of the wave's own;
//   - the waves meet ONCE a step: each has a part of the gradient of all features, in fp64, and after the barrier
//     every wave adds the parts in the same order and updates the same model in its registers (a lane, a feature),
//     so that the digits of y are a wave's own affair again;
//   - exchange words are never cleared.  They count up through the epoch, and who polls one knows what it read there the
//     last time: the difference, modulo 2^64, holds the arrivals above and the sum below.  Two buffers are enough: a
//     wave adds to step t + 2 only after its workgroup has met in step t + 1, so after every workgroup has added to step
//     t + 1, which each did after all its waves had read step t.  Lanes without a sample take part with whatever codes
//     they read, which spares the others the question;
//   - the packed codes are requested directly behind the atomics (before them they hold the sums back, behind the
//     first question for the sums they are in the way of the next one), or copy 1 as soon as the sums have arrived where
//     a step has more than the compute unit takes in while it waits; they are expanded to bytes while the sums of the
//     next step are under way.
#pragma once
#include "zipml_mfma_ops.h"

namespace zipml {

// Digits of r and y.
// FULL = false, for the plans of zipml_sgd_mfma.h (2, 4 and 8 bits, whole blocks of 64 samples): four, as there, 30 bits below
// the wave's largest r, and 30 below the bound of y, which behind a refresh is the sum of the workgroups' largest.  (There 29
// and 29.  The bit more of y is the one that the sum over twice the workgroups takes from 4,097 features on: 512 samples x
// 16,384 features, 4 bits, equal elements: a step's model off by 3.8e-7 with 29, 4e-8 with 30.)
// FULL = true, for the plans of the vector loop, which computes in fp32: eight of r, which hold all bits of a number down
// to 2^-35 of the wave's largest, and six of y, 46 bits below its bound; what is published of their sums ends 42 bits below a
// larger number.  With four, numbers beside a much larger one lose bits (see zipml_sgd_solo.hip): 96 samples x 520 features,
// 8 bits, one residual in 16 larger by 10^6, worst coordinate of the gradient relative to the magnitudes that reach it 1.7e-4
// (four digits), 1.5e-7 (the vector loop), 9.3e-8 (eight).  What the eight cost, us per step with four | eight | in the vector
// loop: 96 samples x 300 features, 4 bits 1.34 | 1.38 | 2.28; 160 x 3,000, 8 bits 1.82 | 1.91 | 3.22; 736 x 1,500, 2 bits 2.09 |
// 2.20 | 3.78, 8 bits (no more registers) 2.95 | 3.41 | 4.40.
template <bool FULL> constexpr int kWaveDigits = FULL ? 8 : 4;
constexpr int kWaveBounds = 16;        // steps between exact refreshes of the magnitude bounds

// LDS bytes: digits of r and y per wave, two sets of gradient parts and of the waves' figures
template <int SB, bool FULL>
constexpr int kWaveLds = kWaves * (1 + SB) * kWaveDigits<FULL> * 64 + 2 * kWaves * 64 * 8 + 2 * kWaves * 4;

// An operand's dwords from a buffer, as one load.
template <int N>
__device__ __forceinline__ void buffer_fetch(__amdgpu_buffer_rsrc_t rsrc, uint32_t off, uint32_t step, uint32_t (&w)[N])
{
    typedef uint32_t v2u __attribute__((ext_vector_type(2)));
    typedef uint32_t v3u __attribute__((ext_vector_type(3)));
    typedef uint32_t v4u __attribute__((ext_vector_type(4)));
    if constexpr (N == 4) {
        const v4u q = __builtin_bit_cast(v4u, __builtin_amdgcn_raw_buffer_load_b128(rsrc, off, step, 0));
#pragma unroll
        for (int k = 0; k < 4; ++k) w[k] = q[k];
    } else if constexpr (N == 3) {
        const v3u q = __builtin_bit_cast(v3u, __builtin_amdgcn_raw_buffer_load_b96(rsrc, off, step, 0));
#pragma unroll
        for (int k = 0; k < 3; ++k) w[k] = q[k];
    } else if constexpr (N == 2) {
        const v2u q = __builtin_bit_cast(v2u, __builtin_amdgcn_raw_buffer_load_b64(rsrc, off, step, 0));
        w[0] = q[0];
        w[1] = q[1];
    } else {
        w[0] = __builtin_amdgcn_raw_buffer_load_b32(rsrc, off, step, 0);
    }
}

// How a wave's load brings the operands of several tiles.  A load instruction costs the compute unit's memory pipeline
// some 16 clocks, however little a lane asks for, so a lane loads whole units where its operand is half a small one:
// 1 and 2 bits: four or two units side by side, which are the rows of four tiles (two of them for each lane of a pair 16
// lanes apart); 3 and 4 bits: one unit, lanes 16 apart those of two tiles; and what a lane holds of the other's operands
// changes hands 16 lanes on (v_permlane16_swap).  Wider codes: an operand is a load.
template <int BITS> constexpr int kWaveLoads = BITS <= 2 ? 1 : BITS <= 4 ? 2 : 4;       // of a block of 64 x 64 codes
template <int BITS> constexpr int kWaveDwords = BITS <= 2 ? 4 : BITS <= 4 ? BITS : kOpDwords<BITS>;
// The row of 16 lanes q4 looks after tile q4; lane n16 of it after this element of the block (so that four neighbouring
// lanes hold the digits of a dword of an operand, at wave_digits_at)
template <int BITS>
__device__ __forceinline__ int wave_element(int q4, int n16)
{
    if (BITS == 1) return 4 * (8 * (n16 >> 3) + 2 * (n16 & 3) + ((n16 >> 2) & 1)) + q4;
    if (BITS == 2) return 4 * n16 + q4;
    return lane_slot<BITS>(16 * q4 + n16);
}
template <int BITS>
__device__ __forceinline__ int wave_digits_at(int q4, int n16)
{
    const int dword = BITS == 1 ? 8 * (n16 >> 3) + 4 * ((n16 >> 2) & 1) + q4 : BITS == 2 ? 4 * (n16 >> 2) + q4 : 4 * q4 + (n16 >> 2);
    return 64 * (n16 & 3) + 4 * dword;
}
// The row (of 64) that a lane's load l begins at.
template <int BITS>
__device__ __forceinline__ int wave_load_row(int q4, int n16, int l)
{
    if (BITS <= 2) return wave_element<BITS>(0, n16) + (BITS == 2 ? 2 * (q4 & 1) : 0);
    return BITS <= 4 ? wave_element<BITS>(2 * l + (q4 & 1), n16) : wave_element<BITS>(l, n16);
}
// Sums of four digits, two to an integer, of the tile that a row of lanes looks after.
__device__ __forceinline__ void pick_tile(const v4i (&c)[4], int q4, int (&sum)[2])
{
    const bool sel1 = q4 & 1, sel2 = q4 & 2;
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        int p[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) p[q] = c[q][2 * k] + (c[q][2 * k + 1] << 8);
        sum[k] = sel2 ? (sel1 ? p[3] : p[2]) : (sel1 ? p[1] : p[0]);
    }
}
// Loads -> the operands of the four tiles (code bytes).
template <int BITS>
__device__ __forceinline__ void wave_operands(const uint32_t (&c)[kWaveLoads<BITS>][kWaveDwords<BITS>], uint32_t shift, v4i (&e)[4])
{
    typedef unsigned int v2u __attribute__((ext_vector_type(2)));
    constexpr int HW = kOpDwords<BITS>;
    uint32_t w[4][HW];
    if constexpr (BITS == 1) {
#pragma unroll
        for (int s = 0; s < 4; ++s) w[s][0] = c[0][s];
    } else if constexpr (BITS == 2) {
        // even rows of lanes: both halves of units 0, 1; odd rows: of 2, 3
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            const v2u v = __builtin_amdgcn_permlane16_swap(c[0][2 * k], c[0][2 * k + 1], false, false);
            w[k][0] = v[0];
            w[2 + k][0] = v[1];
        }
    } else if constexpr (BITS <= 4) {
        // dwords k of half 0 and kOpStride + k of half 1: even rows hold the unit of tile 2 l, odd rows that of 2 l + 1
#pragma unroll
        for (int l = 0; l < 2; ++l)
#pragma unroll
            for (int k = 0; k < HW; ++k) {
                const v2u v = __builtin_amdgcn_permlane16_swap(c[l][k], c[l][kOpStride<BITS> + k], false, false);
                w[2 * l][k] = v[0];
                w[2 * l + 1][k] = v[1];
            }
    } else {
#pragma unroll
        for (int s = 0; s < 4; ++s)
#pragma unroll
            for (int k = 0; k < HW; ++k) w[s][k] = c[s][k];
    }
#pragma unroll
    for (int s = 0; s < 4; ++s) {
        e[s] = expand_codes<BITS>(w[s], shift);
        asm volatile("" : "+v"(e[s]));                  // (here, and not where it is used)
    }
}

template <int BITS, int SB, bool FULL, bool DBG>
__device__ __forceinline__ void sgd_steps_wave(const SgdArgs &a, unsigned char *smem)
{
    constexpr int NL = kWaveLoads<BITS>, LW = kWaveDwords<BITS>, ND = kWaveDigits<FULL>, K = 1 << BITS;
    // Codes of 8 bits are operands 128 below.  FULL: 128 times the sum of the other operand is added to the integers (in the
    // factor of a sum of fp32 numbers a large element that meets the code zero everywhere would leave its rounding errors).
    constexpr int kOff = BITS == 8 && !FULL ? 128 : 0;
    constexpr bool kOffset = BITS == 8 && FULL;
    constexpr double kMagic = 6755399441055744.0;       // 3 2^51: an integer below 2^51 in magnitude added to it is its foot
    const int tid = threadIdx.x, lane = tid & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n16 = lane & 15, q4 = lane >> 4;
    const int B = a.B, W = a.wave_w;
    const int nwv = (B + 64 * SB - 1) / (64 * SB);      // waves that have samples
    if (wave >= nwv) return;                            // (a barrier waits for the waves that are left)
    const int w = blockIdx.x, g0 = 2 * w;               // first feature group of this workgroup
    const int ngroups = a.d32 - g0 < 2 ? a.d32 - g0 : 2;
    const int nrg = B >= 32 ? B / 32 : 1;               // groups of 32 samples in a step
    const int own = wave_element<BITS>(q4, n16);
    const uint32_t shift = op_shift<BITS>(q4 & 1);
    const QuadStore quad(lane);

    // ---- LDS
    int8_t *const rdig = (int8_t *)smem + wave * ((1 + SB) * ND * 64);
    int8_t *const ydig = rdig + SB * ND * 64;
    double *const gpart = (double *)(smem + kWaves * (1 + SB) * ND * 64);           // [2][kWaves][64]
    uint32_t *const info = (uint32_t *)(gpart + 2 * kWaves * 64);                   // [2][kWaves] bits of the wave's max |r|
    const int dig_at = (n16 & (ND - 1)) * 64 + q4 * 16, put_at = wave_digits_at<BITS>(q4, n16);
    // (parts and figures of waves that are not there: read as zeros)
    if (wave == 0)
        for (int p = 0; p < 2; ++p)
            for (int q = nwv; q < kWaves; ++q) {
                if (lane == 0) info[p * kWaves + q] = 0u;
                gpart[(p * kWaves + q) * 64 + lane] = 0.0;
            }

    // A row of 16 lanes looks after one of four tiles.  Its two lower and two upper pairs of digit sums, two to an integer
    // (four digits: in lo only)
    struct Sums {
        int lo[2], hi[2];
    };
    auto pick = [&](const v4i (&c)[4], const v4i &half) __attribute__((always_inline)) {
        Sums s = {};
        if constexpr (ND == 8) {
            int x[2], y[2];
#pragma unroll
            for (int k = 0; k < 2; ++k) {
                int p[4];
#pragma unroll
                for (int q = 0; q < 4; ++q) p[q] = c[q][2 * k] + (c[q][2 * k + 1] << 8);
                x[k] = q4 & 2 ? p[2] : p[0];
                y[k] = q4 & 2 ? p[3] : p[1];
                if constexpr (kOffset) {                // (the same for all tiles)
                    const int on = 2 * (half[2 * k] + (half[2 * k + 1] << 8));
                    x[k] += on;
                    y[k] += on;
                }
            }
            const DigitSums j = join_rows(x, y);
#pragma unroll
            for (int k = 0; k < 2; ++k) { s.lo[k] = j.lo[k]; s.hi[k] = j.hi[k]; }
        } else {
            pick_tile(c, q4, s.lo);
        }
        return s;
    };

    // 64 times the sum of a digit operand
    auto offset = [&](const v4i &digits, v4i half) __attribute__((always_inline)) {
        if constexpr (kOffset) {
            const v4i h = {0x40404040, 0x40404040, 0x40404040, 0x40404040};
            half = __builtin_amdgcn_mfma_i32_16x16x64_i8(digits, h, half, 0, 0, 0);
        }
        return half;
    };

    // ---- bounds that fix the fixed-point scale of a step; every workgroup forms the same numbers (see zipml_sgd_mfma.h)
    float beta = (float)a.bound[0] * 1.00001f, ymax = (float)a.bound[2] * 1.00001f;
    const float lr_abs = fabsf(a.lr) * 1.00002f;
    const float grow = 1.0f + lr_abs * fabsf(a.l2) * 1.00001f;
    const float beta_r = lr_abs * ((float)a.bound[1] * 1.00001f), ymax_r = lr_abs * ((float)a.bound[3] * 1.00001f);
    int kp, kd, ks;                                     // scales of the published sums, of the digits of y, of a published max |y|
    auto set_scales = [&]() __attribute__((always_inline)) {
        const int eb = exponent_of(__float_as_uint(beta)), ey = exponent_of(__float_as_uint(ymax));
        ks = 30 - ey;
        if constexpr (ND == 4) { kp = 42 - eb < ks ? 42 - eb : ks; kd = kp; }
        else { kp = 42 - eb; kd = 46 - ey; }
    };

    // ---- this lane's feature
    const int j = 32 * g0 + own;
    const bool live = (own >> 5) < ngroups && j < a.d;
    const float lo = live ? a.levels[(size_t)j * K] : 0.0f, hi = live ? a.levels[(size_t)j * K + K - 1] : 0.0f;
    const double spacing = ((double)hi - (double)lo) / (double)(K - 1);
    const float dl = (float)spacing, mid = lo + (float)kOff * dl;
    const float maxl = fmaxf(fabsf(lo), fabsf(lo + dl * (float)(K - 1))) * 1.00001f;
    // (eight digits hold more of it than fp32 does; the higher of two levels is itself so, whatever their difference)
    const double dlw = FULL ? spacing : (double)dl;
    const double g_dl = dlw / (double)B, g_mid = (double)mid / (double)B;    // (the mean over the minibatch)
    float x = live ? a.x[j] : 0.0f;
    // What the next exchange takes from the model: digits of y (read back at once as the operand), sum of mid x
    v4i yd;
    float cq = 0.0f;
    auto publish_y = [&]() __attribute__((always_inline)) {
        uint32_t *const at = reinterpret_cast<uint32_t *>(ydig + put_at);
        if constexpr (ND == 4) {
            *at = quad.transpose(signed_digits(__float2int_rn(ldexpf(dl * x, kd))));
        } else {
            // six digits of an integer below 2^46 in magnitude; 128 in the five lower bytes on top (signed_digits)
            const double y = ldexp(dlw * (double)x, kd) + (kMagic + 551911719040.0);
            const uint64_t v = (uint64_t)__double_as_longlong(y);
            at[0] = quad.transpose((uint32_t)v ^ 0x80808080u);
            at[64] = quad.transpose((uint32_t)(v >> 32) ^ 0x80u);      // (two digits; what stands above them is not used)
        }
        asm volatile("" ::: "memory");
        yd = *reinterpret_cast<const v4i *>(ydig + dig_at);
        cq = wave_total(mid * x, AddF());
    };

    // ---- where the operands lie.  Groups of samples or features that are not there lie past the end of the buffer (0xF0000000
    // of 0xE0000000 bytes): zeros, and nothing is read, whether the range check counts a step's scalar offset to the lane's, takes
    // it off the size, or leaves it out; for what is there the two stay below 0xE0000000 together (run_sgd).
    uint32_t at2[SB][NL], at1[SB][NL];
    const uint32_t group_bytes = (uint32_t)(a.nb64 * 64 * 4 * BITS);                // of either copy
#pragma unroll
    for (int sb = 0; sb < SB; ++sb)
#pragma unroll
        for (int l = 0; l < NL; ++l) {
            // the row of this lane's load, and how far into its unit the load begins
            const int row = wave_load_row<BITS>(q4, n16, l);
            const int in_unit = BITS <= 4 ? 0 : (q4 & 1) * kOpStride<BITS> * 4, s0 = 2 * (wave * SB + sb);
            auto at = [&](int f, int s) {
                return f < ngroups && s < nrg ? (uint32_t)f * group_bytes + (uint32_t)((s * 32 + (row & 31)) * 4 * BITS + in_unit) : 0xF0000000u;
            };
            at2[sb][l] = at(q4 >> 1, s0 + (row >> 5));
            at1[sb][l] = at(row >> 5, s0 + (q4 >> 1));
        }
    // Where the groups of samples begin that a step's minibatch lies in (one of 4, 8 or 16 lies inside a group, `k` samples
    // on), in bytes of a group of features and of the labels: of the next step and of the one after, and past the last one that
    // of the last one again.
    struct Window {
        uint32_t codes, labels;
        int k;
    };
    auto next_of = [&](Window w, bool more) {
        const int on = more ? (w.k + B) & ~31 : 0;
        return Window{w.codes + (uint32_t)(on * (4 * BITS)), w.labels + 4u * (uint32_t)on, more ? (w.k + B) & 31 : w.k};
    };
    const uint32_t first = (uint32_t)(a.step0 * B) & ~31u;
    const Window win0 = {first * (4 * BITS), first * 4, (int)(a.step0 * B & 31)};
    Window win1 = next_of(win0, a.nsteps > 1);
    auto buffer = [](const void *p, int64_t at, uint32_t bytes) {
        return __builtin_amdgcn_make_buffer_rsrc((unsigned char *)p + at, 0, (int)bytes, 0x00020000);
    };
    const __amdgpu_buffer_rsrc_t src2 = buffer(a.p2, (int64_t)g0 * group_bytes, 0xE0000000u);
    const __amdgpu_buffer_rsrc_t src1 = buffer(a.p1, (int64_t)g0 * group_bytes, 0xE0000000u);
    const __amdgpu_buffer_rsrc_t srcb = buffer(a.b, 0, 0xE0000000u);
    uint32_t c2[SB][NL][LW], c1[SB][NL][LW];
    auto load2 = [&](const Window &w) __attribute__((always_inline)) {
#pragma unroll
        for (int sb = 0; sb < SB; ++sb)
#pragma unroll
            for (int l = 0; l < NL; ++l) buffer_fetch<LW>(src2, at2[sb][l], w.codes, c2[sb][l]);
    };
    auto load1 = [&](const Window &w) __attribute__((always_inline)) {
#pragma unroll
        for (int sb = 0; sb < SB; ++sb)
#pragma unroll
            for (int l = 0; l < NL; ++l) buffer_fetch<LW>(src1, at1[sb][l], w.codes, c1[sb][l]);
    };
    // this lane has a sample of the minibatch that begins k samples into its window; where its label is (else a neighbour's)
    auto has_sample = [&](int sb, int k) { return (uint32_t)(64 * (wave * SB + sb) + own - k) < (uint32_t)B; };
    uint32_t label_at[SB];
    float label[2][SB];
    auto set_label_at = [&](int k) __attribute__((always_inline)) {
#pragma unroll
        for (int sb = 0; sb < SB; ++sb) label_at[sb] = 4 * (has_sample(sb, k) ? 64 * (wave * SB + sb) + own : k);
    };
    auto load_labels = [&](const Window &w, float (&dst)[SB]) __attribute__((always_inline)) {
#pragma unroll
        for (int sb = 0; sb < SB; ++sb) {
            uint32_t v[1];
            buffer_fetch<1>(srcb, label_at[sb], w.labels, v);
            dst[sb] = __uint_as_float(v[0]);
        }
    };
    // exchange words of this lane's samples, in both buffers: the first of the S that it polls, and the one that it adds to
    const int S = a.wave_split, sub = a.wave_sub;
    const uint32_t mine = (uint32_t)(w % S) * (uint32_t)sub;
    uint64_t *word[2][SB];
#pragma unroll
    for (int sb = 0; sb < SB; ++sb)
#pragma unroll
        for (int p = 0; p < 2; ++p) word[p][sb] = a.acc + (size_t)p * S * sub + xword(64 * (wave * SB + sb) + own, a.wave_sh);
    uint64_t *const side = a.acc + xword(64 * SB * nwv, a.wave_sh) + (lane & 1);

    v4i e2[SB][4], e1[SB][4];
    uint64_t prev[2][SB] = {}, prev_side = 0;
    bool valid[SB];
    auto set_valid = [&](int k) __attribute__((always_inline)) {
#pragma unroll
        for (int sb = 0; sb < SB; ++sb) valid[sb] = has_sample(sb, k);
    };
    int k0 = win0.k;
    set_valid(k0);
    set_label_at(k0);
    load2(win0);
    load1(win0);
    load_labels(win0, label[0]);
    set_label_at(win1.k);
    set_scales();
    publish_y();
#pragma unroll
    for (int sb = 0; sb < SB; ++sb) wave_operands<BITS>(c2[sb], shift, e2[sb]);
    load2(win1);
    FirstPoll first_poll;
    int dead = a.spin_limit == 0;                       // (no polls at all: every wait gives up)
    if (dead != 0) store_dev(a.status, (int)ZIPML_ETIMEOUT);
    int since = 0;                                      // steps since the bounds were exact
    // (asked with a scalar comparison where it is needed, not kept as a mask)
    auto uniform = [](int v) __attribute__((always_inline)) { asm("" : "+s"(v)); return v; };

    auto step = [&](auto parity, int left) __attribute__((always_inline)) {
        constexpr int P = decltype(parity)::value;
        const int kp_pub = kp;
        // ============ dot pass, into the exchange
        {
            // what every sample gets on top, rounded to an integer
            const double base = ldexp((double)cq, kp) + kMagic;
            const v4i half = offset(yd, v4i{0, 0, 0, 0});
#pragma unroll
            for (int sb = 0; sb < SB; ++sb) {
                v4i c[4];
#pragma unroll
                for (int s = 0; s < 4; ++s) c[s] = __builtin_amdgcn_mfma_i32_16x16x64_i8(yd, e2[sb][s], v4i{0, 0, 0, 0}, 0, 0, 0);
                const Sums s = pick(c, half);
                uint64_t q;
                if constexpr (ND == 4) {
                    q = (uint64_t)__double_as_longlong(base) + (uint64_t)((long long)s.lo[0] + ((long long)s.lo[1] << 16));
                } else {
                    // (the six digits' weights: 1, 2^8, 2^16, 2^24 | 2^32, 2^40)
                    const double v = fma((double)s.hi[0], 4294967296.0, fma((double)s.lo[1], 65536.0, (double)s.lo[0]));
                    q = (uint64_t)__double_as_longlong(ldexp(v, kp - kd) + base);
                }
                // below 2^43 in magnitude, whatever the numbers (the count of the arrivals stays intact); bias and arrival
                int hi = (int)(q >> 32) - 0x43380000;
                hi = hi < -2048 ? -2048 : hi > 2047 ? 2047 : hi;
                add_dev(word[P][sb] + mine, (uint64_t)(uint32_t)(hi + (1 << (kCountShift - 32)) + 2048) << 32 | (uint32_t)q);
            }
        }
        __builtin_amdgcn_s_setprio(0);
        const bool side_step = since == kWaveBounds;
        if (side_step && wave == 0) {
            // the bounds travel with this exchange: this workgroup's shares, rounded up
            const float bw = wave_total(maxl * fabsf(x), AddF());
            const uint32_t ym = wave_total(magnitude(dl * x), MaxU());
            const double v = ceil(ldexp((double)(lane & 1 ? __uint_as_float(ym) : bw), lane & 1 ? ks : kp)) + 1.0;
            if (lane < 2) add_dev(side, ((uint64_t)1 << kCountShift) + (uint64_t)fmin(v, 8796093022207.0));
        }
        // ============ while the sums travel: operands of the gradient pass and of the next dot pass, and behind the atomics the
        // requests for later steps
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int sb = 0; sb < SB; ++sb) {
            wave_operands<BITS>(c1[sb], shift, e1[sb]);
            wave_operands<BITS>(c2[sb], shift, e2[sb]);
        }
        __builtin_amdgcn_sched_barrier(0);
        const Window win2 = next_of(win1, left > 2);
        load_labels(win1, label[P ^ 1]);
        load2(win2);
        if (uniform(a.wave_early) == 0) load1(win1);
        __builtin_amdgcn_sched_barrier(0);
        // ============ poll the sums of this lane's samples
        uint64_t diff[SB];
        first_poll.wait();
        // (asked again and again until `answer` has all; false: given up, now or before)
        auto poll = [&](auto answer) __attribute__((always_inline)) {
            uint32_t spins = 0;
#pragma unroll 1
            for (;;) {
                const int missing = __builtin_amdgcn_readfirstlane(__builtin_amdgcn_ballot_w64(!answer()) != 0 ? 1 : 0);
                if (missing == 0 || dead != 0 || ++spins > a.spin_limit) break;
            }
            spins = (uint32_t)__builtin_amdgcn_readfirstlane((int)spins);
            if (spins > a.spin_limit) {
                store_dev(a.status, (int)ZIPML_ETIMEOUT);
                dead = 1;
            }
            return spins;
        };
        const uint32_t again = poll([&]() __attribute__((always_inline)) {
            uint64_t raw[SB];
#pragma unroll
            for (int sb = 0; sb < SB; ++sb) raw[sb] = load_dev(word[P][sb]);
            if (uniform(S) > 1) {
                uint64_t second[SB], third[SB], fourth[SB];
                const bool four = uniform(S) > 2;
#pragma unroll
                for (int sb = 0; sb < SB; ++sb) second[sb] = load_dev(word[P][sb] + sub);
                if (four) {
#pragma unroll
                    for (int sb = 0; sb < SB; ++sb) {
                        third[sb] = load_dev(word[P][sb] + 2 * sub);
                        fourth[sb] = load_dev(word[P][sb] + 3 * sub);
                    }
#pragma unroll
                    for (int sb = 0; sb < SB; ++sb) raw[sb] += third[sb] + fourth[sb];
                }
#pragma unroll
                for (int sb = 0; sb < SB; ++sb) raw[sb] += second[sb];
            }
            bool all = true;
#pragma unroll
            for (int sb = 0; sb < SB; ++sb) {
                diff[sb] = raw[sb] - prev[P][sb];
                all = all && (int)(diff[sb] >> kCountShift) == W;
            }
            return all;
        });
        first_poll.learn(again != 0);
#pragma unroll
        for (int sb = 0; sb < SB; ++sb) prev[P][sb] += diff[sb];
        if (side_step) {
            uint64_t raw = 0;
            (void)poll([&]() __attribute__((always_inline)) {
                raw = load_dev(side) - prev_side;
                return (int)(raw >> kCountShift) == W;
            });
            prev_side += raw;
            const float f = (float)ldexp((double)(raw & kPayloadMask), lane & 1 ? -ks : -kp_pub) * 1.00001f;
            beta = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(f), 0));
            ymax = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(f), 1));
        }
        __builtin_amdgcn_s_setprio(3);
        asm volatile("" ::: "memory");
        // ============ residuals
        float r[SB], rsum = 0.0f;
        uint32_t rmax = 0u;
        // (2^52, whose foot holds the sums of up to 256 workgroups, and their biases)
        const double sum_bias = 4503599627370496.0 + (double)W * 8796093022208.0;
#pragma unroll
        for (int sb = 0; sb < SB; ++sb) {
            const uint64_t foot = (diff[sb] & 0x000FFFFFFFFFFFFFull) | 0x4330000000000000ull;
            const float z = (float)ldexp(__longlong_as_double((long long)foot) - sum_bias, -kp_pub);
            float d = z - label[P][sb];
            asm("" : "+v"(d));                           // (no branch)
            r[sb] = valid[sb] ? d : 0.0f;
            rmax = MaxU()(rmax, magnitude(r[sb]));
            rsum += r[sb];
        }
        if (uniform(a.wave_early) != 0) load1(win1);
        rmax = wave_total(rmax, MaxU());
        const int kr = (ND == 4 ? 30 : 59) - exponent_of(rmax);
#pragma unroll
        for (int sb = 0; sb < SB; ++sb) {
            uint32_t *const at = reinterpret_cast<uint32_t *>(rdig + sb * ND * 64 + put_at);
            if constexpr (ND == 8) {
                const Digits8 dg = digits_of(r[sb], kr);
                at[0] = quad.transpose(dg.lo);
                at[64] = quad.transpose(dg.hi);
            } else {
                at[0] = quad.transpose(signed_digits(__float2int_rn(ldexpf(r[sb], kr))));
            }
        }
        asm volatile("" ::: "memory");
        v4i rd[SB];
#pragma unroll
        for (int sb = 0; sb < SB; ++sb) rd[sb] = *reinterpret_cast<const v4i *>(rdig + sb * ND * 64 + dig_at);
        if (nwv > 1 && lane == 0) info[P * kWaves + wave] = rmax;
        rsum = wave_total(rsum, AddF());
        if constexpr (DBG) {
            if (w == 0 && a.dbg_r)
#pragma unroll
                for (int sb = 0; sb < SB; ++sb)
                    if (valid[sb]) a.dbg_r[64 * (wave * SB + sb) + own - k0] = r[sb];
        }
        if (B < 32) {
            k0 = win1.k;
            set_valid(k0);
            set_label_at(win2.k);
        }
        win1 = win2;
        // ============ gradient pass: this wave's part of the mean gradient
        double G;
        {
            v4i c[4], half = {0, 0, 0, 0};
#pragma unroll
            for (int sb = 0; sb < SB; ++sb) half = offset(rd[sb], half);
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                c[s] = v4i{0, 0, 0, 0};
#pragma unroll
                for (int sb = 0; sb < SB; ++sb) c[s] = __builtin_amdgcn_mfma_i32_16x16x64_i8(rd[sb], e1[sb][s], c[s], 0, 0, 0);
            }
            const Sums s = pick(c, half);
            double v = fma((double)s.lo[1], 65536.0, (double)s.lo[0]);
            if constexpr (ND == 8) v = fma(fma((double)s.hi[1], 65536.0, (double)s.hi[0]), (double)kUpper, v);
            G = fma(g_dl, ldexp(v, -kr), g_mid * (double)rsum);
        }
        float Rmax = __uint_as_float(rmax);
        if (nwv > 1) {
            gpart[(P * kWaves + wave) * 64 + lane] = G;
            lds_barrier();
            const uint4 *const f4 = reinterpret_cast<const uint4 *>(info + P * kWaves);
            const uint4 m0 = f4[0], m1 = f4[1];
            double v[kWaves] = {};
#pragma unroll
            for (int q = 0; q < 4; ++q) v[q] = gpart[(P * kWaves + q) * 64 + lane];
            if (nwv > 4) {
#pragma unroll
                for (int q = 4; q < 8; ++q) v[q] = gpart[(P * kWaves + q) * 64 + lane];
            }
            const MaxU m;
            Rmax = __uint_as_float(m(m(m(m0.x, m0.y), m(m0.z, m0.w)), m(m(m1.x, m1.y), m(m1.z, m1.w))));
            G = ((v[0] + v[1]) + (v[2] + v[3])) + ((v[4] + v[5]) + (v[6] + v[7]));
        }
        // |dx_j| <= lr (maxabs(L_j) max |r| + l2 |x_j|)
        beta = fmaf(beta_r, Rmax, grow * beta);
        ymax = fmaf(ymax_r, Rmax, grow * ymax);
        set_scales();
        since = side_step ? 1 : since + 1;
        // ============ update
        const float g = live ? (float)G : 0.0f;
        if constexpr (DBG) {
            if (a.dbg_g && wave == 0 && live) a.dbg_g[j] = g;
        }
        const float reg = a.l2 * x;
        const float stp = a.lr * (g + reg);
        x = x - stp;
        if (__builtin_expect(a.prox != 0, 0)) x = apply_prox(x, a.prox, a.lr, a.prox_coef);
        publish_y();
    };
    for (int left = a.nsteps;;) {
        step(std::integral_constant<int, 0>(), left);
        if (--left == 0) break;
        step(std::integral_constant<int, 1>(), left);
        if (--left == 0) break;
    }
    if (wave == 0 && live) a.x[j] = x;
}

}  // namespace zipml
