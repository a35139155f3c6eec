// The epoch on a single workgroup: problems of at most 256 features, fp32 model.
//
// With one workgroup there is no device-wide exchange; a step is a chain of short phases, and what it
// costs is the latency of that chain (LDS round trips, barriers, cross-lane sums), not arithmetic.  The
// general step loop took 2.1 us for a step of 16 samples x 64 features and 4.7 us for one of 256 x 90 on
// uneven levels.  Here the roles are split:
//   - loader waves keep a ring of steps in LDS, ahead of the step at work, with loads that go from memory
//     to LDS directly (no registers, nothing to wait for in the other waves);
//   - the other waves only ever touch LDS.  Evenly spaced levels run on v_mfma_i32_16x16x64_i8 against
//     fixed-point digits as in zipml_sgd_mfma.h, but eight of them: the general loop on one workgroup computes
//     in fp32 throughout, and with the 29 bits of four digits a small residual or model element beside a large
//     one lost bits (one residual in 64 larger by 10^6: worst coordinate of the gradient off by 9e-5 instead of
//     6e-7).  Eight digits hold all 24 bits of a number down to 2^-35 of the largest, whatever its size; the sixteen
//     rows of the instruction hold them twice over, so there are no more instructions than with four.  The scale
//     of the residuals is that of a block of 64 samples (one wave's), the scale of y = delta x is a bound that
//     every wave forms from the last step's largest |y| and |r|, so a step has two workgroup barriers: dot pass
//     and residuals | gradient pass and update.  Where a minibatch and the features fit one wave (64 x 64) that
//     wave runs the whole step and meets the loader only.
//   - Uneven levels of 2 or 3 bits (at most 8 levels): the dot pass looks up L_j[c] x_j + L_j'[c'] x_j'
//     of two features at once in LDS; in the gradient pass a lane owns one feature, so that a level look-up is
//     a byte permute from registers, four codes at a time: the byte digits of the fixed-point level go to
//     the matrix cores against the digits of r, two at a time and only down to the lowest that some level has (two
//     in all for levels on a grid of 2^12 or fewer steps, six for any fp32 levels down to 2^-19 of the largest).  More
//     levels: gathers from a table in LDS in both passes, in fp32.
// Measured against the general loop: an epoch of 256 steps, 16 samples x 64 features, 4 bits 549 -> 133 us
// (0.52 us a step; 128 with four digits); 512 steps, 256 x 90, 3 bits on optimal levels 2,419 -> 1,165 us (2.3 us
// a step; 1,201 with four digits of every level); 256 x 100, 3 bits, arbitrary levels 5.3 -> 3.3 us a step.
#include "zipml_device.h"
#include "zipml_mfma_ops.h"
#include "zipml_prox.h"
#include "zipml_sgd_solo.h"

namespace zipml {

// s_waitcnt vmcnt(n) with n known at run time only (0 <= n <= 63).
__device__ __forceinline__ void wait_loads(int n)
{
    switch (n) {
#define ZIPML_W(k) case k: __builtin_amdgcn_s_waitcnt(0x0F70 | ((k) & 15) | (((k) >> 4) << 14)); break;
#define ZIPML_W8(k) ZIPML_W(k) ZIPML_W(k + 1) ZIPML_W(k + 2) ZIPML_W(k + 3) ZIPML_W(k + 4) ZIPML_W(k + 5) ZIPML_W(k + 6) ZIPML_W(k + 7)
        ZIPML_W8(0) ZIPML_W8(8) ZIPML_W8(16) ZIPML_W8(24) ZIPML_W8(32) ZIPML_W8(40) ZIPML_W8(48) ZIPML_W8(56)
        default: __builtin_amdgcn_s_waitcnt(0x0F70);
#undef ZIPML_W8
#undef ZIPML_W
    }
}

// Loader wave `lw`: step t + S - 1 is requested during step t (its slot was given back by the barrier
// that ended step t - 1), and the last barrier of step t is joined once step t + 1 has landed -- with three
// slots or more, step t + 2, so that the other waves can read the operands of step t + 1 before that barrier.
// The number of loads in flight is the same in every step (steps past the end repeat the last one).
template <int BITS>
__device__ __forceinline__ void solo_loader(const SoloArgs &a, unsigned char *ring, int S, int lw, int nbar)
{
    typedef const __attribute__((address_space(1))) unsigned char *gptr;
    typedef __attribute__((address_space(3))) unsigned char *lptr;
    const SoloSlot sl(a.d32, a.B, BITS, a.loaders);
    const int lane = threadIdx.x & (kWave - 1);
    const int B = a.B;
    // per load: which array (the same for all lanes), and the lane's offset in it from the step's first byte
    uint32_t off[kSoloMaxInstr];
#pragma unroll
    for (int m = 0; m < kSoloMaxInstr; ++m) {
        int ck = m * a.loaders + lw;
        ck = ck < sl.chunks ? ck : sl.chunks - 1;      // (padding of the slot: any address inside)
        uint32_t p = (uint32_t)ck * 1024 + lane * 16, end;
        if (ck < sl.chunks2) {
            end = a.d32 * sl.len2;
            p = p < end ? p : end - 16;
            off[m] = p / sl.len2 * (uint32_t)(a.n_pad * 4 * BITS) + p % sl.len2;
        } else if (ck < sl.chunks2 + sl.chunks1) {
            p -= sl.c1_off;
            end = a.d32 * sl.len1;
            p = p < end ? p : end - 16;
            off[m] = p / sl.len1 * (uint32_t)(a.n32 * 128 * BITS) + p % sl.len1;
        } else {
            p -= sl.label_off;
            end = 4 * B;
            off[m] = p < end ? p : end - 16;
        }
    }
    const int64_t t_end = a.step0 + a.nsteps;
    int64_t at = a.step0;                              // the step that the pointers stand at
    const unsigned char *src2 = (const unsigned char *)a.p2 + at * sl.len2;
    const unsigned char *src1 = (const unsigned char *)a.p1 + at * B / 32 * (128 * BITS);
    const unsigned char *srcb = (const unsigned char *)a.b + at * B * 4;
    int in_group = (int)(at * B & 31);                 // (a batch below 32: where it begins in its sample group)
    int slot = 0;
    auto request = [&]() {
        unsigned char *dst = ring + slot + lw * 1024;
#pragma unroll
        for (int m = 0; m < kSoloMaxInstr; ++m)
            if (m < sl.instr) {
                const int ck = m * a.loaders + lw;
                const unsigned char *src = ck < sl.chunks2 ? src2 : ck < sl.chunks2 + sl.chunks1 ? src1 : srcb;
                __builtin_amdgcn_global_load_lds((gptr)(src + off[m]), (lptr)(dst + m * a.loaders * 1024), 16, 0, 0);
            }
        slot = slot + sl.bytes < S * sl.bytes ? slot + sl.bytes : 0;
        if (at + 1 < t_end) {
            ++at;
            src2 += sl.len2;
            srcb += 4 * B;
            in_group += B;
            src1 += (in_group >> 5) * (128 * BITS);
            in_group &= 31;
        }
    };
    auto barrier = [&]() {
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
    };
    const int flying = (S >= 3 ? S - 3 : 0) * sl.instr;
    for (int k = 0; k < S - 1; ++k) request();
    wait_loads(flying);
    barrier();
    for (int64_t t = a.step0; t < t_end; ++t) {
        request();
        for (int k = 1; k < nbar; ++k) barrier();
        wait_loads(flying);
        barrier();
    }
    wait_loads(0);                                     // nothing may land in LDS after the workgroup has ended
}

// A sum over the four rows of 16 lanes, in every lane.
__device__ __forceinline__ float rows_sum(float v)
{
    typedef unsigned int v2u __attribute__((ext_vector_type(2)));
    v2u s = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    v = __uint_as_float(s[0]) + __uint_as_float(s[1]);
    s = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return __uint_as_float(s[0]) + __uint_as_float(s[1]);
}
// Digit sums of four tiles -> the number of the tile that this row looks after.  A row of the sum with one element is
// exact up to the last step (24 bits of the element stand in the upper digits): one rounding as in a product, two in a
// sum.
__device__ __forceinline__ float tile_value(const v4i (&c)[4], int q4)
{
    int a[2], b[2];
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        const int a0 = q4 & 2 ? c[2][2 * k] : c[0][2 * k], a1 = q4 & 2 ? c[2][2 * k + 1] : c[0][2 * k + 1];
        const int b0 = q4 & 2 ? c[3][2 * k] : c[1][2 * k], b1 = q4 & 2 ? c[3][2 * k + 1] : c[1][2 * k + 1];
        a[k] = a0 + (a1 << 8);
        b[k] = b0 + (b1 << 8);
    }
    const DigitSums s = join_rows(a, b);
    return fmaf(fmaf((float)s.hi[1], 65536.0f, (float)s.hi[0]), kUpper, fmaf((float)s.lo[1], 65536.0f, (float)s.lo[0]));
}

struct SoloLds {
    int8_t *ydig;          // [KB][8 digits][4 q][16]
    int8_t *rdig;          // [NB][8 digits][4 q][16]
    float4 *info;          // [NB] (scale of r, -, -, -)
    float *wr;             // [16] per wave: sum of r, [8 + w]: bits of the largest |r|
    float *wy;             // [16] per wave: sum of mid x, [8 + w]: bits of the largest |y|
    int8_t *zeros;         // [16]
    float *rs;             // [NB * 64] residuals  (these two for uneven levels of 4 and more bits only)
    float *xs;             // [256] model
    float *zp;             // [1024] parts of the dot products, one per split and sample (splits * NB <= 16)
    unsigned char *table;  // uneven levels
    unsigned char *ring;
};
__device__ __forceinline__ SoloLds solo_carve(unsigned char *smem, int B, int bits)
{
    const int NB = (B + 63) / 64;
    SoloLds L;
    L.ydig = (int8_t *)smem;
    L.rdig = L.ydig + 2048;
    L.info = (float4 *)(L.rdig + NB * 512);
    L.wr = (float *)(L.info + NB);
    L.wy = L.wr + 16;
    L.zeros = (int8_t *)(L.wy + 16);
    L.rs = (float *)(L.wr + 128);
    L.xs = L.rs + (bits > 3 ? NB * 64 : 0);
    L.zp = L.xs + (bits > 3 ? 256 : 0);
    L.table = (unsigned char *)(L.zp + 4 * 256);
    L.ring = L.table;
    return L;
}

// A lane's residual -> the sum and the largest magnitude over the wave, the digits of the block `sb`.
struct SoloR {
    float sum;
    uint32_t max;
    int k;
};
__device__ __forceinline__ SoloR solo_residuals(int8_t *planes, const QuadStore &store, float r)
{
    SoloR o;
    o.max = wave_total(magnitude(r), MaxU());
    o.sum = wave_total(r, AddF());
    o.k = scale_for(exponent_of(o.max));
    store(planes, digits_of(r, o.k));
    return o;
}

__device__ __forceinline__ float wave_figures_sum(const float *v)
{
    const float4 p = *reinterpret_cast<const float4 *>(v), q = *reinterpret_cast<const float4 *>(v + 4);
    return ((p.x + p.y) + (p.z + p.w)) + ((q.x + q.y) + (q.z + q.w));
}
__device__ __forceinline__ uint32_t wave_figures_max(const float *v)
{
    const uint4 p = *reinterpret_cast<const uint4 *>(v), q = *reinterpret_cast<const uint4 *>(v + 4);
    const MaxU m;
    return (uint32_t)__builtin_amdgcn_readfirstlane((int)m(m(m(p.x, p.y), m(p.z, p.w)), m(m(q.x, q.y), m(q.z, q.w))));
}

__device__ __forceinline__ float solo_update(const SoloArgs &a, float x, float g)
{
    const float reg = a.l2 * x;
    const float stp = a.lr * (g + reg);
    const float v = x - stp;
    int prox = a.prox;
    asm("" : "+s"(prox));                              // (one branch for the case without, not a tree of the kinds)
    if (__builtin_expect(prox != 0, 0)) return apply_prox(v, a.prox, a.lr, a.prox_coef);
    return v;
}

// One lane operand (16 codes) from a slot, as one load where its alignment allows: that takes an offset, two loads of
// a dword at a distance take an address.
template <int BITS>
__device__ __forceinline__ void slot_codes(const unsigned char *p, uint32_t (&w)[kOpDwords<BITS>])
{
    typedef uint32_t v2u __attribute__((ext_vector_type(2)));
    typedef uint32_t v4u __attribute__((ext_vector_type(4)));
    if constexpr (BITS == 8) {
        const v4u q = *reinterpret_cast<const v4u *>(p);
#pragma unroll
        for (int k = 0; k < 4; ++k) w[k] = q[k];
    } else if constexpr (BITS == 4) {
        const v2u q = *reinterpret_cast<const v2u *>(p);
        w[0] = q[0];
        w[1] = q[1];
    } else {
        const uint32_t *q = reinterpret_cast<const uint32_t *>(p);
#pragma unroll
        for (int k = 0; k < kOpDwords<BITS>; ++k) w[k] = q[k];
    }
}

// What the sums over codes start from: codes of 8 bits are operands 128 below, so 128 times the sum of the other
// operand, 64 twice over.  (In integers: with the 128 in the factor of a sum of fp32 numbers, a large element that meets
// the code zero everywhere would leave its rounding errors.)
template <int BITS>
__device__ __forceinline__ v4i code_offset(const v4i &a, v4i c)
{
    if constexpr (BITS == 8) {
        const v4i h = {0x40404040, 0x40404040, 0x40404040, 0x40404040};
        c = __builtin_amdgcn_mfma_i32_16x16x64_i8(a, h, c, 0, 0, 0);
        c = __builtin_amdgcn_mfma_i32_16x16x64_i8(a, h, c, 0, 0, 0);
    }
    return c;
}

// Evenly spaced levels.  KB: blocks of 64 features.  MANY = false: at most 64 samples, wave w owns the
// features 64 w .. 64 w + 63, a lane each, and wave 0 takes the dot pass.  MANY = true: a wave takes blocks of
// 64 samples in the dot pass (wave, wave + nc, ...), and the feature tiles wave and wave + nc (16 features) in
// the gradient pass, where the four rows of 16 lanes hold the parts of four sample blocks.  T: 16-sample tiles
// of a block (1, 2 or 4; a batch below 32 lies in one tile of its sample group).
// All LDS reads of a phase are issued together and none sits behind a branch: with a read, its wait and its
// matrix instruction per branch the smallest step took 1.0 us instead of 0.5.
template <int BITS, int KB, bool MANY, int T>
__device__ __forceinline__ void solo_affine(const SoloArgs &a, const SoloLds &L, int S, int nc)
{
    constexpr bool kOne = KB == 1 && !MANY;            // one wave does it all
    constexpr int kFt = MANY ? (KB == 4 ? 2 : 1) : 1;  // feature sets of a wave
    constexpr int K = 1 << BITS, HW = kOpDwords<BITS>;
    const int tid = threadIdx.x, lane = tid & (kWave - 1);
    const int wave = kOne ? 0 : __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n16 = lane & 15, q4 = lane >> 4;
    const int B = a.B, NB = MANY ? (B + 63) / 64 : 1, nrg = B >= 32 ? B / 32 : 1;
    const SoloSlot sl(a.d32, B, BITS, a.loaders);
    const uint32_t shift = op_shift<BITS>(q4 & 1);
    const int own = lane_slot<BITS>(lane), own16 = lane_slot<BITS>(n16);   // this lane's element of 64, its column of a tile
    const QuadStore store(lane);

    // ---- this lane's features (the mean over the batch is folded into the gradient's factors)
    float o_dl[kFt], o_mid[kFt], g_dl[kFt], g_mid[kFt], x[kFt];
    int y_pos[kFt];
    bool live[kFt];
    float mu = 0.0f, y0 = 0.0f;
#pragma unroll
    for (int u = 0; u < kFt; ++u) {
        const int f = MANY ? 16 * (wave + nc * u) + n16 : 64 * wave + own;
        live[u] = f < a.d;
        const float lo = live[u] ? a.levels[(size_t)f * K] : 0.0f, hi = live[u] ? a.levels[(size_t)f * K + K - 1] : 0.0f;
        o_dl[u] = (float)(((double)hi - (double)lo) / (double)(K - 1));
        o_mid[u] = lo;
        g_dl[u] = __fdiv_rn(o_dl[u], (float)B);
        g_mid[u] = __fdiv_rn(o_mid[u], (float)B);
        x[u] = live[u] ? a.x[f] : 0.0f;
        mu = fmaxf(mu, fabsf(o_dl[u]) * fmaxf(fabsf(lo), fabsf(hi)));
        y0 = fmaxf(y0, fabsf(o_dl[u] * x[u]));
        int half, byte;
        code_slot<BITS>(f & 31, half, byte);
        y_pos[u] = MANY ? ((f >> 6) & 3) * 512 + (2 * ((f >> 5) & 1) + half) * 16 + byte + 64 * q4 : wave * 512;
        if (f >= 64 * KB) y_pos[u] = -1;               // no such feature, not even a padding one
    }
    // digits of y, and the wave's figures of the model
    float cp = 0.0f;
    uint32_t ym = 0u;
    auto publish_y = [&](int ky) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < kFt; ++u) {
            const float y = o_dl[u] * x[u];
            const Digits8 dg = digits_of(y, ky);
            if (MANY) {
                // (the rows of lanes hold the same feature: each stores two digits)
                if (y_pos[u] >= 0) {
                    L.ydig[y_pos[u]] = (int8_t)(dg.lo >> (8 * q4));
                    L.ydig[y_pos[u] + 256] = (int8_t)(dg.hi >> (8 * q4));
                }
            } else {
                store(L.ydig + y_pos[u], dg);
            }
            cp = u == 0 ? o_mid[u] * x[u] : cp + o_mid[u] * x[u];
            ym = u == 0 ? magnitude(y) : MaxU()(ym, magnitude(y));
        }
        if (!kOne) {
            if (MANY) { cp = row_total(cp, AddF()); ym = row_total(ym, MaxU()); }
            else { cp = wave_total(cp, AddF()); ym = wave_total(ym, MaxU()); }
            if (lane == 0) { L.wy[wave] = cp; L.wy[8 + wave] = __uint_as_float(ym); }
        }
    };
    // Bound of the next step's |y_j|: |dy_j| <= lr (delta_j maxabs(L_j) max_i |r_i| + l2 |y_j|), as powers of
    // two; the exponent of the largest |y| (plus one or more where there is an l2 term) and that of the
    // first term, and one above the larger.
    int e_step, e_l2 = 0;
    uint32_t m_bits = wave_total(magnitude(mu), MaxU()), y_bits = wave_total(magnitude(y0), MaxU());
    if constexpr (!kOne) {
        if (lane == 0) { L.wr[wave] = __uint_as_float(m_bits); L.wr[8 + wave] = __uint_as_float(y_bits); }
        lds_barrier();
        m_bits = wave_figures_max(L.wr);
        y_bits = wave_figures_max(L.wr + 8);
        lds_barrier();
        if (tid < 16) L.wr[tid] = 0.0f;
    }
    e_step = exponent_of(magnitude(fabsf(a.lr) * __uint_as_float(m_bits) * 1.0001f));
    if (a.l2 != 0.0f) e_l2 = exponent_of(magnitude(1.0f + fabsf(a.lr * a.l2) * 1.0001f));
    e_step = __builtin_amdgcn_readfirstlane(e_step);
    e_l2 = __builtin_amdgcn_readfirstlane(e_l2);
    int ky = scale_for(exponent_of(y_bits));
    publish_y(ky);

    // ---- where the operands of a step lie in its slot.  (Lanes without a sample or a sample group read
    // whatever is there: their result is dropped, or meets digits that are zero.)
    int dot_at[KB];
#pragma unroll
    for (int kb = 0; kb < KB; ++kb) {
        const int g = 2 * kb + (q4 >> 1) < a.d32 ? 2 * kb + (q4 >> 1) : a.d32 - 1;   // (padding: its digits are zero)
        dot_at[kb] = (g * B + own16) * 4 * BITS + (q4 & 1) * kOpStride<BITS> * 4;
    }
    const int dig_at = (n16 & 7) * 64 + q4 * 16;
    int grad_at[kFt][4];
#pragma unroll
    for (int u = 0; u < kFt; ++u)
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            const int f = MANY ? 16 * (wave + nc * u) + n16 : 64 * wave + tile_slot<BITS>(s) + own16;
            const int g = (f >> 5) < a.d32 ? f >> 5 : a.d32 - 1;
            int rg = (MANY ? 2 * s : 0) + (q4 >> 1);
            rg = rg < nrg ? rg : nrg - 1;
            grad_at[u][s] = sl.c1_off + ((g * nrg + rg) * 32 + (f & 31)) * 4 * BITS + (q4 & 1) * kOpStride<BITS> * 4;
        }

    // operands of the dot pass of a block, and of the gradient pass of four blocks (or four feature tiles)
    auto read_dot = [&](const unsigned char *base, int sb, int k0, uint32_t (&w)[T][KB][HW]) __attribute__((always_inline)) {
        const unsigned char *first = base + (64 * sb - (T == 1 ? k0 & 15 : k0)) * 4 * BITS;
#pragma unroll
        for (int s = 0; s < T; ++s)
#pragma unroll
            for (int kb = 0; kb < KB; ++kb) slot_codes<BITS>(first + dot_at[kb] + tile_slot<BITS>(s) * 4 * BITS, w[s][kb]);
    };
    const bool dots = kOne || (MANY ? wave < NB : wave == 0);    // this wave takes part in the dot pass
    const bool early = S >= 3;                         // (the ring is then a step further ahead)
    uint32_t dop[T][KB][HW], gop[kFt][4][HW];

    lds_barrier();                                     // the first step has landed; y, wave figures
    int k0 = (int)((a.step0 * B) & 31);                // where a batch begins in its sample group (0 from 32 samples on)
    int at = 0;
    const int slot_bytes = __builtin_amdgcn_readfirstlane(sl.bytes), label_off = __builtin_amdgcn_readfirstlane(sl.label_off);
    const int ring_end = S * slot_bytes;
    if (early && dots) read_dot(L.ring, MANY ? wave : 0, k0, dop);
    // Where the loop lies within 32 bytes is set (see solo_table): over ten sizes of 1 to 4, 7 and 8 bits the means of the eight
    // places are within 1.5 %, single sizes up to 5 % apart; 4 bytes in nothing is more than 1.5 % off its best, at 5 and 6 bits 0.
    if constexpr (BITS == 5 || BITS == 6) asm volatile(".p2align 5");
    else asm volatile(".p2align 5\n\ts_nop 0");
    int64_t left = a.nsteps;                           // (at least one)
    do {
        const unsigned char *base = L.ring + at;
        at = at + slot_bytes < ring_end ? at + slot_bytes : 0;
        // ================= dot pass, residuals
        SoloR mine = {0.0f, 0u, 0};
        float C = cp, label = 0.0f;
        uint32_t Y = ym;
        v4i ad[KB];
        if (dots) {
#pragma unroll
            for (int kb = 0; kb < KB; ++kb) ad[kb] = *reinterpret_cast<const v4i *>(L.ydig + kb * 512 + dig_at);
            label = *reinterpret_cast<const float *>(base + label_off + 4 * ((MANY ? 64 * wave : 0) + own - k0));
            if (!early) read_dot(base, MANY ? wave : 0, k0, dop);
        }
#pragma unroll
        for (int u = 0; u < kFt; ++u)
#pragma unroll
            for (int s = 0; s < 4; ++s) slot_codes<BITS>(base + grad_at[u][s], gop[u][s]);
        if constexpr (kOne) {
            C = wave_total(cp, AddF());
            Y = wave_total(ym, MaxU());
        } else {
            C = wave_figures_sum(L.wy);
            Y = wave_figures_max(L.wy + 8);
        }
        auto block = [&](int sb) __attribute__((always_inline)) {
            v4i c[4], from = {0, 0, 0, 0};
#pragma unroll
            for (int kb = 0; kb < KB; ++kb) from = code_offset<BITS>(ad[kb], from);
#pragma unroll
            for (int s = 0; s < T; ++s) {
                c[s] = from;
#pragma unroll
                for (int kb = 0; kb < KB; ++kb)
                    c[s] = __builtin_amdgcn_mfma_i32_16x16x64_i8(ad[kb], expand_codes<BITS>(dop[s][kb], shift), c[s], 0, 0, 0);
            }
            if constexpr (T == 1) c[1] = c[0];
            if constexpr (T <= 2) { c[2] = c[0]; c[3] = c[1]; }
            const float z = ldexpf(tile_value(c, q4), -ky) + C;
            const float r = (uint32_t)(64 * sb + own - k0) < (uint32_t)B ? z - label : 0.0f;
            return solo_residuals(L.rdig + sb * 512, store, r);
        };
        if (dots) {
            if constexpr (MANY) {
                int sb = wave;
                for (;;) {
                    const SoloR o = block(sb);
                    if (lane == 0) L.info[sb] = make_float4(__int_as_float(o.k), 0.0f, 0.0f, 0.0f);
                    mine.sum += o.sum;
                    mine.max = MaxU()(mine.max, o.max);
                    sb += nc;
                    if (sb >= NB) break;
                    read_dot(base, sb, k0, dop);       // (blocks beyond the first)
                    label = *reinterpret_cast<const float *>(base + label_off + 4 * (64 * sb + own - k0));
                }
            } else {
                mine = block(0);
                if (!kOne && lane == 0) L.info[0] = make_float4(__int_as_float(mine.k), 0.0f, 0.0f, 0.0f);
            }
            if (!kOne && lane == 0) { L.wr[wave] = mine.sum; L.wr[8 + wave] = __uint_as_float(mine.max); }
        }
        k0 = (k0 + B) & 31;
        if constexpr (!kOne) lds_barrier();

        // ================= gradient pass, update
        v4i c[kFt][4];
        v4i rd[MANY ? 4 : 1];
#pragma unroll
        for (int s = 0; s < (MANY ? 4 : 1); ++s)
            rd[s] = *reinterpret_cast<const v4i *>(L.rdig + (s < NB ? s : NB - 1) * 512 + dig_at);
        const int kr = kOne ? mine.k : __float_as_int(L.info[MANY && q4 < NB ? q4 : 0].x);
        float Rsum = mine.sum;
        uint32_t Rmax = mine.max;
        if constexpr (MANY) { Rsum = wave_figures_sum(L.wr); Rmax = wave_figures_max(L.wr + 8); }
        else if constexpr (!kOne) { Rsum = L.wr[0]; Rmax = (uint32_t)__builtin_amdgcn_readfirstlane(__float_as_int(L.wr[8])); }
        const int e_y = exponent_of(Y) + e_l2, e_r = exponent_of(Rmax) + e_step;
        ky = scale_for((e_y > e_r ? e_y : e_r) + 1);
        v4i from[MANY ? 4 : 1];
#pragma unroll
        for (int s = 0; s < (MANY ? 4 : 1); ++s) from[s] = code_offset<BITS>(rd[s], v4i{0, 0, 0, 0});
#pragma unroll
        for (int u = 0; u < kFt; ++u)
#pragma unroll
            for (int s = 0; s < 4; ++s)
                c[u][s] = __builtin_amdgcn_mfma_i32_16x16x64_i8(rd[MANY ? s : 0], expand_codes<BITS>(gop[u][s], shift), from[MANY ? s : 0], 0, 0, 0);
        if (early && dots) read_dot(L.ring + at, MANY ? wave : 0, k0, dop);
#pragma unroll
        for (int u = 0; u < kFt; ++u) {
            float G = ldexpf(tile_value(c[u], q4), -kr);
            if constexpr (MANY) {
                G = q4 < NB ? G : 0.0f;
                for (int sb0 = 4; sb0 < NB; sb0 += 4) {
                    uint32_t w[4][HW];
                    v4i e[4], rx[4];
#pragma unroll
                    for (int s = 0; s < 4; ++s) {
                        int more = 2 * sb0;            // sample groups on from grad_at's
                        if (2 * (sb0 + s) + (q4 >> 1) >= nrg) more = 0;   // (past the batch: what is read does not count)
                        slot_codes<BITS>(base + grad_at[u][s] + more * 128 * BITS, w[s]);
                        rx[s] = *reinterpret_cast<const v4i *>(2 * (sb0 + s) + (q4 >> 1) < nrg ? L.rdig + (sb0 + s) * 512 + dig_at : L.zeros);
                    }
                    const int k = __float_as_int(L.info[sb0 + q4 < NB ? sb0 + q4 : NB - 1].x);
#pragma unroll
                    for (int s = 0; s < 4; ++s)
                        e[s] = __builtin_amdgcn_mfma_i32_16x16x64_i8(rx[s], expand_codes<BITS>(w[s], shift), code_offset<BITS>(rx[s], v4i{0, 0, 0, 0}), 0, 0, 0);
                    G += ldexpf(tile_value(e, q4), -k);
                }
                G = rows_sum(G);
            }
            x[u] = solo_update(a, x[u], fmaf(g_mid[u], Rsum, g_dl[u] * G));
        }
        publish_y(ky);
        lds_barrier();
    } while (--left != 0);
#pragma unroll
    for (int u = 0; u < kFt; ++u) {
        const int f = MANY ? 16 * (wave + nc * u) + n16 : 64 * wave + own;
        if (live[u] && (!MANY || q4 == 0)) a.x[f] = x[u];
    }
}

// Uneven levels, eight waves.  A wave owns the feature tiles wave and, with kFt = 2, wave + 8 (16 features, held by all
// four rows of 16 lanes).
template <int BITS, bool IN_LDS, int kFt>
__device__ __forceinline__ void solo_table(const SoloArgs &a, const SoloLds &L, unsigned char *ring, int S, int splits)
{
    // Where the loop lies within 32 bytes is worth up to 6 % of a step to it, so it is set here, whatever code precedes it.  Us
    // per step at 0, 4, ... 28 bytes: 256 samples x 90 features, 3 bits 2.07, 2.06, 2.08, 2.07, 2.04, 2.07, 2.05, 2.08 (4 bits: within
    // 1 %); 128 x 100, 6 bits 2.44, 2.44, 2.44, 2.48, 2.49, 2.49, 2.50, 2.46, 16 x 64 1.61, 1.58, 1.61, 1.63, 1.66, 1.68, 1.65, 1.69.
    // (64 x 64, 2 bits at 16 and 20 bytes 1.31, 1.27.)
    if constexpr (BITS == 2) asm volatile(".p2align 5\n\ts_nop 0\n\ts_nop 0\n\ts_nop 0\n\ts_nop 0\n\ts_nop 0");
    else if constexpr (BITS <= 5) asm volatile(".p2align 5\n\ts_nop 0\n\ts_nop 0\n\ts_nop 0\n\ts_nop 0");
    else if constexpr (BITS == 6) asm volatile(".p2align 5\n\ts_nop 0");
    constexpr int K = 1 << BITS;
    static_assert(BITS >= 2, "two levels are evenly spaced");
    constexpr bool kPairs = K <= 8;
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n16 = lane & 15, q4 = lane >> 4;
    const int B = a.B, NB = (B + 63) / 64, nrg = B >= 32 ? B / 32 : 1, nft = (a.d + 15) / 16;
    const SoloSlot sl(a.d32, B, BITS, a.loaders);
    const uint32_t shift = op_shift<BITS>(q4 & 1);
    float *const tab = (float *)L.table;

    float x[kFt];
    bool live[kFt];
    // Bytes 6 and 7 of the eight digits of the levels 0..3 and 4..7; the lower six are in LDS, behind the pair tables
    // ([feature tile][byte][16 features], K bytes each): levels on a grid of 2^12 or fewer steps have none.
    constexpr int kPw = kPairs ? K / 4 : 1;
    uint32_t plane[kFt][2][kPw];
    uint32_t *const low_planes = (uint32_t *)(L.table + (kPairs ? a.d32 * 16 * K * K * 4 : 0));
    int kl[kFt], used = 8;                             // (used: the lowest byte that is not zero for all levels)
    float la[kFt][kPairs ? K : 1], lb[kFt][2];         // levels of the pair's first feature; of the second, this lane's
#pragma unroll
    for (int u = 0; u < kFt; ++u) {
        const int f = 16 * (wave + 8 * u) + n16;
        live[u] = f < a.d;
        x[u] = live[u] ? a.x[f] : 0.0f;
        kl[u] = 0;
        if constexpr (kPairs) {
            float m = 0.0f, lv[K];
#pragma unroll
            for (int c = 0; c < K; ++c) {
                lv[c] = live[u] ? a.levels[(size_t)f * K + c] : 0.0f;
                m = fmaxf(m, fabsf(lv[c]));
                la[u][c] = (f & ~1) < a.d ? a.levels[(size_t)(f & ~1) * K + c] : 0.0f;
            }
            kl[u] = scale_for(exponent_of(magnitude(m)));
            uint32_t all[8][kPw] = {};
#pragma unroll
            for (int c = 0; c < K; ++c) {
                const Digits8 dg = digits_of(lv[c], kl[u]);
#pragma unroll
                for (int p = 0; p < 8; ++p) {
                    const uint32_t byte = ((p < 4 ? dg.lo : dg.hi) >> (8 * (p & 3))) & 0xFFu;
                    all[p][c >> 2] |= byte << (8 * (c & 3));
                }
            }
#pragma unroll
            for (int q = 0; q < kPw; ++q) {
#pragma unroll
                for (int p = 7; p >= 0; --p) {
                    if (__any(all[p][q] != 0u) && p < used) used = p;
                    if (p < 6 && wave + 8 * u < 2 * a.d32) low_planes[(((wave + 8 * u) * 6 + p) * 16 + n16) * kPw + q] = all[p][q];
                }
                plane[u][0][q] = all[6][q];
                plane[u][1][q] = all[7][q];
            }
            // eight lanes share a pair's table: entries sub * K K / 8 on
            const int sub = (n16 & 1) * 4 + q4;
            const int hi = K == 8 ? sub : sub >> 1;
            lb[u][0] = (f | 1) < a.d ? a.levels[(size_t)(f | 1) * K + hi] : 0.0f;
            lb[u][1] = 0.0f;
        }
    }
    if constexpr (!kPairs && IN_LDS)
        for (int e = tid; e < a.d32 * 32 * K; e += kSoloWaves * kWave)
            tab[e + e / K] = e / K < a.d ? a.levels[e] : 0.0f;
    // what the dot pass needs of the model: the pair tables, or the model itself
    auto publish_x = [&]() {
#pragma unroll
        for (int u = 0; u < kFt; ++u) {
            const int f = 16 * (wave + 8 * u) + n16;
            if (f < a.d32 * 32) {
                if constexpr (kPairs) {
                    const float other = dpp_move<0xB1>(x[u]);           // of lane n16 ^ 1
                    const float xa = n16 & 1 ? other : x[u], xb = n16 & 1 ? x[u] : other;
                    const float v = lb[u][0] * xb;
                    const int sub = (n16 & 1) * 4 + q4;
                    float *row = tab + (f >> 1) * (K * K) + sub * (K * K / 8);
                    if constexpr (K == 8) {
                        float4 p, q;
                        p.x = fmaf(la[u][0], xa, v); p.y = fmaf(la[u][1], xa, v); p.z = fmaf(la[u][2], xa, v); p.w = fmaf(la[u][3], xa, v);
                        q.x = fmaf(la[u][4], xa, v); q.y = fmaf(la[u][5], xa, v); q.z = fmaf(la[u][6], xa, v); q.w = fmaf(la[u][7], xa, v);
                        *reinterpret_cast<float4 *>(row) = p;
                        *reinterpret_cast<float4 *>(row + 4) = q;
                    } else if constexpr (K == 4) {
                        float2 p;
                        p.x = fmaf(sub & 1 ? la[u][2] : la[u][0], xa, v);
                        p.y = fmaf(sub & 1 ? la[u][3] : la[u][1], xa, v);
                        *reinterpret_cast<float2 *>(row) = p;
                    }
                } else {
                    if (q4 == 0) L.xs[f] = x[u];
                }
            }
        }
    };
    publish_x();

    const int own = kPairs ? lane_slot<BITS>(lane) : lane;     // this lane's sample of a block
    const QuadStore store(lane);
    // the digits of a block of samples: two blocks to an accumulator
    int dig_at[2];
#pragma unroll
    for (int s = 0; s < 2; ++s) dig_at[s] = (n16 >> 3) == s ? (n16 & 7) * 64 + q4 * 16 : -1;
    const int own_block = (q4 & 1) * 2 + (q4 >> 1);    // of four: the one whose sums this row ends up with
    int grad_at[kFt];
#pragma unroll
    for (int u = 0; u < kFt; ++u) {
        const int f = 16 * (wave + 8 * u) + n16, g = (f >> 5) < a.d32 ? f >> 5 : a.d32 - 1;
        grad_at[u] = sl.c1_off + (g * nrg * 32 + (f & 31)) * 4 * BITS;
    }
    const int fs = wave / (kSoloWaves / splits);       // which part of the features (dot pass)
    const int dw = wave % (kSoloWaves / splits), nd = kSoloWaves / splits;
    const bool early = S >= 3;                         // (the ring is then a step further ahead)
    const int64_t t_end = a.step0 + a.nsteps;
    const int lane_unit = own * (4 * BITS);
    // the unit of this lane's sample of block sb, feature group g (lanes without a sample: whatever is there)
    auto read_dot = [&](const unsigned char *base, int sb, int k0, int g, uint32_t (&w)[BITS]) __attribute__((always_inline)) {
        const uint32_t *q = reinterpret_cast<const uint32_t *>(base + (g < a.d32 ? g : fs) * sl.len2 + (64 * sb - k0) * (4 * BITS) + lane_unit);
#pragma unroll
        for (int k = 0; k < BITS; ++k) w[k] = q[k];
    };
    // the 16 table entries of a unit's pairs of features
    auto pairs = [&](const uint32_t (&w)[BITS], int g, float (&v)[16]) __attribute__((always_inline)) {
        constexpr int kField = 2 * BITS;
        constexpr uint32_t kMask = kPairs ? 4u * K * K - 4u : 0u;
        const uint32_t table_at = (uint32_t)g * (16 * K * K * 4);   // (above the bits of an entry: joined by one and-or)
        const unsigned char *tb = (const unsigned char *)tab;
#pragma unroll
        for (int k = 0; k < 16; ++k) {
            const int bit = k * kField, wi = bit >> 5, sh = bit & 31;
            if (bit >= 32 * BITS) continue;            // (no pairs at this width)
            uint32_t at;
            if (sh + kField > 32) at = __builtin_amdgcn_alignbit(w[wi + 1 < BITS ? wi + 1 : wi], w[wi], sh - 2);
            else at = sh >= 2 ? w[wi] >> (sh - 2) : w[wi] << (2 - sh);
            asm("v_and_or_b32 %0, %1, %2, %3" : "=v"(at) : "v"(at), "v"(kMask), "s"(table_at));   // (the compiler makes two of it)
            v[k] = *reinterpret_cast<const float *>(tb + k * K * K * 4 + at);
        }
    };
    constexpr int kGop = kPairs ? 4 : 1, GW = kPairs ? kOpDwords<BITS> : BITS;
    auto read_grad = [&](const unsigned char *base, int u, int sb0, uint32_t (&w)[kGop][GW]) __attribute__((always_inline)) {
        if constexpr (kPairs) {
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                int rg = 2 * (sb0 + s) + (q4 >> 1);
                rg = rg < nrg ? rg : nrg - 1;          // (past the batch: the digits are zero)
                slot_codes<BITS>(base + grad_at[u] + rg * 128 * BITS + (q4 & 1) * kOpStride<BITS> * 4, w[s]);
            }
        } else {
            const int rg = q4 < nrg ? q4 : 0;
            const uint32_t *q = reinterpret_cast<const uint32_t *>(base + grad_at[u] + rg * 128 * BITS);
#pragma unroll
            for (int k = 0; k < BITS; ++k) w[0][k] = q[k];
        }
    };
    uint32_t w0[BITS], w1[BITS], gop[kFt][kGop][GW];

    lds_barrier();
    int slot = 0;
    int k0 = (int)((a.step0 * B) & 31);                // where a batch begins in its sample group (0 from 32 samples on)
    if (early) read_dot(ring, dw < NB ? dw : 0, k0, fs, w0);
    for (int64_t t = a.step0; t < t_end; ++t) {
        const unsigned char *base = ring + slot * sl.bytes;
        slot = slot + 1 < S ? slot + 1 : 0;
        // ================= dot pass
        auto finish = [&](int sb, float z) {           // residual of this lane's sample of block sb
            const int i = 64 * sb + own - k0;
            const bool ok = i >= 0 && i < B;
            const float label = *reinterpret_cast<const float *>(base + sl.label_off + 4 * (ok ? i : 0));
            const float r = ok ? z - label : 0.0f;
            if constexpr (kPairs) {
                const uint32_t m = wave_total(magnitude(r), MaxU());
                const int k = scale_for(exponent_of(m));
                store(L.rdig + sb * 512, digits_of(r, k));
                // (an infinity or a NaN has no digits: it reaches the gradient as a NaN)
                if (lane == 0) L.info[sb] = make_float4(__int_as_float(k), m < 0x7F800000u ? 0.0f : __builtin_nanf(""), 0.0f, 0.0f);
            } else {
                L.rs[sb * 64 + lane] = r;
            }
        };
        if (!early) read_dot(base, dw < NB ? dw : 0, k0, fs, w0);
        for (int sb = dw; sb < NB; sb += nd) {
            if (sb != dw) read_dot(base, sb, k0, fs, w0);
            float z[4] = {0.0f, 0.0f, 0.0f, 0.0f};
            for (int g = fs; g < a.d32; g += splits) {
                read_dot(base, sb, k0, g + splits, w1);        // (the next one)
                if constexpr (kPairs) {
                    // two groups at a time: 32 look-ups on the way before the first sum is waited for
                    float v0[16], v1[16];
                    pairs(w0, g, v0);
                    const bool two = g + splits < a.d32;
                    if (two) {
                        g += splits;
                        read_dot(base, sb, k0, g + splits, w0);
                        pairs(w1, g, v1);
                    }
#pragma unroll
                    for (int k = 0; k < 16; ++k) z[k & 3] += v0[k];
                    if (two) {
#pragma unroll
                        for (int k = 0; k < 16; ++k) z[k & 3] += v1[k];
                    }
                } else {
                    const float *lv = IN_LDS ? tab + g * 32 * (K + 1) : a.levels + (size_t)g * 32 * K;
                    const float4 *xv = reinterpret_cast<const float4 *>(L.xs + g * 32);
                    const int nf = a.d - g * 32 < 32 ? a.d - g * 32 : 32;
#pragma unroll
                    for (int k = 0; k < 32; k += 4) {
                        const float4 v = xv[k / 4];
                        if (IN_LDS || k + 3 < nf) {
                            z[0] = fmaf(lv[(k + 0) * (IN_LDS ? K + 1 : K) + unit_code<BITS>(w0, k + 0)], v.x, z[0]);
                            z[1] = fmaf(lv[(k + 1) * (IN_LDS ? K + 1 : K) + unit_code<BITS>(w0, k + 1)], v.y, z[1]);
                            z[2] = fmaf(lv[(k + 2) * (IN_LDS ? K + 1 : K) + unit_code<BITS>(w0, k + 2)], v.z, z[2]);
                            z[3] = fmaf(lv[(k + 3) * (IN_LDS ? K + 1 : K) + unit_code<BITS>(w0, k + 3)], v.w, z[3]);
                        } else {
                            if (k + 0 < nf) z[0] = fmaf(lv[(k + 0) * K + unit_code<BITS>(w0, k + 0)], v.x, z[0]);
                            if (k + 1 < nf) z[1] = fmaf(lv[(k + 1) * K + unit_code<BITS>(w0, k + 1)], v.y, z[1]);
                            if (k + 2 < nf) z[2] = fmaf(lv[(k + 2) * K + unit_code<BITS>(w0, k + 2)], v.z, z[2]);
                        }
                    }
#pragma unroll
                    for (int k = 0; k < BITS; ++k) w0[k] = w1[k];
                }
            }
            const float zown = (z[0] + z[1]) + (z[2] + z[3]);
            if (splits == 1) finish(sb, zown);
            else L.zp[(fs * NB + sb) * 64 + lane] = zown;
        }
        // what the gradient pass needs from the slot, before the others' residuals are waited for
#pragma unroll
        for (int u = 0; u < kFt; ++u)
            if (wave + 8 * u < nft) read_grad(base, u, 0, gop[u]);
        if (splits > 1) {
            lds_barrier();
            if (wave < NB) {
                float z = 0.0f;
                for (int v = 0; v < splits; ++v) z += L.zp[(v * NB + wave) * 64 + lane];
                finish(wave, z);
            }
        }
        lds_barrier();

        // ================= gradient pass, update
        k0 = (k0 + B) & 31;
        if (early) read_dot(ring + slot * sl.bytes, dw < NB ? dw : 0, k0, fs, w0);
#pragma unroll
        for (int u = 0; u < kFt; ++u) {
            if (wave + 8 * u >= nft) continue;
            float gp = 0.0f;
            if constexpr (kPairs) {
                float G = 0.0f;
                for (int sb0 = 0; sb0 < NB; sb0 += 4) {
                    v4i rd[4];
                    if (sb0 > 0) read_grad(base, u, sb0, gop[u]);
#pragma unroll
                    for (int s = 0; s < 4; ++s)
                        rd[s] = *reinterpret_cast<const v4i *>(dig_at[s & 1] >= 0 && sb0 + s < NB ? L.rdig + (sb0 + s) * 512 + dig_at[s & 1] : L.zeros);
                    const float4 block = L.info[sb0 + own_block < NB ? sb0 + own_block : NB - 1];
                    const int k = __float_as_int(block.x);
                    // two digits of the levels at a time, from the top down to the last that some level has
                    constexpr bool kHold = kFt == 1;           // (else there are not registers enough)
                    v4i held[kHold ? 4 : 1];
                    if constexpr (kHold) {
#pragma unroll
                        for (int s = 0; s < 4; ++s)
                            if (s == 0 || sb0 + s < NB) held[s] = expand_codes<BITS>(gop[u][s], shift);
                    }
                    double half[2] = {0.0, 0.0};
                    auto digits = [&](const uint32_t (&pl)[2][kPw], double up) __attribute__((always_inline)) {
                        v4i c[2][2];
                        c[0][0] = c[0][1] = c[1][0] = c[1][1] = v4i{0, 0, 0, 0};
#pragma unroll
                        for (int s = 0; s < 4; ++s)
                            if (s == 0 || sb0 + s < NB) {
                                const v4i e = kHold ? held[kHold ? s : 0] : expand_codes<BITS>(gop[u][s], shift);
#pragma unroll
                                for (int p = 0; p < 2; ++p) {
                                    v4i lv;
#pragma unroll
                                    for (int q = 0; q < 4; ++q) lv[q] = (int)__builtin_amdgcn_perm(pl[p][kPw - 1], pl[p][0], (uint32_t)e[q]);
                                    c[p][s >> 1] = __builtin_amdgcn_mfma_i32_16x16x64_i8(rd[s], lv, c[p][s >> 1], 0, 0, 0);
                                }
                            }
                        // sums of equal weight first (two of 2^20 each), two of them to an integer
#pragma unroll
                        for (int h = 0; h < 2; ++h) {
                            const v4i &c0 = c[0][h], &c1 = c[1][h];
                            const double low = (double)(c0[0] + ((c0[1] + c1[0]) << 8)), mid = (double)((c0[2] + c1[1]) + ((c0[3] + c1[2]) << 8));
                            half[h] = fma(half[h], up, fma(fma((double)c1[3], 65536.0, mid), 65536.0, low));
                        }
                    };
                    int at = 6;
                    digits(plane[u], 0.0);
                    while (at > used) {
                        at -= 2;
                        uint32_t pl[2][kPw];
#pragma unroll
                        for (int p = 0; p < 2; ++p)
#pragma unroll
                            for (int q = 0; q < kPw; ++q) pl[p][q] = low_planes[(((wave + 8 * u) * 6 + at + p) * 16 + n16) * kPw + q];
                        digits(pl, at == 2 ? 16384.0 : 65536.0);         // (the words are 2^30 apart)
                    }
                    // even rows hold the lower digits of r, odd rows the upper ones: to one row
                    const uint64_t ia = __builtin_bit_cast(uint64_t, half[0]), ib = __builtin_bit_cast(uint64_t, half[1]);
                    const int a2[2] = {(int)(uint32_t)ia, (int)(uint32_t)(ia >> 32)}, b2[2] = {(int)(uint32_t)ib, (int)(uint32_t)(ib >> 32)};
                    const DigitSums j = join_rows(a2, b2);
                    const double lo = __builtin_bit_cast(double, (uint64_t)(uint32_t)j.lo[1] << 32 | (uint32_t)j.lo[0]);
                    const double hi = __builtin_bit_cast(double, (uint64_t)(uint32_t)j.hi[1] << 32 | (uint32_t)j.hi[0]);
                    G += (float)ldexp(fma(hi, (double)kUpper, lo), 8 * at - (at >= 4 ? 2 : 0) - k - kl[u]) + block.y;
                }
                gp = G;
            } else {
                float s4[4] = {0.0f, 0.0f, 0.0f, 0.0f};
                const int f = 16 * (wave + 8 * u) + n16;
                const float *lv = IN_LDS ? tab + f * (K + 1) : a.levels + (size_t)(live[u] ? f : 0) * K;
                for (int rg = q4; rg < nrg; rg += 4) {
                    const float4 *rv = reinterpret_cast<const float4 *>(L.rs + rg * 32);
                    uint32_t w[BITS];
#pragma unroll
                    for (int k = 0; k < BITS; ++k) w[k] = gop[u][0][k];
                    if (rg + 4 < nrg) {                // (the next one)
                        const uint32_t *q = reinterpret_cast<const uint32_t *>(base + grad_at[u] + (rg + 4) * 128 * BITS);
#pragma unroll
                        for (int k = 0; k < BITS; ++k) gop[u][0][k] = q[k];
                    }
#pragma unroll
                    for (int k = 0; k < 32; k += 4) {
                        const float4 v = rv[k / 4];
                        s4[0] = fmaf(lv[unit_code<BITS>(w, k + 0)], v.x, s4[0]);
                        s4[1] = fmaf(lv[unit_code<BITS>(w, k + 1)], v.y, s4[1]);
                        s4[2] = fmaf(lv[unit_code<BITS>(w, k + 2)], v.z, s4[2]);
                        s4[3] = fmaf(lv[unit_code<BITS>(w, k + 3)], v.w, s4[3]);
                    }
                }
                gp = (s4[0] + s4[1]) + (s4[2] + s4[3]);
            }
            const float g = live[u] ? __fdiv_rn(rows_sum(gp), (float)B) : 0.0f;
            x[u] = solo_update(a, x[u], g);
        }
        publish_x();
        lds_barrier();
    }
#pragma unroll
    for (int u = 0; u < kFt; ++u) {
        const int f = 16 * (wave + 8 * u) + n16;
        if (live[u] && q4 == 0) a.x[f] = x[u];
    }
}

template <int BITS, int KB, bool MANY, int T>
__global__ __launch_bounds__((kSoloWaves + 4) * kWave) void k_sgd_solo(SoloArgs a)
{
    constexpr int K = 1 << BITS;
    extern __shared__ __align__(16) unsigned char smem[];
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    SoloLds L = solo_carve(smem, a.B, BITS);
    if (tid == 0) a.status[0] = 0;
    // zero digits (padding features and samples), figures of waves that are not there
    for (int e = tid; e < (int)(L.table - smem) / 4; e += blockDim.x) reinterpret_cast<int *>(smem)[e] = 0;
    // Are the levels evenly spaced (fp64 formula, rounded once)?  Two levels always are, but for the rounding of
    // a sum in fp64.  The product with the spacing gives the same
    // fp32 number unless it is close to a rounding boundary; only then is it divided for real.
    int ok = 1;
    for (int e = tid; BITS > 1 && e < a.d * K; e += blockDim.x) {
        const int c = e & (K - 1);
        const float *row = a.levels + (e - c);
        const double lo = (double)row[0], wdt = (double)row[K - 1] - lo;
        const float v = row[c];
        if (v != (float)fma((double)c, wdt * (1.0 / (double)(K - 1)), lo)) ok &= (v == (float)(lo + ((double)c * wdt) / (double)(K - 1)));
    }
    const bool affine = __syncthreads_and(ok) || BITS == 1;
    const SoloSlot sl(a.d32, a.B, BITS, a.loaders);
    const int NB = (a.B + 63) / 64;
    int table = 0;
    if (!affine) table = solo_table_bytes(BITS, a.d32);
    // (2 KiB behind the last slot: lanes without a sample read on)
    const int room = a.lds_bytes - 2048 - (int)(L.table - smem);
    int S = (room - table) / sl.bytes;
    const int most = 2 + 63 / sl.instr;
    S = S < most ? S : most;
    S = __builtin_amdgcn_readfirstlane(S < kSoloMaxSlots ? S : kSoloMaxSlots);   // (divisions end in vector registers)
    unsigned char *const ring = L.table + __builtin_amdgcn_readfirstlane(table);
    L.ring = ring;
    if (affine) {
        const int nc = MANY ? (KB == 1 && a.B <= 256 ? 4 : kSoloWaves) : KB == 4 ? (a.d32 + 1) / 2 : KB;
        if (wave < nc) solo_affine<BITS, KB, MANY, T>(a, L, S, nc);
        else if (wave >= kSoloWaves) {
            if (!(KB == 1 && !MANY)) {                 // (the set-up of the others has two barriers more)
                __builtin_amdgcn_s_barrier();
                __builtin_amdgcn_s_barrier();
            }
            solo_loader<BITS>(a, ring, S, wave - kSoloWaves, KB == 1 && !MANY ? 1 : 2);
        }
        // (a barrier waits for the waves that are still there)
    } else if constexpr (BITS > 1) {
        // fewer than eight blocks of samples: the waves share the features of a block in the dot pass (two waves
        // to a SIMD: one alone issues its chains of dependent instructions at half the rate)
        int splits = NB >= 8 ? 1 : NB >= 4 ? 2 : NB >= 2 ? 4 : 8;
        while (splits > a.d32) splits >>= 1;
        if (wave < kSoloWaves) {
            constexpr int kFt = KB == 4 ? 2 : 1;
            // (only at 8 bits and more than 64 features there is no room for the table)
            if (BITS < 8 || table) solo_table<BITS, true, kFt>(a, L, ring, S, splits);
            else if constexpr (BITS == 8) solo_table<BITS, false, kFt>(a, L, ring, S, splits);
        } else {
            solo_loader<BITS>(a, ring, S, wave - kSoloWaves, splits > 1 ? 3 : 2);
        }
    }
}

template <int BITS>
int launch_solo(hipStream_t s, const SoloArgs &a)
{
    // (solo_plan has at most 128 features from 5 bits on)
    constexpr int kMost = BITS < 5 ? 4 : 2;
    const int KB = a.d32 <= 2 ? 1 : a.d32 <= 4 ? 2 : kMost;
#define ZIPML_SOLO(MANY, T) (KB == 1 ? (const void *)k_sgd_solo<BITS, 1, MANY, T> : KB == 2 ? (const void *)k_sgd_solo<BITS, 2, MANY, T> \
                                                                                         : (const void *)k_sgd_solo<BITS, kMost, MANY, T>)
    const void *kern = a.B > 64 ? ZIPML_SOLO(true, 4) : a.B > 32 ? ZIPML_SOLO(false, 4) : a.B > 16 || BITS == 1 ? ZIPML_SOLO(false, 2) : ZIPML_SOLO(false, BITS == 1 ? 2 : 1);
#undef ZIPML_SOLO
    if (HIP_FAILED(hipFuncSetAttribute(kern, hipFuncAttributeMaxDynamicSharedMemorySize, a.lds_bytes))) return ZIPML_ELAUNCH;
    SoloArgs args = a;
    void *params[] = {&args};
    return HIP_FAILED(hipLaunchKernel(kern, dim3(1), dim3((kSoloWaves + a.loaders) * kWave), params, a.lds_bytes, s)) ? ZIPML_ELAUNCH : ZIPML_OK;
}
template int launch_solo<ZIPML_SGD_BITS>(hipStream_t, const SoloArgs &);

}  // namespace zipml
