// Operand helpers of the matrix-core paths (v_mfma_i32_16x16x64_i8 on packed low-bit codes against
// fixed-point digits): shared by the SGD step loops and the loss kernel.
//
// Operand layout of the instruction (checked against a host reference on the device):
//   A: lane l holds row l%16, k = 16*(l/16) .. +15 (16 bytes);  B: lane l holds column l%16, same k;
//   C: lane l holds column l%16, rows 4*(l/16) .. +3.
// A lane's 16 codes are half a packed unit; code_slot() says which half and which byte of the operand
// a code of the unit lands in, and the digit operands are laid out in LDS with the same map.
#pragma once
#include "zipml_device.h"

#include <math.h>

namespace zipml {

typedef int v4i __attribute__((ext_vector_type(4)));

// The dwords of a unit that hold a half's codes: kOpDwords<BITS> of them from dword h * kOpStride<BITS> on.
// Odd widths: half 1 begins 16 bits into its first dword (1 bit: both halves read the same dword).
template <int BITS> constexpr int kOpDwords = (BITS + 1) / 2;
template <int BITS> constexpr int kOpStride = BITS / 2;
// the alignment of such an operand in bytes: the largest power of two in the stride, at most 16
template <int BITS> constexpr int kOpAlign = BITS == 8 ? 16 : BITS == 4 ? 8 : 4;
// expand_codes' shift for half h
template <int BITS>
__device__ __forceinline__ uint32_t op_shift(int h)
{
    return BITS == 1 ? 4u * (uint32_t)h : (BITS & 1) ? 16u * (uint32_t)h : 0u;
}

// Code f (0..31) of a packed unit -> (half: which lane operand of 16 codes, byte inside it).
template <int BITS>
__device__ __forceinline__ void code_slot(int f, int &half, int &byte)
{
    if (BITS == 4) {            // packed dword pd holds codes 8pd..8pd+7; low nibbles -> one operand
        const int pd = f >> 3, e = f & 7;    // dword, high nibbles -> the next
        half = pd >> 1;
        byte = (2 * (pd & 1) + (e & 1)) * 4 + (e >> 1);
    } else if (BITS == 2) {     // one packed dword per half; operand dword D = (p >> 2D) & 0x03..
        const int e = f & 15;
        half = f >> 4;
        byte = (e & 3) * 4 + (e >> 2);
    } else if (BITS == 1) {     // one dword for both halves; operand dword D of half h = (p >> (4h + D)) & 0x01..
        half = (f >> 2) & 1;
        byte = (f & 3) * 4 + (f >> 3);
    } else if (BITS == 3) {     // codes 24 bits apart share a shift: 2D, 2D + 8, 2D + 1, 2D + 9
        const int e = f & 15;
        half = f >> 4;
        byte = 4 * ((e & 7) >> 1) + 2 * (e & 1) + (e >> 3);
    } else if (BITS == 6) {     // the same in each half of the 16: 0, 4, 1, 5 and 2, 6, 3, 7
        const int e = f & 15;
        half = f >> 4;
        byte = 8 * (e >> 3) + 4 * ((e >> 1) & 1) + 2 * (e & 1) + ((e >> 2) & 1);
    } else {                    // in order
        half = f >> 4;
        byte = f & 15;
    }
}

// The other way: the code whose byte is i of dword D of a half.
template <int BITS>
__device__ __forceinline__ int slot_code(int half, int D, int i)
{
    if (BITS == 4) return 16 * half + 8 * (D >> 1) + 2 * i + (D & 1);
    if (BITS == 2) return 16 * half + 4 * i + D;
    if (BITS == 1) return 8 * i + 4 * half + D;
    if (BITS == 3) return 16 * half + 2 * D + (i >> 1) + 8 * (i & 1);
    if (BITS == 6) return 16 * half + 8 * (D >> 1) + 2 * (D & 1) + (i >> 1) + 4 * (i & 1);
    return 16 * half + 4 * D + i;
}

// Byte k of dword i <-> byte i of dword k.
__device__ __forceinline__ void bytes_transpose(uint32_t (&v)[4])
{
    const uint32_t a = __builtin_amdgcn_perm(v[1], v[0], 0x05010400u), b = __builtin_amdgcn_perm(v[1], v[0], 0x07030602u);
    const uint32_t c = __builtin_amdgcn_perm(v[3], v[2], 0x05010400u), d = __builtin_amdgcn_perm(v[3], v[2], 0x07030602u);
    v[0] = __builtin_amdgcn_perm(c, a, 0x05040100u);
    v[1] = __builtin_amdgcn_perm(c, a, 0x07060302u);
    v[2] = __builtin_amdgcn_perm(d, b, 0x05040100u);
    v[3] = __builtin_amdgcn_perm(d, b, 0x07060302u);
}

// The 16 codes of a half -> 16 signed bytes (code - off; off = 128 at 8 bits, else 0).  shift: op_shift<BITS>(half).
template <int BITS>
__device__ __forceinline__ v4i expand_codes(const uint32_t (&p)[kOpDwords<BITS>], uint32_t shift = 0)
{
    v4i r;
    if constexpr (BITS == 8) {
        r[0] = (int)(p[0] ^ 0x80808080u);
        r[1] = (int)(p[1] ^ 0x80808080u);
        r[2] = (int)(p[2] ^ 0x80808080u);
        r[3] = (int)(p[3] ^ 0x80808080u);
    } else if constexpr (BITS == 4) {
        r[0] = (int)(p[0] & 0x0F0F0F0Fu);
        r[1] = (int)((p[0] >> 4) & 0x0F0F0F0Fu);
        r[2] = (int)(p[1] & 0x0F0F0F0Fu);
        r[3] = (int)((p[1] >> 4) & 0x0F0F0F0Fu);
    } else if constexpr (BITS == 2) {
        r[0] = (int)(p[0] & 0x03030303u);
        r[1] = (int)((p[0] >> 2) & 0x03030303u);
        r[2] = (int)((p[0] >> 4) & 0x03030303u);
        r[3] = (int)((p[0] >> 6) & 0x03030303u);
    } else if constexpr (BITS == 1) {
        const uint32_t q = p[0] >> shift;
        r[0] = (int)(q & 0x01010101u);
        r[1] = (int)((q >> 1) & 0x01010101u);
        r[2] = (int)((q >> 2) & 0x01010101u);
        r[3] = (int)((q >> 3) & 0x01010101u);
    } else if constexpr (BITS == 3 || BITS == 6) {
        // Two codes that are 24 bits apart are bytes 0 and 3 once the first stands at bit 0: some 1 operation a code
        // (64 samples x 1,000 features, 6 bits, in the order of the codes 1.64 us a step, now 1.52).
        constexpr uint32_t kMask = ((1u << BITS) - 1u) * 0x01010101u;
        constexpr int N = kOpDwords<BITS>;
        uint32_t q[N + 1];
#pragma unroll
        for (int k = 0; k < N; ++k)
            q[k] = (BITS & 1) ? __builtin_amdgcn_alignbit(k + 1 < N ? p[k + 1] : 0u, p[k], shift) : p[k];
        q[N] = 0u;
        uint32_t x[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            const int bit = BITS == 3 ? 3 * k : 48 * (k >> 2) + 6 * (k & 3), wi = bit >> 5, sh = bit & 31;
            x[k] = sh == 0 ? q[wi] : sh + 24 + BITS <= 32 ? q[wi] >> sh : __builtin_amdgcn_alignbit(q[wi + 1], q[wi], sh);
        }
#pragma unroll
        for (int m = 0; m < 4; ++m) r[m] = (int)(__builtin_amdgcn_perm(x[2 * m + 1], x[2 * m], 0x07040300u) & kMask);
    } else {
        // Four codes of b bits at a time.  x: the 32 bits from the first of them on; t: codes 0 and 1 at
        // the foot of the low half-word, 2 and 3 of the high one; then the upper code of each pair moves up to
        // its byte.  Some 1.5 operations a code (what is chosen by a mask as one instruction, 0xCA; the compiler makes two).
        constexpr int N = kOpDwords<BITS>;
        constexpr int kMask = (int)(((1u << BITS) - 1u) * 0x01010101u);
        uint32_t q[N];
#pragma unroll
        for (int k = 0; k < N; ++k)
            q[k] = (BITS & 1) ? __builtin_amdgcn_alignbit(k + 1 < N ? p[k + 1] : 0u, p[k], shift) : p[k];
#pragma unroll
        for (int m = 0; m < 4; ++m) {
            const int bit = 4 * BITS * m, wi = bit >> 5, sh = bit & 31;
            const uint32_t x = sh == 0 ? q[wi]
                             : sh + 4 * BITS <= 32 ? q[wi] >> sh
                                                   : __builtin_amdgcn_alignbit(q[wi + 1 < N ? wi + 1 : wi], q[wi], sh);
            const int t = __builtin_amdgcn_bitop3_b32((int)0xFFFF0000u, (int)(x << (16 - 2 * BITS)), (int)x, 0xCA);
            r[m] = __builtin_amdgcn_bitop3_b32((int)0xFF00FF00u, (int)((uint32_t)t << (8 - BITS)), t, 0xCA) & kMask;
        }
    }
    return r;
}

// v = d0 + 256 d1 + 65536 d2 + 2^24 d3 with signed bytes d_k (|v| < 2^30): adding 128 to each of
// the three low bytes (carries included) leaves d_k + 128 in byte k, and x + 128 -> x is a flip of
// the top bit.  Returns the four digits as the bytes of one dword.
__device__ __forceinline__ uint32_t signed_digits(int v)
{
    return ((uint32_t)v + 0x00808080u) ^ 0x00808080u;
}
// N signed base-256 digits, the bytes of the result (|v| < 2^(8 N - 1) - 2^(8 N - 8)).
template <int N>
__device__ __forceinline__ uint64_t signed_digits_64(long long v)
{
    constexpr uint64_t kHalf = 0x8080808080808080ull >> (8 * (9 - N));       // 128 in the N - 1 lower bytes
    return ((uint64_t)v + kHalf) ^ kHalf;
}
// Digit k of an element goes to plane k: 64 bytes apart.
__device__ __forceinline__ void store_digits(int8_t *plane0, uint32_t dg)
{
    plane0[0] = (int8_t)(dg & 0xFF);
    plane0[64] = (int8_t)((dg >> 8) & 0xFF);
    plane0[128] = (int8_t)((dg >> 16) & 0xFF);
    plane0[192] = (int8_t)(dg >> 24);
}

__device__ __forceinline__ long long combine_digits(const v4i &c)
{
    return (long long)c[0] + ((long long)c[1] << 8) + ((long long)c[2] << 16) + ((long long)c[3] << 24);
}

// int64 (|v| < 2^53) times 2^-k as fp32, rounded once.
__device__ __forceinline__ float fixed_to_float(long long v, int k)
{
    const double d = (double)(int)(v >> 32) * 4294967296.0 + (double)(uint32_t)v;
    return (float)ldexp(d, -k);
}

// Largest k (clamped to +-60) with 2^k * v < 2^bits, for finite v >= 0.
__device__ __forceinline__ int scale_exponent(float v, int bits)
{
    if (!(v > 0.0f)) return 60;
    int e = 0;
    (void)frexpf(v, &e);     // v = m 2^e, 0.5 <= m < 1
    const int k = bits - e;
    return k < -60 ? -60 : k > 60 ? 60 : k;
}

// Reductions of 0 as the neutral element (sums, maxima of unsigned numbers): a row of 16 lanes, or the wave
// by two row broadcasts more, the result in lane 63 and from there in a scalar register.  Magnitudes are
// compared as bit patterns, which takes one instruction per step where fmaxf takes three.
template <typename T, typename Op>
__device__ __forceinline__ T row_total(T v, Op op)
{
    v = op(v, dpp_move<0xB1>(v));
    v = op(v, dpp_move<0x4E>(v));
    v = op(v, dpp_move<0x141>(v));
    return op(v, dpp_move<0x140>(v));
}
template <typename T, typename Op>
__device__ __forceinline__ T wave_total(T v, Op op)
{
    v = row_total(v, op);
    int i = __builtin_bit_cast(int, v);
    v = op(v, __builtin_bit_cast(T, __builtin_amdgcn_update_dpp(0, i, 0x142, 0xA, 0xF, false)));   // row_bcast15 into rows 1, 3
    i = __builtin_bit_cast(int, v);
    v = op(v, __builtin_bit_cast(T, __builtin_amdgcn_update_dpp(0, i, 0x143, 0xC, 0xF, false)));   // row_bcast31 into rows 2, 3
    return __builtin_bit_cast(T, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), 63));
}
struct AddF { __device__ __forceinline__ float operator()(float p, float q) const { return p + q; } };
struct MaxU { __device__ __forceinline__ uint32_t operator()(uint32_t p, uint32_t q) const { return p > q ? p : q; } };
__device__ __forceinline__ uint32_t magnitude(float v) { return __float_as_uint(v) & 0x7FFFFFFFu; }
// v < 2^exponent_of(v) for the bits of a finite v >= 0
__device__ __forceinline__ int exponent_of(uint32_t bits) { return (int)(bits >> 23) - 126; }
// Fixed point in two words of four signed base-256 digits, upper * 2^30 + lower: k such that 2^k v < 2^59 for
// v < 2^e ...
__device__ __forceinline__ int scale_for(int e) { return 59 - e; }
constexpr float kUpper = 1073741824.0f;            // weight of the upper four digits, see digits_of
// ... and the digits of 2^k v, the bytes of the two words (a |v| of one binade more has room, too).  A number down
// to 2^-35 of 2^e keeps all the bits that it has in fp32; below that it is rounded to 2^-59 of 2^e.
struct Digits8 {
    uint32_t lo, hi;
};
__device__ __forceinline__ Digits8 digits_of(float v, int k)
{
    const float t = ldexpf(v, k - 30), whole = rintf(t);   // (the difference is exact)
    return {signed_digits((int)((t - whole) * kUpper)), signed_digits((int)whole)};
}
// Where an element stands in an operand of 64 (a plane of 64 bytes) is where its lane stands in the wave: lane l looks
// after element lane_slot(l) of a group, so that four neighbouring lanes hold the bytes of a dword.  They exchange
// their digits and store two dwords each; eight byte stores a lane were 70 ns of the smallest step.
template <int BITS>
__device__ __forceinline__ int lane_slot(int l)
{
    return (l & 32) + slot_code<BITS>((l >> 4) & 1, (l >> 2) & 3, l & 3);
}
// lane_slot(16 s + i) = tile_slot(s) + lane_slot(i) for i < 16
template <int BITS> constexpr int tile_slot(int s) { return BITS == 1 ? 32 * (s >> 1) + 4 * (s & 1) : 16 * s; }
struct QuadStore {
    uint32_t sel1, sel2;
    int at;
    __device__ __forceinline__ explicit QuadStore(int lane)
    {
        sel1 = lane & 1 ? 0x03070105u : 0x06020400u;
        sel2 = lane & 2 ? 0x03020706u : 0x05040100u;
        at = 64 * (lane & 3) + (lane & ~3);
    }
    __device__ __forceinline__ uint32_t transpose(uint32_t v) const
    {
        v = __builtin_amdgcn_perm(dpp_move<0xB1>(v), v, sel1);
        return __builtin_amdgcn_perm(dpp_move<0x4E>(v), v, sel2);
    }
    // digit p of the lane's element -> planes + 64 p + lane (all lanes of the wave)
    __device__ __forceinline__ void operator()(int8_t *planes, Digits8 dg) const
    {
        *reinterpret_cast<uint32_t *>(planes + at) = transpose(dg.lo);
        *reinterpret_cast<uint32_t *>(planes + at + 256) = transpose(dg.hi);
    }
};

// a and b hold the sums of the lower four digits in the even rows of 16 lanes and of the upper four in the odd rows,
// each at most 2^22 in magnitude, two to an integer: row r gets those of a (r even) or b (r odd).
struct DigitSums {
    int lo[2], hi[2];
};
__device__ __forceinline__ DigitSums join_rows(const int (&a)[2], const int (&b)[2])
{
    typedef unsigned int v2u __attribute__((ext_vector_type(2)));
    DigitSums s;
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        const v2u v = __builtin_amdgcn_permlane16_swap((uint32_t)a[k], (uint32_t)b[k], false, false);
        s.lo[k] = (int)v[0];
        s.hi[k] = (int)v[1];
    }
    return s;
}

}  // namespace zipml
