// What the host needs to know of the single-workgroup epoch kernel (zipml_sgd_solo.hip).
#pragma once
#include "zipml_host.h"

namespace zipml {

struct SoloArgs {
    const uint32_t *p1, *p2;
    const float *levels, *b;
    float *x;
    int64_t n_pad, n32;
    int d, d32;
    int B;
    int64_t step0, nsteps;
    float lr, l2;
    int prox;
    float prox_coef;
    int *status;
    int loaders;           // waves that bring the packed codes into LDS: 1, 2 or 4
    int lds_bytes;
};

// One step's packed codes and labels in LDS: copy 2 (d32 groups of B units), copy 1 (d32 groups of the step's
// sample groups), labels, each in chunks of 1 KiB (one load of a wave; a load never mixes two arrays).
struct SoloSlot {
    int len2, len1;                // bytes per feature group of copy 2 and of copy 1
    int chunks2, chunks1, chunks;  // chunks of copy 2, of copy 1, of all three
    int c1_off, label_off, instr, bytes;
    __host__ __device__ SoloSlot(int d32, int B, int bits, int loaders)
    {
        len2 = B * 4 * bits;
        len1 = (B >= 32 ? B / 32 : 1) * 128 * bits;
        chunks2 = (d32 * len2 + 1023) / 1024;
        chunks1 = (d32 * len1 + 1023) / 1024;
        chunks = chunks2 + chunks1 + (4 * B + 1023) / 1024;
        c1_off = chunks2 * 1024;
        label_off = c1_off + chunks1 * 1024;
        instr = (chunks + loaders - 1) / loaders;      // loads per loader wave
        bytes = instr * loaders * 1024;
    }
};
constexpr int kSoloWaves = 8;          // consumer waves of a launch (some leave at once)
constexpr int kSoloMaxInstr = 16;      // loads per loader wave and step
constexpr int kSoloMaxSlots = 16;
constexpr int kSoloMaxBatch = 2048;

// LDS beside the ring of slots and the level tables: digits of y (at most 4 blocks of 64 features) and of
// r, per-block and per-wave figures, residuals and model (uneven levels of 4 and more bits), the parts of the dot
// products
__host__ __device__ inline int solo_fixed_lds(int B, int bits)
{
    const int NB = (B + 63) / 64;
    return 2048 + NB * 512 + NB * 16 + 512 + (bits > 3 ? NB * 256 + 1024 : 0) + 4 * 256 * 4 + 64;
}

// Bytes of the tables of the uneven-level loop: pair tables of the dot pass and the lower digits of the levels (at most
// 8 levels), or the level rows K + 1 words apart (0: they stay in memory).
__host__ __device__ inline int solo_table_bytes(int bits, int d32)
{
    const int K = 1 << bits, d_pad = 32 * d32;
    if (K <= 8) return d_pad / 2 * K * K * 4 + d_pad * 6 * K;
    const int rows = d_pad * (K + 1) * 4;
    return rows <= 72 * 1024 ? (rows + 15) & ~15 : 0;
}

// The launch for a problem, false if it does not fit: the layout's fields, B, loaders and lds_bytes are set.
inline bool solo_plan(const Layout &lay, int B, int lds_limit, SoloArgs &a)
{
    // (the loaders' offsets inside a packed copy are 32 bits wide)
    if (lay.d32 > 8 || B > kSoloMaxBatch || lay.bytes() >= ((size_t)1 << 32)) return false;
    // Where the general loop is the faster one (us a step here, there; the line is drawn by uneven levels, and even
    // ones, which the host cannot tell, follow it): the pair tables of uneven 3-bit levels are rebuilt every step,
    // whatever the batch (256 features, 32 samples: 3.85, 2.62; 128 samples 5.2, 5.0, even levels 3.4, 3.5); the
    // bytes of wide codes on many features pass through LDS twice (7 bits, 256 features, 128 samples: 6.5, 4.0; 8
    // bits, 128 features, 8 samples, uneven: 4.6, 3.8); one group of features leaves most waves without a
    // feature tile when the batch is large (7 bits, 12 features, 1,024 samples: 5.6, 4.2).
    const bool pow2 = lay.bits == 1 || lay.bits == 2 || lay.bits == 4;
    if (lay.bits == 3 && (lay.d32 > 4 ? B <= 64 : lay.d32 > 3 && B <= 32)) return false;
    if (lay.bits >= 5 && lay.d32 > 4) return false;
    if (lay.bits == 8 && lay.d32 > 2 && B <= 32) return false;
    if (!pow2 && lay.d32 == 1 && B > 256) return false;
    a.n_pad = lay.n_pad;
    a.n32 = lay.n32;
    a.d32 = (int)lay.d32;
    a.B = B;
    a.lds_bytes = lds_limit - 1024;                    // (static LDS of the kernel)
    // one loader where it has at most four requests per step, else two, else four
    a.loaders = 1;
    while (a.loaders < 4 && SoloSlot(a.d32, B, lay.bits, a.loaders).instr > 4) a.loaders *= 2;
    const SoloSlot sl(a.d32, B, lay.bits, a.loaders);
    if (sl.instr > kSoloMaxInstr) return false;
    // (a table that gives way to the slots is read from memory: 7 bits, 64 features, 512 samples 13.1, 6.1)
    const int table = lay.bits > 1 ? solo_table_bytes(lay.bits, a.d32) : 0;
    return solo_fixed_lds(B, lay.bits) + 2048 + table + 2 * sl.bytes <= a.lds_bytes;
}

template <int BITS> int launch_solo(hipStream_t s, const SoloArgs &a);

}  // namespace zipml
