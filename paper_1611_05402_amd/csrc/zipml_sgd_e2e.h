// Step loop of the epoch kernel in the end-to-end mode (Supp. C-E): the model is quantised before
// the dot pass (Q3), the mean gradient before the update (Q4), both with row scaling by the l2
// norm (Supp. A.3), so a step has three device-wide exchanges that depend on each other:
//     ||x||_2  ->  Q3, integer dot products  ->  residuals, gradient, ||g||_2  ->  Q4, update.
// Production launch only (persistent, more than one workgroup); included by zipml_sgd.hip and
// built on its SgdArgs / Lds / exchange-word helpers.  The stepwise and single-workgroup launches
// stay on sgd_steps<kInt>.
//
// Each exchange is ONE trip to the coherence point:
//   - the integer dot products travel like the fp32 ones (one 64-bit atomic per workgroup and
//     sample carrying arrival count and sum; every thread polls the words of its own samples);
//   - a norm is exchanged through one 64-bit slot per workgroup that holds the bits of the
//     workgroup's sum of squares PLUS ONE (sums are >= 0, so the bits never wrap; a zero slot means
//     "not there yet"): one store delivers value and arrival, and the waves that own features poll
//     all slots and add them up in registers.  The slots rotate over four buffers and are cleared
//     two steps ahead together with the dot-product words.
// The sums of squares are taken in fp64 in a fixed adjacent-pair tree over the feature index
// (inside a wave: butterfly over lanes, which is that tree because fp addition is commutative;
// then waves, then workgroups, pairwise), so the fp32 norm has the same bits on every workgroup
// and as a plain pairwise sum over the padded vector.
//
// Arithmetic per code: the dot pass adds G[j][code] * m_j.  On the matrix cores (DX: at most eight levels, 64 features to
// a workgroup) the grid index is a polynomial of the code's bits, G[j][c] = sum over the subsets s of the bits of a_js
// (1 where all bits of s are set in c), so the sum is 2^bits - 1 products of 0/1 bytes with the digits of a_js m_j, in exact
// integers like the others.  Else from a table T[j][code] = G[j][code] * m_j, rebuilt by the owner of feature j after Q3 (one
// LDS gather and one integer add per code; for wide level sets the product is formed on the fly): 512 samples x 64
// features, 3 bits 1.56 us from the table, 0.66 so; the whole step of 512 x 4,096 with that and with two exchange words for
// a sample 8.43 -> 7.66.  The mean gradient that Q4 quantises is the exact mean rounded to
// fp32, whatever the order: the gradient pass adds L[j][code] * r_i either in fp64 (products of two fp32
// numbers are exact there) or, for at most 16 levels and whole sample groups (MX), in integers on the matrix
// cores: r and a feature's levels in eight signed bytes each (24 bits at the top of 62, so that a number is exact
// down to 2^-38 of the largest residual of the step, or the largest level of the feature, and off by 2^-62 of that
// below: less than one rounding of the fp64 sum as soon as that largest one has a part in it).  A lane owns one
// feature, so a look-up is a byte permute of the level's bytes from registers, four codes at a time;
// the eight bytes of r fill half of the sixteen rows of v_mfma_i32_16x16x64_i8, one instruction per byte of
// the levels, by pairs down to the lowest byte that some level has (one pair for levels on a grid of 2^14 or fewer
// steps).  In fp64 the pass took, per code, a field extraction, an LDS gather with bank conflicts, two
// conversions and a multiply-add: a step of 512 samples x 4,096 features at 3 bits took 12.8 us, 9.6 with this
// pass and with the draws of the two quantisations made while the norms travel.
#pragma once

namespace zipml {

// Sum over the 64 lanes in the adjacent-pair tree (lane order); every lane gets the result (fp
// addition is commutative, so the butterfly lane ^ 1, ^ 2, ... forms exactly that tree).  DPP row
// operations for the four levels inside a row of 16 lanes (after the two quad steps all lanes of
// a quad hold the quad's sum, so the mirror steps pair neighbouring quads and half rows), the
// cross-lane network for the rows.
template <int CTRL>
__device__ __forceinline__ double dpp_move_f64(double x)
{
    const long long b = __double_as_longlong(x);
    int blo = (int)(uint32_t)b, bhi = (int)(uint32_t)((uint64_t)b >> 32);
    asm volatile("" : "+v"(blo), "+v"(bhi));     // the source of a DPP move must sit in vector registers
    int lo = __builtin_amdgcn_update_dpp(0, blo, CTRL, 0xF, 0xF, true);
    int hi = __builtin_amdgcn_update_dpp(0, bhi, CTRL, 0xF, 0xF, true);
    asm volatile("" : "+v"(lo), "+v"(hi));       // (and the moves stay moves: no folding into the fp64 add)
    return __longlong_as_double((long long)(((uint64_t)(uint32_t)hi << 32) | (uint64_t)(uint32_t)lo));
}
__device__ __forceinline__ double wave_tree_sum_f64(double v)
{
    v = v + dpp_move_f64<0xB1>(v);     // lane ^ 1
    v = v + dpp_move_f64<0x4E>(v);     // lane ^ 2
    v = v + dpp_move_f64<0x141>(v);    // the other quad of the half row
    v = v + dpp_move_f64<0x140>(v);    // the other half row
    v = v + __shfl_xor(v, 16, kWave);  // the neighbouring row
    v = v + __shfl_xor(v, 32, kWave);  // the other pair of rows
    return v;
}

// A float as a fixed-point number whose unit is 2^(emax - 150 - top), emax >= 1 the largest biased exponent
// that is met: exact where its own exponent is at most `top` below, cut off beyond.
__device__ __forceinline__ long long fixed_from_float(float v, int emax, int top)
{
    const uint32_t b = __float_as_uint(v);
    const int e = (int)((b >> 23) & 255u);
    const uint32_t m = (b & 0x7FFFFFu) | (e ? 0x800000u : 0u);
    const int sh = (e ? e : 1) - emax + top;
    const long long f = sh >= 0 ? (long long)((uint64_t)m << sh) : (long long)(m >> (sh > -31 ? -sh : 31));
    return (b >> 31) ? -f : f;
}
constexpr int kDigits = 8, kTop = 38;       // residuals and levels: 24 + 38 bits

// Slots per buffer of the norm exchange: beside the matrix-core dot pass up to 64 workgroups eight to 256 bytes, up to 128 eight
// to 128 (xword; everybody asks for all of them, and the memory side answers for one stretch after the other); else side
// by side (5 bits, 160 samples x 179 8.23 us a step spread, 8.13 so).
constexpr int kNormSlots = 256;
template <bool SPREAD>
__device__ __forceinline__ int norm_slot(int w, int W) { return SPREAD ? xword(w, W <= 64 ? 2 : W <= 128 ? 1 : 0) : w; }

// The monomials of up to three bits: bit b of `set` says whether bit b of the code is a factor.
template <int BITS> constexpr int kMonomials = (1 << BITS) - 1;

// MX: the gradient pass on the matrix cores (at most 16 levels, B >= 32, GQ <= 4).
// DX: the dot pass, too (at most 8 levels, GQ <= 2, 32 <= B <= 512, and the lanes' offsets in copy 2 within 32 bits).
// SPLIT: two exchange words for a sample (asked of the host at run time it cost the launches of few workgroups 3 %).
// OWNERS: so many waves own the features of a workgroup: 1 (at most 64 features, no barrier before a norm), 2 (128 features),
// 0: not known here.  (Us per step, asked at run time | known: 128 samples x 3,000 features, 4 bits 7.79 | 7.38, 64 x 4,000, 3
// bits 7.10 | 6.64, 512 x 4,096, 3 bits 7.79 | 7.66.)
template <int BITS, int UPT, bool MX, bool DX, bool SPLIT, int OWNERS>
__device__ __forceinline__ void sgd_steps_e2e(const SgdArgs &a, const Lds &L)
{
    constexpr int K = 1 << BITS;
    constexpr bool kTable = BITS <= 4 && !DX;        // T[j][c] = G[j][c] * m_j kept in LDS
    const int tid = threadIdx.x;
    const int lane = tid & (kWave - 1), wave = tid >> 6;
    const int w = blockIdx.x;
    const int W = a.W, GQ = OWNERS == 2 ? 4 : a.GQ, CW = 32 * GQ, B = a.B;
    const int nrg = B >= 32 ? B / 32 : 1;
    const int j0 = w * CW;
    const int ngroups = (a.d32 - w * GQ) < GQ ? (a.d32 - w * GQ) : GQ;
    const float *Lg = a.levels + (size_t)j0 * K;
    float *const xs = L.xs, *const rs = L.rs;
    double *const red = L.red;
    double *const gpart = reinterpret_cast<double *>(L.gpart);
    int *const tq = L.tq;
    const bool is_owner = tid < CW;                  // this thread owns feature j0 + tid
    const int owner_waves = OWNERS ? OWNERS : (CW + kWave - 1) / kWave;
    const bool owner_wave = wave < owner_waves;
    const int jme = j0 + tid;
    const bool live = is_owner && jme < a.d;
    const int s_m = (1 << (a.model_bits - 1)) - 1;
    const int s_g = a.grad_bits > 0 ? (1 << (a.grad_bits - 1)) - 1 : 1;
    const int nq = (W + kWave - 1) / kWave;          // norm slots per lane (W <= 256: at most 4)
    // exchange words of a sample: one, or two of them, apart by `sub`, and the workgroups in turn add to either
    constexpr int split = SPLIT ? 2 : 1;
    const int sub = a.acc_words / split, mine_at = (w % split) * sub;
    // The sum of the model's codes: one word behind the samples', or among many workgroups one for each of the waves that ask
    // for it, apart (one for all would be asked for eight times as often as any other).
    constexpr int apart = SPLIT ? 8 : 0;

    // ---- the units this thread owns, the same in every step (as in sgd_steps)
    int d_i[UPT], d_g[UPT];
#pragma unroll
    for (int k = 0; k < UPT; ++k) {
        int i = tid + k * kThreads, g = 0;
        while (i >= B && g < GQ) { i -= B; ++g; }
        d_i[k] = i;
        d_g[k] = g;
    }
    // all units of a thread belong to one sample (B == kThreads): their sums meet in a register
    bool one_sample = B == kThreads && ngroups <= UPT;
    const int nsl = kThreads / CW;
    const int g_c = tid % CW, g_sl = tid / CW;
    const int g_gq = g_c >> 5, g_cin = g_c & 31;
    const bool g_live = g_gq < ngroups;

    // ---- matrix-core gradient pass: the feature tiles of 16 are shared out over the waves, waves that share a
    // tile take every KSS-th block of 64 samples.  A lane's operand m: half a packed unit.
    constexpr int HW = kOpDwords<BITS>;
    constexpr int kOps = 2 * UPT;                    // (B GQ <= 512 UPT: at most this many blocks per wave)
    constexpr int kPlaneWords = (K + 3) / 4;         // registers that hold one byte of all levels
    const int n16 = lane & 15, q4 = lane >> 4;
    const int FT = MX ? 2 * GQ : 8, KSS = kWaves / FT, wave_u = __builtin_amdgcn_readfirstlane(wave);
    const int x_ft = wave_u % FT, x_kh = wave_u / FT;
    const int xc = 16 * x_ft + n16;                  // this lane's feature, inside the workgroup
    int8_t *const rdig = reinterpret_cast<int8_t *>(gpart + 2 * kWaves * 16);   // [blocks][8][64], behind the waves' sums
    uint32_t *const wmax = reinterpret_cast<uint32_t *>(L.wsum + kWaves);
    uint32_t plane[MX ? kDigits : 1][MX ? kPlaneWords : 1];
    int r_pos = 0, el_own = 1, lowest = kDigits - 2;     // lowest: the lowest pair of bytes that is looked at
    if constexpr (MX) {
        auto level_exponent = [&](int c) {
            uint32_t m = 0;
            for (int q = 0; q < K; ++q) {
                const uint32_t b = j0 + c < a.d ? __float_as_uint(Lg[(size_t)c * K + q]) & 0x7FFFFFFFu : 0u;
                m = b > m ? b : m;
            }
            return (int)(m >> 23) > 1 ? (int)(m >> 23) : 1;
        };
        if (is_owner) el_own = level_exponent(tid);
        const int el = level_exponent(xc);
#pragma unroll
        for (int p = 0; p < kDigits; ++p)
#pragma unroll
            for (int q = 0; q < kPlaneWords; ++q) plane[p][q] = 0u;
#pragma unroll
        for (int c = 0; c < K; ++c) {
            const float lv = j0 + xc < a.d ? Lg[(size_t)xc * K + c] : 0.0f;
            const uint64_t dg = signed_digits_64<kDigits>(fixed_from_float(lv, el, kTop));
#pragma unroll
            for (int p = 0; p < kDigits; ++p) plane[p][c >> 2] |= (uint32_t)((dg >> (8 * p)) & 0xFFu) << (8 * (c & 3));
        }
#pragma unroll
        for (int p = kDigits - 4; p >= 0; p -= 2)
#pragma unroll
            for (int q = 0; q < kPlaneWords; ++q)
                if (__any((plane[p][q] | plane[p + 1][q]) != 0u)) lowest = p;
        lowest = __builtin_amdgcn_readfirstlane(lowest);
        // sample i: block i / 64, and this byte of each of its digit rows (i = tid + 512 q: the same for every q)
        int half, byte;
        code_slot<BITS>(tid & 31, half, byte);
        r_pos = (tid >> 6) * 512 + (2 * ((tid >> 5) & 1) + half) * 16 + byte;
        for (int e = tid; e < (B + 63) / 64 * 128; e += kThreads) reinterpret_cast<uint32_t *>(rdig)[e] = 0u;
        if (tid < kWaves) wmax[tid] = 0u;
        // (the exchange of the first step has barriers enough before they are used)
    }
    auto load_grad_ops = [&](int64_t t, uint32_t (&dst)[kOps][HW]) {
        const int64_t g = (int64_t)w * GQ + (x_ft >> 1), rg0 = t * B / 32;
#pragma unroll
        for (int m = 0; m < kOps; ++m) {
            const int rg = 2 * (x_kh + KSS * m) + (q4 >> 1);
            if (rg < nrg && (x_ft >> 1) < ngroups) {
                const uint32_t *q = static_cast<const uint32_t *>(__builtin_assume_aligned(
                    a.p1 + ((g * a.n32 + rg0 + rg) * 32 + (xc & 31)) * BITS + (q4 & 1) * kOpStride<BITS>, kOpAlign<BITS>));
#pragma unroll
                for (int k = 0; k < HW; ++k) dst[m][k] = q[k];
            }
        }
    };

    // ---- matrix-core dot pass: a wave takes a block of 64 samples (zipml_sgd_wave.h: how the operands are loaded, and which
    // sample and feature a lane looks after)
    constexpr int NL = kWaveLoads<BITS>, LW = kWaveDwords<BITS>, kSets = DX ? kMonomials<BITS> : 1;
    const int own = wave_element<BITS>(q4, n16);
    int8_t *const mdig = reinterpret_cast<int8_t *>(tq);           // [kSets][4 digits][64 features]
    uint32_t at2[NL], codes2[NL][LW];
    v4i bits2[4][DX ? BITS : 1];                       // a bit of the codes each, in a byte
    int coef[kSets], coef0 = 0;                        // of the grid indices of feature `own`, as a polynomial of the bits
    __amdgpu_buffer_rsrc_t src2;
    if constexpr (DX) {
        const uint32_t group_bytes = (uint32_t)(a.nb64 * 64 * 4 * BITS);
        src2 = __builtin_amdgcn_make_buffer_rsrc((unsigned char *)a.p2 + (int64_t)w * GQ * group_bytes, 0, (int)0xE0000000u, 0x00020000);
#pragma unroll
        for (int l = 0; l < NL; ++l) {
            const int row = wave_load_row<BITS>(q4, n16, l), s = 2 * wave + (row >> 5);
            at2[l] = (q4 >> 1) < ngroups && s < nrg ? (uint32_t)(q4 >> 1) * group_bytes + (uint32_t)((s * 32 + (row & 31)) * 4 * BITS) : 0xF0000000u;
        }
        auto grid = [&](int c) { return own >= CW || j0 + own >= a.d ? 0 : a.ident_grid ? c : (int)a.grid[(size_t)(j0 + own) * K + c]; };
        coef0 = grid(0);
#pragma unroll
        for (int set = 1; set < K; ++set) {
            int v = 0;                                 // sum over the subsets, signs by how many bits are left out
#pragma unroll
            for (int c = 0; c < K; ++c)
                if ((c & set) == c) v += __builtin_popcount(set ^ c) & 1 ? -grid(c) : grid(c);
            coef[set - 1] = v;
        }
    }
    auto load_dot_codes = [&](int64_t t) __attribute__((always_inline)) {
        const uint32_t step = (uint32_t)(t * B) * (4 * BITS);
#pragma unroll
        for (int l = 0; l < NL; ++l) buffer_fetch<LW>(src2, at2[l], step, codes2[l]);
    };
    auto expand_dot_codes = [&]() __attribute__((always_inline)) {
        if constexpr (DX) {
            v4i e[4];
            wave_operands<BITS>(codes2, op_shift<BITS>(q4 & 1), e);
#pragma unroll
            for (int s = 0; s < 4; ++s)
#pragma unroll
                for (int b = 0; b < BITS; ++b) {
#pragma unroll
                    for (int q = 0; q < 4; ++q) bits2[s][b][q] = (int)(((uint32_t)e[s][q] >> b) & 0x01010101u);
                    asm volatile("" : "+v"(bits2[s][b]));
                }
        }
    };

    auto load_dot_units = [&](int64_t t, uint32_t (&dst)[UPT][BITS]) {
        const int64_t row0 = t * B;
#pragma unroll
        for (int k = 0; k < UPT; ++k) {
            if (d_g[k] < ngroups) {
                const int64_t row = row0 + d_i[k];
                const int64_t g = (int64_t)w * GQ + d_g[k];
                load_unit<BITS>(a.p2 + (g * a.nb64 * 64 + row) * BITS, dst[k]);
            }
        }
    };
    auto load_grad_units = [&](int64_t t, uint32_t (&dst)[UPT][BITS]) {
        const int64_t rg0 = (t * B) / 32;
#pragma unroll
        for (int k = 0; k < UPT; ++k) {
            const int rgl = g_sl + k * nsl;
            if (g_live && rgl < nrg) {
                const int64_t g = (int64_t)w * GQ + g_gq;
                load_unit<BITS>(a.p1 + ((g * a.n32 + rg0 + rgl) * 32 + g_cin) * BITS, dst[k]);
            }
        }
    };
    auto load_labels = [&](int64_t t, float (&dst)[UPT]) {
#pragma unroll
        for (int k = 0; k < UPT; ++k) {
            const int i = tid + k * kThreads;
            if (i < B) dst[k] = a.b[t * B + i];
        }
    };

    bool dead = false;
    FirstPoll first_poll, first_norm[2];
    // (Without a barrier in front of its slot the owner is sooner on its way, and the other waves sooner at what stands in the
    // way of its polls.  Us per step with it | without: 4 bits, 96 samples x 294 6.98 | 6.79, 192 x 376 7.21 | 6.96; look-ups,
    // 2 bits, 256 x 244 6.90 | 7.03, 5 bits, 160 x 179 8.13 | 8.23.)
    // One trip of the norm exchange.  sq: this thread's square (owners; 0 elsewhere), fp64.
    // Returns the l2 norm over all workgroups as fp32, to the owner waves (others get 0).
    // meanwhile(): work of the owner waves that does not need the norm, done while it travels.
    auto exchange_norm = [&](double sq, uint64_t *slots, FirstPoll &first, auto meanwhile) -> float {
        // (one owner wave needs nobody: the barriers of a step are enough for what else it shares)
        if constexpr (OWNERS == 1) {
            if (owner_wave) {
                sq = wave_tree_sum_f64(sq);
                if (lane == 0) store_dev(slots + norm_slot<DX>(w, W), (uint64_t)((uint64_t)__double_as_longlong(sq) + 1ull));
            }
        } else {
            if (owner_wave) {
                sq = wave_tree_sum_f64(sq);
                if (lane == 0) red[wave] = sq;
            }
            lds_barrier();
            if (tid == 0) {
                // (as one expression the choice is made after four reads: 160 samples x 3,684, 5 bits 7.79 us a step, so 7.60)
                double own = red[0];
                if (owner_waves == 2) own = red[0] + red[1];
                else if (owner_waves == 4) own = (red[0] + red[1]) + (red[2] + red[3]);
                store_dev(slots + norm_slot<DX>(w, W), (uint64_t)((uint64_t)__double_as_longlong(own) + 1ull));
            }
        }
        if (!owner_wave) return 0.0f;
        meanwhile();
        first.wait();
        uint64_t raw[4] = {1ull, 1ull, 1ull, 1ull};   // (bits of 0.0) + 1 for the slots past W
        uint32_t spins = 0;
#pragma unroll 1
        for (;;) {
            bool all = true;
#pragma unroll
            for (int q = 0; q < 4; ++q)
                if (q < nq && lane + kWave * q < W) {
                    raw[q] = load_dev(slots + norm_slot<DX>(lane + kWave * q, W));
                    all = all && raw[q] != 0ull;
                }
            if (__builtin_amdgcn_ballot_w64(!all) == 0ull || dead) break;
            if (++spins > a.spin_limit) {
                store_dev(a.status, (int)ZIPML_ETIMEOUT);
                dead = true;
            }
        }
        first.learn(spins != 0);
        double s[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int q = 0; q < 4; ++q)
            if (q < nq) s[q] = wave_tree_sum_f64(__longlong_as_double((long long)(raw[q] - 1ull)));
        const double S = nq <= 1 ? s[0] : nq == 2 ? s[0] + s[1] : (s[0] + s[1]) + (s[2] + s[3]);
        return (float)sqrt(S);
    };

    const int64_t t_end = a.step0 + a.nsteps;
    uint32_t c2cur[UPT][BITS], c2nxt[UPT][BITS];
    uint32_t c1cur[MX ? kOps : UPT][MX ? HW : BITS], c1nxt[MX ? kOps : UPT][MX ? HW : BITS];
    auto load_grad = [&](int64_t t) {
        if constexpr (MX) load_grad_ops(t, c1nxt);
        else load_grad_units(t, c1nxt);
    };
    if constexpr (MX) {
        // (operands that are never loaded meet residual digits that are zero, or features that do not exist)
#pragma unroll
        for (int m = 0; m < kOps; ++m)
#pragma unroll
            for (int k = 0; k < HW; ++k) c1nxt[m][k] = 0u;
    }
    float bnext[UPT], bfut[UPT];
#pragma unroll
    for (int k = 0; k < UPT; ++k) bnext[k] = bfut[k] = 0.0f;
    if constexpr (DX) {
        load_dot_codes(a.step0);
        if (wave_u == 0) {
            expand_dot_codes();
            if (a.step0 + 1 < t_end) load_dot_codes(a.step0 + 1);
        }
    } else {
        load_dot_units(a.step0, c2cur);
        if (a.step0 + 1 < t_end) load_dot_units(a.step0 + 1, c2nxt);
    }
    load_grad(a.step0);
    load_labels(a.step0, bnext);

    float x_own = is_owner ? xs[tid] : 0.0f;         // the owner keeps its weight in a register
    uint64_t *const slot_base = reinterpret_cast<uint64_t *>(a.nrm);

#ifdef ZIPML_PHASE_TIMING
    long long prof_[12] = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
    long long last_ = wall_clock64();
#endif
    for (int64_t t = a.step0; t < t_end; ++t) {
        uint64_t *const acc = a.acc + (size_t)(t & 3) * a.acc_words;
        uint64_t *const xn = slot_base + (size_t)(t & 3) * kNormSlots;
        uint64_t *const gn = slot_base + (size_t)(4 + (t & 3)) * kNormSlots;
        const int k0 = B >= 32 ? 0 : (int)((t * B) % 32);

        // ================= ||x||_2, Q3, the table of the dot pass
        // (the draws of Q3 and Q4 do not depend on the norms: they are made while those travel, 0.2 us each)
        float draw = 0.0f;
        auto draw_for = [&](uint32_t stream) {
            return [&, stream]() {
                const Philox4 r = philox_block(a.seed, a.epoch, (uint64_t)t, (uint32_t)jme >> 2, stream);
                draw = u24(philox_word(r, (uint32_t)jme & 3u));
                asm volatile("" : "+v"(draw));       // (here, not where it is used)
            };
        };
        const float Mx = exchange_norm(live ? (double)x_own * (double)x_own : 0.0, xn, first_norm[0], draw_for(3u));
        ZIPML_TICK(0);
        if constexpr (DX) {
            if (wave_u != 0) expand_dot_codes();
        }
        const float sigma = Mx > 0.0f ? __fdiv_rn(Mx, (float)s_m) : 0.0f;
        if (owner_wave) {
            int mine = 0;
            if (live) {
                mine = qvec_code(x_own, Mx, s_m, draw);
                if (a.dbg_m) a.dbg_m[jme] = mine;
            }
            if (is_owner) {
                L.ms[tid] = mine;
                if constexpr (kTable) {
#pragma unroll
                    for (int c = 0; c < K; ++c)
                        tq[tid * K + c] = (a.ident_grid ? c : (int)L.Gs[tid * K + c]) * mine;
                }
            }
            if constexpr (DX) {
                // what multiplies a monomial: an integer below 2^25 in magnitude, in four digits
                const int m = __shfl(mine, own, kWave);
                const QuadStore quad(lane);
                int8_t *const at = mdig + wave_digits_at<BITS>(q4, n16);
#pragma unroll
                for (int k = 0; k < kSets; ++k) *reinterpret_cast<uint32_t *>(at + 256 * k) = quad.transpose(signed_digits(coef[k] * m));
                const int low = wave_sum_dpp(coef0 * m);
                if (lane == 0) L.isum[1] = low;
            }
            const int part = wave_sum_dpp(mine);
            if (lane == 0) L.isum[wave] = part;
            if (tid == 0) L.wsum[0] = sigma;          // for the threads outside the owner waves
        }
        lds_barrier();      // ms / tq / isum / sigma
        const float sigma_b = L.wsum[0];
        ZIPML_TICK(1);
        if (tid == 0 || (SPLIT && tid < kWaves && tid * kWave < B)) {
            int tot = 0;
            for (int q = 0; q < owner_waves; ++q) tot += L.isum[q];
            add_dev(acc + mine_at + xword(B + apart * tid, a.acc_sh), pack_int(tot));
        }

        // ================= dot pass: acc_i = sum_j G[j][c2_ij] m_j over the owned features
        if constexpr (DX) {
            const int low = L.isum[1];
            v4i md[kSets];
#pragma unroll
            for (int k = 0; k < kSets; ++k) md[k] = *reinterpret_cast<const v4i *>(mdig + 256 * k + (n16 & 3) * 64 + q4 * 16);
            const int i = 64 * wave + own;
            if (64 * wave_u < B) {
                v4i c[4];
#pragma unroll
                for (int s = 0; s < 4; ++s) {
                    c[s] = v4i{0, 0, 0, 0};
#pragma unroll
                    for (int set = 1; set < K; ++set) {
                        v4i e = {-1, -1, -1, -1};
#pragma unroll
                        for (int b = 0; b < BITS; ++b)
                            if (set >> b & 1) e &= bits2[s][b];
                        c[s] = __builtin_amdgcn_mfma_i32_16x16x64_i8(md[set - 1], e, c[s], 0, 0, 0);
                    }
                }
                int sum[2];
                pick_tile(c, q4, sum);
                if (i < B) add_dev(acc + mine_at + xword(i, a.acc_sh), pack_int((long long)sum[0] + ((long long)sum[1] << 16) + low));
            }
        } else {
            int pi[UPT];
#pragma unroll
            for (int k = 0; k < UPT; ++k) {
                pi[k] = 0;
                if (d_g[k] < ngroups) {
                    const int jb = d_g[k] * 32;
                    if constexpr (kTable) {
                        // (all lanes look up the same feature q at a time: K neighbouring words)
                        const int *T = tq + jb * K;
#pragma unroll
                        for (int q = 0; q < 32; ++q) {
                            pi[k] += T[q * K + (int)unit_code<BITS>(c2cur[k], q)];
                            if ((q & 15) == 15) asm volatile("" ::: "memory");   // sixteen look-ups in flight
                        }
                    } else {
                        pi[k] = unit_dot_int<BITS>(c2cur[k], a.ident_grid ? nullptr : L.Gs + jb * K, L.ms + jb, 0);
                    }
                }
            }
            if (one_sample) {
                int tot = 0;
#pragma unroll
                for (int k = 0; k < UPT; ++k) tot += pi[k];
                add_dev(acc + mine_at + xword(tid, a.acc_sh), pack_int(tot));
            } else if (ngroups > 1) {
#pragma unroll
                for (int k = 0; k < UPT; ++k)
                    if (d_g[k] < ngroups) L.zp[d_g[k] * B + d_i[k]] = (uint32_t)pi[k];
                lds_barrier();
                for (int i = tid; i < B; i += kThreads) {
                    int tot = 0;
                    for (int gq = 0; gq < ngroups; ++gq) tot += (int)L.zp[gq * B + i];
                    add_dev(acc + mine_at + xword(i, a.acc_sh), pack_int(tot));
                }
            } else {
#pragma unroll
                for (int k = 0; k < UPT; ++k)
                    if (d_g[k] < ngroups) add_dev(acc + mine_at + xword(d_i[k], a.acc_sh), pack_int(pi[k]));
            }
        }
        ZIPML_TICK(2);
        // The last wave of every workgroup clears its share of the exchange words, and its own norm
        // slots, of step t+2 (four buffers in rotation).  The workgroup is past the ||x|| exchange of
        // step t, so every workgroup has finished step t-1 and with it every read of step t-2, the
        // last user of these buffers; the stores are complete before this wave's poll below returns
        // (a wave's memory operations complete in order), hence before the workgroup contributes to
        // any later exchange, and nobody reaches step t+2 without those contributions.
        if (wave == kWaves - 1) {
            uint64_t *nxt = a.acc + (size_t)((t + 2) & 3) * a.acc_words;
            const int words = B + 1 + (kWaves - 1) * apart, per = (words + W - 1) / W, hi = (w + 1) * per < words ? (w + 1) * per : words;
            for (int i = w * per + lane; i < hi; i += kWave) {
                store_dev(nxt + xword(i, a.acc_sh), (uint64_t)0);
                if (split > 1) store_dev(nxt + sub + xword(i, a.acc_sh), (uint64_t)0);
            }
            if (lane == 0) {
                store_dev(slot_base + (size_t)((t + 2) & 3) * kNormSlots + norm_slot<DX>(w, W), (uint64_t)0);
                store_dev(slot_base + (size_t)(4 + ((t + 2) & 3)) * kNormSlots + norm_slot<DX>(w, W), (uint64_t)0);
            }
            if (!(tid < B)) vm_wait_all();
        }
        // rotate the register sets; request what later steps need right behind the atomics
#pragma unroll
        for (int k = 0; k < (MX ? kOps : UPT); ++k)
#pragma unroll
            for (int q = 0; q < (MX ? HW : BITS); ++q) c1cur[k][q] = c1nxt[k][q];
        if constexpr (!DX) {
#pragma unroll
            for (int k = 0; k < UPT; ++k)
#pragma unroll
                for (int q = 0; q < BITS; ++q) c2cur[k][q] = c2nxt[k][q];
        }
        if (t + 1 < t_end) {
            load_grad(t + 1);
            load_labels(t + 1, bfut);
        }
        if constexpr (DX) {
            // the wave that owns the features expands the codes of the next step here, requested in the last one; the others
            // have time when it waits for the norm of the model
            if (wave_u == 0) {
                expand_dot_codes();
                if (t + 2 < t_end) load_dot_codes(t + 2);
            } else if (t + 1 < t_end) {
                load_dot_codes(t + 1);
            }
        } else {
            if (t + 2 < t_end) load_dot_units(t + 2, c2nxt);
        }
        ZIPML_TICK(3);

        // ================= residuals: every thread polls the words of its own samples
        float rown[UPT];
#pragma unroll
        for (int q = 0; q < UPT; ++q) rown[q] = 0.0f;
        if (tid < B) {
            uint64_t raw[UPT], rawm = 0;
            uint32_t spins = 0;
            first_poll.wait();
#pragma unroll 1
            for (;;) {
#pragma unroll
                for (int q = 0; q < UPT; ++q) {
                    const int i = tid + q * kThreads;
                    raw[q] = load_dev(acc + xword(i < B ? i : B - 1, a.acc_sh));
                }
                rawm = load_dev(acc + xword(B + apart * wave_u, a.acc_sh));
                if (split > 1) {
                    uint64_t second[UPT];
#pragma unroll
                    for (int q = 0; q < UPT; ++q) {
                        const int i = tid + q * kThreads;
                        second[q] = load_dev(acc + sub + xword(i < B ? i : B - 1, a.acc_sh));
                    }
                    rawm += load_dev(acc + sub + xword(B + apart * wave_u, a.acc_sh));
#pragma unroll
                    for (int q = 0; q < UPT; ++q) raw[q] += second[q];
                }
                bool all = (int)(rawm >> kCountShift) == W;
#pragma unroll
                for (int q = 0; q < UPT; ++q) all = all && (int)(raw[q] >> kCountShift) == W;
                if (all || dead) break;
                if (++spins > a.spin_limit) {
                    store_dev(a.status, (int)ZIPML_ETIMEOUT);
                    dead = true;
                }
            }
            first_poll.learn(__builtin_amdgcn_ballot_w64(spins != 0) != 0);
            ZIPML_TICK(8);
            const double summ = (double)unpack_sum(rawm, W);
#pragma unroll
            for (int q = 0; q < UPT; ++q) {
                const int i = tid + q * kThreads;
                if (i < B) {
                    const int av = (int)unpack_sum(raw[q], W);
                    const double z = (double)sigma_b * ((double)a.grid_lo * summ + (double)a.grid_step * (double)av);
                    const float r = (float)z - bnext[q];
                    if constexpr (MX) rown[q] = r;
                    else rs[k0 + i] = r;
                    if (w == 0) {
                        if (a.dbg_acc) a.dbg_acc[i] = av;
                        if (a.dbg_r) a.dbg_r[i] = r;
                    }
                }
            }
        }
#pragma unroll
        for (int q = 0; q < UPT; ++q) bnext[q] = bfut[q];
        if constexpr (MX) {
            // the largest residual gives the unit of all, then each becomes digits
            uint32_t m = 0;
#pragma unroll
            for (int q = 0; q < UPT; ++q) {
                const uint32_t b = __float_as_uint(rown[q]) & 0x7FFFFFFFu;
                m = b > m ? b : m;
            }
            m = wave_reduce_dpp(m, [](uint32_t p, uint32_t q) { return p > q ? p : q; });
            if (lane == 0) wmax[wave] = m;
        }
        ZIPML_TICK(9);
        lds_barrier();    // rs[], or the waves' largest residuals
        ZIPML_TICK(10);
        int er = 1;
        if constexpr (MX) {
            uint32_t m = 0;
#pragma unroll
            for (int q = 0; q < kWaves; ++q) m = wmax[q] > m ? wmax[q] : m;
            er = (int)(m >> 23) > 1 ? (int)(m >> 23) : 1;
#pragma unroll
            for (int q = 0; q < UPT; ++q)
                if (tid + q * kThreads < B) {
                    const uint64_t dg = signed_digits_64<kDigits>(fixed_from_float(rown[q], er, kTop));
                    int8_t *at = rdig + q * (kThreads / 64 * 512) + r_pos;
#pragma unroll
                    for (int k = 0; k < kDigits; ++k) at[64 * k] = (int8_t)(dg >> (8 * k));
                }
            lds_barrier();    // the digits
        }
        ZIPML_TICK(4);

        // ================= gradient pass
        if constexpr (MX) {
            v4i c[kDigits];
#pragma unroll
            for (int p = 0; p < kDigits; ++p) c[p] = v4i{0, 0, 0, 0};
            const uint32_t shift = op_shift<BITS>(q4 & 1);
#pragma unroll
            for (int m = 0; m < kOps; ++m) {
                const int sb = x_kh + KSS * m;
                if (2 * sb < nrg) {
                    // (rows 8 .. 15 repeat the others: their results are not used)
                    const v4i rd = *reinterpret_cast<const v4i *>(rdig + sb * 512 + (n16 & 7) * 64 + q4 * 16);
                    v4i e = expand_codes<BITS>(c1cur[m], shift), up = {0, 0, 0, 0};
                    if constexpr (K == 16) {
#pragma unroll
                        for (int q = 0; q < 4; ++q) {
                            const uint32_t top = ((uint32_t)e[q] >> 3) & 0x01010101u;
                            up[q] = (int)((top << 8) - top);          // 0xFF where the code is 8 or more
                            e[q] &= 0x07070707;
                        }
                    }
#pragma unroll
                    for (int p0 = kDigits - 2; p0 >= 0; p0 -= 2)
                        if (p0 >= lowest) {
#pragma unroll
                            for (int p = p0; p < p0 + 2; ++p) {
                                v4i lv;
#pragma unroll
                                for (int q = 0; q < 4; ++q) {
                                    uint32_t v = __builtin_amdgcn_perm(plane[p][K >= 8 ? 1 : 0], plane[p][0], (uint32_t)e[q]);
                                    if constexpr (K == 16) {
                                        const uint32_t h = __builtin_amdgcn_perm(plane[p][3], plane[p][2], (uint32_t)e[q]);
                                        v = ((uint32_t)up[q] & h) | (~(uint32_t)up[q] & v);
                                    }
                                    lv[q] = (int)v;
                                }
                                c[p] = __builtin_amdgcn_mfma_i32_16x16x64_i8(rd, lv, c[p], 0, 0, 0);
                            }
                        }
                }
            }
            // Rows 0 .. 3 are in the first sixteen lanes, rows 4 .. 7 in the next.  Sums of equal weight first: each
            // below 2^26, so that four of them join exactly in a double.
            if (q4 < 2) {
                int v[kDigits + 4];
#pragma unroll
                for (int s = 0; s < kDigits + 4; ++s) v[s] = 0;
#pragma unroll
                for (int p = 0; p < kDigits; ++p)
#pragma unroll
                    for (int s = 0; s < 4; ++s) v[p + s] += c[p][s];
                auto four = [&](int s) {
                    return fma(fma((double)v[s + 3], 256.0, (double)v[s + 2]), 65536.0, fma((double)v[s + 1], 256.0, (double)v[s]));
                };
                const double sum = fma(fma(four(8), 4294967296.0, four(4)), 4294967296.0, four(0));
                gpart[(2 * x_kh + q4) * CW + xc] = sum * (q4 ? 4294967296.0 : 1.0);
            }
        } else {
            double part[UPT];
#pragma unroll
            for (int k = 0; k < UPT; ++k) {
                part[k] = 0.0;
                const int rgl = g_sl + k * nsl;
                if (g_live && rgl < nrg) {
                    // (rows of the LDS copy are K + 1 apart: lanes hold different features, and
                    // rows K apart would put all their look-ups on a few banks)
                    // (two loops: one pointer that may be LDS or global memory would be a generic one)
                    const float *rr = rs + rgl * 32;
                    double acc = 0.0;
                    if (a.lds_levels) {
                        const float *Lj = L.Lp + g_c * (K + 1);
#pragma unroll
                        for (int q = 0; q < 32; ++q) {
                            acc = fma((double)Lj[unit_code<BITS>(c1cur[k], q)], (double)rr[q], acc);
                            if ((q & 15) == 15) asm volatile("" ::: "memory");   // sixteen look-ups in flight
                        }
                    } else {
                        // (no rows for padding features in memory; their sums are dropped)
                        acc = unit_grad_table_f64<BITS>(c1cur[k], Lg + (size_t)(j0 + g_c < a.d ? g_c : a.d - 1 - j0) * K, rr);
                    }
                    part[k] = acc;
                }
            }
#pragma unroll
            for (int k = 0; k < UPT; ++k) {
                const int rgl = g_sl + k * nsl;
                if (rgl < nrg) gpart[rgl * CW + g_c] = part[k];
            }
        }
        lds_barrier();    // gpart[]
        ZIPML_TICK(5);
        float g = 0.0f;
        if (is_owner) {
            double sacc = 0.0;
            const int nparts = MX ? 2 * KSS : nrg;
            for (int r0 = 0; r0 < nparts; r0 += 8) {
                double v[8];
#pragma unroll
                for (int q = 0; q < 8; ++q) v[q] = gpart[(r0 + q < nparts ? r0 + q : r0) * CW + tid];
#pragma unroll
                for (int q = 0; q < 8; ++q)
                    if (r0 + q < nparts) sacc += v[q];
            }
            if constexpr (MX) {
                sacc = ldexp(sacc, er + el_own - (300 + 2 * kTop));
                if (er == 255) sacc = __longlong_as_double(0x7FF8000000000000ll);    // an infinity or a NaN among the residuals
            }
            g = live ? (float)(sacc / (double)B) : 0.0f;      // the mean, rounded once
            if (a.dbg_g && live) a.dbg_g[jme] = g;
        }
        if (B < 32) {
            // a short batch shares its sample group with its neighbours: clear its residuals
            // (every read of rs[] is behind the barrier above; the next write is barriers away)
            for (int i = tid; i < B; i += kThreads) rs[k0 + i] = 0.0f;
        }

        ZIPML_TICK(6);
        // ================= ||g||_2, Q4, update
        if (a.grad_bits > 0) {
            const float Mg = exchange_norm(is_owner ? (double)g * (double)g : 0.0, gn, first_norm[1], draw_for(4u));
            const float sg = Mg > 0.0f ? __fdiv_rn(Mg, (float)s_g) : 0.0f;
            if (live) {
                const int code = qvec_code(g, Mg, s_g, draw);
                if (a.dbg_gq) a.dbg_gq[jme] = code;
                const float gh = sg * (float)code;
                const float stp = a.lr * gh;
                x_own = x_own - stp;
            }
        } else if (live) {
            const float stp = a.lr * g;
            x_own = x_own - stp;
        }
        ZIPML_TICK(7);
    }
    if (is_owner) xs[tid] = x_own;
    lds_barrier();
#ifdef ZIPML_PHASE_TIMING
    if (w == 0 && tid == 0)
        for (int k = 0; k < 12; ++k) ((long long *)(a.nrm + 2048))[k] = prof_[k];
#endif
}

}  // namespace zipml
