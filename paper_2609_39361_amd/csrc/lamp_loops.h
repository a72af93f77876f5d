// lamp_loops.h -- the logit loops of the LampAttention forward pass.
//
// Every lane owns QPL query rows; a pass accumulates over the D channels the
// logits of groups of 4 keys, one rank-1 matrix instruction per channel, group
// and row slot: v_mfma_f32_4x4x1_16b_f32 computes 16 blocks of 4 x 4 outer
// products D = A B + C, and with the A operand of one block broadcast to all
// (cbsz 4, the block chosen by abid) its four results are, in every lane, the
// FP32 FMAs fma(k_i, q, c_i) of four keys i with that lane's own query value.
// Each is one fused multiply-add with one rounding, bit for bit v_fma_f32
// (subnormals and signed zeros included), so chained over the channels it is
// the FMA chain of the method's definition.  A wave reads its keys once: lane
// l of a key operand holds key (l mod 16) of channel group (l / 16) of a
// 16-channel block, and abid = 4 * group + g broadcasts keys 4g .. 4g+3.
//
// What bounds it: VALU issue.  The fp32 matrix instructions do not overlap the
// VALU's conversions (neither of their own wave nor of another), but feed the
// keys for free.  Measured in one run, ns per wave and SIMD (they move together
// by some 4 % from run to run): the matrix instruction 3.60, 0.90 per 64
// multiply-adds, against 1.78 for an FMA that reads its key through a DPP
// broadcast and 1.09 for one on plain registers; decoding a code pair 1.96,
// rounding a value pair to e4m3 3.39.  Per 64 multiply-adds the parts of the
// 8-bit step come to 0.90 + (1.96 + 3.39) / 2 = 3.58, and the step takes 3.72:
// nothing overlaps, and the changes between the two kinds cost the rest.  With
// broadcast FMAs the parts come to 4.45.  The 16-bit accumulation takes 0.90.
// (Decoding on the fp8 matrix instructions instead was no faster: 0.93 to 1.01
// of the step's time.)
#pragma once
#include <utility>

#include "lamp_device.h"

namespace lamp {

typedef float f32x4_t __attribute__((ext_vector_type(4)));

// acc + bcast_i(kv) * q with one rounding, key i of each 16-lane row by DPP
// (the stochastic-rounding loop).
template <int I>
__device__ __forceinline__ float fmac_bc(float acc, float kv, float q)
{
    asm("v_fmac_f32_dpp %0, %1, %2 row_newbcast:%3 row_mask:0xf bank_mask:0xf" : "+v"(acc) : "v"(kv), "v"(q), "n"(I));
    return acc;
}

// c_i + k_i * q for the 4 keys i that lanes 4*ABID .. 4*ABID+3 of kv hold.
template <int ABID>
__device__ __forceinline__ f32x4_t rank1(float kv, float q, f32x4_t c)
{
    return __builtin_amdgcn_mfma_f32_4x4x1f32(kv, q, c, 4, ABID, 0);
}

// A key that orders the nonzero magnitudes (zero last): the pattern without its
// sign, doubled, minus one; bits [31:24] are at most the biased exponent.
__device__ __forceinline__ uint32_t min_bits(float x) { return (__builtin_bit_cast(uint32_t, x) << 1) - 1u; }
__device__ __forceinline__ uint32_t min_u32(uint32_t a, uint32_t b) { return a < b ? a : b; }

// Where the loops find the fp32 queries and keys.  Row layout ([row][D]): the
// 4-channel group g of a row is at offset 4g and consecutive keys are D apart.
// Grouped layout (the pipelined kernel): queries in blocks of 64 rows and keys
// in blocks of 16, each block stored [group][row][4], so that one 4-channel
// group of a block is contiguous: group g of a query row is at 256g, of a key
// row at 64g, and consecutive keys of a block are 4 apart.
template <int QS_, int KS_, int KR_>
struct Lay {
    static constexpr int QS = QS_, KS = KS_, KR = KR_;   // query / key group stride, key row stride
};
template <int D>
using RowLay = Lay<4, 4, D>;
using GrpLay = Lay<256, 64, 4>;

// The query rows of a wave: slot s of a lane at base[s] (uniform) + off bytes
// (the lane's own), so that the loads keep one offset register.
// SIM profile only: qmin, min_bits over each row (set_qmin), and whether the
// 8-bit loop has left the range of its fast rounding (uniform).
template <int QPL>
struct QRows {
    const float *base[QPL];
    uint32_t off;
    uint32_t qmin[QPL];
    bool exact;
    __device__ __forceinline__ const float *row(int s) const
    {
        return reinterpret_cast<const float *>(reinterpret_cast<const char *>(base[s]) + off);
    }
};

// A key operand: group 0 of this lane's key at base (uniform) + off bytes; the
// lane reads channel group 4j + lane/16 of every 16-channel block j.
struct KRows {
    const float *base;
    uint32_t off;
};

// The 16 consecutive keys at k32.
template <class LY>
__device__ __forceinline__ KRows keys16(const float *k32)
{
    const uint32_t l = __lane_id();
    return {k32, 4u * ((l & 15u) * LY::KR + (l >> 4) * LY::KS)};
}

// The key at element offset `key_off` of this lane (the caller's choice of
// keys: groups of four in lanes 4g .. 4g+3 of every 16-lane row).
template <class LY>
__device__ __forceinline__ KRows keys_at(const float *k32, uint32_t key_off)
{
    return {k32, 4u * (key_off + (__lane_id() >> 4) * LY::KS)};
}

__device__ __forceinline__ float4 load4(const float *p) { return *reinterpret_cast<const float4 *>(p); }
__device__ __forceinline__ f32x4_t load4v(const float *base, uint32_t off)
{
    return *reinterpret_cast<const f32x4_t *>(reinterpret_cast<const char *>(base) + off);
}
__device__ __forceinline__ float4 load4(const float *base, uint32_t off)
{
    const f32x4_t v = load4v(base, off);
    return make_float4(v.x, v.y, v.z, v.w);
}

// Two wait states that nothing is scheduled across, at the top of every loop
// whose DPP instructions read loaded registers: the register allocator may
// copy such a register with a VALU move where a loop is entered or left, and a
// DPP read of a VGPR needs two wait states after a VALU write of it.  The
// build check verifies the result.
__device__ __forceinline__ void dpp_guard_fenced()
{
    asm volatile("s_nop 1");
    __builtin_amdgcn_sched_barrier(0);
}

// 8-bit logits of 16 keys: e4m3 codes, four per word (word g: keys 4g .. 4g+3),
// or, in the SIM profile, bf16 patterns two per word.
template <bool SIMP>
constexpr int Y8_WORDS = SIMP ? 8 : 4;

// c_g <- fma(k, q, c_g) for NG groups g of 4 keys (channel group R of the key operand).
template <int R, int NG, int... G>
__device__ __forceinline__ void fma_groups(float kv, float q, f32x4_t (&c)[NG], std::integer_sequence<int, G...>)
{
    ((c[G] = rank1<4 * R + G>(kv, q, c[G])), ...);
}

// One channel of the 8-bit accumulation of 16 keys of one query row,
// acc <- RN_e4m3(RN32(q * k + acc)), and of the FMA chains of NM groups of 4
// keys of kr.  In three batches that nothing is scheduled across -- decode the
// four code words, the matrix instructions back to back, round back -- because
// every change between the VALU and the matrix instructions costs some 8
// cycles: alternating them one by one took 1.18 times as long as the batches (all
// eight words of two rows in one batch: the same time, with 16 more registers).
template <int R, bool SAT, int NM>
__device__ __forceinline__ void emu8_row(float ke, float kr, float q, uint32_t (&w)[4], f32x4_t (&acc)[NM > 0 ? NM : 1])
{
    f32x4_t t[4];
#pragma unroll
    for (int g = 0; g < 4; ++g) {
        const float2 lo = unpk_e4m3x4(w[g], 0), hi = unpk_e4m3x4(w[g], 1);
        t[g] = f32x4_t{lo.x, lo.y, hi.x, hi.y};
    }
    __builtin_amdgcn_sched_barrier(0);
    fma_groups<R>(ke, q, t, std::make_integer_sequence<int, 4>());
    if constexpr (NM > 0) fma_groups<R>(kr, q, acc, std::make_integer_sequence<int, NM>());
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int g = 0; g < 4; ++g) {
        if constexpr (SAT) w[g] = pk_e4m3_sat(t[g][0], t[g][1], w[g]);
        else w[g] = pk_e4m3(t[g][0], t[g][1], w[g]);
    }
#pragma unroll
    for (int g = 0; g < 4; ++g) {
        if constexpr (SAT) w[g] = pk_e4m3_sat_hi(t[g][2], t[g][3], w[g]);
        else w[g] = pk_e4m3_hi(t[g][2], t[g][3], w[g]);
    }
    __builtin_amdgcn_sched_barrier(0);
}

// The 8-bit SIM rounding of a value that is 0 or has 2^-126 <= |t| < 2^107, in
// two FMA-class operations instead of three integer ones (the step of one
// multiply-add takes 2.95 ns per 64 and SIMD, 0.90 of it the matrix
// instruction; the integer operations alone took 4.8).  With t = m 2^(e-23) and
// q = 2^(e-3) the quantum to round to, t (2^20 - 1) = (m - m 2^-20) q rounded to FP32 is m - RN(m 2^-20) quanta,
// ties to even since m is even there, and t 2^20 = m q minus it is t rounded
// (Dekker's splitting).  Below 2^23 quanta, m < 2^23 + 8, the product's ulp is
// q/2, but m 2^-20 then lies within 2^-17 of 8 and rounds to it all the same; a
// factor 2^20 + 1 would not do: above 2^24 quanta its ulp is 2q, and an odd m
// rounds to 15 instead of 16.  c1 = -(2^20 - 1), c2 = 2^20.
__device__ __forceinline__ float rn_sim3_normal(float t, float c1, float c2)
{
    const float s = t * c1;
    return __builtin_fmaf(t, c2, s);
}

// The loop over the channels: the 8-bit accumulation of the 16 keys of ke
// (EMU; in the SIM profile on FP32 values in e8, otherwise on the codes w8;
// EXACT: saturating, or in the SIM profile the rounding that holds for every
// FP32 value) and the FMA chains of NM groups of 4 keys of kr, sharing
// the query loads.  The queries come PD 4-channel groups ahead, the keys a
// 16-channel block ahead (the last block's loads wrap to the first channels
// and are not used).
template <int D, int QPL, int NM, bool EMU, bool SIMP, bool EXACT, int PD, class LY>
__device__ __forceinline__ void logit_loop(const QRows<QPL> &qr, const KRows &ke, const KRows &kr,
                                           uint32_t (&w8)[QPL][4], f32x4_t (&e8)[QPL][SIMP && EMU ? 4 : 1],
                                           f32x4_t (&acc)[QPL][NM > 0 ? NM : 1], uint32_t &kmin)
{
    static_assert(D % 16 == 0 && (PD == 2 || PD == 4), "16-channel blocks");
    f32x4_t q4[PD][QPL], kea, keb, kra, krb;
    uint32_t qoff = qr.off, eoff = ke.off, roff = kr.off;
    auto ldk = [&](int c, f32x4_t &e, f32x4_t &r) {
        if constexpr (EMU) e = load4v(ke.base + (c / 4) * LY::KS, eoff);
        if constexpr (NM > 0) r = load4v(kr.base + (c / 4) * LY::KS, roff);
    };
    auto ldq = [&](int g, f32x4_t (&q)[QPL]) {
#pragma unroll
        for (int s = 0; s < QPL; ++s) q[s] = load4v(qr.base[s] + g * LY::QS, qoff);
    };
    float c1 = -1048575.0f, c2 = 1048576.0f;   // kept in vector registers (a scalar operand issues slower)
    if constexpr (EMU && SIMP && !EXACT) asm volatile("" : "+v"(c1), "+v"(c2));
    ldk(0, kea, kra);
#pragma unroll
    for (int r = 0; r < PD; ++r) ldq(r, q4[r]);
    auto group = [&](auto r_c, int c, const f32x4_t &e, const f32x4_t &k) {
        constexpr int R = decltype(r_c)::value;
#pragma unroll
        for (int cc = 0; cc < 4; ++cc)
#pragma unroll
            for (int s = 0; s < QPL; ++s) {
                const float q = q4[R % PD][s][cc];
                if constexpr (EMU && !SIMP) {
                    emu8_row<R, EXACT, NM>(e[cc], NM > 0 ? k[cc] : 0.0f, q, w8[s], acc[s]);
                } else {
                    if constexpr (EMU) fma_groups<R>(e[cc], q, e8[s], std::make_integer_sequence<int, 4>());
                    if constexpr (NM > 0) fma_groups<R>(k[cc], q, acc[s], std::make_integer_sequence<int, NM>());
                    if constexpr (EMU) {
                        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                        for (int g = 0; g < 4; ++g)
#pragma unroll
                            for (int i = 0; i < 4; ++i)
                                e8[s][g][i] = EXACT ? rn_sim<3>(e8[s][g][i]) : rn_sim3_normal(e8[s][g][i], c1, c2);
                        __builtin_amdgcn_sched_barrier(0);
                    }
                }
            }
        const int g = c / 4 + R + PD;
        ldq(g < D / 4 ? g : g - D / 4, q4[R % PD]);
    };
#pragma nounroll
    for (int c = 0; c < D; c += 16) {
        // opaque to the compiler, so that the loads keep the form of a scalar
        // base plus a 32-bit lane offset
        asm volatile("" : "+v"(qoff), "+v"(eoff), "+v"(roff));
        ldk(c + 16 < D ? c + 16 : 0, keb, krb);
        if constexpr (EMU && SIMP && !EXACT) {
#pragma unroll
            for (int i = 0; i < 4; ++i) kmin = min_u32(kmin, min_bits(kea[i]));
        }
        group(std::integral_constant<int, 0>(), c, kea, kra);
        group(std::integral_constant<int, 1>(), c, kea, kra);
        group(std::integral_constant<int, 2>(), c, kea, kra);
        group(std::integral_constant<int, 3>(), c, kea, kra);
        if constexpr (EMU) kea = keb;
        if constexpr (NM > 0) kra = krb;
    }
}

// Y8 of one 16-key chunk for QPL query rows of this lane (Sec. 4.1:
// acc <- RN_e4m3(RN32(q_tilde * k + acc)), channels ascending, from +0).
template <int D, int QPL, bool SAT, class LY = RowLay<D>>
__device__ __forceinline__ void emu8_pass(const QRows<QPL> &qr, const KRows &ke, uint32_t (&w)[QPL][4])
{
    f32x4_t none[QPL][1];
#pragma unroll
    for (int s = 0; s < QPL; ++s)
#pragma unroll
        for (int g = 0; g < 4; ++g) w[s][g] = 0u;
    uint32_t kmin;
    logit_loop<D, QPL, 0, true, false, SAT, 2, LY>(qr, ke, ke, w, none, none, kmin);
}

// Nonzero iff one of the four codes of a word is a NaN code (bits 7, 15, 23, 31).
__device__ __forceinline__ uint32_t e4m3x4_nan_bits(uint32_t w) { return ((w & 0x7F7F7F7Fu) + 0x01010101u) & 0x80808080u; }

// Keys whose 8-bit code is a NaN after the non-saturating pass, one bit per
// key (bit i: key i of the 16).  Such a chain overflowed in some step, which
// is exactly when the saturating recursion clamps to +-448: the two recursions
// agree up to that step.
template <int QPL>
__device__ __forceinline__ void nan_keys(const uint32_t (&w)[QPL][4], uint32_t (&sat)[QPL])
{
#pragma unroll
    for (int s = 0; s < QPL; ++s) {
        uint32_t m = 0;
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            const uint32_t r = e4m3x4_nan_bits(w[s][g]);
#pragma unroll
            for (int i = 0; i < 4; ++i) m |= ((r >> (8 * i + 7)) & 1u) << (4 * g + i);
        }
        sat[s] = m;
    }
}

// After the non-saturating pass: if any lane of the wave overflowed somewhere
// (a NaN code at the end of a chain), the chunk is recomputed with the
// saturating conversion.  sat[s] receives the keys of slot s whose
// accumulation saturated (nan_keys), 0 when none did.
template <int D, int QPL, class LY>
__device__ __forceinline__ void emu8_check(const QRows<QPL> &qr, const KRows &ke, uint32_t (&w)[QPL][4],
                                           uint32_t (&sat)[QPL])
{
    uint32_t nan = 0;
#pragma unroll
    for (int s = 0; s < QPL; ++s) {
        sat[s] = 0u;
#pragma unroll
        for (int g = 0; g < 4; ++g) nan |= e4m3x4_nan_bits(w[s][g]);
    }
    if (wave_any(nan != 0)) {
        nan_keys<QPL>(w, sat);
        emu8_pass<D, QPL, true, LY>(qr, ke, w);
    }
}

// ---- the SIM profile (Sec. 4.1): FP32 range, 3 / 11 mantissa bits, no saturation
// Smallest nonzero magnitudes of a lane's query rows.
template <int D, int QPL, class LY>
__device__ __forceinline__ void set_qmin(QRows<QPL> &qr)
{
#pragma unroll
    for (int s = 0; s < QPL; ++s) {
        uint32_t m = 0xFFFFFFFFu;
        for (int g = 0; g < D / 4; ++g) {
            const f32x4_t v = load4v(qr.base[s] + g * LY::QS, qr.off);
#pragma unroll
            for (int i = 0; i < 4; ++i) m = min_u32(m, min_bits(v[i]));
        }
        qr.qmin[s] = m;
    }
    qr.exact = false;
}

// Whether a pass with rn_sim3_normal rounded some step outside its range (then
// the chunk is recomputed with rn_sim).  Above: an overflow gives an infinity or
// a NaN, which stays to the end of the chain.  Below: every sum and every
// rounded value is a multiple of the product of the smallest quanta of the row
// and the keys, 2^(eq-23) and 2^(ek-7) (bf16 keys), so with eq + ek >= -96 a
// nonzero one is at least 2^-126.
template <int QPL>
__device__ __forceinline__ bool sim8_out_of_range(const QRows<QPL> &qr, uint32_t kmin, const f32x4_t (&e8)[QPL][4])
{
#pragma unroll
    for (int m = 1; m < 64; m <<= 1) kmin = min_u32(kmin, (uint32_t)__shfl_xor((int)kmin, m, 64));
    bool bad = false;
#pragma unroll
    for (int s = 0; s < QPL; ++s) {
        bad |= (qr.qmin[s] >> 24) + (kmin >> 24) < 2 * 127 - 96;
#pragma unroll
        for (int g = 0; g < 4; ++g)
#pragma unroll
            for (int i = 0; i < 4; ++i) bad |= !(__builtin_fabsf(e8[s][g][i]) < __builtin_inff());
    }
    return wave_any(bad);
}

// Two SIM 8-bit logits as their bf16 patterns (exact: 3 mantissa bits).
__device__ __forceinline__ uint32_t pack_sim8(float a, float b)
{
    return (__builtin_bit_cast(uint32_t, a) >> 16) | (__builtin_bit_cast(uint32_t, b) & 0xFFFF0000u);
}

// The 16-bit logits of the FP32 chains in acc, rounded once to e4m11 (SIM
// profile: to 11 mantissa bits), as FP32 values.
template <bool SIMP, int QPL, int NM>
__device__ __forceinline__ void round16(const f32x4_t (&acc)[QPL][NM], float (&y)[QPL][4 * NM])
{
#pragma unroll
    for (int s = 0; s < QPL; ++s)
#pragma unroll
        for (int i = 0; i < 4 * NM; ++i)
            y[s][i] = SIMP ? rn_sim<11>(acc[s][i / 4][i % 4]) : rn_e4m11(acc[s][i / 4][i % 4]);
}

// The 8-bit logits of the 16 keys ke (EMU; with the overflow check) and the
// 16-bit logits of NKEY keys kr in one loop that shares the query loads.  The
// forward kernel uses it to run the 8-bit logits of the next key tile together
// with the speculative 16-bit recompute of the current one.  a8 receives the
// 8-bit logits (Y8_WORDS), y16 the 16-bit ones as FP32 values, sat the saturated keys of the
// 8-bit chunk (0 in the SIM profile, which does not saturate).
template <int D, int QPL, int NKEY, bool EMU, bool SIMP, class LY = RowLay<D>>
__device__ __forceinline__ void fused_pass(QRows<QPL> &qr, const KRows &ke, const KRows &kr,
                                           uint32_t (&a8)[QPL][Y8_WORDS<SIMP>], float (&y16)[QPL][NKEY > 0 ? NKEY : 1],
                                           uint32_t (&sat)[QPL])
{
    static_assert(EMU || NKEY > 0, "something to compute");
    static_assert(NKEY == 0 || NKEY == 4 || NKEY == 8 || NKEY == 12 || NKEY == 16, "0, 4, 8, 12 or 16 keys");
    constexpr int NM = NKEY / 4, NA = NM > 0 ? NM : 1, NE = SIMP && EMU ? 4 : 1;
    uint32_t w8[QPL][4];
    f32x4_t acc[QPL][NA], e8[QPL][NE];
#pragma unroll
    for (int s = 0; s < QPL; ++s) {
        sat[s] = 0u;
#pragma unroll
        for (int g = 0; g < 4; ++g) w8[s][g] = 0u;
#pragma unroll
        for (int g = 0; g < NA; ++g) acc[s][g] = f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int g = 0; g < NE; ++g) e8[s][g] = f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};
    }
    uint32_t kmin = 0xFFFFFFFFu;
    if (!(EMU && SIMP) || !qr.exact)
        logit_loop<D, QPL, NM, EMU, SIMP, false, EMU ? 2 : 4, LY>(qr, ke, kr, w8, e8, acc, kmin);
    if constexpr (EMU && SIMP) {
        // out of range once: the rest of this wave's tiles at once exactly
        f32x4_t none[QPL][1];
        if (qr.exact) {
            if constexpr (NM > 0) logit_loop<D, QPL, NM, false, true, false, 4, LY>(qr, kr, kr, w8, none, acc, kmin);
        } else {
            qr.exact = sim8_out_of_range<QPL>(qr, kmin, e8);
        }
        if (qr.exact) {
#pragma unroll
            for (int s = 0; s < QPL; ++s)
#pragma unroll
                for (int g = 0; g < 4; ++g) e8[s][g] = f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};
            logit_loop<D, QPL, 0, true, true, true, 2, LY>(qr, ke, ke, w8, e8, none, kmin);
        }
#pragma unroll
        for (int s = 0; s < QPL; ++s)
#pragma unroll
            for (int p = 0; p < 8; ++p) a8[s][p] = pack_sim8(e8[s][p / 2][2 * (p & 1)], e8[s][p / 2][2 * (p & 1) + 1]);
    } else if constexpr (EMU) {
        emu8_check<D, QPL, LY>(qr, ke, w8, sat);
#pragma unroll
        for (int s = 0; s < QPL; ++s)
#pragma unroll
            for (int g = 0; g < 4; ++g) a8[s][g] = w8[s][g];
    }
    if constexpr (NM > 0) round16<SIMP>(acc, y16);
}

// Y8 of a 16-key chunk in either profile (sat as in emu8_check).
template <int D, int QPL, bool SIMP, class LY = RowLay<D>>
__device__ __forceinline__ void emu8_any(QRows<QPL> &qr, const KRows &ke, uint32_t (&a8)[QPL][Y8_WORDS<SIMP>],
                                         uint32_t (&sat)[QPL])
{
    float none[QPL][1];
    fused_pass<D, QPL, 0, true, SIMP, LY>(qr, ke, ke, a8, none, sat);
}

// Y16 of NKEY keys (NKEY in {4, 8, 12, 16}) for QPL query rows: the FP32 FMA
// chain over the channels in ascending order from +0, rounded once to e4m11
// (saturating), as FP32 values.  Lane l of every 16-lane row of kr supplies key
// (l mod 16) and must hold key (l mod NKEY) (lanes past NKEY are not read).
template <int D, int QPL, int NKEY, bool SIMP = false, class LY = RowLay<D>>
__device__ __forceinline__ void rec16_values(QRows<QPL> &qr, const KRows &kr, float (&y)[QPL][NKEY])
{
    uint32_t none[QPL][Y8_WORDS<SIMP>], sat[QPL];
    fused_pass<D, QPL, NKEY, false, SIMP, LY>(qr, kr, kr, none, y, sat);
}

// The same as e4m11 codes: codes[s][p] holds keys 2p (bits [15:0]) and 2p+1.
template <int D, int QPL, int NKEY, class LY = RowLay<D>>
__device__ __forceinline__ void rec16_keys(QRows<QPL> &qr, const KRows &kr, uint32_t (&codes)[QPL][NKEY / 2])
{
    float y[QPL][NKEY];
    rec16_values<D, QPL, NKEY, false, LY>(qr, kr, y);
#pragma unroll
    for (int s = 0; s < QPL; ++s)
#pragma unroll
        for (int p = 0; p < NKEY / 2; ++p) codes[s][p] = e4m11_code(y[s][2 * p]) | e4m11_code(y[s][2 * p + 1]) << 16;
}

// Whether the 16-bit logit of one (query row, key) saturates: its FP32 FMA
// chain (channels ascending from +0, the recursion rec16_keys runs) rounds
// beyond 511.875, the largest e4m11 value, i.e. |sum| >= 511.9375 (a tie
// goes to the even 512).  Used only where a 16-bit code is at that maximum.
template <int D, class LY>
__device__ __forceinline__ bool y16_saturates(const float *qrow, const float *krow)
{
    float a = 0.0f;
#pragma unroll 4
    for (int c = 0; c < D; ++c) a = __builtin_fmaf(qrow[(c / 4) * LY::QS + c % 4], krow[(c / 4) * LY::KS + c % 4], a);
    return __builtin_fabsf(a) >= 511.9375f;
}

} // namespace lamp
