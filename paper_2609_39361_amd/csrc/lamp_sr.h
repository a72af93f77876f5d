// lamp_sr.h -- stochastic rounding of the 8-bit logit accumulation.
//
// Sec. 3.3 ("Floating-point formats") names stochastic rounding (Croci et al.
// 2022) as the alternative to round-to-nearest for the e4m3 accumulation, to
// counter swamping.  The paper fixes neither the generator nor the number of
// random bits; the library's reading:
//   - each step rounds the FP32 FMA result t to one of its two e4m3
//     neighbours: a = min(|t|, 448), lo the e4m3 number next to a toward zero,
//     u its spacing; the step goes to lo + u when floor(2^16 (a - lo) / u) +
//     r >= 2^16 and to lo otherwise, with the sign of t; r is a uniform
//     16-bit integer;
//   - r comes from the counter-based generator Philox4x32-10 (Salmon, Moraes,
//     Dror and Shaw, "Parallel random numbers: as easy as 1, 2, 3", SC 2011)
//     under key (seed mod 2^32, seed / 2^32) at counter (j, i, b*Hq + h,
//     c / 8) for query row j, key i, query head h of batch b and channel c;
//     each of the four 32-bit outputs holds two 16-bit fields, channel c
//     taking the low half (c even) or the high half (c odd) of output
//     (c mod 8) / 2, so one call serves eight channels.
// The random numbers depend on the logit and the channel only, so the 8-bit
// logits are the same under every blocking and in the logits entry point.
//
// The rounding itself is gfx950's stochastic fp32 -> fp8 conversion
// (v_cvt_sr_fp8_f32) on the value clamped to +-448: it adds the top 20 bits
// of its 32-bit random operand to the 20 bits of the FP32 significand below
// e4m3's last bit (below 2^-6: to the bits below the 2^-9 quantum) and
// truncates, which with the operand r << 16 is the rounding above (the low 4
// of those 20 random bits are zero, so they never carry); the library's tests
// check it against the oracle's rounding.
#pragma once
#include <stdint.h>
#include <utility>

#include "lamp_device.h"
#include "lamp_loops.h"

namespace lamp {

// Philox4x32-10: ten rounds of the 4x32 round function; the key is bumped by
// the Weyl constants before every round after the first.
__device__ __forceinline__ void philox4x32_10(uint32_t (&c)[4], uint32_t k0, uint32_t k1)
{
    constexpr uint32_t M0 = 0xD2511F53u, M1 = 0xCD9E8D57u;
    constexpr uint32_t W0 = 0x9E3779B9u, W1 = 0xBB67AE85u;
#pragma unroll
    for (int r = 0; r < 10; ++r) {
        if (r > 0) {
            k0 += W0;
            k1 += W1;
        }
        const uint64_t p0 = (uint64_t)M0 * c[0], p1 = (uint64_t)M1 * c[2];
        // three-input exclusive or in one VALU instruction (bitop3 truth table 0x96)
        const uint32_t n0 = __builtin_amdgcn_bitop3_b32((uint32_t)(p1 >> 32), c[1], k0, 0x96);
        const uint32_t n2 = __builtin_amdgcn_bitop3_b32((uint32_t)(p0 >> 32), c[3], k1, 0x96);
        c[1] = (uint32_t)p1;
        c[3] = (uint32_t)p0;
        c[0] = n0;
        c[2] = n2;
    }
}

// Channels cb .. cb+7 of the two chains of keys 2P, 2P+1 of each of QPL query
// rows, whose codes share word acc[s][P] (bits 7:0, 15:8): one Philox call per
// chain, then 8 steps of both, each decoding the pair, running both FP32 FMAs
// (the keys by row broadcast) and rounding each value stochastically into its
// byte.  Without CLAMP a |t| above 448 gives +-448 as well or, rounded up, a
// NaN code, which the NaN carries to the end of the chain (the caller then
// re-runs with CLAMP, which is the saturating recursion: the two agree up to
// that step).  COUNT: bit i of sat[s] is set when a step of key i had |t| > 448.
template <int P, int QPL, bool CLAMP, bool COUNT>
__device__ __forceinline__ void sr8_pair8(const float4 &k0, const float4 &k1, const float4 (&q0)[QPL],
                                          const float4 (&q1)[QPL], const int (&j)[QPL], uint32_t key0,
                                          uint32_t bh, uint32_t g, uint32_t s0, uint32_t s1, uint32_t (&acc)[QPL][8],
                                          uint32_t (&sat)[QPL])
{
    const float kv[8] = {k0.x, k0.y, k0.z, k0.w, k1.x, k1.y, k1.z, k1.w};
#pragma unroll
    for (int s = 0; s < QPL; ++s) {
        // the query index through an empty statement the compiler cannot move:
        // the generator's rounds stay here, next to their use, instead of being
        // hoisted for every pair and block at once (which exhausts the registers)
        uint32_t js = (uint32_t)j[s];
        asm volatile("" : "+v"(js));
        uint32_t wa[4] = {js, key0 + 2 * P, bh, g};
        uint32_t wb[4] = {js, key0 + 2 * P + 1, bh, g};
        philox4x32_10(wa, s0, s1);
        philox4x32_10(wb, s0, s1);
        const float qv[8] = {q0[s].x, q0[s].y, q0[s].z, q0[s].w, q1[s].x, q1[s].y, q1[s].z, q1[s].w};
        uint32_t word = acc[s][P];
        float ma = 0.0f, mb = 0.0f;
#pragma unroll
        for (int c = 0; c < 8; ++c) {
            const uint32_t ra = (c & 1) ? (wa[c / 2] & 0xFFFF0000u) : (wa[c / 2] << 16);
            const uint32_t rb = (c & 1) ? (wb[c / 2] & 0xFFFF0000u) : (wb[c / 2] << 16);
            const float2 f = unpk_e4m3(word);
            float ta = fmac_bc<2 * P>(f.x, kv[c], qv[c]);
            float tb = fmac_bc<2 * P + 1>(f.y, kv[c], qv[c]);
            if constexpr (COUNT) {
                ma = __builtin_fmaxf(ma, __builtin_fabsf(ta));
                mb = __builtin_fmaxf(mb, __builtin_fabsf(tb));
            }
            if (CLAMP) {
                ta = __builtin_amdgcn_fmed3f(ta, -448.0f, 448.0f);
                tb = __builtin_amdgcn_fmed3f(tb, -448.0f, 448.0f);
            }
            word = (uint32_t)__builtin_amdgcn_cvt_sr_fp8_f32(ta, (int)ra, (int)word, 0);
            word = (uint32_t)__builtin_amdgcn_cvt_sr_fp8_f32(tb, (int)rb, (int)word, 1);
        }
        acc[s][P] = word;
        if constexpr (COUNT) sat[s] |= (ma > 448.0f ? 1u << (2 * P) : 0u) | (mb > 448.0f ? 2u << (2 * P) : 0u);
    }
}

// Y8 with stochastic rounding of one 16-key chunk for QPL query rows of this
// lane, keys read by DPP row broadcast (k32 at the chunk's first
// key, layout LY; slot s of qr the pre-scaled query row of query index j[s];
// key index key0 + i; bh = b*Hq + h).  The loop runs 8 channels of every
// chain at a time, so that each Philox call feeds its 8 steps at once, one key
// pair after the other (a loop, not unrolled, over a switch on the pair: the
// broadcast lane is an immediate, and one pair's chains at a time keep the
// registers of the surrounding kernel free); the loads run 8 channels ahead in
// two buffers written only by loads.  acc[s][p] receives the codes of keys
// 2p (bits 7:0) and 2p+1 (bits 15:8), sat[s] (COUNT) the saturated keys.
template <int D, int QPL, bool CLAMP, bool COUNT, class LY>
__device__ __forceinline__ void sr8_pass(const QRows<QPL> &qr, const float *k32, const int (&j)[QPL], uint32_t key0,
                                         uint32_t bh, uint64_t seed, uint32_t (&acc)[QPL][8], uint32_t (&sat)[QPL])
{
    static_assert(D % 16 == 0, "pairs of 8-channel blocks");
#pragma unroll
    for (int s = 0; s < QPL; ++s) {
        sat[s] = 0u;
#pragma unroll
        for (int p = 0; p < 8; ++p) acc[s][p] = 0u;
    }
    const uint32_t s0 = (uint32_t)seed, s1 = (uint32_t)(seed >> 32);
    const float *krow = k32 + (size_t)(__lane_id() & 15) * LY::KR;
    float4 ka0, ka1, kb0, kb1, qa0[QPL], qa1[QPL], qb0[QPL], qb1[QPL];
    auto ld = [&](int c, float4 &k0, float4 &k1, float4 (&q0)[QPL], float4 (&q1)[QPL]) {
        k0 = load4(krow + (c / 4) * LY::KS);
        k1 = load4(krow + (c / 4 + 1) * LY::KS);
#pragma unroll
        for (int s = 0; s < QPL; ++s) {
            q0[s] = load4(qr.base[s] + (c / 4) * LY::QS, qr.off);
            q1[s] = load4(qr.base[s] + (c / 4 + 1) * LY::QS, qr.off);
        }
    };
    auto run = [&](int c, const float4 &k0, const float4 &k1, const float4 (&q0)[QPL], const float4 (&q1)[QPL]) {
        const uint32_t g = (uint32_t)(c / 8);
#pragma nounroll
        for (int p = 0; p < 8; ++p) {
            switch (p) {
            case 0: sr8_pair8<0, QPL, CLAMP, COUNT>(k0, k1, q0, q1, j, key0, bh, g, s0, s1, acc, sat); break;
            case 1: sr8_pair8<1, QPL, CLAMP, COUNT>(k0, k1, q0, q1, j, key0, bh, g, s0, s1, acc, sat); break;
            case 2: sr8_pair8<2, QPL, CLAMP, COUNT>(k0, k1, q0, q1, j, key0, bh, g, s0, s1, acc, sat); break;
            case 3: sr8_pair8<3, QPL, CLAMP, COUNT>(k0, k1, q0, q1, j, key0, bh, g, s0, s1, acc, sat); break;
            case 4: sr8_pair8<4, QPL, CLAMP, COUNT>(k0, k1, q0, q1, j, key0, bh, g, s0, s1, acc, sat); break;
            case 5: sr8_pair8<5, QPL, CLAMP, COUNT>(k0, k1, q0, q1, j, key0, bh, g, s0, s1, acc, sat); break;
            case 6: sr8_pair8<6, QPL, CLAMP, COUNT>(k0, k1, q0, q1, j, key0, bh, g, s0, s1, acc, sat); break;
            default: sr8_pair8<7, QPL, CLAMP, COUNT>(k0, k1, q0, q1, j, key0, bh, g, s0, s1, acc, sat); break;
            }
        }
    };
    ld(0, ka0, ka1, qa0, qa1);
    for (int c = 0; c < D - 16; c += 16) {
        dpp_guard_fenced();
        ld(c + 8, kb0, kb1, qb0, qb1);
        run(c, ka0, ka1, qa0, qa1);
        ld(c + 16, ka0, ka1, qa0, qa1);
        run(c + 8, kb0, kb1, qb0, qb1);
    }
    ld(D - 8, kb0, kb1, qb0, qb1);
    dpp_guard_fenced();
    run(D - 16, ka0, ka1, qa0, qa1);
    run(D - 8, kb0, kb1, qb0, qb1);
}

// sr8_pass without saturation first; if any lane of the wave overflowed (a
// NaN code at the end of a chain), the chunk again with the clamp.  w[s][p]
// receives the codes of keys 4p .. 4p+3, one per byte.  COUNT and count
// (uniform): the pass with the clamp alone, and sat[s] the keys of slot s with a
// |t| > 448 (one in (448, 480) may round to 448 and leave no NaN); else sat is 0.
// Kept to the kernels' observing instantiations: in the others the third pass
// changes the register allocation (8K prefill 38.96 to 39.45 ms).
template <int D, int QPL, class LY, bool COUNT = false>
__device__ __forceinline__ void sr8_chunk_bc(const QRows<QPL> &qr, const float *k32, const int (&j)[QPL],
                                             uint32_t key0, uint32_t bh, uint64_t seed, uint32_t (&w)[QPL][4],
                                             uint32_t (&sat)[QPL], bool count = false)
{
    uint32_t acc[QPL][8];
    auto pack = [&] {
#pragma unroll
        for (int s = 0; s < QPL; ++s)
#pragma unroll
            for (int p = 0; p < 4; ++p) w[s][p] = (acc[s][2 * p] & 0xFFFFu) | (acc[s][2 * p + 1] << 16);
    };
    if constexpr (COUNT)
        if (count) {
            sr8_pass<D, QPL, true, true, LY>(qr, k32, j, key0, bh, seed, acc, sat);
            pack();
            return;
        }
    sr8_pass<D, QPL, false, false, LY>(qr, k32, j, key0, bh, seed, acc, sat);
    pack();
    uint32_t nan = 0;
#pragma unroll
    for (int s = 0; s < QPL; ++s)
#pragma unroll
        for (int p = 0; p < 4; ++p) nan |= e4m3x4_nan_bits(w[s][p]);
    if (wave_any(nan != 0)) {
        sr8_pass<D, QPL, true, false, LY>(qr, k32, j, key0, bh, seed, acc, sat);
        pack();
    }
}

} // namespace lamp
