// lamp_kernels.hip -- auxiliary HIP kernels of liblamp.so for gfx950: the
// prepass (pre-scaled Q, K in fp32), the exponential
// tables, the stand-alone logit kernels and the self tests.  The forward
// kernel is in lamp_fwd.hip, the logit loops in lamp_loops.h.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "lamp_device.h"
#include "lamp_kernels.h"
#include "lamp_loops.h"
#include "lamp_sr.h"

namespace lamp {

static_assert(SIM8_ENTRIES == SIM8_N && SIM16_TABLE == SIM16_N && SIM8_N <= SIM8_TABLE, "SIM table sizes");

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// ------------------------------------------------------------------ prepass
// One thread per 4 channels of one row of one head.  u (below rows * D/4)
// indexes the float4 groups of a head's output in storage order: the row
// layout (blk = 0) stores [rows][D]; the grouped layout stores blocks of blk
// rows, each [D/4][blk][4], so that one 4-channel group of a block is
// contiguous.  Returns the row j and group g of u.
__device__ __forceinline__ void rg_of(int u, int G, int blk, int &j, int &g)
{
    if (blk == 0) {
        j = u / G;
        g = u % G;
        return;
    }
    const int per = blk * G, r = u % per;
    j = (u / per) * blk + r % blk;
    g = r / blk;
}

// 4 bf16 values (8 bytes) as fp32, times s (s = 1: exact conversion)
__device__ __forceinline__ float4 bf16x4_scaled(const uint2 w, float s)
{
    return make_float4(bf16_value(w.x & 0xFFFFu) * s, bf16_value(w.x >> 16) * s, bf16_value(w.y & 0xFFFFu) * s,
                       bf16_value(w.y >> 16) * s);
}

// Nonzero iff one of the bf16 values in a word has an all-ones exponent
// (an infinity or a NaN).
__device__ __forceinline__ uint32_t bf16_nonfinite(uint32_t w)
{
    return ((w & 0x7F80u) == 0x7F80u) | ((w & 0x7F800000u) == 0x7F800000u);
}

// Or `bit` into *bad once per wave if any lane saw a non-finite value.
__device__ __forceinline__ void flag_nonfinite(unsigned *bad, bool seen, unsigned bit)
{
    if (__ballot(seen) != 0ull && __lane_id() == (unsigned)__builtin_ctzll(__ballot(seen))) atomicOr(bad, bit);
}

// Rows x [BH][N][D] as fp32 times scale (RN32; 1 converts exactly), padded with
// zeros from N to Np rows: y [BH][Np][D] in the row or grouped layout (blk rows
// a block).  Workgroup (bx, by) of (gx, gy): bx over the float4 groups of a
// head, by over heads (both grid-stride).  Returns whether an element is not
// finite.
__device__ __forceinline__ bool rows_to_f32(const uint16_t *__restrict__ x, float *__restrict__ y, float scale, int N,
                                            int Np, int D, int BH, int blk, unsigned bx, unsigned by, unsigned gx,
                                            unsigned gy)
{
    const int G = D / 4, n4 = Np * G;
    bool seen = false;
    for (unsigned bh = by; bh < (unsigned)BH; bh += gy)
        for (int u = bx * 256 + threadIdx.x; u < n4; u += gx * 256) {
            int j, g;
            rg_of(u, G, blk, j, g);
            const uint2 w = j < N ? *reinterpret_cast<const uint2 *>(x + ((size_t)bh * N + j) * D + 4 * g)
                                  : make_uint2(0u, 0u);
            seen |= (bf16_nonfinite(w.x) | bf16_nonfinite(w.y)) != 0u;
            reinterpret_cast<float4 *>(y + (size_t)bh * Np * D)[u] = bf16x4_scaled(w, scale);
        }
    return seen;
}

// V^T [B*Hkv][D][Nk] from V [B*Hkv][N][D] (bf16), keys padded with zeros from N
// to Nk: the 64 x 64 tile number t (key tiles innermost) through LDS.  Nk and D
// are multiples of 64.
__device__ __forceinline__ bool transpose_v_tile(const uint16_t *__restrict__ v, uint16_t *__restrict__ vt, int N,
                                                 int Nk, int D, unsigned t, uint16_t (&tile)[64][66])
{
    const unsigned nt = (unsigned)Nk / 64, ct = (unsigned)D / 64;
    const size_t bh = t / (nt * ct);
    const int n0 = (int)(t % nt) * 64, c0 = (int)(t / nt % ct) * 64;
    const uint16_t *src = v + bh * (size_t)N * D;
    uint16_t *dst = vt + bh * (size_t)D * Nk;
    bool seen = false;
    for (int e = threadIdx.x; e < 64 * 64; e += 256) {
        const int r = e / 64, c = e % 64;
        const uint16_t x = n0 + r < N ? src[(size_t)(n0 + r) * D + c0 + c] : (uint16_t)0;
        seen |= (x & 0x7F80u) == 0x7F80u;
        tile[r][c] = x;
    }
    __syncthreads();
    for (int e = threadIdx.x; e < 64 * 64; e += 256) {
        const int c = e / 64, r = e % 64;
        dst[(size_t)(c0 + c) * Nk + n0 + r] = tile[r][c];
    }
    return seen;
}

// The prepass in one launch: the pre-scaled queries q~ = RN32(q * s), the keys
// in fp32 and (v not null) V transposed, each on its own range of workgroups.
// Three launches cost a short call some 10 us of gaps and of devices nearly
// empty (300 tokens, 32 heads: 17 us, one launch 7).
// bad (may be null): bits 0, 1, 2 are or-ed into *bad if an element of q, k, v
// is not finite.
struct PrepassParams {
    const uint16_t *q, *k, *v;
    float *qt, *kt32;
    uint16_t *vt;
    int N, Nq, Nk, D, BHq, BHk, blkq, blkk;
    float scale;
    dim3 gq, gk;       // workgroups of the queries and keys
    unsigned nv;       // workgroups of V
    unsigned *bad;
};

__global__ __launch_bounds__(256) void prepass_kernel(PrepassParams a)
{
    __shared__ uint16_t tile[64][66];
    const unsigned nq = a.gq.x * a.gq.y, nk = a.gk.x * a.gk.y;
    unsigned i = blockIdx.x, bit;
    bool seen;
    if (i < nq) {
        seen = rows_to_f32(a.q, a.qt, a.scale, a.N, a.Nq, a.D, a.BHq, a.blkq, i % a.gq.x, i / a.gq.x, a.gq.x, a.gq.y);
        bit = 1u;
    } else if (i < nq + nk) {
        i -= nq;
        seen = rows_to_f32(a.k, a.kt32, 1.0f, a.N, a.Nk, a.D, a.BHk, a.blkk, i % a.gk.x, i / a.gk.x, a.gk.x, a.gk.y);
        bit = 2u;
    } else {
        const unsigned tiles = (unsigned)(a.Nk / 64) * (unsigned)(a.D / 64) * (unsigned)a.BHk;
        seen = false;
        for (unsigned t = i - nq - nk; t < tiles; t += a.nv) {
            seen |= transpose_v_tile(a.v, a.vt, a.N, a.Nk, a.D, t, tile);
            __syncthreads();   // the next tile's values replace this one's
        }
        bit = 4u;
    }
    if (a.bad) flag_nonfinite(a.bad, seen, bit);
}

// ------------------------------------------------------------------ tables
// Exponential tables: E = RN(exp(-s)) for every shift code s, correctly
// rounded (Sec. 3.3 LUT exp; Sec. 4.1 exponentials correctly rounded).  exp
// is evaluated with exp_doc (error below 2^-50 relative); an entry whose
// enclosure straddles a rounding midpoint is counted in *ambiguous and the
// library refuses to run.
__device__ __forceinline__ double rn_grid(double y, int mbits, int emin)
{
    int e = __builtin_amdgcn_frexp_exp(y) - 1;
    int qe = (e > emin ? e : emin) - mbits;
    double c = __builtin_amdgcn_ldexp(1.5, 52 + qe);
    return (y + c) - c;
}

__device__ __forceinline__ uint32_t grid_code(double r, int mbits, int emin, int bias)
{
    if (r < __builtin_amdgcn_ldexp(1.0, emin))
        return (uint32_t)(r * __builtin_amdgcn_ldexp(1.0, mbits - emin));
    uint32_t hi = (uint32_t)(__builtin_bit_cast(uint64_t, r) >> 32);
    uint32_t ex = (hi >> 20) - 1023u + (uint32_t)bias;
    return (ex << mbits) | ((hi >> (20 - mbits)) & ((1u << mbits) - 1u));
}

__device__ __forceinline__ double grid_value(uint32_t c, int mbits, int bias)
{
    uint32_t ex = c >> mbits, m = c & ((1u << mbits) - 1u);
    if (ex == 0) return __builtin_amdgcn_ldexp((double)m, 1 - bias - mbits);
    return __builtin_amdgcn_ldexp((double)((1u << mbits) | m), (int)ex - bias - mbits);
}

__global__ void build_tables_kernel(uint8_t *__restrict__ lut8, uint16_t *__restrict__ lut8e,
                                    uint16_t *__restrict__ exp16, uint32_t *__restrict__ exp16hl,
                                    unsigned *__restrict__ ambiguous)
{
    unsigned c = blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= 65536u + 256u) return;
    bool small = c >= 65536u;
    unsigned code = small ? c - 65536u : c;
    int mb = small ? 3 : 11;
    double s = grid_value(code, mb, 15);
    double y = exp_doc(-s);
    double lo = y * (1.0 - 0x1p-48), hi = y * (1.0 + 0x1p-48);
    double r = rn_grid(y, mb, -30);
    if (rn_grid(lo, mb, -30) != r || rn_grid(hi, mb, -30) != r) atomicAdd(ambiguous, 1u);
    uint32_t e = grid_code(r, mb, -30, 31);
    if (small) {
        lut8[code] = (uint8_t)e;
        lut8e[code] = (uint16_t)bf16_bits((float)r);   // E8 is exact in bf16
    } else {
        exp16[code] = (uint16_t)e;
        uint32_t eh, el;   // the same value as exact bf16 high and low parts, for P.V
        split_bf16((float)r, eh, el);
        exp16hl[code] = eh | (el << 16);
    }
}

// Exponential tables of the SIM profile (layout in lamp_device.h): entry
// ((e - EMIN) << P) | m is RN_P(exp(-s)), s = (2^P + m) 2^(e-P), rounded to P
// mantissa bits in FP32's exponent range (quantum 2^(-126-P) below 2^-126);
// the same enclosure check as above.  sim8 holds 256 entries, those past
// SIM8_N being 0.
__global__ void build_sim_tables_kernel(uint16_t *__restrict__ sim8, uint32_t *__restrict__ sim16,
                                        unsigned *__restrict__ ambiguous)
{
    unsigned c = blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= (unsigned)SIM16_N + (unsigned)SIM8_TABLE) return;
    const bool small = c >= (unsigned)SIM16_N;
    const unsigned idx = small ? c - (unsigned)SIM16_N : c;
    if (small && idx >= (unsigned)SIM8_N) {   // padding of the 256-entry copy
        sim8[idx] = 0;
        return;
    }
    const int P = small ? 3 : 11;
    const int e = (small ? SIM8_EMIN : SIM16_EMIN) + (int)(idx >> P);
    const double s = __builtin_amdgcn_ldexp((double)((1u << P) | (idx & ((1u << P) - 1u))), e - P);
    const double y = exp_doc(-s);
    const double lo = y * (1.0 - 0x1p-48), hi = y * (1.0 + 0x1p-48);
    const double r = rn_grid(y, P, -126);
    if (rn_grid(lo, P, -126) != r || rn_grid(hi, P, -126) != r) atomicAdd(ambiguous, 1u);
    if (small) sim8[idx] = (uint16_t)bf16_bits((float)r);   // 4 significant bits: exact in bf16
    else sim16[idx] = __builtin_bit_cast(uint32_t, (float)r);
}

// ------------------------------------------------------------------ logits entry kernels
// One wave: 64 rows x (16*NC) keys.  grid.x = B*Hq*ceil(nrows/64), grid.y = N/(16*NC).
template <int D, int NC, bool SR>
__global__ __launch_bounds__(64, 2) void logits8_kernel(LogitsParams p)
{
    const int lane = threadIdx.x;
    const int nrg = (p.nrows + 63) / 64;
    const int bh = blockIdx.x / nrg;
    const int rg = blockIdx.x % nrg;
    const int b = bh / p.Hq, h = bh % p.Hq;
    const int hk = h / (p.Hq / p.Hkv);
    const int r = rg * 64 + lane;
    const int rr = r < p.nrows ? r : p.nrows - 1;
    const int j = p.row0 + rr;
    QRows<1> qr = {{p.qt + (((size_t)b * p.Hq + h) * p.N + p.row0) * D}, (uint32_t)rr * D * 4u, {0u}, false};
    for (int g = 0; g < NC; ++g) {
        const int key0 = (blockIdx.y * NC + g) * 16;
        const float *kt = p.kt32 + (((size_t)b * p.Hkv + hk) * p.N + key0) * (size_t)D;
        uint32_t acc[1][4], sat[1];
        if constexpr (SR) {
            const int jq[1] = {j};
            sr8_chunk_bc<D, 1, RowLay<D>>(qr, kt, jq, (uint32_t)key0, (uint32_t)bh, p.seed, acc, sat);
        } else {
            emu8_any<D, 1, false>(qr, keys16<RowLay<D>>(kt), acc, sat);
        }
        if (r < p.nrows) {
            uint8_t *out = p.y8 + (((size_t)b * p.Hq + h) * p.nrows + r) * p.N + key0;
#pragma unroll
            for (int t = 0; t < 16; ++t) {
                const int i = key0 + t;
                const bool vis = !(p.causal && i > j) && !(p.window > 0 && i <= j - p.window);
                out[t] = vis ? (uint8_t)(acc[0][t >> 2] >> (8 * (t & 3))) : (uint8_t)0xFF;
            }
        }
    }
}

template <int D>
__global__ __launch_bounds__(64, 2) void logits16_kernel(LogitsParams p)
{
    const int lane = threadIdx.x;
    const int nrg = (p.nrows + 63) / 64;
    const int bh = blockIdx.x / nrg;
    const int rg = blockIdx.x % nrg;
    const int b = bh / p.Hq, h = bh % p.Hq;
    const int hk = h / (p.Hq / p.Hkv);
    const int r = rg * 64 + lane;
    const int rr = r < p.nrows ? r : p.nrows - 1;
    const int j = p.row0 + rr;
    const int key0 = blockIdx.y * 16;
    QRows<1> qr = {{p.qt + (((size_t)b * p.Hq + h) * p.N + p.row0) * D}, (uint32_t)rr * D * 4u, {0u}, false};
    const float *kt = p.kt32 + (((size_t)b * p.Hkv + hk) * p.N + key0) * (size_t)D;
    uint32_t codes[1][8];
    rec16_keys<D, 1, 16>(qr, keys16<RowLay<D>>(kt), codes);
    if (r >= p.nrows) return;
    uint16_t *out = p.y16 + (((size_t)b * p.Hq + h) * p.nrows + r) * p.N + key0;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        const int key = key0 + i;
        const bool vis = !(p.causal && key > j) && !(p.window > 0 && key <= j - p.window);
        out[i] = vis ? (uint16_t)(codes[0][i >> 1] >> (16 * (i & 1))) : (uint16_t)0xFFFF;
    }
}

// SIM profile logit values: one wave, 64 rows x 16 keys.
template <int D, bool HIGH>
__global__ __launch_bounds__(64, 2) void logits_sim_kernel(LogitsParams p)
{
    const int lane = threadIdx.x;
    const int nrg = (p.nrows + 63) / 64;
    const int bh = blockIdx.x / nrg;
    const int rg = blockIdx.x % nrg;
    const int b = bh / p.Hq, h = bh % p.Hq;
    const int hk = h / (p.Hq / p.Hkv);
    const int r = rg * 64 + lane;
    const int rr = r < p.nrows ? r : p.nrows - 1;
    const int j = p.row0 + rr;
    const int key0 = blockIdx.y * 16;
    QRows<1> qr = {{p.qt + (((size_t)b * p.Hq + h) * p.N + p.row0) * D}, (uint32_t)rr * D * 4u, {0u}, false};
    const float *kt = p.kt32 + (((size_t)b * p.Hkv + hk) * p.N + key0) * (size_t)D;
    float val[16];
    if constexpr (HIGH) {
        float y[1][16];
        rec16_values<D, 1, 16, true>(qr, keys16<RowLay<D>>(kt), y);
#pragma unroll
        for (int i = 0; i < 16; ++i) val[i] = y[0][i];
    } else {
        uint32_t w[1][8], sat[1];
        set_qmin<D, 1, RowLay<D>>(qr);
        emu8_any<D, 1, true>(qr, keys16<RowLay<D>>(kt), w, sat);
        // the fast rounding loses the sign of a zero, which this entry returns
        bool zero = false;
#pragma unroll
        for (int i = 0; i < 16; ++i) zero |= (w[0][i >> 1] >> (16 * (i & 1)) & 0x7FFFu) == 0u;
        if (wave_any(zero)) {
            qr.exact = true;
            emu8_any<D, 1, true>(qr, keys16<RowLay<D>>(kt), w, sat);
        }
#pragma unroll
        for (int i = 0; i < 16; ++i) val[i] = bf16_value((w[0][i >> 1] >> (16 * (i & 1))) & 0xFFFFu);
    }
    if (r >= p.nrows) return;
    float *out = p.ysim + (((size_t)b * p.Hq + h) * p.nrows + r) * p.N + key0;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        const int key = key0 + i;
        const bool vis = !(p.causal && key > j) && !(p.window > 0 && key <= j - p.window);
        out[i] = vis ? val[i] : __builtin_nanf("");
    }
}

// ------------------------------------------------------------------ self tests
// e4m3 codes of fp32 values by the emulator's sequence: the non-saturating
// conversion, then the saturating one where the first gave NaN.  raw (may be
// null) receives the non-saturating codes.
__global__ void selftest_e4m3_kernel(const float *__restrict__ in, uint8_t *__restrict__ out,
                                     uint8_t *__restrict__ raw, size_t n)
{
    size_t i = ((size_t)blockIdx.x * blockDim.x + threadIdx.x) * 2;
    if (i >= n) return;
    float a = in[i], b = (i + 1 < n) ? in[i + 1] : 0.0f;
    uint32_t r = pk_e4m3(a, b);
    uint32_t f = e4m3_nan_bits(r) ? pk_e4m3_sat(a, b) : r;
    out[i] = (uint8_t)f;
    if (raw) raw[i] = (uint8_t)r;
    if (i + 1 < n) {
        out[i + 1] = (uint8_t)(f >> 8);
        if (raw) raw[i + 1] = (uint8_t)(r >> 8);
    }
}

__global__ void selftest_exp_doc_kernel(const double *__restrict__ x, double *__restrict__ y, size_t n)
{
    size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) y[i] = exp_doc(x[i]);
}

// ------------------------------------------------------------------ launchers
// Workgroups of a part of the prepass: 256-thread ones over one head's float4
// groups (x) and over the heads (y); capped (the kernel strides over the rest),
// so that the launch stays below 2^32 threads.
constexpr unsigned PREPASS_MAX = 1u << 21;

static dim3 prepass_grid(int BH, int rows, int D)
{
    const long n4 = (long)rows * (D / 4);
    const long gx = (n4 + 255) / 256;
    const unsigned x = (unsigned)(gx < 4096 ? (gx > 0 ? gx : 1) : 4096), my = PREPASS_MAX / x;
    return dim3(x, (unsigned)BH < my ? (BH > 0 ? (unsigned)BH : 1u) : my);
}

hipError_t launch_prepass(const uint16_t *q, const uint16_t *k, const uint16_t *v, float *qt, float *kt32, uint16_t *vt,
                          int B, int Hq, int Hkv, int N, int Nq, int Nk, int D, float scale, hipStream_t s, bool grouped,
                          unsigned *bad)
{
    const uint64_t tiles = v ? (uint64_t)(Nk / 64) * (uint64_t)(D / 64) * (uint64_t)B * Hkv : 0;
    PrepassParams a{q, k, v, qt, kt32, vt, N, Nq, Nk, D, B * Hq, B * Hkv, grouped ? 64 : 0, grouped ? 16 : 0, scale,
                    prepass_grid(B * Hq, Nq, D), prepass_grid(B * Hkv, Nk, D),
                    (unsigned)(tiles < PREPASS_MAX ? tiles : PREPASS_MAX), bad};
    hipLaunchKernelGGL(prepass_kernel, dim3(a.gq.x * a.gq.y + a.gk.x * a.gk.y + a.nv), dim3(256), 0, s, a);
    return hipGetLastError();
}

template <bool SR>
static void launch_logits8_t(const LogitsParams &p, int D, hipStream_t s)
{
    const unsigned gx = (unsigned)(p.B * p.Hq * ((p.nrows + 63) / 64));
    if (p.N % 64 == 0) {
        dim3 grid(gx, (unsigned)(p.N / 64));
        if (D == 64) hipLaunchKernelGGL((logits8_kernel<64, 4, SR>), grid, dim3(64), 0, s, p);
        else if (D == 128) hipLaunchKernelGGL((logits8_kernel<128, 4, SR>), grid, dim3(64), 0, s, p);
        else hipLaunchKernelGGL((logits8_kernel<256, 4, SR>), grid, dim3(64), 0, s, p);
    } else {
        dim3 grid(gx, (unsigned)(p.N / 16));
        if (D == 64) hipLaunchKernelGGL((logits8_kernel<64, 1, SR>), grid, dim3(64), 0, s, p);
        else if (D == 128) hipLaunchKernelGGL((logits8_kernel<128, 1, SR>), grid, dim3(64), 0, s, p);
        else hipLaunchKernelGGL((logits8_kernel<256, 1, SR>), grid, dim3(64), 0, s, p);
    }
}

hipError_t launch_logits8(const LogitsParams &p, int D, hipStream_t s, bool sr)
{
    if (sr) launch_logits8_t<true>(p, D, s);
    else launch_logits8_t<false>(p, D, s);
    return hipGetLastError();
}

hipError_t launch_logits16(const LogitsParams &p, int D, hipStream_t s)
{
    dim3 grid((unsigned)(p.B * p.Hq * ((p.nrows + 63) / 64)), (unsigned)(p.N / 16));
    if (D == 64) hipLaunchKernelGGL(logits16_kernel<64>, grid, dim3(64), 0, s, p);
    else if (D == 128) hipLaunchKernelGGL(logits16_kernel<128>, grid, dim3(64), 0, s, p);
    else hipLaunchKernelGGL(logits16_kernel<256>, grid, dim3(64), 0, s, p);
    return hipGetLastError();
}

hipError_t launch_logits_sim(const LogitsParams &p, int D, int high, hipStream_t s)
{
    dim3 grid((unsigned)(p.B * p.Hq * ((p.nrows + 63) / 64)), (unsigned)(p.N / 16));
    if (high) {
        if (D == 64) hipLaunchKernelGGL((logits_sim_kernel<64, true>), grid, dim3(64), 0, s, p);
        else if (D == 128) hipLaunchKernelGGL((logits_sim_kernel<128, true>), grid, dim3(64), 0, s, p);
        else hipLaunchKernelGGL((logits_sim_kernel<256, true>), grid, dim3(64), 0, s, p);
    } else {
        if (D == 64) hipLaunchKernelGGL((logits_sim_kernel<64, false>), grid, dim3(64), 0, s, p);
        else if (D == 128) hipLaunchKernelGGL((logits_sim_kernel<128, false>), grid, dim3(64), 0, s, p);
        else hipLaunchKernelGGL((logits_sim_kernel<256, false>), grid, dim3(64), 0, s, p);
    }
    return hipGetLastError();
}

hipError_t launch_build_sim_tables(uint16_t *sim8, uint32_t *sim16, unsigned *ambiguous, hipStream_t s)
{
    hipLaunchKernelGGL(build_sim_tables_kernel, dim3((SIM16_N + SIM8_TABLE + 255) / 256), dim3(256), 0, s, sim8, sim16,
                       ambiguous);
    return hipGetLastError();
}

hipError_t launch_build_tables(uint8_t *lut8, uint16_t *lut8e, uint16_t *exp16, uint32_t *exp16hl, unsigned *ambiguous,
                              hipStream_t s)
{
    hipLaunchKernelGGL(build_tables_kernel, dim3((65536 + 256 + 255) / 256), dim3(256), 0, s, lut8, lut8e, exp16,
                       exp16hl, ambiguous);
    return hipGetLastError();
}

hipError_t launch_selftest_e4m3(const float *in, uint8_t *out, uint8_t *raw, size_t n, hipStream_t s)
{
    size_t pairs = (n + 1) / 2;
    hipLaunchKernelGGL(selftest_e4m3_kernel, dim3((unsigned)((pairs + 255) / 256)), dim3(256), 0, s, in, out, raw, n);
    return hipGetLastError();
}

hipError_t launch_selftest_exp_doc(const double *x, double *y, size_t n, hipStream_t s)
{
    hipLaunchKernelGGL(selftest_exp_doc_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, x, y, n);
    return hipGetLastError();
}

} // namespace lamp
