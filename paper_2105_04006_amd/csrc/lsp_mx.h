// lsp_mx.h -- FP32 sums on the matrix cores, shared by the FP32 form's kernels
// (lsp_mx.hip) and the coarse spectra of the features (lsp_features.hip).
//
// A lane-per-bin loop spends six vector instructions per (observation, bin).
// Here the sums become matrix products.  A bin's frequency is written as a
// block centre plus or minus an offset, f = g_a +- h_m, with 64 bins per block
// (h_m = (m + 1/2) df, m = 0..31), and the angle-addition formulas split every
// sum over the observations j into products of a factor that depends on
// (a, j) and one that depends on (m, j):
//   sum y cos wt = sum (y cos g_a)(cos h_m) -+ sum (y sin g_a)(sin h_m),
//   sum y sin wt = sum (y sin g_a)(cos h_m) +- sum (y cos g_a)(sin h_m),
// and the same with 2wt and without y for sum cos 2wt, sum sin 2wt.  Four
// products give both bins g_a + h_m and g_a - h_m, so a (bin, observation)
// pair costs two multiply-adds for the sums with y and two for those at 2wt.
//
// Precision: every factor v is split as v = hi + lo with hi = f16(v) and
// lo = f16(v - hi) (22 significant bits), and a product is taken as
// hi hi + hi lo + lo hi on v_mfma_f32_32x32x16_f16, whose products are exact
// and whose accumulators are FP32.  What is dropped, lo lo, is at most 2^-24
// of the factors' range.  Every factor's phase is one FP64 product, reduced
// exactly in FP64, into the hardware sine and cosine, so no error grows along
// a recurrence.  The magnitudes are scaled by a power of two per object
// (ObjMeta::exps) into the range where f16 keeps both halves normal.
//
// Work per 32 x 32 tile (2,048 bins) and 16 observations: 24 matrix
// instructions; one factor pair (sine and cosine, double angle, splits) per
// (a, j) and per (m, j).  A wave makes its own centre factors straight into
// the registers the matrix instructions read; the offset factors are the same
// for every block of an object, so a workgroup's waves make a quarter each and
// share them through LDS.
//
// What bounds it: the card's power.  With all slices' operands in registers and
// nothing but these matrix instructions the clock falls to 1.6 GHz (a large
// FP16 library product reaches 1.09 PFLOP/s); a long object's slice takes
// 0.74 us per SIMD, the same rate.  Taken without gain for that reason: fewer
// vector instructions for the factors (-13 %), the next slice's factors made
// between the matrix instructions, eight waves sharing the offset factors.
// Around the slices a tile costs 2.7 us per SIMD (staging, first factors, the
// powers of its bins).
//
// Measured, vector kernels -> here: 2,500 objects of 20..500 points on 250,000
// bins 19.3 -> 4.1 ms (8.5e12 -> 4.0e13 (observation, bin) pairs a second);
// 4,096 points on 500,000 bins 287 -> 70 us; error against 64 bits 1e-6 -> 2e-7.
#pragma once

#include "lsp_common.h"

namespace lsp {
namespace mx {

typedef _Float16 h8 __attribute__((ext_vector_type(8)));
typedef _Float16 h2 __attribute__((ext_vector_type(2)));
typedef float f2 __attribute__((ext_vector_type(2)));
typedef float f16v __attribute__((ext_vector_type(16)));

constexpr int kSlice = 16;                    // observations per matrix instruction
constexpr int kOffs = 32;                     // offsets h_m per block
constexpr int kBlk = 2 * kOffs;               // bins per block
constexpr int kRowsA = 32;                    // blocks per wave tile
constexpr int kWaveBins = kBlk * kRowsA;      // 2,048 bins
constexpr int kFix = kMxTile;                 // bins per fix-up tile

// hi and lo halves of two values: hi = f16(x), lo = f16(x - hi); x - hi is exact.
// Two mixed-precision fused multiply-adds (where the compiler does not know
// that their factor is -1) and a conversion of the pair.  Never as inline
// assembly: the compiler does not see what such an instruction writes, and in a
// generalized kernel it left one of the two wait states that the matrix
// instruction after it needs.  (v_fma_mixlo_f16 and v_fma_mixhi_f16, written
// so, were also slower: a survey batch 4,285 -> 4,194 us.)
__device__ __forceinline__ void split2(float x, float y, h2& hi, h2& lo) {
    hi = __builtin_convertvector((f2){x, y}, h2);
    float m1 = -1.0f;
    asm("" : "+s"(m1));
    lo = h2{(_Float16)fmaf((float)hi.x, m1, x), (_Float16)fmaf((float)hi.y, m1, y)};
}

__device__ __forceinline__ void put2(h8& v, int p, h2 x) {
    v[2 * p] = x.x;
    v[2 * p + 1] = x.y;
}

__device__ __forceinline__ void sincos_rev(double f, double tau, float& s, float& c) {
    double ph = f * tau;
    ph -= rint(ph);
    const float r = (float)ph;
    s = __builtin_amdgcn_sinf(r);
    c = __builtin_amdgcn_cosf(r);
}

// The factors of 8 observations: q[0..3] hi halves, q[4..7] lo halves of
// (u c, u s, (cos 2)/2 = c^2 - 1/2, (sin 2)/2 = c s).
struct Frag {
    h8 q[8];
};

// A side: u = the scaled magnitudes.
__device__ __forceinline__ void gen_a(Frag& F, double f, const double* tau, const float* u) {
#pragma unroll
    for (int p = 0; p < 4; ++p) {
        float s0, c0, s1, c1;
        sincos_rev(f, tau[2 * p], s0, c0);
        sincos_rev(f, tau[2 * p + 1], s1, c1);
        h2 hi, lo;
        split2(u[2 * p] * c0, u[2 * p + 1] * c1, hi, lo);
        put2(F.q[0], p, hi);
        put2(F.q[4], p, lo);
        split2(u[2 * p] * s0, u[2 * p + 1] * s1, hi, lo);
        put2(F.q[1], p, hi);
        put2(F.q[5], p, lo);
        split2(fmaf(c0, c0, -0.5f), fmaf(c1, c1, -0.5f), hi, lo);
        put2(F.q[2], p, hi);
        put2(F.q[6], p, lo);
        split2(c0 * s0, c1 * s1, hi, lo);
        put2(F.q[3], p, hi);
        put2(F.q[7], p, lo);
    }
}

// The offset factors of two observations, as pairs: hi halves v[0..3], lo v[4..7].
__device__ __forceinline__ void gen_b2(h2 (&v)[8], double h, const double* tau) {
    float s0, c0, s1, c1;
    sincos_rev(h, tau[0], s0, c0);
    sincos_rev(h, tau[1], s1, c1);
    split2(c0, c1, v[0], v[4]);
    split2(s0, s1, v[1], v[5]);
    split2(fmaf(c0, c0, -0.5f), fmaf(c1, c1, -0.5f), v[2], v[6]);
    split2(c0 * s0, c1 * s1, v[3], v[7]);
}

// Zero factors for the observations from `valid` on: the padding of an
// object's last slice.  (Only that slice is trimmed: a mask on every factor
// cost a sixth of the factors' instructions.)
__device__ __forceinline__ void trim_b2(h2 (&v)[8], int valid) {
    const uint32_t keep = valid >= 2 ? ~0u : valid == 1 ? 0xFFFFu : 0u;
#pragma unroll
    for (int q = 0; q < 8; ++q)
        v[q] = __builtin_bit_cast(h2, __builtin_bit_cast(uint32_t, v[q]) & keep);
}

// B side.  The caller trims the slice that holds padding.
__device__ __forceinline__ void gen_b(Frag& F, double h, const double* tau) {
#pragma unroll
    for (int p = 0; p < 4; ++p) {
        h2 v[8];
        gen_b2(v, h, tau + 2 * p);
#pragma unroll
        for (int q = 0; q < 8; ++q) put2(F.q[q], p, v[q]);
    }
}

__device__ __forceinline__ void trim_b(Frag& F, int valid) {
    typedef uint32_t u4 __attribute__((ext_vector_type(4)));
#pragma unroll
    for (int q = 0; q < 8; ++q) {
        u4 v = __builtin_bit_cast(u4, F.q[q]);
#pragma unroll
        for (int p = 0; p < 4; ++p)
            v[p] &= valid >= 2 * p + 2 ? ~0u : valid == 2 * p + 1 ? 0xFFFFu : 0u;
        F.q[q] = __builtin_bit_cast(h8, v);
    }
}

__device__ __forceinline__ f16v mm(h8 a, h8 b, f16v c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_f16(a, b, c, 0, 0, 0);
}

// acc[0..3]: (u c)(c), (u s)(s), (u s)(c), (u c)(s); acc[4..7]: the same at
// the double angle, times 1/4.  Accumulator element (row, column) is (block,
// offset), or (offset, block) with OFFS_FIRST.
template <bool OFFS_FIRST = false>
__device__ __forceinline__ void accumulate(f16v (&acc)[8], const Frag& A, const Frag& B) {
    // the three partial products of each sum, the four sums in turn, so that
    // consecutive instructions do not wait for each other
#pragma unroll
    for (int g = 0; g < 2; ++g)
#pragma unroll
        for (int part = 0; part < 3; ++part) {  // hi hi, lo hi, hi lo
            const h8 a0 = A.q[2 * g + (part == 1 ? 4 : 0)], a1 = A.q[2 * g + 1 + (part == 1 ? 4 : 0)];
            const h8 b0 = B.q[2 * g + (part == 2 ? 4 : 0)], b1 = B.q[2 * g + 1 + (part == 2 ? 4 : 0)];
            auto add = [&](int k, h8 a, h8 b) {
                acc[4 * g + k] = OFFS_FIRST ? mm(b, a, acc[4 * g + k]) : mm(a, b, acc[4 * g + k]);
            };
            add(0, a0, b0);
            add(1, a1, b1);
            add(2, a1, b0);
            add(3, a0, b1);
        }
}

// The factor from the power in scaled magnitudes to the reported one, in two
// parts: unnormalised powers of magnitudes of 1e-18 are ordinary floats, the
// factor is not.  The first is a power of two, so a power that needs one part
// rounds as it would with the whole factor.
struct PowerScale {
    float two, rest;
};

__device__ __forceinline__ PowerScale power_scale(double f) {
    const int e = f > 0.0 ? ilogb(f) / 2 : 0;
    return PowerScale{(float)ldexp(1.0, e), (float)ldexp(f, -e)};
}

// Power of one bin from its sums, the double-angle sums at 1/4 (power32 with
// N/4 for N): P = (A N - B R) / (N^2 - R^2), `ill` as in power32.
__device__ __forceinline__ float power_mx(float xc, float xs, float c2, float s2, float n4,
                                          PowerScale scale4, bool& ill) {
    const float r2 = fmaf(c2, c2, s2 * s2);
    const float n2 = n4 * n4;
    ill = !(r2 < (1.0f - kIllTheta) * (1.0f - kIllTheta) * n2);
    const float a = fmaf(xc, xc, xs * xs);
    const float br = fmaf(fmaf(xc, xc, -(xs * xs)), c2, 2.0f * xc * xs * s2);
    return fmaxf(fmaf(a, n4, -br), 0.0f) * __builtin_amdgcn_rcpf(n2 - r2) * scale4.two *
           scale4.rest;
}

}  // namespace mx
}  // namespace lsp
