// lsp_fx.h -- FP64 sums on the matrix cores, shared by the FP64 form and the
// FP64 fix-up of the FP32 forms.
//
// As in lsp_mx.hip, a bin's frequency is a block centre plus or minus an
// offset, f = G_a +- H_m (32 bins per block), and the angle-addition formulas
// turn the sums over observations into products of centre factors and offset
// factors, here in FP64 on v_mfma_f64_16x16x4_f64.  Every factor is an FP64
// sine and cosine of an exactly reduced phase (fx_sincos), one pair per
// (block or offset, observation) instead of one per (bin, observation).
//
// The grid's frequencies are rounded (grid_freq), so f_i = G_a +- H_m + e with a
// residual e of about one unit in the last place, which the phases of a long
// span can see (2 pi e tau ~ 1e-10).  It is applied to first order,
//   sum v exp(2 pi i f tau) = S + 2 pi i e D,   D = sum v tau exp(2 pi i (G +- H) tau),
// and since e is that small D needs few digits: it is accumulated from f16
// factors on v_mfma_f32_16x16x32_f16.  Where 2 pi e tau could exceed 1e-9
// (kFxResidual), so that D's rounding or the second order could show, the bins
// are evaluated one by one instead (fx_direct), as are those of objects of a
// few points (fx_few), whose moment matrix is often close to singular.
//
// Per four observations a 512-bin tile takes eight matrix instructions (512
// cycles at their rate of 16 multiply-adds a cycle) and about 70 FP64 vector
// instructions for its factors, which the FP64 units execute in turn: the two
// bound it together.  Measured, a sine and cosine per (bin, observation) ->
// here: 48 objects of 50..1,000 points on 40,000 bins 2,250 -> 330 us; 256
// points on 10,000 bins 82 -> 24 us; 100 objects of 520 points on 40,000 bins
// 3.9e12 (observation, bin) pairs a second; the FP64 recompute of 300
// asteroid-like objects 1370 -> 78 us.  The error against an extended-
// precision evaluation is unchanged (3.8e-15 of the 2-norm).
//
// A bin whose smaller denominator (N - R, or T - R) is at most N/256 loses more
// than two digits of it to cancellation; it goes to a list of the workgroup's,
// and its sums are taken again term by term when the matrix sums are done
// (fx_direct).
#pragma once

#include "lsp_common.h"

namespace lsp {

typedef double fx_d4 __attribute__((ext_vector_type(4)));
typedef float fx_f4 __attribute__((ext_vector_type(4)));
typedef float fx_f2 __attribute__((ext_vector_type(2)));
typedef double fx_d2 __attribute__((ext_vector_type(2)));
typedef _Float16 fx_h2 __attribute__((ext_vector_type(2)));
typedef _Float16 fx_h8 __attribute__((ext_vector_type(8)));

constexpr int kFxOffs = 16;             // offsets per block
constexpr int kFxBlk = 2 * kFxOffs;     // bins per block
constexpr int kFxBins = 16 * kFxBlk;    // 512 bins of a wave tile
constexpr int kFxSteps = 8;             // FP64 matrix steps (four observations) per f16 product
constexpr int kFxObs = 256;             // observations staged per pass
constexpr double kFxResidual = 1e-9;
constexpr double kFxIll = 1.0 / 256.0;
// Objects of up to this many points are evaluated bin by bin, in a tile of their
// own and in the fix-up, whose waves share one.  Measured, bin by bin / matrix
// (us): 2,000 objects on 10,000 bins, 4 points 317 / 428, 5 points 346 / 266, with
// errors 6 points 330 / 354, 8 points 391 / 292; fix-up of 300 objects of two to four
// clumps on 20,000 bins, 16 points 970 / 1,106, 24 points 1,270 / 1,211, with errors
// 32 points 783 / 905, 48 points 1,016 / 948.
constexpr int fx_few(bool gen) { return gen ? 6 : 4; }
constexpr int fx_few_fix(bool gen) { return gen ? 32 : 20; }

// Sums of a wave tile.  Complex sums: the standard form has sum y e and
// sum e^2 / 2, the generalized one sum w e, sum w yw e and sum w e^2 / 2
// (e = exp(2 pi i f tau)).  x[4 g + ..]: the four products of sum g,
// d: the same with tau, in scaled units.
template <bool GEN>
struct FxSums {
    static constexpr int kSums = GEN ? 3 : 2;
    fx_d4 x[4 * kSums];
    fx_f4 d[4 * kSums];
};

// Staged observations (LDS).  u: y - ybar (standard) or w (yw and w: w yw, w);
// the float values are those times tau, scaled into f16's range.
template <bool GEN>
struct FxStage {
    double hi[kFxObs], lo[kFxObs];
    double u[kFxObs];                 // y - ybar, or w (y - ybar)
    double w[GEN ? kFxObs : 1];       // generalized: weights
    float ut[kFxObs];                 // u tau
    float wt[kFxObs];                 // tau, or w tau
};

struct FxScales {
    double up_u, up_w, up_t;  // powers of two: u, w and tau into f16's range
};

template <bool GEN>
__device__ __forceinline__ FxScales fx_scales(const ObjMeta& m) {
    FxScales s;
    s.up_u = ldexp(1.0, mx_exp_y(m));
    s.up_w = GEN ? ldexp(1.0, mx_exp_w(m)) : 1.0;
    s.up_t = ldexp(1.0, -mx_exp_reach(m));  // |tau| up_t <= 1
    return s;
}

// Steps of a wave with a tile of its own that are taken together, without a
// branch between them, so that their chains of dependent FP64 operations
// overlap; a pass is padded to whole groups with observations that weigh nothing.
// Steps alone, in twos, in fours: 48 objects of 50 to 1,000 points on 40,000 bins
// 357, 301 and 312 us (kernel); 1,000 generalized ones on 50,000 bins 4.47, 3.90
// and 3.79 ms.
constexpr int fx_group(bool gen) { return gen ? 4 : 2; }

template <bool GEN>
__device__ __forceinline__ void fx_stage(FxStage<GEN>& S, const ObjMeta& m,
                                         const double* __restrict__ t,
                                         const double* __restrict__ y,
                                         const double* __restrict__ dy, int64_t jt, int cnt,
                                         const FxScales& sc, int threads) {
    constexpr int kGroup = 4 * fx_group(GEN);
    const int padded = (cnt + kGroup - 1) / kGroup * kGroup;
    for (int q = threadIdx.x; q < padded; q += threads) {
        const int64_t j = m.j0 + jt + q;
        double hi = 0.0, lo = 0.0, u = 0.0, w = 0.0;
        if (q < cnt) {
            recentre64(t[j], m.t0, &hi, &lo);
            w = GEN ? gen_weight(dy, j, m.wnorm) : 1.0;
            u = w * (y[j] - m.ybar);
        }
        S.hi[q] = hi;
        S.lo[q] = lo;
        S.u[q] = u;
        if (GEN) S.w[q] = w;
        const double ts = hi * sc.up_t;
        S.ut[q] = (float)(u * sc.up_u * ts);
        S.wt[q] = (float)(w * sc.up_w * ts);
    }
}

// The operand of the lane that holds row 4 b + a, for a lane of row 4 a + b.
__device__ __forceinline__ fx_h8 fx_transpose_rows(fx_h8 v, int lane) {
    typedef int i4 __attribute__((ext_vector_type(4)));
    const int from = (lane & 48) | ((lane & 3) << 2) | ((lane >> 2) & 3);
    i4 x = __builtin_bit_cast(i4, v);
#pragma unroll
    for (int k = 0; k < 4; ++k) x[k] = __builtin_amdgcn_ds_bpermute(from << 2, x[k]);
    return __builtin_bit_cast(fx_h8, x);
}

// sin and cos of 2 pi f (hi + lo), the phase reduced exactly as in
// sincos_cycles64, then to a quarter turn about zero, |x| <= pi/4, and the
// Taylor series there: to x^17 and x^16, whose first dropped terms are below
// 2^-60.  The library function spends as many FP64 operations and, on its
// selections for arguments that cannot occur here, about forty more.
__device__ __forceinline__ void fx_sincos(double f, double hi, double lo, double* sn, double* cs) {
    double r;
    {
#pragma clang fp contract(off)
        const double p = f * hi;
        const double e = fma(f, hi, -p);
        r = (p - rint(p)) + fma(f, lo, e);
    }
    const double k = rint(4.0 * r);
    const double x = kTwoPi * fma(-0.25, k, r);
    const double z = x * x;
    double ps = fma(z, 1.0 / 355687428096000.0, -1.0 / 1307674368000.0);
    ps = fma(z, ps, 1.0 / 6227020800.0);
    ps = fma(z, ps, -1.0 / 39916800.0);
    ps = fma(z, ps, 1.0 / 362880.0);
    ps = fma(z, ps, -1.0 / 5040.0);
    ps = fma(z, ps, 1.0 / 120.0);
    ps = fma(z, ps, -1.0 / 6.0);
    const double s0 = fma(x * z, ps, x);
    double pc = fma(z, 1.0 / 20922789888000.0, -1.0 / 87178291200.0);
    pc = fma(z, pc, 1.0 / 479001600.0);
    pc = fma(z, pc, -1.0 / 3628800.0);
    pc = fma(z, pc, 1.0 / 40320.0);
    pc = fma(z, pc, -1.0 / 720.0);
    pc = fma(z, pc, 1.0 / 24.0);
    pc = fma(z, pc, -0.5);
    const double c0 = fma(z, pc, 1.0);
    // rotate by k quarter turns: swap on odd k, then the signs
    const int q = (int)(float)k;
    const double sx = (q & 1) ? c0 : s0, cx = (q & 1) ? s0 : c0;
    const uint64_t top = 1ull << 63;
    *sn = __longlong_as_double(__double_as_longlong(sx) ^ ((q & 2) ? top : 0ull));
    *cs = __longlong_as_double(__double_as_longlong(cx) ^ (((q + 1) & 2) ? top : 0ull));
}

// Offset factors of one round of steps, in two buffers, for the waves of a
// workgroup that have tiles of one row: the FP64 cosine and sine, and the four
// f16 factors.
struct FxOffsets {
    fx_d2 x[2][kFxSteps][kWave];
    fx_h8 h[2][4][kWave];
};

struct FxOffset {
    double c, s;
    _Float16 h[4];
};

__device__ __forceinline__ FxOffset fx_make_offset(double H, double th, double tl) {
    FxOffset o;
    fx_sincos(H, th, tl, &o.s, &o.c);
    const float cf = (float)o.c, sf = (float)o.s;
    const fx_h2 b1 = __builtin_convertvector((fx_f2){cf, sf}, fx_h2);
    o.h[0] = b1.x;
    o.h[1] = b1.y;
    o.h[2] = (_Float16)fmaf(cf, cf, -0.5f);
    o.h[3] = (_Float16)(cf * sf);
    return o;
}

// Add the steps [lo, hi) of four staged observations each to the wave's sums.
// Lane (row or column lane % 16, quarter lane / 16) supplies observation
// 4 step + quarter to both operands; eight steps feed one f16 product.
// WAVES > 0: all WAVES waves of the workgroup call with the same steps and H,
// make the offset factors of 8 / WAVES steps each and share them through O
// (48 objects of 50 to 1,000 points on 40,000 bins: 379 -> 357 us).  A wave
// without a tile (idle) makes its share only.
template <bool GEN, int WAVES = 0>
__device__ __forceinline__ void fx_accumulate(FxSums<GEN>& A, const FxStage<GEN>& S, int cnt,
                                              int lo, int hi, double G, double H, int lane,
                                              FxOffsets* O = nullptr, int wave = 0,
                                              bool idle = false) {
    constexpr int NG = FxSums<GEN>::kSums;
    const int quarter = lane >> 4;
    for (int s0 = lo; s0 < hi; s0 += kFxSteps) {
        const int steps = hi - s0 < kFxSteps ? hi - s0 : kFxSteps;
        fx_h8 ah[2 * NG], bh[4];
        const int buf = ((s0 - lo) / kFxSteps) & 1;
        if constexpr (WAVES > 0) {
            constexpr int kMine = kFxSteps / WAVES;
            _Float16 mine[4][kMine];
#pragma unroll
            for (int e = 0; e < kMine; ++e) {
                const int s = wave * kMine + e;
                const int j = 4 * (s < steps ? s0 + s : s0) + quarter;  // (past the end: unused)
                const FxOffset o = fx_make_offset(H, S.hi[j], S.lo[j]);
                O->x[buf][s][lane] = fx_d2{o.c, o.s};
#pragma unroll
                for (int q = 0; q < 4; ++q) mine[q][e] = o.h[q];
            }
#pragma unroll
            for (int q = 0; q < 4; ++q)
#pragma unroll
                for (int e = 0; e < kMine; ++e)
                    reinterpret_cast<_Float16*>(&O->h[buf][q][lane])[wave * kMine + e] = mine[q][e];
            __syncthreads();
            if (idle) continue;
        }
#pragma unroll
        for (int q = 0; q < 2 * NG; ++q) ah[q] = fx_h8{0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
        for (int q = 0; q < 4; ++q)
            bh[q] = WAVES > 0 ? O->h[buf][q][lane] : fx_h8{0, 0, 0, 0, 0, 0, 0, 0};
        constexpr int kGroup = WAVES > 0 ? fx_group(GEN) : 1;
#pragma unroll
        for (int sg = 0; sg < kFxSteps; sg += kGroup) {
            if (sg >= steps) break;
#pragma unroll
            for (int s = sg; s < sg + kGroup; ++s) {
                const int j = 4 * (s0 + s) + quarter;
                const double th = S.hi[j], tl = S.lo[j], u = S.u[j];
                const double one = j < cnt ? 1.0 : 0.0;  // padding weighs nothing
                double sn, cs;
                fx_sincos(G, th, tl, &sn, &cs);
                const double w = GEN ? S.w[j] : one;
                const double c2 = w * fma(cs, cs, -0.5), s2 = w * (cs * sn);
                double a[2 * NG];
                a[0] = (GEN ? w : u) * cs;
                a[1] = (GEN ? w : u) * sn;
                if (GEN) {
                    a[2] = u * cs;
                    a[3] = u * sn;
                }
                a[2 * NG - 2] = c2;
                a[2 * NG - 1] = s2;
                const float cf = (float)cs, sf = (float)sn, ut = S.ut[j], wt = S.wt[j];
                ah[0][s] = (_Float16)((GEN ? wt : ut) * cf);
                ah[1][s] = (_Float16)((GEN ? wt : ut) * sf);
                if (GEN) {
                    ah[2][s] = (_Float16)(ut * cf);
                    ah[3][s] = (_Float16)(ut * sf);
                }
                ah[2 * NG - 2][s] = (_Float16)(wt * fmaf(cf, cf, -0.5f));
                ah[2 * NG - 1][s] = (_Float16)(wt * (cf * sf));
                double bs, bc;
                if constexpr (WAVES > 0) {
                    const fx_d2 b = O->x[buf][s][lane];
                    bc = b[0];
                    bs = b[1];
                } else {
                    const FxOffset o = fx_make_offset(H, th, tl);
                    bc = o.c;
                    bs = o.s;
#pragma unroll
                    for (int q = 0; q < 4; ++q) bh[q][s] = o.h[q];
                }
                const double b2c = fma(bc, bc, -0.5), b2s = bc * bs;
#pragma unroll
                for (int g = 0; g < NG; ++g) {
                    const double c = g + 1 == NG ? b2c : bc, z = g + 1 == NG ? b2s : bs;
                    A.x[4 * g + 0] =
                        __builtin_amdgcn_mfma_f64_16x16x4f64(a[2 * g], c, A.x[4 * g + 0], 0, 0, 0);
                    A.x[4 * g + 1] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[2 * g + 1], z,
                                                                         A.x[4 * g + 1], 0, 0, 0);
                    A.x[4 * g + 2] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[2 * g + 1], c,
                                                                         A.x[4 * g + 2], 0, 0, 0);
                    A.x[4 * g + 3] =
                        __builtin_amdgcn_mfma_f64_16x16x4f64(a[2 * g], z, A.x[4 * g + 3], 0, 0, 0);
                }
            }
        }
        // the FP64 product leaves block row 4 r + quarter in element r, the f16
        // one row 4 quarter + r: transpose the rows that feed the latter
#pragma unroll
        for (int q = 0; q < 2 * NG; ++q) ah[q] = fx_transpose_rows(ah[q], lane);
#pragma unroll
        for (int g = 0; g < NG; ++g) {
            const fx_h8 c = bh[g + 1 == NG ? 2 : 0], z = bh[g + 1 == NG ? 3 : 1];
            A.d[4 * g + 0] =
                __builtin_amdgcn_mfma_f32_16x16x32_f16(ah[2 * g], c, A.d[4 * g + 0], 0, 0, 0);
            A.d[4 * g + 1] =
                __builtin_amdgcn_mfma_f32_16x16x32_f16(ah[2 * g + 1], z, A.d[4 * g + 1], 0, 0, 0);
            A.d[4 * g + 2] =
                __builtin_amdgcn_mfma_f32_16x16x32_f16(ah[2 * g + 1], c, A.d[4 * g + 2], 0, 0, 0);
            A.d[4 * g + 3] =
                __builtin_amdgcn_mfma_f32_16x16x32_f16(ah[2 * g], z, A.d[4 * g + 3], 0, 0, 0);
        }
    }
}

template <bool GEN>
__device__ __forceinline__ void fx_zero(FxSums<GEN>& A) {
#pragma unroll
    for (int q = 0; q < 4 * FxSums<GEN>::kSums; ++q) {
        A.x[q] = fx_d4{0.0, 0.0, 0.0, 0.0};
        A.d[q] = fx_f4{0.0f, 0.0f, 0.0f, 0.0f};
    }
}

// Power of the bin at frequency f (cycles) = G + side H + e from the products
// x and d of its block and offset (side -1 or +1).  `ill`: its sums have to be
// taken term by term (fx_direct).
template <bool GEN>
__device__ __forceinline__ double fx_power(const double (&x)[4 * FxSums<GEN>::kSums],
                                           const float (&d)[4 * FxSums<GEN>::kSums], double f,
                                           double G, double H, double side, const ObjMeta& m,
                                           const FxScales& sc, bool& ill) {
    constexpr int NG = FxSums<GEN>::kSums;
    const double h = side * H;
    double e;  // f - (G + h), the sum's rounding error included (two-sum)
    {
#pragma clang fp contract(off)
        const double s = G + h;
        const double bb = s - G;
        const double err = (G - (s - bb)) + (h - bb);
        e = (f - s) - err;
    }
    double re[NG], im[NG];
#pragma unroll
    for (int g = 0; g < NG; ++g) {
        const bool weighted = GEN ? g == 1 : g == 0;  // sums of u, else of w
        const double back = (kTwoPi * e) * (1.0 / ((weighted ? sc.up_u : sc.up_w) * sc.up_t)) *
                            (g + 1 == NG ? 2.0 : 1.0);
        const double dr = (double)d[4 * g] - side * (double)d[4 * g + 1];
        const double di = (double)d[4 * g + 2] + side * (double)d[4 * g + 3];
        re[g] = fma(-back, di, x[4 * g] - side * x[4 * g + 1]);
        im[g] = fma(back, dr, x[4 * g + 2] + side * x[4 * g + 3]);
    }
    // the double-angle factors are halves on both sides
    const double c2 = 4.0 * re[NG - 1], s2 = 4.0 * im[NG - 1];
    const double n = (double)m.n;
    double p, tr = n, dd = c2, ee = s2;  // trace, and the difference R = |(dd, ee)|
    if (GEN) {
        const double rn = 1.0 / n;
        tr = n - (re[0] * re[0] + im[0] * im[0]) * rn;
        dd = c2 - (re[0] * re[0] - im[0] * im[0]) * rn;
        ee = s2 - 2.0 * re[0] * im[0] * rn;
        p = power64_gen(SumsGen64{re[0], im[0], re[1], im[1], 0.5 * (n + c2), 0.5 * (n - c2),
                                  0.5 * s2},
                        n, m.scale);
    } else {
        p = power64_shifted(re[0], im[0], c2, s2, n, n, m.scale);
    }
    const double edge = tr - kFxIll * n;
    ill = !(edge > 0.0 && dd * dd + ee * ee < edge * edge);
    return p;
}

// Bins (from the first of a workgroup's) left to fx_direct.
template <int N>
struct FxList {
    int count;
    uint16_t bin[N];
};

// Adds the lanes' bins where `bad` holds.  Called by all lanes of a wavefront.
template <int N>
__device__ __forceinline__ void fx_list(FxList<N>& L, int bin, bool bad, int lane) {
    const unsigned long long bits = __ballot(bad);
    if (!bits) return;
    int base = 0;
    if (lane == 0) base = atomicAdd(&L.count, __popcll(bits));
    base = uniform_i32(base);
    if (bad) L.bin[base + __popcll(bits & ((1ull << lane) - 1))] = (uint16_t)bin;
}

// Powers of `count` bins term by term, bin(q) the q-th, each handed to
// offer(bin, power) by one thread; called by all threads of the workgroup.  A
// thread takes four bins at a time, so that their chains of FP64 operations
// overlap; where there are fewer bins than that, groups of up to 64 lanes share
// four bins and split the observations.  `staged`: S holds the object's only pass.
// Bound by the FP64 units, as the plain FP64 kernel is.  Measured, each lane its
// bin from global memory, or each listed bin by a wavefront of its own -> here:
// 48 objects of 500 points on 40,000 bins past the residual's range 2,543 -> 1,407
// us (two bins at a time 1,516), with errors 3,515 -> 1,519; 300 objects of 200
// points in two clumps with errors 4,783 -> 1,137 us; 300 of six points 3,659 -> 146.
constexpr int kFxTogether = 4;

template <bool GEN, int THREADS, typename Bin, typename Offer>
__device__ __forceinline__ void fx_direct(FxStage<GEN>& S, bool staged, const ObjMeta& m,
                                          const double* __restrict__ t,
                                          const double* __restrict__ y,
                                          const double* __restrict__ dy, const FxScales& sc,
                                          double f_min, double df, double to_cyc, int count,
                                          Bin bin, Offer offer) {
    constexpr int NV = GEN ? 7 : 5, KB = kFxTogether;
    int log_g = 0;
    while (log_g < 6 && (count << log_g) <= THREADS * KB / 2) ++log_g;
    const int per = THREADS >> log_g;  // groups of lanes
    const int sub = threadIdx.x & ((1 << log_g) - 1), group = threadIdx.x >> log_g;
    for (int r0 = 0; r0 < count; r0 += KB * per) {
        int64_t i[KB];
        double f[KB], v[KB][NV];
#pragma unroll
        for (int e = 0; e < KB; ++e) {
            const int q = r0 + e * per + group;
            i[e] = bin(q < count ? q : r0);
            f[e] = grid_freq(f_min, df, i[e]) * to_cyc;
            if (q >= count) i[e] = -1;
#pragma unroll
            for (int k = 0; k < NV; ++k) v[e][k] = 0.0;
        }
        for (int64_t jt = 0; jt < m.n; jt += kFxObs) {
            const int cnt = uniform_i32((int)(m.n - jt < kFxObs ? m.n - jt : kFxObs));
            if (!staged) {
                __syncthreads();
                fx_stage(S, m, t, y, dy, jt, cnt, sc, THREADS);
                __syncthreads();
                staged = m.n <= kFxObs;
            }
            for (int q = sub; q < cnt; q += 1 << log_g) {
                const double th = S.hi[q], tl = S.lo[q], u = S.u[q];
#pragma unroll
                for (int e = 0; e < KB; ++e) {
                    double sn, cs;
                    fx_sincos(f[e], th, tl, &sn, &cs);
                    v[e][0] = fma(u, cs, v[e][0]);
                    v[e][1] = fma(u, sn, v[e][1]);
                    double wc = cs, ws = sn;
                    if (GEN) {
                        const double w = S.w[q];
                        wc *= w;
                        ws *= w;
                        v[e][5] += wc;
                        v[e][6] += ws;
                    }
                    v[e][2] = fma(wc, cs, v[e][2]);
                    v[e][3] = fma(ws, sn, v[e][3]);
                    v[e][4] = fma(wc, sn, v[e][4]);
                }
            }
        }
        for (int o = (1 << log_g) >> 1; o > 0; o >>= 1)
#pragma unroll
            for (int e = 0; e < KB; ++e)
#pragma unroll
                for (int k = 0; k < NV; ++k) v[e][k] += __shfl_xor(v[e][k], o, kWave);
        if (sub == 0) {
#pragma unroll
            for (int e = 0; e < KB; ++e) {
                if (i[e] < 0) continue;
                double p;
                if constexpr (GEN)
                    p = power64_gen(SumsGen64{v[e][5], v[e][6], v[e][0], v[e][1], v[e][2], v[e][3],
                                              v[e][4]},
                                    (double)m.n, m.scale);
                else
                    p = power64(Sums64{v[e][0], v[e][1], v[e][2], v[e][3], v[e][4]}, (double)m.n,
                                m.scale);
                offer(i[e], p);
            }
        }
    }
}

// Whether the object's bins, whose frequencies (cycles) are at most f_top in
// size, go through the matrix cores: the first-order residual covers them, and
// there are more than `few` points.
__device__ __forceinline__ bool fx_covers(double f_top, const ObjMeta& m, int few) {
    return m.n > few && kTwoPi * 2.220446049250313e-16 * f_top * ldexp(1.0, mx_exp_reach(m)) <= kFxResidual;
}

// Wave w's share [lo, hi) of the steps of cnt staged observations.
template <int W>
__device__ __forceinline__ void fx_share(int cnt, int wave, int* lo, int* hi) {
    const int steps = (cnt + 3) / 4, per = (steps + W - 1) / W;
    *lo = wave * per < steps ? wave * per : steps;
    *hi = *lo + per < steps ? *lo + per : steps;
}

// The sums over the W waves of a workgroup, in wave order, of accumulator row
// `wave` (of the lane's four; waves from 4 on take part in the exchange only).
// Each round passes two of the products through LDS (d: four, as floats).
template <bool GEN, int W>
__device__ __forceinline__ void fx_gather(const FxSums<GEN>& A, double (*buf)[8][kWave], int wave,
                                          int lane, double (&x)[4 * FxSums<GEN>::kSums],
                                          float (&d)[4 * FxSums<GEN>::kSums]) {
    constexpr int NQ = 4 * FxSums<GEN>::kSums;
#pragma unroll
    for (int q = 0; q < NQ; q += 2) {
        __syncthreads();
#pragma unroll
        for (int r = 0; r < 8; ++r) buf[wave][r][lane] = A.x[q + r / 4][r % 4];
        __syncthreads();
        if (wave < 4) {
            double v0 = 0.0, v1 = 0.0;
#pragma unroll
            for (int w = 0; w < W; ++w) {
                v0 += buf[w][wave][lane];
                v1 += buf[w][4 + wave][lane];
            }
            x[q] = v0;
            x[q + 1] = v1;
        }
    }
    float (*fbuf)[16][kWave] = reinterpret_cast<float (*)[16][kWave]>(buf);
#pragma unroll
    for (int q = 0; q < NQ; q += 4) {
        __syncthreads();
#pragma unroll
        for (int r = 0; r < 16; ++r) fbuf[wave][r][lane] = A.d[q + r / 4][r % 4];
        __syncthreads();
        if (wave < 4)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                float v = 0.0f;
#pragma unroll
                for (int w = 0; w < W; ++w) v += fbuf[w][4 * e + wave][lane];
                d[q + e] = v;
            }
    }
}

// Centre frequency of a block row, and offset of a column, in cycles, for the
// tile whose first bin is w0.  Never contracted: the sums and the residual
// (fx_power) must see the same value.
__device__ __forceinline__ double fx_centre(double f_min, double df, double to_cyc, int64_t w0,
                                            int row) {
#pragma clang fp contract(off)
    return (f_min + df * ((double)(w0 + (int64_t)row * kFxBlk) + (kFxOffs - 0.5))) * to_cyc;
}
__device__ __forceinline__ double fx_offset(double df, double to_cyc, int col) {
#pragma clang fp contract(off)
    return (df * to_cyc) * ((double)col + 0.5);
}
// Accumulator element r of lane l holds block row 4 r + l / 16, offset l % 16.
__device__ __forceinline__ int fx_row(int r, int lane) { return 4 * r + (lane >> 4); }

}  // namespace lsp
