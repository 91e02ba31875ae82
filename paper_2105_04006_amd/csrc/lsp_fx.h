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
// and since e is that small D needs few digits: it is accumulated on the f16
// matrix cores from factors of two f16 halves each (22 significant bits; hi hi
// + hi lo + lo hi).  Where 2 pi e tau could exceed 1e-9 (kFxResidual), so that
// D's rounding (2^-22 of it) or the second order could show, the bins are
// evaluated one by one instead (fx_direct), as are those of objects of a few
// points (fx_few), whose moment matrix is often close to singular.  (With single
// f16 factors the error grew with the frequency, from 1.2e-15 at 12 to 3.7e-14 at
// 340 cycles a day on ten years.)
//
// Per four observations a 512-bin tile takes eight matrix instructions (512
// cycles at their rate of 16 multiply-adds a cycle) and about 70 FP64 vector
// instructions for its factors, which the FP64 units execute in turn: the two
// bound it together.  Measured, a sine and cosine per (bin, observation) ->
// here: 48 objects of 50..1,000 points on 40,000 bins 2,250 -> 319 us; 256
// points on 10,000 bins 82 -> 23 us; the FP64 recompute of 300 asteroid-like
// objects 1370 -> 78 us.  (The residual's second halves cost the first 2 %.)
// Error against an extended-precision evaluation (2-norm of a tile, ten years, 60
// and 1,000 points; the same arithmetic on the host): 2.4e-16 and 4.5e-16 from 12 to 340 cycles a day, term by term
// 2.1e-16 and 6.3e-16.
//
// A bin whose smaller denominator (N - R, or T - R) is at most N/256 loses more
// than two digits of it to cancellation; it goes to a list of the workgroup's,
// and its sums are taken again term by term when the matrix sums are done
// (fx_direct).
#pragma once

#include <type_traits>

#include "lsp_common.h"

namespace lsp {

typedef double fx_d4 __attribute__((ext_vector_type(4)));
typedef float fx_f4 __attribute__((ext_vector_type(4)));
typedef double fx_d2 __attribute__((ext_vector_type(2)));
typedef float fx_f2 __attribute__((ext_vector_type(2)));
typedef _Float16 fx_h2 __attribute__((ext_vector_type(2)));
typedef _Float16 fx_h4 __attribute__((ext_vector_type(4)));
typedef _Float16 fx_h8 __attribute__((ext_vector_type(8)));

constexpr int kFxOffs = 16;             // offsets per block
constexpr int kFxBlk = 2 * kFxOffs;     // bins per block
constexpr int kFxBins = 16 * kFxBlk;    // 512 bins of a wave tile
// FP64 matrix steps (four observations) per f16 product: eight of the waves that
// share their offset factors, four of those that make their own, whose f16
// operands would not fit the registers.
constexpr int kFxSteps = 8;
constexpr int kFxOwnSteps = 4;
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
    int back_u, back_w;       // exponents that take u tau and w tau back
};

template <bool GEN>
__device__ __forceinline__ FxScales fx_scales(const ObjMeta& m) {
    FxScales s;
    s.up_u = ldexp(1.0, mx_exp_y(m));
    s.up_w = GEN ? ldexp(1.0, mx_exp_w(m)) : 1.0;
    s.up_t = ldexp(1.0, -mx_exp_reach(m));  // |tau| up_t <= 1
    s.back_u = mx_exp_reach(m) - mx_exp_y(m);
    s.back_w = mx_exp_reach(m) - (GEN ? mx_exp_w(m) : 0);
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

__device__ __forceinline__ fx_f4 fx_mm(fx_h8 a, fx_h8 b, fx_f4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ fx_f4 fx_mm(fx_h4 a, fx_h4 b, fx_f4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x16f16(a, b, c, 0, 0, 0);
}

// sin and cos of 2 pi f (hi + lo), the phase reduced exactly as in
// sincos_cycles64, then to a quarter turn about zero, |x| <= pi/4, and the
// Taylor series there: to x^17 and x^16, whose first dropped terms are below
// 2^-63 and 2^-58.  The library function spends as many FP64 operations and, on its
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
// workgroup that have tiles of one row: the FP64 cosine and sine, and the f16
// halves of the four factors.
struct FxOffsets {
    fx_d2 x[2][kFxSteps][kWave];
    fx_h8 h[2][8][kWave];
};

struct FxOffset {
    double c, s;
    float v[4];  // the f16 factors
};

__device__ __forceinline__ FxOffset fx_make_offset(double H, double th, double tl) {
    FxOffset o;
    fx_sincos(H, th, tl, &o.s, &o.c);
    const float cf = (float)o.c, sf = (float)o.s;
    o.v[0] = cf;
    o.v[1] = sf;
    o.v[2] = fmaf(cf, cf, -0.5f);
    o.v[3] = cf * sf;
    return o;
}

// hi and lo halves of two values: hi = f16(x), lo = f16(x - hi) (lsp_mx.h).
__device__ __forceinline__ void fx_halves(float x, float y, fx_h2& hi, fx_h2& lo) {
    hi = __builtin_convertvector((fx_f2){x, y}, fx_h2);
    float m1 = -1.0f;
    asm("" : "+s"(m1));
    lo = __builtin_convertvector((fx_f2){fmaf((float)hi.x, m1, x), fmaf((float)hi.y, m1, y)}, fx_h2);
}

// The same into elements s and s + 1 of two operands.
template <typename H>
__device__ __forceinline__ void fx_put(H& hi, H& lo, int s, float x, float y) {
    fx_h2 a, b;
    fx_halves(x, y, a, b);
    hi[s] = a.x;
    hi[s + 1] = a.y;
    lo[s] = b.x;
    lo[s + 1] = b.y;
}

// Add the steps [lo, hi) of four staged observations each to the wave's sums.
// Lane (row or column lane % 16, quarter lane / 16) supplies observation
// 4 step + quarter to both operands.
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
    constexpr int kSteps = WAVES > 0 ? kFxSteps : kFxOwnSteps;
    typedef typename std::conditional<(WAVES > 0), fx_h8, fx_h4>::type Halves;
    const int quarter = lane >> 4;
    for (int s0 = lo; s0 < hi; s0 += kSteps) {
        const int steps = hi - s0 < kSteps ? hi - s0 : kSteps;
        Halves ah[4 * NG], bh[8];  // hi, then lo halves
        const int buf = ((s0 - lo) / kSteps) & 1;
        if constexpr (WAVES > 0) {
            static_assert(kSteps == 2 * WAVES, "a wave makes the factors of two steps");
            FxOffset o[2];
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                const int s = 2 * wave + e;
                const int j = 4 * (s < steps ? s0 + s : s0) + quarter;  // (past the end: unused)
                o[e] = fx_make_offset(H, S.hi[j], S.lo[j]);
                O->x[buf][s][lane] = fx_d2{o[e].c, o[e].s};
            }
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                fx_h2 a, b;
                fx_halves(o[0].v[q], o[1].v[q], a, b);
                reinterpret_cast<fx_h2*>(&O->h[buf][q][lane])[wave] = a;
                reinterpret_cast<fx_h2*>(&O->h[buf][q + 4][lane])[wave] = b;
            }
            __syncthreads();
            if (idle) continue;
        }
#pragma unroll
        for (int q = 0; q < 4 * NG; ++q) ah[q] = Halves{};
#pragma unroll
        for (int q = 0; q < 8; ++q) bh[q] = Halves{};
        float av[2 * NG][kSteps], bv[4][kSteps];
#pragma unroll
        for (int s = 0; s < kSteps; ++s) {
#pragma unroll
            for (int q = 0; q < 2 * NG; ++q) av[q][s] = 0.0f;
#pragma unroll
            for (int q = 0; q < 4; ++q) bv[q][s] = 0.0f;
        }
        constexpr int kGroup = WAVES > 0 ? fx_group(GEN) : 1;
#pragma unroll
        for (int sg = 0; sg < kSteps; sg += kGroup) {
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
                av[0][s] = (GEN ? wt : ut) * cf;
                av[1][s] = (GEN ? wt : ut) * sf;
                if (GEN) {
                    av[2][s] = ut * cf;
                    av[3][s] = ut * sf;
                }
                av[2 * NG - 2][s] = wt * fmaf(cf, cf, -0.5f);
                av[2 * NG - 1][s] = wt * (cf * sf);
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
                    for (int q = 0; q < 4; ++q) bv[q][s] = o.v[q];
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
            if constexpr (kGroup % 2 == 0)
#pragma unroll
                for (int s = sg; s < sg + kGroup; s += 2)
#pragma unroll
                    for (int q = 0; q < 2 * NG; ++q)
                        fx_put(ah[q], ah[q + 2 * NG], s, av[q][s], av[q][s + 1]);
        }
        if constexpr (kGroup == 1)
#pragma unroll
            for (int s = 0; s < kSteps; s += 2) {
#pragma unroll
                for (int q = 0; q < 2 * NG; ++q)
                    fx_put(ah[q], ah[q + 2 * NG], s, av[q][s], av[q][s + 1]);
#pragma unroll
                for (int q = 0; q < 4; ++q) fx_put(bh[q], bh[q + 4], s, bv[q][s], bv[q][s + 1]);
            }
        if constexpr (WAVES > 0)
#pragma unroll
            for (int q = 0; q < 8; ++q) bh[q] = O->h[buf][q][lane];
#pragma unroll
        for (int part = 0; part < 3; ++part) {  // hi hi, lo hi, hi lo
            const int ao = part == 1 ? 2 * NG : 0, bo = part == 2 ? 4 : 0;
#pragma unroll
            for (int g = 0; g < NG; ++g) {
                const Halves a0 = ah[ao + 2 * g], a1 = ah[ao + 2 * g + 1];
                const Halves c = bh[bo + (g + 1 == NG ? 2 : 0)], z = bh[bo + (g + 1 == NG ? 3 : 1)];
                A.d[4 * g + 0] = fx_mm(a0, c, A.d[4 * g + 0]);
                A.d[4 * g + 1] = fx_mm(a1, z, A.d[4 * g + 1]);
                A.d[4 * g + 2] = fx_mm(a1, c, A.d[4 * g + 2]);
                A.d[4 * g + 3] = fx_mm(a0, z, A.d[4 * g + 3]);
            }
        }
    }
}

// The FP64 product leaves block row 4 r + lane / 16 in element r, the f16 one row
// 4 (lane / 16) + r: the sums d of a whole tile, in x's places.  (Their operands'
// rows turned at each product instead took 328 us where this takes 319: 48 objects
// of 50 to 1,000 points on 40,000 bins.)
template <bool GEN>
__device__ __forceinline__ void fx_turn(FxSums<GEN>& A) {
    auto swap = [](auto f, float& a, float& b) {
        const auto r = f(__float_as_uint(a), __float_as_uint(b));
        a = __uint_as_float(r[0]);
        b = __uint_as_float(r[1]);
    };
    auto halves = [](uint32_t a, uint32_t b) {
        return __builtin_amdgcn_permlane32_swap(a, b, false, false);
    };
    auto rows = [](uint32_t a, uint32_t b) {
        return __builtin_amdgcn_permlane16_swap(a, b, false, false);
    };
#pragma unroll
    for (int q = 0; q < 4 * FxSums<GEN>::kSums; ++q) {
        float v[4] = {A.d[q][0], A.d[q][1], A.d[q][2], A.d[q][3]};
        swap(halves, v[0], v[2]);
        swap(halves, v[1], v[3]);
        swap(rows, v[0], v[1]);
        swap(rows, v[2], v[3]);
        A.d[q] = fx_f4{v[0], v[1], v[2], v[3]};
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
        const double back =
            ldexp(kTwoPi * e, (weighted ? sc.back_u : sc.back_w) + (g + 1 == NG ? 1 : 0));
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
    while (log_g < 6 && (count << log_g) <= THREADS * KB / 2 && (1 << log_g) < m.n) ++log_g;
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
        // the powers, which cost as much as a few terms: a bin for each of the
        // group's lanes, as far as they go
        const int share = 1 << log_g < KB ? 1 << log_g : KB;
#pragma unroll 1
        for (int j = 0; j < KB; j += share) {
            int64_t own = i[0];
            double w[NV];
#pragma unroll
            for (int k = 0; k < NV; ++k) w[k] = v[0][k];
#pragma unroll
            for (int e = 1; e < KB; ++e) {
                const bool it = j + sub == e;
                own = it ? i[e] : own;
#pragma unroll
                for (int k = 0; k < NV; ++k) w[k] = it ? v[e][k] : w[k];
            }
            if (sub >= share || own < 0) continue;
            if constexpr (GEN)
                offer(own, power64_gen(SumsGen64{w[5], w[6], w[0], w[1], w[2], w[3], w[4]},
                                       (double)m.n, m.scale));
            else
                offer(own, power64(Sums64{w[0], w[1], w[2], w[3], w[4]}, (double)m.n, m.scale));
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
    const int from = 16 * wave + (lane & 15);  // d's places are other than x's (fx_turn)
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
                for (int w = 0; w < W; ++w) v += fbuf[w][4 * e + (lane >> 4)][from];
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
