// lsp_features.hip -- per-object features for the learned band proposal.
//
// The paper evaluates every bin of every object.  The learned path first
// computes, per object, 1,088 cheap features and lets a small network propose
// the few frequency bands worth evaluating.  Two kernels fill one feature row
// per object:
//
//   coarse_kernel : the object is cut into seasons (a new season at every gap
//     longer than `season_gap`), and consecutive seasons are grouped until a
//     group holds at least `min_season_obs` observations (a trailing group
//     with fewer is dropped).  For each group, the normalised Lomb-Scargle
//     power of Section 2 (Eq. 1-2 without tau) of the object's
//     centred magnitudes y - ybar is evaluated on 8,192 bins over
//     [f_min, f_max), max-pooled over runs of 8 bins and averaged over the
//     groups -> features [0, 1024).  The group's own mean is not removed
//     again: that only changes power near zero frequency, and it keeps the
//     sums those of the FP32 form, taken the same way on the matrix cores
//     (lsp_mx.h), with the same FP64 recompute of bins FP32 cannot resolve.
//   window_kernel : one workgroup per object computes sampling and magnitude
//     statistics in FP64 and the spectral window at 53 probe frequencies
//     (FP64 phases, hardware FP32 sin/cos, FP64 sums) -> features [1024, 1088).
//
// Objects whose status is not OK get an all-zero row.
#include <math.h>

#include <cmath>

#include "lsp_mx.h"

namespace lsp {
namespace {

constexpr int kCoarseW = 4;      // wavefronts per workgroup, 2,048 bins each
constexpr int kCoarseBins = LSP_FEAT_COARSE * LSP_FEAT_POOL;
constexpr int kRound = 4;        // slices of offset factors made at a time
constexpr int kProbes = LSP_FEAT_WINDOW - 11;
constexpr int kWindowStage = 1024;  // observations per pass of the window kernel

static_assert(LSP_FEAT_POOL == 8, "a pool is two runs of four accumulator rows");
constexpr int kCoarseParts = kCoarseBins / (kCoarseW * mx::kWaveBins);  // workgroups per object

struct FeatParams {
    const ObjMeta* meta;
    const double* t;
    const double* y;
    double f_min, df, to_cyc;  // coarse grid: df = (f_max - f_min) / 8192
    double gap;
    int64_t n_obj;
    int32_t min_obs;
    int32_t pad;
    float* out;            // [n_obj][LSP_FEAT_DIM]
    double probe[kProbes];  // spectral-window probe frequencies, 10^-3 .. 30 log-spaced
};

// Normalised power of the observations [g0, g0 + n) of one object (magnitudes
// centred on the object's mean, normalised by the group's own sum of
// squares) at f_cyc cycles per time unit, in FP64 as the main kernel's FP64
// form computes it: exact re-centred phases, library sin/cos, Eq. 1-2 through
// power64 with its drop rule.  Not inlined: its FP64 registers stay out of
// the coarse kernel's hot loop.
__device__ __noinline__ double group_power64(const double* __restrict__ t, const double* __restrict__ y,
                                double t0, double ybar, int64_t g0, int64_t n, double f_cyc) {
    Sums64 a = {0.0, 0.0, 0.0, 0.0, 0.0};
    double syy = 0.0;
    for (int64_t j = g0; j < g0 + n; ++j) {
        double s, c, hi, lo;
        recentre64(t[j], t0, &hi, &lo);
        sincos_cycles64(f_cyc, hi, lo, &s, &c);
        const double yj = y[j] - ybar;
        sums64_add(a, yj, s, c);
        syy = fma(yj, yj, syy);
    }
    return syy > 0.0 ? power64(a, (double)n, 2.0 / syy) : 0.0;
}

// The larger of the two half-wavefronts' values: `lo` pooled in lanes 0..31,
// `hi` in lanes 32..63 (one lane exchange for both).
__device__ __forceinline__ float pool_halves(float lo, float hi) {
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(lo), __float_as_uint(hi), false,
                                                    false);
    return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}

// The exponent e for which the largest of |u[q .. b)| times 2^e is in [2^13, 2^14),
// at most 100; the same in every lane.
__device__ __forceinline__ int run_exp(const float* u, int q, int b, int lane) {
    float top = 0.0f;
    for (int j = q + lane; j < b; j += kWave) top = fmaxf(top, fabsf(u[j]));
#pragma unroll
    for (int o = kWave / 2; o > 0; o >>= 1) top = fmaxf(top, __shfl_xor(top, o, kWave));
    const int e = 13 + 127 - (uniform_i32(__float_as_int(top)) >> 23);
    return e < 100 ? e : 100;
}

// One workgroup per object; a wave owns 2,048 of the 8,192 bins as a 32 x 32
// tile whose accumulator rows are the offsets and whose columns the blocks, so
// that a lane holds runs of four neighbouring bins and the pooling is one
// exchange of half-wavefronts.  The observations of a group are walked in
// slices of 16; the offset factors of up to four slices are made by the four
// waves together, in units of two observations, and shared through LDS.
// A group of 27 points costs two slices (48 matrix instructions a wave, 1,536
// cycles) and as many cycles again for its 32 powers a lane; what bounds it is
// the chain staging -> offset factors -> slices -> powers of one group after
// another, two waves a SIMD (some 80 registers of the group ends and the pass
// set-up are kept in scratch, none in the slices).  Measured, lane per bin -> here: 1,500 objects of
// 50..500 points 876 -> 330 us; one or two waves per workgroup 383 and 354 us.
__global__ __launch_bounds__(kWave* kCoarseW, 2) void coarse_kernel(const FeatParams P) {
    using namespace mx;
    __shared__ double s_tau[kTile + kSlice];
    __shared__ float s_u[kTile + kSlice];
    __shared__ h8 s_b[2][kRound][8][kWave];
    __shared__ unsigned long long s_starts[kTile / kWave];  // new-season flags, one bit each
    __shared__ unsigned long long s_large[kTile / kWave];   // magnitudes of 1 (scaled) and more

    const int64_t block = linear_block();
    if (block >= P.n_obj * kCoarseParts) return;
    const int64_t item = xcd_remap(block, P.n_obj * kCoarseParts);
    const int64_t obj = item / kCoarseParts;
    const int part = (int)(item - obj * kCoarseParts);
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
    const int sub = lane & 31, half = lane >> 5;
    float* out = P.out + obj * LSP_FEAT_DIM;
    const ObjMeta m = P.meta[obj];
    if (m.status != LSP_OBJ_OK) {
        constexpr int kOut = LSP_FEAT_COARSE / kCoarseParts;
        for (int q = tid; q < kOut; q += kWave * kCoarseW) out[part * kOut + q] = 0.0f;
        return;
    }
    const int w0 = (part * kCoarseW + wave) * kWaveBins;
    const double fa =
        (P.f_min + P.df * ((double)(w0 + sub * kBlk) + (kOffs - 0.5))) * P.to_cyc;
    const double hb = (P.df * P.to_cyc) * ((double)sub + 0.5);
    const double up = ldexp(1.0, mx_exp_y(m));

    f16v acc[8];
    auto clear = [&]() {
#pragma unroll
        for (int q = 0; q < 8; ++q)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[q][r] = 0.0f;
    };
    clear();
    // pooled sums of the groups' powers: bins 32 + 8 g .. of the lane's block
    // (lanes 0..31), or 24 - 8 g .. (lanes 32..63)
    float feat[4] = {0.0f, 0.0f, 0.0f, 0.0f};
    int n_good = 0, buf = 0;
    // the current group: its observation count, first observation and sum of
    // squares (this lane's share)
    int ns = 0;
    int64_t g0 = m.j0;
    float syy = 0.0f;
    // 2^e_group scales the group's magnitudes on top of the object's scale: a group
    // whose largest one is below 2^-14 of the object's keeps its bits in f16
    int e_group = 0;

    const int64_t j_end = m.j0 + m.n;
    for (int64_t jt = m.j0;; jt += kTile) {
        const bool over = jt >= j_end;
        const int cnt = over ? 0 : (int)(j_end - jt < kTile ? j_end - jt : kTile);
        if (!over) {
            __syncthreads();
#pragma unroll
            for (int r = wave; r < kTile / kWave; r += kCoarseW) {
                const int q = r * kWave + lane;
                const int64_t j = jt + q;
                bool starts = false;
                double tc = 0.0;
                float u = 0.0f;
                if (q < cnt) {
                    // (the previous time is loaded unconditionally, clamped to
                    // the object's first observation, so the two loads go out
                    // together)
                    const double tj = P.t[j], tprev = P.t[j > m.j0 ? j - 1 : j];
                    tc = tj - m.t0;
                    u = (float)((P.y[j] - m.ybar) * up);
                    starts = j > m.j0 && tj - tprev > P.gap;
                }
                s_tau[q] = tc;
                s_u[q] = u;
                const unsigned long long word = __ballot(starts), large = __ballot(fabsf(u) >= 1.0f);
                if (lane == 0) {
                    s_starts[r] = word;
                    s_large[r] = large;
                }
            }
            if (tid < kSlice) {  // a slice may read past the pass
                s_tau[kTile + tid] = 0.0;
                s_u[kTile + tid] = 0.0f;
            }
            __syncthreads();
        }
        int q = 0;
        do {
            // A season boundary closes the group once it holds min_obs
            // observations (sparser seasons merge with the next).
            bool close = over;
            if (!over) {
                const uint64_t here = (uint64_t)uniform_i64((int64_t)s_starts[q / kWave]);
                close = ((here >> (q % kWave)) & 1ull) && ns >= P.min_obs;
            }
            if (close) {
                if (ns >= P.min_obs) {
                    float sq = syy;
#pragma unroll
                    for (int o = kWave / 2; o > 0; o >>= 1) sq += __shfl_xor(sq, o, kWave);
                    const float n4 = 0.25f * (float)ns, n2 = n4 * n4;
                    const float edge = (1.0f - kIllTheta) * (1.0f - kIllTheta) * n2;
                    // scaled magnitudes in sums and norm alike, so no scale back
                    const float scale4 = sq > 0.0f ? 0.25f * 2.0f / sq : 0.0f;
#pragma unroll
                    for (int g = 0; g < 4; ++g) {
                        float best[2];
#pragma unroll
                        for (int side = 0; side < 2; ++side) {
                            // four neighbouring bins: power_mx without its scale
                            // and clamp, which follow the pooling
                            float p[4], r2[4];
                            const float z = side ? 1.0f : -1.0f;
#pragma unroll
                            for (int e = 0; e < 4; ++e) {
                                const int r = 4 * g + e;
                                const float xc = fmaf(-z, acc[1][r], acc[0][r]);
                                const float xs = fmaf(z, acc[3][r], acc[2][r]);
                                const float c2 = fmaf(-z, acc[5][r], acc[4][r]);
                                const float s2 = fmaf(z, acc[7][r], acc[6][r]);
                                r2[e] = fmaf(c2, c2, s2 * s2);
                                const float qc = xc * xc, qs = xs * xs;
                                const float br = fmaf(qc - qs, c2, (xc + xc) * (xs * s2));
                                p[e] = fmaf(qc + qs, n4, -br) * __builtin_amdgcn_rcpf(n2 - r2[e]);
                            }
                            const float top = fmaxf(fmaxf(r2[0], r2[1]), fmaxf(r2[2], r2[3]));
                            if (__any(!(top < edge))) {
                                // what FP32 cannot resolve (power_mx's `ill`)
#pragma unroll 1
                                for (int e = 0; e < 4; ++e) {
                                    const float re = e == 0 ? r2[0] : e == 1 ? r2[1] : e == 2 ? r2[2] : r2[3];
                                    if (!(re < edge)) {
                                        const int off = 8 * g + 4 * half + e;
                                        const int i = w0 + sub * kBlk +
                                                      (side ? kOffs + off : kOffs - 1 - off);
                                        const double f = grid_freq(P.f_min, P.df, i) * P.to_cyc;
                                        const float v = (float)group_power64(P.t, P.y, m.t0, m.ybar,
                                                                             g0, ns, f) / scale4;
#pragma unroll
                                        for (int k = 0; k < 4; ++k) p[k] = k == e ? v : p[k];
                                    }
                                }
                            }
                            best[side] = fmaxf(fmaxf(p[0], p[1]), fmaxf(p[2], p[3]));
                        }
                        feat[g] += fminf(fmaxf(pool_halves(best[1], best[0]) * scale4, 0.0f), 1.0f);
                    }
                    ++n_good;
                }
                if (over) break;
                clear();
                e_group = 0;
                ns = 0;
                g0 = jt + q;
                syy = 0.0f;
            }
            // the run to the first boundary after q at which the group is large
            // enough, or to the pass's end
            int b = cnt;
            for (int w = (q + 1) / kWave; w * kWave < cnt; ++w) {
                uint64_t bits = (uint64_t)uniform_i64((int64_t)s_starts[w]);
                if (w == (q + 1) / kWave) bits &= ~0ull << ((q + 1) % kWave);
                const int least = q + P.min_obs - ns;  // first index that may close it
                if (least > w * kWave) {
                    const int skip = least - w * kWave;
                    bits = skip >= kWave ? 0ull : bits & (~0ull << skip);
                }
                if (bits) {
                    b = w * kWave + (int)__builtin_ctzll(bits);
                    break;
                }
            }
            bool large = false;
            for (int w = q / kWave; w * kWave < b; ++w) {
                uint64_t bits = (uint64_t)uniform_i64((int64_t)s_large[w]);
                if (w == q / kWave) bits &= ~0ull << (q % kWave);
                if ((w + 1) * kWave > b) bits &= ~(~0ull << (b % kWave));
                large |= bits != 0ull;
            }
            if (!large || e_group != 0) {  // rare
                const int e = large ? 0 : run_exp(s_u, q, b, lane);
                if (ns == 0) {
                    e_group = e;
                } else if (e < e_group) {
                    const float down = ldexpf(1.0f, e - e_group);
                    syy = syy * down * down;
#pragma unroll
                    for (int k = 0; k < 4; ++k)
#pragma unroll
                        for (int r = 0; r < 16; ++r) acc[k][r] *= down;
                    e_group = e;
                }
                const float scale = ldexpf(1.0f, e_group);
                __syncthreads();
                for (int j = q + tid; j < b; j += kWave * kCoarseW) s_u[j] *= scale;
                __syncthreads();
            }
            for (int j = q + lane; j < b; j += kWave) syy = fmaf(s_u[j], s_u[j], syy);
            for (int c0 = q; c0 < b; c0 += kRound * kSlice) {
                const int left = b - c0;
                const int slices =
                    left < kRound * kSlice ? (left + kSlice - 1) / kSlice : kRound;
                for (int unit = wave; unit < 4 * slices; unit += kCoarseW) {
                    const int sl = unit >> 2, pair = unit & 3;
                    const int j = c0 + sl * kSlice + 8 * half + 2 * pair;
                    h2 v[8];
                    gen_b2(v, hb, s_tau + j);
                    if (left < (sl + 1) * kSlice) trim_b2(v, b - j);
#pragma unroll
                    for (int k = 0; k < 8; ++k)
                        reinterpret_cast<h2*>(&s_b[buf][sl][k][lane])[pair] = v[k];
                }
                __syncthreads();
                for (int sl = 0; sl < slices; ++sl) {
                    Frag A, B;
                    const int j = c0 + sl * kSlice + 8 * half;
                    gen_a(A, fa, s_tau + j, s_u + j);
#pragma unroll
                    for (int k = 0; k < 8; ++k) B.q[k] = s_b[buf][sl][k][lane];
                    accumulate<true>(acc, A, B);
                }
                buf ^= 1;
            }
            ns += b - q;
            q = b;
        } while (q < cnt);
        if (over) break;
    }

    const float inv = n_good > 0 ? 1.0f / (float)n_good : 0.0f;
    const int base = (w0 + sub * kBlk) / LSP_FEAT_POOL;
#pragma unroll
    for (int g = 0; g < 4; ++g) out[base + (half ? 3 - g : 4 + g)] = feat[g] * inv;
}

__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
    for (int o = kWave / 2; o > 0; o >>= 1) v += __shfl_xor(v, o, kWave);
    return v;
}

__device__ __forceinline__ double wave_max(double v) {
#pragma unroll
    for (int o = kWave / 2; o > 0; o >>= 1) v = fmax(v, __shfl_xor(v, o, kWave));
    return v;
}

__device__ __forceinline__ double wave_min(double v) {
#pragma unroll
    for (int o = kWave / 2; o > 0; o >>= 1) v = fmin(v, __shfl_xor(v, o, kWave));
    return v;
}

// One workgroup of four wavefronts per object.  The statistics are a pass over
// the object with all threads; then lane 11 + p of each wavefront sums probe p
// over a quarter of the observations, whose times it reads from LDS as
// broadcasts, so that no probe's sum is reduced across lanes.  Bound by
// latency (a few passes over 500 points at most): 1,500 objects of 50..500
// points take 28 us, against 75 us with one wavefront per object and a pair of
// wavefront reductions per probe.
constexpr int kWinW = 4;
constexpr int kWinThreads = kWinW * kWave;

struct WinStats {
    double tmin, tmax, m3, m4, amax, dsum, lsum, lsq, dcnt;
};

__global__ __launch_bounds__(kWinThreads) void window_kernel(const FeatParams P) {
    __shared__ double s_tc[kWindowStage];
    __shared__ unsigned long long s_starts[kWindowStage / kWave];  // new-season flags
    __shared__ WinStats s_stat[kWinW];
    __shared__ double s_sum[kWinW][2][kWave];
    const int64_t obj = linear_block();
    if (obj >= P.n_obj) return;
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
    float* out = P.out + obj * LSP_FEAT_DIM + LSP_FEAT_COARSE;
    const ObjMeta m = P.meta[obj];
    if (m.status != LSP_OBJ_OK) {
        if (wave == 0) out[lane] = 0.0f;
        return;
    }
    const int64_t j0 = m.j0, n = m.n, j1 = j0 + n;

    // Time span, moments of y - ybar, within-season spacings and seasons; the
    // spectral window |sum_j exp(2 pi i f_p t_j)|^2 / N^2 with phases taken
    // from the object's mid-span origin (the modulus does not depend on it),
    // reduced to [-1/2, 1/2] cycles in FP64, then the hardware FP32 sin/cos
    // (argument in revolutions) as in the periodogram kernels, summed in FP64.
    WinStats st = {__builtin_inf(), -__builtin_inf(), 0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
    int64_t n_seasons = 1, n_good = 0, good_obs = 0, start = j0;
    const double f = lane >= 11 ? P.probe[lane - 11] : 0.0;
    double sc = 0.0, ss = 0.0;
    for (int64_t jb = j0; jb < j1; jb += kWindowStage) {
        const int cnt = (int)(j1 - jb < kWindowStage ? j1 - jb : kWindowStage);
        __syncthreads();
        for (int q0 = wave * kWave; q0 < cnt; q0 += kWinThreads) {
            const int q = q0 + lane;
            bool begins = false;
            if (q < cnt) {
                const int64_t j = jb + q;
                const double tj = P.t[j], tprev = P.t[j > j0 ? j - 1 : j];
                const double yc = P.y[j] - m.ybar;
                s_tc[q] = tj - m.t0;
                st.tmin = fmin(st.tmin, tj);
                st.tmax = fmax(st.tmax, tj);
                const double y2 = yc * yc;
                st.m3 += y2 * yc;
                st.m4 += y2 * y2;
                st.amax = fmax(st.amax, fabs(yc));
                const double d = tj - tprev;
                begins = j > j0 && d > P.gap;
                if (j > j0 && !begins) {
                    const double l = log10(fmax(d, 1e-6));
                    st.dsum += d;
                    st.lsum += l;
                    st.lsq += l * l;
                    st.dcnt += 1.0;
                }
            }
            const unsigned long long word = __ballot(begins);
            if (lane == 0) s_starts[q0 / kWave] = word;
        }
        __syncthreads();
        // the season starts, in order (every thread walks the same words)
        for (int w = 0; w * kWave < cnt; ++w) {
            uint64_t mask = (uint64_t)uniform_i64((int64_t)s_starts[w]);
            while (mask) {
                const int64_t s = jb + w * kWave + __builtin_ctzll(mask);
                mask &= mask - 1;
                ++n_seasons;
                if (s - start >= P.min_obs) {
                    ++n_good;
                    good_obs += s - start;
                }
                start = s;
            }
        }
#pragma unroll 4
        for (int q = uniform_i32(wave); q < cnt; q += kWinW) {
            double ph = f * s_tc[q];
            ph -= rint(ph);
            const float r = (float)ph;
            sc += (double)__builtin_amdgcn_cosf(r);
            ss += (double)__builtin_amdgcn_sinf(r);
        }
    }
    if (j1 - start >= P.min_obs) {
        ++n_good;
        good_obs += j1 - start;
    }
    st.tmin = wave_min(st.tmin);
    st.tmax = wave_max(st.tmax);
    st.m3 = wave_sum(st.m3);
    st.m4 = wave_sum(st.m4);
    st.amax = wave_max(st.amax);
    st.dsum = wave_sum(st.dsum);
    st.lsum = wave_sum(st.lsum);
    st.lsq = wave_sum(st.lsq);
    st.dcnt = wave_sum(st.dcnt);
    if (lane == 0) s_stat[wave] = st;
    s_sum[wave][0][lane] = sc;
    s_sum[wave][1][lane] = ss;
    __syncthreads();
    if (wave != 0) return;
    st = s_stat[0];
    sc = s_sum[0][0][lane];
    ss = s_sum[0][1][lane];
#pragma unroll
    for (int w = 1; w < kWinW; ++w) {
        const WinStats o = s_stat[w];
        st.tmin = fmin(st.tmin, o.tmin);
        st.tmax = fmax(st.tmax, o.tmax);
        st.m3 += o.m3;
        st.m4 += o.m4;
        st.amax = fmax(st.amax, o.amax);
        st.dsum += o.dsum;
        st.lsum += o.lsum;
        st.lsq += o.lsq;
        st.dcnt += o.dcnt;
        sc += s_sum[w][0][lane];
        ss += s_sum[w][1][lane];
    }

    const double nd = (double)n;
    const double var = m.syy / nd;
    const double sigma = sqrt(var);
    double w = 0.0;
    switch (lane) {
        case 0: w = log10(nd); break;
        case 1: w = log10(fmax(st.tmax - st.tmin, 1e-3)); break;
        case 2: w = (double)n_seasons; break;
        case 3: w = (double)n_good; break;
        case 4: w = st.dcnt > 0.0 ? log10(fmax(st.dsum / st.dcnt, 1e-6)) : 0.0; break;
        case 5: {
            if (st.dcnt > 0.0) {
                const double mu = st.lsum / st.dcnt;
                w = sqrt(fmax(st.lsq / st.dcnt - mu * mu, 0.0));
            }
            break;
        }
        case 6: w = (double)good_obs / nd; break;
        case 7: w = sigma > 0.0 ? log10(sigma) : -30.0; break;
        case 8: w = sigma > 0.0 ? (st.m3 / nd) / (var * sigma) : 0.0; break;
        case 9: w = sigma > 0.0 ? (st.m4 / nd) / (var * var) - 3.0 : 0.0; break;
        case 10: w = sigma > 0.0 ? st.amax / sigma : 0.0; break;
        default: w = (sc * sc + ss * ss) / (nd * nd); break;
    }
    out[lane] = (float)w;
}

}  // namespace

static hipError_t launch_features(const ObjMeta* meta, const double* t, const double* y,
                                  double f_min, double f_max, int unit, double gap, int min_obs,
                                  int64_t n_obj, float* out, hipStream_t s) {
    if (n_obj <= 0) return hipSuccess;
    FeatParams p;
    p.meta = meta;
    p.t = t;
    p.y = y;
    p.f_min = f_min;
    p.df = (f_max - f_min) / (double)kCoarseBins;
    p.to_cyc = unit == LSP_UNIT_CYCLES ? 1.0 : kInvTwoPi;
    p.gap = gap;
    p.n_obj = n_obj;
    p.min_obs = min_obs;
    p.pad = 0;
    p.out = out;
    const double lstep = (log10(30.0) + 3.0) / (double)(kProbes - 1);
    for (int q = 0; q < kProbes; ++q) p.probe[q] = pow(10.0, -3.0 + (double)q * lstep);
    hipLaunchKernelGGL(coarse_kernel, grid_for(n_obj * kCoarseParts), dim3(kWave * kCoarseW), 0, s, p);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(window_kernel, grid_for(n_obj), dim3(kWinThreads), 0, s, p);
    return hipGetLastError();
}

}  // namespace lsp

extern "C" {

lsp_feature_options lsp_default_feature_options(void) {
    lsp_feature_options o = {};
    o.season_gap = 60.0;
    o.min_season_obs = 8;
    return o;
}

size_t lsp_features_workspace_bytes(int64_t n_obj) {
    if (n_obj < 1) return 0;
    // per-object statistics and 256 bytes to spare
    return ((size_t)n_obj * sizeof(lsp::ObjMeta) + 255) / 256 * 256 + 256;
}

lsp_status lsp_features(const int64_t* offsets, int64_t n_obj, int64_t n_obs, const double* t,
                        const double* y, const lsp_grid* grid, const lsp_feature_options* fopt_in,
                        float* features, void* workspace, size_t workspace_bytes, void* stream) {
    if (!offsets || !grid || !features || !workspace) return LSP_EINVAL;
    if (n_obj < 1 || n_obs < 0 || (n_obs > 0 && (!t || !y))) return LSP_EINVAL;
    if (!(std::isfinite(grid->f_min) && std::isfinite(grid->f_max) && grid->f_max > grid->f_min) ||
        !(grid->unit == LSP_UNIT_CYCLES || grid->unit == LSP_UNIT_ANGULAR))
        return LSP_EINVAL;
    const lsp_feature_options fo = fopt_in ? *fopt_in : lsp_default_feature_options();
    if (!(std::isfinite(fo.season_gap) && fo.season_gap >= 0.0) || fo.min_season_obs < 2)
        return LSP_EINVAL;
    if (reinterpret_cast<uintptr_t>(workspace) % 256) return LSP_EINVAL;
    if (workspace_bytes < lsp_features_workspace_bytes(n_obj)) return LSP_ENOMEM;
    if (n_obj > (((int64_t)1 << 31) - 1) / LSP_FEAT_POOL) return LSP_EUNSUPPORTED;
    hipStream_t s = static_cast<hipStream_t>(stream);
    lsp::PrepParams pp;
    pp.offsets = offsets;
    pp.t = t;
    pp.y = y;
    pp.n_obj = n_obj;
    pp.n_obs = n_obs;
    pp.subtract_mean = 1;
    pp.normalize = 1;
    pp.meta = static_cast<lsp::ObjMeta*>(workspace);
    if (lsp::launch_prep(pp, s) != hipSuccess) return LSP_EHIP;
    if (lsp::launch_features(pp.meta, t, y, grid->f_min, grid->f_max, grid->unit, fo.season_gap,
                             fo.min_season_obs, n_obj, features, s) != hipSuccess)
        return LSP_EHIP;
    return LSP_OK;
}

}  // extern "C"
