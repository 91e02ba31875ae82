// lsp_mx.hip -- the FP32 form's sums on the matrix cores.
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
// Measured, vector kernels -> here: 2,500 objects of 20..500 points on 250,000
// bins 19.6 -> 4.3 ms (8.3e12 -> 3.8e13 (observation, bin) pairs a second);
// 4,096 points on 500,000 bins 295 -> 76 us; error against 64 bits 1e-6 -> 2e-7.
#include "lsp_common.h"

namespace lsp {
namespace {

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

// hi and lo halves of two values: hi = f16(x), lo = f16(x - hi).
__device__ __forceinline__ void split2(float x, float y, h2& hi, h2& lo) {
    hi = __builtin_convertvector((f2){x, y}, h2);
    const float m1 = -1.0f;
    float lx, ly;
    // x - hi in one instruction each (a mixed-precision fused multiply-add)
    asm("v_fma_mix_f32 %0, %1, %2, %3 op_sel_hi:[1,0,0]" : "=v"(lx) : "v"(hi), "v"(m1), "v"(x));
    asm("v_fma_mix_f32 %0, %1, %2, %3 op_sel:[1,0,0] op_sel_hi:[1,0,0]"
        : "=v"(ly)
        : "v"(hi), "v"(m1), "v"(y));
    lo = __builtin_convertvector((f2){lx, ly}, h2);
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

// B side: observations from `valid` on are padding and get zero factors.
__device__ __forceinline__ void gen_b(Frag& F, double h, const double* tau, int valid) {
#pragma unroll
    for (int p = 0; p < 4; ++p) {
        float s0, c0, s1, c1;
        sincos_rev(h, tau[2 * p], s0, c0);
        sincos_rev(h, tau[2 * p + 1], s1, c1);
        const float w0 = 2 * p < valid ? 1.0f : 0.0f;
        const float w1 = 2 * p + 1 < valid ? 1.0f : 0.0f;
        c0 *= w0;
        s0 *= w0;
        c1 *= w1;
        s1 *= w1;
        h2 hi, lo;
        split2(c0, c1, hi, lo);
        put2(F.q[0], p, hi);
        put2(F.q[4], p, lo);
        split2(s0, s1, hi, lo);
        put2(F.q[1], p, hi);
        put2(F.q[5], p, lo);
        split2(fmaf(c0, c0, -0.5f * w0), fmaf(c1, c1, -0.5f * w1), hi, lo);
        put2(F.q[2], p, hi);
        put2(F.q[6], p, lo);
        split2(c0 * s0, c1 * s1, hi, lo);
        put2(F.q[3], p, hi);
        put2(F.q[7], p, lo);
    }
}

__device__ __forceinline__ f16v mm(h8 a, h8 b, f16v c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_f16(a, b, c, 0, 0, 0);
}

// acc[0..3]: (u c)(c), (u s)(s), (u s)(c), (u c)(s); acc[4..7]: the same at
// the double angle, times 1/4.
__device__ __forceinline__ void accumulate(f16v (&acc)[8], const Frag& A, const Frag& B) {
#pragma unroll
    for (int g = 0; g < 2; ++g) {
        const int o = 2 * g;
        // the three partial products of each sum, the four sums in turn, so
        // that consecutive instructions do not wait for each other
        acc[4 * g + 0] = mm(A.q[o], B.q[o], acc[4 * g + 0]);
        acc[4 * g + 1] = mm(A.q[o + 1], B.q[o + 1], acc[4 * g + 1]);
        acc[4 * g + 2] = mm(A.q[o + 1], B.q[o], acc[4 * g + 2]);
        acc[4 * g + 3] = mm(A.q[o], B.q[o + 1], acc[4 * g + 3]);
        acc[4 * g + 0] = mm(A.q[o + 4], B.q[o], acc[4 * g + 0]);
        acc[4 * g + 1] = mm(A.q[o + 5], B.q[o + 1], acc[4 * g + 1]);
        acc[4 * g + 2] = mm(A.q[o + 5], B.q[o], acc[4 * g + 2]);
        acc[4 * g + 3] = mm(A.q[o + 4], B.q[o + 1], acc[4 * g + 3]);
        acc[4 * g + 0] = mm(A.q[o], B.q[o + 4], acc[4 * g + 0]);
        acc[4 * g + 1] = mm(A.q[o + 1], B.q[o + 5], acc[4 * g + 1]);
        acc[4 * g + 2] = mm(A.q[o + 1], B.q[o + 4], acc[4 * g + 2]);
        acc[4 * g + 3] = mm(A.q[o], B.q[o + 5], acc[4 * g + 3]);
    }
}

// Power of one bin from its sums, the double-angle sums at 1/4 (power32 with
// N/4 for N): P = (A N - B R) / (N^2 - R^2), `ill` as in power32.
__device__ __forceinline__ float power_mx(float xc, float xs, float c2, float s2, float n4,
                                          float scale4, bool& ill) {
    const float r2 = fmaf(c2, c2, s2 * s2);
    const float n2 = n4 * n4;
    ill = !(r2 < (1.0f - kIllTheta) * (1.0f - kIllTheta) * n2);
    const float a = fmaf(xc, xc, xs * xs);
    const float br = fmaf(fmaf(xc, xc, -(xs * xs)), c2, 2.0f * xc * xs * s2);
    return fmaxf(fmaf(a, n4, -br), 0.0f) * __builtin_amdgcn_rcpf(n2 - r2) * scale4;
}

// The best bin of a lane: larger power first; bins are offered in increasing
// index, so a strict comparison keeps the lowest of equals.
struct LaneBest {
    float p;
    uint32_t i;
};

__device__ __forceinline__ unsigned long long lane_key(const LaneBest& b) {
    return b.p >= 0.0f ? ((unsigned long long)__float_as_uint(b.p > 0.0f ? b.p : 0.0f) << 32) |
                             (uint32_t)(0xFFFFFFFFu - b.i)
                       : 0ull;
}

struct Finish {
    float n4, scale4;
    int64_t f_lo, f_hi;  // the row's bins
    int64_t out;         // first periodogram element of the object
    void* pgram;
    int32_t f64;
};

// Both bins of (block row a, offset m) from their eight sums; i0 is the
// block's first bin.
__device__ __forceinline__ void finish_pair(const Finish& R, const float (&v)[8], int64_t i0, int m,
                                            LaneBest& best, bool& ill) {
    const int64_t im = i0 + (kOffs - 1 - m), ip = i0 + (kOffs + m);
    bool i_m, i_p;
    const float pm = power_mx(v[0] + v[1], v[2] - v[3], v[4] + v[5], v[6] - v[7], R.n4, R.scale4,
                              i_m);
    const float pp = power_mx(v[0] - v[1], v[2] + v[3], v[4] - v[5], v[6] + v[7], R.n4, R.scale4,
                              i_p);
    if (im < R.f_hi) {
        ill |= i_m;
        if (R.pgram) store_pgram(R.pgram, R.f64, R.out + im, (double)pm);
        if (pm > best.p) best = LaneBest{pm, (uint32_t)im};
    }
    if (ip < R.f_hi) {
        ill |= i_p;
        if (R.pgram) store_pgram(R.pgram, R.f64, R.out + ip, (double)pp);
        if (pp > best.p) best = LaneBest{pp, (uint32_t)ip};
    }
}

__device__ __forceinline__ Finish make_finish(const MainParams& P, const ObjMeta& m,
                                              const RowRange& rr) {
    Finish R;
    const double back = ldexp(1.0, -mx_exp_y(m));
    R.n4 = 0.25f * (float)m.n;
    R.scale4 = (float)(0.25 * (m.scale * back * back));
    R.f_lo = rr.f_lo;
    R.f_hi = rr.f_hi;
    R.out = rr.obj * P.n_f;
    R.pgram = P.pgram;
    R.f64 = P.pgram_f64;
    return R;
}

// Fill values of an object without a periodogram, bins [lo, hi).
__device__ __forceinline__ void fill_bins(const MainParams& P, const RowRange& rr, int32_t status,
                                          int64_t lo, int64_t hi, int threads) {
    if (!P.pgram) return;
    const double v = fill_value(status);
    if (hi > rr.f_hi) hi = rr.f_hi;
    for (int64_t i = lo + threadIdx.x; i < hi; i += threads)
        store_pgram(P.pgram, P.pgram_f64, rr.obj * P.n_f + i, v);
}

// W waves per workgroup, each with its own 32 x 32 tile (W consecutive runs of
// 2,048 bins of one row); they share the offset factors through LDS.
template <int W>
__global__ __launch_bounds__(kWave* W, 2) void mx_tile_kernel(const MainParams P) {
    __shared__ double s_tau[kTile];
    __shared__ float s_u[kTile];
    __shared__ h8 s_b[2][W][8][kWave];  // two buffers of W slices

    const int64_t b = linear_block();
    if (b >= P.n_items) return;
    const int64_t item = xcd_remap(b, P.n_items);
    const int64_t rank = item / P.chunks_per_row;
    const int64_t chunk = item - rank * P.chunks_per_row;
    const int64_t row = item_row(P.row_perm, rank);
    const RowRange rr =
        decode_row(P.row_obj, P.row_band, P.band_bins, P.rows_per_group, P.n_obj, P.n_f, row);
    const int64_t g0 = rr.f_lo + chunk * (int64_t)(W * kWaveBins);
    if (rr.obj < 0 || g0 >= rr.f_hi) return;
    const ObjMeta m = P.meta[rr.obj];
    if (m.status != LSP_OBJ_OK) {
        fill_bins(P, rr, m.status, g0, g0 + W * kWaveBins, kWave * W);
        return;
    }
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = threadIdx.x / kWave;
    const int sub = lane & 31, half = lane >> 5;
    const int64_t w0 = g0 + (int64_t)wave * kWaveBins;  // the wave's first bin
    // block centre of this lane's row, and this lane's offset, in cycles
    const double fa = (P.f_min + P.df * ((double)(w0 + (int64_t)sub * kBlk) + (kOffs - 0.5))) * P.to_cyc;
    const double hb = (P.df * P.to_cyc) * ((double)sub + 0.5);
    const double up = ldexp(1.0, mx_exp_y(m));

    f16v acc[8];
#pragma unroll
    for (int q = 0; q < 8; ++q)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[q][r] = 0.0f;

    int buf = 0;
    for (int64_t jt = 0; jt < m.n; jt += kTile) {
        const int cnt = (int)(m.n - jt < kTile ? m.n - jt : kTile);
        const int slices = (cnt + kSlice - 1) / kSlice;
        __syncthreads();
        for (int q = threadIdx.x; q < slices * kSlice; q += kWave * W) {
            const bool in = q < cnt;
            s_tau[q] = in ? P.t[m.j0 + jt + q] - m.t0 : 0.0;
            s_u[q] = in ? (float)((P.y[m.j0 + jt + q] - m.ybar) * up) : 0.0f;
        }
        __syncthreads();
        for (int s0 = 0; s0 < slices; s0 += W) {
            const int mine = s0 + wave;
            if (mine < slices) {
                Frag B;
                const int j = mine * kSlice + half * 8;
                gen_b(B, hb, s_tau + j, cnt - j);
#pragma unroll
                for (int q = 0; q < 8; ++q) s_b[buf][wave][q][lane] = B.q[q];
            }
            __syncthreads();
            const int todo = slices - s0 < W ? slices - s0 : W;
            for (int s = 0; s < todo; ++s) {
                Frag A, B;
                const int j = (s0 + s) * kSlice + half * 8;
                gen_a(A, fa, s_tau + j, s_u + j);
#pragma unroll
                for (int q = 0; q < 8; ++q) B.q[q] = s_b[buf][s][q][lane];
                accumulate(acc, A, B);
            }
            buf ^= 1;
        }
    }

    const Finish R = make_finish(P, m, rr);
    unsigned long long best = 0ull;
#pragma unroll
    for (int t = 0; t < kWaveBins / kFix; ++t) {
        LaneBest lb{-1.0f, 0u};
        bool ill = false;
#pragma unroll
        for (int r = 8 * t; r < 8 * t + 8; ++r) {
            const int a = 8 * (r / 4) + 4 * half + (r & 3);
            float v[8];
#pragma unroll
            for (int q = 0; q < 8; ++q) v[q] = acc[q][r];
            finish_pair(R, v, w0 + (int64_t)a * kBlk, sub, lb, ill);
        }
        if (__any(ill)) {
            const int64_t tile = row * P.tiles_per_row + (w0 - rr.f_lo) / kFix + t;
            if (lane == 0) atomicOr(&P.ill_bits[tile >> 5], 1u << (tile & 31));
        } else {
            best = umax64(best, lane_key(lb));
        }
    }
    best = wave_max_u64(best);
    if (lane == 0 && best != 0ull) atomicMax(&P.keys[row / P.rows_per_group], best);
}

// One 32 x 32 tile per workgroup of eight waves, which share out the
// observations in slices and add their sums through LDS in wave order: for a
// single series, whose tiles alone are too few to fill the chip.
constexpr int kSplitW = 8;
constexpr int kSplitObs = 1024;  // observations staged per pass

__global__ __launch_bounds__(kWave* kSplitW, 2) void mx_split_kernel(const MainParams P) {
    __shared__ double s_tau[kSplitObs];
    __shared__ float s_u[kSplitObs];
    __shared__ float s_sum[2][kSplitW][16][kWave];
    __shared__ unsigned long long s_key[kSplitW];
    __shared__ int s_ill[kSplitW];

    const int64_t b = linear_block();
    if (b >= P.n_items) return;
    const int64_t rank = b / P.chunks_per_row;
    const int64_t chunk = b - rank * P.chunks_per_row;
    const int64_t row = item_row(P.row_perm, rank);
    const RowRange rr =
        decode_row(P.row_obj, P.row_band, P.band_bins, P.rows_per_group, P.n_obj, P.n_f, row);
    const int64_t w0 = rr.f_lo + chunk * (int64_t)kWaveBins;
    if (rr.obj < 0 || w0 >= rr.f_hi) return;
    const ObjMeta m = P.meta[rr.obj];
    if (m.status != LSP_OBJ_OK) {
        fill_bins(P, rr, m.status, w0, w0 + kWaveBins, kWave * kSplitW);
        return;
    }
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = threadIdx.x / kWave;
    const int sub = lane & 31, half = lane >> 5;
    const double fa = (P.f_min + P.df * ((double)(w0 + (int64_t)sub * kBlk) + (kOffs - 0.5))) * P.to_cyc;
    const double hb = (P.df * P.to_cyc) * ((double)sub + 0.5);
    const double up = ldexp(1.0, mx_exp_y(m));

    f16v acc[8];
#pragma unroll
    for (int q = 0; q < 8; ++q)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[q][r] = 0.0f;

    for (int64_t jt = 0; jt < m.n; jt += kSplitObs) {
        const int cnt = (int)(m.n - jt < kSplitObs ? m.n - jt : kSplitObs);
        const int slices = (cnt + kSlice - 1) / kSlice;
        __syncthreads();
        for (int q = threadIdx.x; q < slices * kSlice; q += kWave * kSplitW) {
            const bool in = q < cnt;
            s_tau[q] = in ? P.t[m.j0 + jt + q] - m.t0 : 0.0;
            s_u[q] = in ? (float)((P.y[m.j0 + jt + q] - m.ybar) * up) : 0.0f;
        }
        __syncthreads();
        for (int s = uniform_i32(wave); s < slices; s += kSplitW) {
            Frag A, B;
            const int j = s * kSlice + half * 8;
            gen_b(B, hb, s_tau + j, cnt - j);
            gen_a(A, fa, s_tau + j, s_u + j);
            accumulate(acc, A, B);
        }
    }

    // wave w adds the eight waves' sums of accumulator rows 2w and 2w + 1
    float sum[8][2];
#pragma unroll
    for (int q = 0; q < 8; ++q) {
#pragma unroll
        for (int r = 0; r < 16; ++r) s_sum[q & 1][wave][r][lane] = acc[q][r];
        __syncthreads();
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            float v = s_sum[q & 1][0][2 * wave + e][lane];
#pragma unroll
            for (int w = 1; w < kSplitW; ++w) v += s_sum[q & 1][w][2 * wave + e][lane];
            sum[q][e] = v;
        }
    }

    const Finish R = make_finish(P, m, rr);
    LaneBest lb{-1.0f, 0u};
    bool ill = false;
#pragma unroll
    for (int e = 0; e < 2; ++e) {
        const int r = 2 * wave + e;
        const int a = 8 * (r / 4) + 4 * half + (r & 3);
        float v[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) v[q] = sum[q][e];
        finish_pair(R, v, w0 + (int64_t)a * kBlk, sub, lb, ill);
    }
    const unsigned long long key = wave_max_u64(lane_key(lb));
    const bool any = __any(ill);
    if (lane == 0) {
        s_key[wave] = key;
        s_ill[wave] = any;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        // rows 0..7 of the accumulators (waves 0..3) are the first fix-up tile
        unsigned long long best = 0ull;
        for (int t = 0; t < kWaveBins / kFix; ++t) {
            int bad = 0;
            unsigned long long k = 0ull;
            for (int w = 4 * t; w < 4 * t + 4; ++w) {
                bad |= s_ill[w];
                k = umax64(k, s_key[w]);
            }
            if (bad) {
                const int64_t tile = row * P.tiles_per_row + (w0 - rr.f_lo) / kFix + t;
                atomicOr(&P.ill_bits[tile >> 5], 1u << (tile & 31));
            } else {
                best = umax64(best, k);
            }
        }
        if (best != 0ull) atomicMax(&P.keys[row / P.rows_per_group], best);
    }
}

}  // namespace

int64_t mx_item_bins(int waves, bool split) {
    return split ? kWaveBins : (int64_t)waves * kWaveBins;
}

hipError_t launch_mx(const MainParams& p, int waves, bool split, hipStream_t s) {
    if (p.n_items <= 0) return hipSuccess;
    const dim3 grid = grid_for(p.n_items);
    if (split) {
        hipLaunchKernelGGL(mx_split_kernel, grid, dim3(kWave * kSplitW), 0, s, p);
    } else if (waves == 4) {
        hipLaunchKernelGGL(mx_tile_kernel<4>, grid, dim3(kWave * 4), 0, s, p);
    } else if (waves == 2) {
        hipLaunchKernelGGL(mx_tile_kernel<2>, grid, dim3(kWave * 2), 0, s, p);
    } else {
        return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

}  // namespace lsp
