// lsp_mx.hip -- the FP32 form on the matrix cores (lsp_mx.h): the standard and
// the generalized periodogram, one tile of bins per wave or one per workgroup
// whose waves split the observations.
#include "lsp_mx.h"

#include <type_traits>

namespace lsp {
namespace {

using namespace mx;

// The end of a tile: a wave holds the sums of its bins in its accumulators,
// some bins a lane.  All powers are computed first and without a branch, so
// that their chains (a reciprocal each) overlap; the best is tracked as the
// number of the lane's bin; a stored periodogram goes out in a pass of its own.
// (With a bounds check and a store branch at every bin this took 6.8 us per
// wave, a quarter of the time of a tile of 260 observations.)
struct LaneBest {
    float p = -1.0f;
    int bin = 0;  // from the tile's first

    // Bins are offered in increasing order, so a strict comparison keeps the
    // lowest of equals.
    __device__ __forceinline__ void offer(float v, int b) {
        const bool more = v > p;
        p = more ? v : p;
        bin = more ? b : bin;
    }
};

// Key of the wave's best bin (0 where no lane has one): larger power first,
// then the lower index; w0 is the tile's first bin.
__device__ __forceinline__ unsigned long long wave_key(const LaneBest& b, int64_t w0) {
    float m = b.p;
    auto up = [&](auto ctrl) {
        const int v = __builtin_amdgcn_update_dpp(__float_as_int(-1.0f), __float_as_int(m),
                                                  decltype(ctrl)::value, 0xF, 0xF, false);
        m = fmaxf(m, __int_as_float(v));
    };
    // maximum over each row of 16 lanes into its last, then over the rows
    up(std::integral_constant<int, 0x111>{});  // row_shr:1
    up(std::integral_constant<int, 0x112>{});  // row_shr:2
    up(std::integral_constant<int, 0x114>{});  // row_shr:4
    up(std::integral_constant<int, 0x118>{});  // row_shr:8
    up(std::integral_constant<int, 0x142>{});  // row_bcast:15
    up(std::integral_constant<int, 0x143>{});  // row_bcast:31
    const float top = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(m), kWave - 1));
    if (!(top >= 0.0f)) return 0ull;
    int least = 0x7FFFFFFF;
    for (unsigned long long ties = __ballot(b.p == top); ties; ties &= ties - 1) {
        const int bin = __builtin_amdgcn_readlane(b.bin, (int)__builtin_ctzll(ties));
        least = bin < least ? bin : least;
    }
    return ((unsigned long long)__float_as_uint(top > 0.0f ? top : 0.0f) << 32) |
           (uint32_t)(0xFFFFFFFFu - (uint32_t)(w0 + least));
}

struct Finish {
    float n4;
    PowerScale scale4;
    void* pgram;   // periodogram at the object's first bin, or NULL
    int32_t f64;
    int left;      // the row's bins from the tile's first, at most a tile

    __device__ __forceinline__ void store(int64_t w0, int bin, float p) const {
        if (bin >= left) return;
        if (f64)
            static_cast<double*>(pgram)[w0 + bin] = (double)p;
        else
            static_cast<float*>(pgram)[w0 + bin] = p;
    }
};

__device__ __forceinline__ void* object_pgram(const MainParams& P, int64_t obj) {
    if (!P.pgram) return nullptr;
    return P.pgram_f64 ? static_cast<void*>(static_cast<double*>(P.pgram) + obj * P.n_f)
                       : static_cast<void*>(static_cast<float*>(P.pgram) + obj * P.n_f);
}

// The sums of one of the two bins (side 0: minus, 1: plus the offset) of a block's
// offset from its eight products: with y at the cosine and sine, then at 2wt (1/4).
__device__ __forceinline__ void bin_sums(const float (&v)[8], int side, float (&b)[4]) {
    const float z = side ? 1.0f : -1.0f;
    b[0] = fmaf(-z, v[1], v[0]);
    b[1] = fmaf(z, v[3], v[2]);
    b[2] = fmaf(-z, v[5], v[4]);
    b[3] = fmaf(z, v[7], v[6]);
}

// Both bins' powers.
__device__ __forceinline__ void pair_power(const Finish& R, const float (&v)[8], float (&p)[2],
                                           bool (&ill)[2]) {
#pragma unroll
    for (int side = 0; side < 2; ++side) {
        float b[4];
        bin_sums(v, side, b);
        p[side] = power_mx(b[0], b[1], b[2], b[3], R.n4, R.scale4, ill[side]);
    }
}

// Bin of (block a, offset m, side) from the tile's first.
__device__ __forceinline__ int tile_bin(int a, int m, int side) {
    return a * kBlk + (side ? kOffs + m : kOffs - 1 - m);
}

__device__ __forceinline__ Finish make_finish(const MainParams& P, const ObjMeta& m,
                                              const RowRange& rr, int64_t w0) {
    Finish R;
    const double back = ldexp(1.0, -mx_exp_y(m));
    R.n4 = 0.25f * (float)m.n;
    R.scale4 = power_scale(0.25 * (m.scale * back * back));
    R.pgram = object_pgram(P, rr.obj);
    R.f64 = P.pgram_f64;
    R.left = (int)(rr.f_hi - w0 < kWaveBins ? rr.f_hi - w0 : kWaveBins);
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

// A wave's whole tile from its accumulators: stores and marks what has to be,
// and returns the key of the best bin.  WHOLE: all of its bins are the row's.
template <bool WHOLE>
__device__ __forceinline__ unsigned long long finish_wave(const MainParams& P, const Finish& R,
                                                          const f16v (&acc)[8], int64_t row,
                                                          int64_t w0, int64_t f_lo, int lane) {
    const int sub = lane & 31, half = lane >> 5;
    constexpr int kRowsFix = 16 * kFix / kWaveBins;  // accumulator rows of a fix-up tile
    float p[16][2];
    LaneBest lb;
#pragma unroll
    for (int t = 0; t < kWaveBins / kFix; ++t) {
        LaneBest lt;
        bool ill = false;
#pragma unroll
        for (int r = kRowsFix * t; r < kRowsFix * (t + 1); ++r) {
            float v[8];
#pragma unroll
            for (int q = 0; q < 8; ++q) v[q] = acc[q][r];
            bool bad[2];
            pair_power(R, v, p[r], bad);
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                const int a = 8 * (r / 4) + 4 * half + (r & 3);
                const bool in = WHOLE || tile_bin(a, sub, e) < R.left;
                ill |= bad[e] & in;
                lt.offer(in ? p[r][e] : -1.0f, 2 * r + e);
            }
        }
        if (__any(ill)) {  // the fix-up's: it offers the tile's bins itself
            const int64_t tile = row * P.tiles_per_row + (w0 - f_lo) / kFix + t;
            if (lane == 0) atomicOr(&P.ill_bits[tile >> 5], 1u << (tile & 31));
        } else {
            lb.offer(lt.p, lt.bin);
        }
    }
    const int r = lb.bin >> 1;
    lb.bin = tile_bin(8 * (r >> 2) + 4 * half + (r & 3), sub, lb.bin & 1);
    const unsigned long long best = wave_key(lb, w0);
    if (R.pgram)
#pragma unroll
        for (int r = 0; r < 16; ++r)
#pragma unroll
            for (int e = 0; e < 2; ++e)
                R.store(w0, tile_bin(8 * (r / 4) + 4 * half + (r & 3), sub, e), p[r][e]);
    return best;
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
    const int64_t item = mx_item(P.row_perm, P.row_obj, b, P.n_items);
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
                gen_b(B, hb, s_tau + j);
                if (cnt < (mine + 1) * kSlice) trim_b(B, cnt - j);
#pragma unroll
                for (int q = 0; q < 8; ++q) s_b[buf][wave][q][lane] = B.q[q];
            }
            __syncthreads();
            // (a wave past the row's end only makes its share of the factors)
            const int todo = w0 >= rr.f_hi ? 0 : slices - s0 < W ? slices - s0 : W;
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

    const Finish R = make_finish(P, m, rr, w0);
    if (R.left <= 0) return;
    const unsigned long long best = R.left == kWaveBins
                                        ? finish_wave<true>(P, R, acc, row, w0, rr.f_lo, lane)
                                        : finish_wave<false>(P, R, acc, row, w0, rr.f_lo, lane);
    if (lane == 0 && best != 0ull) atomicMax(&P.keys[row / P.rows_per_group], best);
}

// A workgroup's part of a long series' observations, in whole slices (P.n_split
// parts, the series' own [0, n) where there is one).
__device__ __forceinline__ void part_range(const MainParams& P, int64_t n, int part, int slice,
                                           int64_t* lo, int64_t* hi) {
    const int64_t slices = (n + slice - 1) / slice;
    const int64_t per = (slices + P.n_split - 1) / P.n_split * slice;
    *lo = part * per < n ? part * per : n;
    *hi = *lo + per < n ? *lo + per : n;
}

// One 32 x 32 tile per workgroup of eight waves, which share out the
// observations in slices and add their sums through LDS in wave order: for
// calls whose tiles alone are too few to fill the chip.  Where even so there are
// few workgroups and the one series is long, its observations are split over
// P.n_split of them too, which leave their bins' sums for mx_combine_kernel.
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
    const int part = P.n_split > 1 ? (int)(b / P.chunks_per_row) : 0;
    const int64_t rank = P.n_split > 1 ? 0 : b / P.chunks_per_row;
    const int64_t chunk = b - (P.n_split > 1 ? part : rank) * P.chunks_per_row;
    const int64_t row = item_row(P.row_perm, rank);
    const RowRange rr =
        decode_row(P.row_obj, P.row_band, P.band_bins, P.rows_per_group, P.n_obj, P.n_f, row);
    const int64_t w0 = rr.f_lo + chunk * (int64_t)kWaveBins;
    if (rr.obj < 0 || w0 >= rr.f_hi) return;
    const ObjMeta m = P.meta[rr.obj];
    if (m.status != LSP_OBJ_OK) {
        if (P.n_split == 1) fill_bins(P, rr, m.status, w0, w0 + kWaveBins, kWave * kSplitW);
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

    int64_t j_lo, j_hi;
    part_range(P, m.n, part, kSlice, &j_lo, &j_hi);
    for (int64_t jt = j_lo; jt < j_hi; jt += kSplitObs) {
        const int cnt = (int)(j_hi - jt < kSplitObs ? j_hi - jt : kSplitObs);
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
            gen_b(B, hb, s_tau + j);
            if (cnt < (s + 1) * kSlice) trim_b(B, cnt - j);
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

    const Finish R = make_finish(P, m, rr, w0);
    if (P.n_split > 1) {
        float* const out = P.part + (int64_t)part * 4 * P.n_f + w0;
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            const int r = 2 * wave + e;
            float v[8];
#pragma unroll
            for (int q = 0; q < 8; ++q) v[q] = sum[q][e];
#pragma unroll
            for (int side = 0; side < 2; ++side) {
                const int bin = tile_bin(8 * (r / 4) + 4 * half + (r & 3), sub, side);
                float b4[4];
                bin_sums(v, side, b4);
                if (bin < R.left)
#pragma unroll
                    for (int q = 0; q < 4; ++q) out[q * P.n_f + bin] = b4[q];
            }
        }
        return;
    }
    LaneBest lb;
    bool ill = false;
    float p[2][2];
#pragma unroll
    for (int e = 0; e < 2; ++e) {
        const int r = 2 * wave + e;
        const int a = 8 * (r / 4) + 4 * half + (r & 3);
        float v[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) v[q] = sum[q][e];
        bool bad[2];
        pair_power(R, v, p[e], bad);
#pragma unroll
        for (int side = 0; side < 2; ++side) {
            const int bin = tile_bin(a, sub, side);
            const bool in = bin < R.left;
            ill |= bad[side] & in;
            lb.offer(in ? p[e][side] : -1.0f, bin);
            if (R.pgram) R.store(w0, bin, p[e][side]);
        }
    }
    const unsigned long long key = wave_key(lb, w0);
    const bool any = __any(ill);
    if (lane == 0) {
        s_key[wave] = key;
        s_ill[wave] = any;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        // eight rows of the accumulators (four waves) are a fix-up tile
        constexpr int kPer = kSplitW * kFix / kWaveBins;
        unsigned long long best = 0ull;
        for (int t = 0; t < kWaveBins / kFix; ++t) {
            int bad = 0;
            unsigned long long k = 0ull;
            for (int w = kPer * t; w < kPer * (t + 1); ++w) {
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

// ---------------------------------------------------------------------------
// Generalized periodogram (errors and a floating mean).  With weights w and
// weighted-mean-centred magnitudes yw the sums are sum w e^{iwt}, sum w yw
// e^{iwt} and sum w e^{2iwt}: three complex sums, six centre factors
//   w c, w s, w yw c, w yw s, w (cos 2)/2, w (sin 2)/2
// against the same four offset factors.  Twelve accumulators of a 32 x 32 tile
// would leave one wave per SIMD, so a wave's tile is 16 blocks x 32 offsets
// (1,024 bins, two fix-up tiles) on v_mfma_f32_16x16x32_f16: 72 matrix
// instructions per 32 observations.  Measured, vector kernels -> here: 4,096
// points with errors on 500,000 bins 413 -> 112 us; error 1.1e-6 -> 2.3e-7.
typedef float f4v __attribute__((ext_vector_type(4)));

constexpr int kGSlice = 32;                  // observations per matrix instruction
constexpr int kGRows = 16;                   // blocks per wave tile
constexpr int kGBins = kBlk * kGRows;        // 1,024 bins
constexpr int kFixG = kMxTileGen;            // bins per fix-up tile
static_assert(kGBins == 2 * kFixG, "a generalized wave tile is two fix-up tiles");

// Centre factors of 8 observations: q[0..5] hi, q[6..11] lo halves.
struct FragG {
    h8 q[12];
};

__device__ __forceinline__ void gen_a_g(FragG& F, double f, const double* tau, const float* w,
                                        const float* wy) {
#pragma unroll
    for (int p = 0; p < 4; ++p) {
        float s0, c0, s1, c1;
        sincos_rev(f, tau[2 * p], s0, c0);
        sincos_rev(f, tau[2 * p + 1], s1, c1);
        const float w0 = w[2 * p], w1 = w[2 * p + 1];
        const float y0 = wy[2 * p], y1 = wy[2 * p + 1];
        const float v[6][2] = {{w0 * c0, w1 * c1},
                               {w0 * s0, w1 * s1},
                               {y0 * c0, y1 * c1},
                               {y0 * s0, y1 * s1},
                               {w0 * fmaf(c0, c0, -0.5f), w1 * fmaf(c1, c1, -0.5f)},
                               {w0 * c0 * s0, w1 * c1 * s1}};
#pragma unroll
        for (int q = 0; q < 6; ++q) {
            h2 hi, lo;
            split2(v[q][0], v[q][1], hi, lo);
            put2(F.q[q], p, hi);
            put2(F.q[q + 6], p, lo);
        }
    }
}

__device__ __forceinline__ f4v mm16(h8 a, h8 b, f4v c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(a, b, c, 0, 0, 0);
}

// acc[4 g + ..] for the three complex sums g: (A0)(c), (A1)(s), (A1)(c), (A0)(s).
__device__ __forceinline__ void accumulate_g(f4v (&acc)[12], const FragG& A, const Frag& B) {
#pragma unroll
    for (int part = 0; part < 3; ++part) {  // hi hi, lo hi, hi lo
        const int ao = part == 1 ? 6 : 0, bo = part == 2 ? 4 : 0;
#pragma unroll
        for (int g = 0; g < 3; ++g) {
            const h8 a0 = A.q[ao + 2 * g], a1 = A.q[ao + 2 * g + 1];
            const h8 b0 = B.q[bo + (g == 2 ? 2 : 0)], b1 = B.q[bo + (g == 2 ? 3 : 1)];
            acc[4 * g + 0] = mm16(a0, b0, acc[4 * g + 0]);
            acc[4 * g + 1] = mm16(a1, b1, acc[4 * g + 1]);
            acc[4 * g + 2] = mm16(a1, b0, acc[4 * g + 2]);
            acc[4 * g + 3] = mm16(a0, b1, acc[4 * g + 3]);
        }
    }
}

// Power of one bin: with all sums in units where the weights sum to n, the
// trace T = n - (c1^2 + s1^2)/n of the moment matrix, its eigenvalue difference
// R (R^2 = D^2 + E^2) and Q = yc^2 + ys^2, power32_gen's two terms are
// (Q T - ((yc^2 - ys^2) D + 2 yc ys E)) / (T^2 - R^2): one reciprocal and no
// square root.  `ill` as there: T - R <= n/32.  c2, s2 are sum w cos 2wt and
// sum w sin 2wt.
__device__ __forceinline__ float power_mx_gen(float c1, float s1, float yc, float ys, float c2,
                                              float s2, float n, float rn, PowerScale scale,
                                              bool& ill) {
    const float tr = fmaf(-rn, fmaf(c1, c1, s1 * s1), n);
    const float d = fmaf(-rn, fmaf(c1, c1, -(s1 * s1)), c2);
    const float e = fmaf(-2.0f * rn * c1, s1, s2);
    const float r2 = fmaf(d, d, e * e);
    const float edge = tr - kIllTheta * n;
    ill = !(edge > 0.0f && r2 < edge * edge);
    const float q = fmaf(yc, yc, ys * ys);
    const float t = fmaf(fmaf(yc, yc, -(ys * ys)), d, 2.0f * yc * ys * e);
    return fmaxf(fmaf(q, tr, -t), 0.0f) * __builtin_amdgcn_rcpf(fmaf(tr, tr, -r2)) * scale.two *
           scale.rest;
}

struct FinishG {
    float n, rn;
    PowerScale scale;
    Finish out;
};

__device__ __forceinline__ FinishG make_finish_g(const MainParams& P, const ObjMeta& m,
                                                 const RowRange& rr, int64_t w0) {
    FinishG R;
    const double up_w = ldexp(1.0, mx_exp_w(m)), back = ldexp(1.0, -mx_exp_y(m));
    R.n = (float)((double)m.n * up_w);
    R.rn = (float)(1.0 / ((double)m.n * up_w));
    R.scale = power_scale(m.scale * back * back * up_w);
    R.out.pgram = object_pgram(P, rr.obj);
    R.out.f64 = P.pgram_f64;
    R.out.left = (int)(rr.f_hi - w0 < kGBins ? rr.f_hi - w0 : kGBins);
    return R;
}

// One of the two bins of an offset: the centre minus (side 0) or plus (side 1) it.
// Its sums of w, of w yw and (four times the products) of w at 2wt.
__device__ __forceinline__ void bin_sums_g(const float (&v)[12], int side, float (&b)[6]) {
    const float z = side ? 1.0f : -1.0f;
#pragma unroll
    for (int g = 0; g < 3; ++g) {
        b[2 * g] = (g == 2 ? 4.0f : 1.0f) * fmaf(-z, v[4 * g + 1], v[4 * g]);
        b[2 * g + 1] = (g == 2 ? 4.0f : 1.0f) * fmaf(z, v[4 * g + 3], v[4 * g + 2]);
    }
}

__device__ __forceinline__ float sums_power_g(const FinishG& R, const float (&b)[6], bool& ill) {
    return power_mx_gen(b[0], b[1], b[2], b[3], b[4], b[5], R.n, R.rn, R.scale, ill);
}

__device__ __forceinline__ float bin_power_g(const FinishG& R, const float (&v)[12], int side,
                                             bool& ill) {
    float b[6];
    bin_sums_g(v, side, b);
    return sums_power_g(R, b, ill);
}

// Stage observations [jt, jt + cnt) of the object, padded with zeros to whole slices.
__device__ __forceinline__ void stage_g(const MainParams& P, const ObjMeta& m, int64_t jt, int cnt,
                                        int padded, double up_w, double up_y, double* s_tau,
                                        float* s_w, float* s_wy, int threads) {
    for (int q = threadIdx.x; q < padded; q += threads) {
        const int64_t j = m.j0 + jt + q;
        const bool in = q < cnt;
        const double w = in ? gen_weight(P.dy, j, m.wnorm) : 0.0;
        s_tau[q] = in ? P.t[j] - m.t0 : 0.0;
        s_w[q] = (float)(w * up_w);
        s_wy[q] = in ? (float)(w * (P.y[j] - m.ybar) * up_y) : 0.0f;
    }
}

// The first fix-up tile of a wave's 1,024 bins is in lanes 0..31 (blocks 0..7),
// the second in the others: bit h of the result is set where half h has an
// ill-conditioned bin.
__device__ __forceinline__ uint32_t ill_halves(bool ill) {
    const unsigned long long m = __ballot(ill);
    return ((uint32_t)m ? 1u : 0u) | ((uint32_t)(m >> 32) ? 2u : 0u);
}

// Leaves fix-up tiles `tile` and `tile` + 1 to the fix-up, by bit.
__device__ __forceinline__ void mark_ill(const MainParams& P, int64_t tile, uint32_t bad,
                                         int lane) {
    if (lane < 2 && ((bad >> lane) & 1u))
        atomicOr(&P.ill_bits[(tile + lane) >> 5], 1u << ((tile + lane) & 31));
}

// Finish one wave's 1,024 bins from complete sums acc[offset half][12].
template <bool WHOLE>
__device__ __forceinline__ void finish_tile_g(const MainParams& P, const FinishG& R, int64_t row,
                                              int64_t tile, int64_t w0, const f4v (&acc)[2][12],
                                              int lane) {
    LaneBest lb;
    bool ill = false;
    float p[4][4];
    // in increasing bins of the lane: minus the larger offset, minus the
    // smaller, plus the smaller, plus the larger
    auto bin_of = [&](int r, int e) {
        const int h = e == 0 || e == 3;
        return tile_bin(4 * (lane >> 4) + r, 16 * h + (lane & 15), e >= 2);
    };
#pragma unroll
    for (int r = 0; r < 4; ++r) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int h = e == 0 || e == 3;
            float v[12];
#pragma unroll
            for (int q = 0; q < 12; ++q) v[q] = acc[h][q][r];
            bool bad;
            p[r][e] = bin_power_g(R, v, e >= 2, bad);
            const bool in = WHOLE || bin_of(r, e) < R.out.left;
            ill |= bad & in;
            lb.offer(in ? p[r][e] : -1.0f, 4 * r + e);
        }
    }
    lb.bin = bin_of(lb.bin >> 2, lb.bin & 3);
    const uint32_t bad = ill_halves(ill);
    mark_ill(P, row * P.tiles_per_row + tile, bad, lane);
    if ((bad >> (lane >> 5)) & 1u) lb.p = -1.0f;
    const unsigned long long best = wave_key(lb, w0);
    if (lane == 0 && best != 0ull) atomicMax(&P.keys[row / P.rows_per_group], best);
    if (R.out.pgram)
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
            for (int e = 0; e < 4; ++e) R.out.store(w0, bin_of(r, e), p[r][e]);
}

// Four waves, each with its own tile; the offset factors of two slices at a
// time are made one quarter (a slice's half of the offsets) per wave.
constexpr int kGW = 4;

__global__ __launch_bounds__(kWave* kGW, 2) void mx_gen_tile_kernel(const MainParams P) {
    __shared__ double s_tau[kTile];
    __shared__ float s_w[kTile], s_wy[kTile];
    __shared__ h8 s_b[2][2][2][8][kWave];  // buffer, slice, offset half, factor

    const int64_t b = linear_block();
    if (b >= P.n_items) return;
    const int64_t item = mx_item(P.row_perm, P.row_obj, b, P.n_items);
    const int64_t rank = item / P.chunks_per_row;
    const int64_t chunk = item - rank * P.chunks_per_row;
    const int64_t row = item_row(P.row_perm, rank);
    const RowRange rr =
        decode_row(P.row_obj, P.row_band, P.band_bins, P.rows_per_group, P.n_obj, P.n_f, row);
    const int64_t g0 = rr.f_lo + chunk * (int64_t)(kGW * kGBins);
    if (rr.obj < 0 || g0 >= rr.f_hi) return;
    const ObjMeta m = P.meta[rr.obj];
    if (m.status != LSP_OBJ_OK) {
        fill_bins(P, rr, m.status, g0, g0 + kGW * kGBins, kWave * kGW);
        return;
    }
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = threadIdx.x / kWave;
    const int sub = lane & 15, quarter = lane >> 4;
    const int64_t w0 = g0 + (int64_t)wave * kGBins;
    const double fa =
        (P.f_min + P.df * ((double)(w0 + (int64_t)sub * kBlk) + (kOffs - 0.5))) * P.to_cyc;
    const double hb = (P.df * P.to_cyc) * ((double)(16 * (wave & 1) + sub) + 0.5);
    const double up_w = ldexp(1.0, mx_exp_w(m)), up_y = ldexp(1.0, mx_exp_y(m));

    f4v acc[2][12];
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int q = 0; q < 12; ++q) acc[h][q] = f4v{0.0f, 0.0f, 0.0f, 0.0f};

    int buf = 0;
    for (int64_t jt = 0; jt < m.n; jt += kTile) {
        const int cnt = (int)(m.n - jt < kTile ? m.n - jt : kTile);
        const int slices = (cnt + kGSlice - 1) / kGSlice;
        __syncthreads();
        stage_g(P, m, jt, cnt, slices * kGSlice, up_w, up_y, s_tau, s_w, s_wy, kWave * kGW);
        __syncthreads();
        for (int s0 = 0; s0 < slices; s0 += 2) {
            const int mine = s0 + (wave >> 1);
            if (mine < slices) {
                Frag B;
                const int j = mine * kGSlice + quarter * 8;
                gen_b(B, hb, s_tau + j);  // (padding has no weight: nothing to trim)
#pragma unroll
                for (int q = 0; q < 8; ++q) s_b[buf][wave >> 1][wave & 1][q][lane] = B.q[q];
            }
            __syncthreads();
            // (a wave past the row's end only makes its share of the factors)
            const int todo = w0 >= rr.f_hi ? 0 : slices - s0 < 2 ? slices - s0 : 2;
            for (int s = 0; s < todo; ++s) {
                FragG A;
                const int j = (s0 + s) * kGSlice + quarter * 8;
                gen_a_g(A, fa, s_tau + j, s_w + j, s_wy + j);
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    Frag B;
#pragma unroll
                    for (int q = 0; q < 8; ++q) B.q[q] = s_b[buf][s][h][q][lane];
                    accumulate_g(acc[h], A, B);
                }
            }
            buf ^= 1;
        }
    }
    const FinishG R = make_finish_g(P, m, rr, w0);
    if (R.out.left <= 0) return;
    const int64_t tile = (w0 - rr.f_lo) / kFixG;
    if (R.out.left == kGBins)
        finish_tile_g<true>(P, R, row, tile, w0, acc, lane);
    else
        finish_tile_g<false>(P, R, row, tile, w0, acc, lane);
}

// One tile per workgroup, the observations shared out over its eight waves and
// the sums added through LDS in wave order; wave w finishes a half row of the
// tile's accumulators.
constexpr int kGSplitObs = 1024;

__global__ __launch_bounds__(kWave* kSplitW, 2) void mx_gen_split_kernel(const MainParams P) {
    __shared__ double s_tau[kGSplitObs];
    __shared__ float s_w[kGSplitObs], s_wy[kGSplitObs];
    __shared__ float s_sum[2][kSplitW][8][kWave];  // 8 = offset halves x accumulator rows
    __shared__ unsigned long long s_key[kSplitW];
    __shared__ uint32_t s_ill[kSplitW];

    const int64_t b = linear_block();
    if (b >= P.n_items) return;
    const int part = P.n_split > 1 ? (int)(b / P.chunks_per_row) : 0;
    const int64_t rank = P.n_split > 1 ? 0 : b / P.chunks_per_row;
    const int64_t chunk = b - (P.n_split > 1 ? part : rank) * P.chunks_per_row;
    const int64_t row = item_row(P.row_perm, rank);
    const RowRange rr =
        decode_row(P.row_obj, P.row_band, P.band_bins, P.rows_per_group, P.n_obj, P.n_f, row);
    const int64_t w0 = rr.f_lo + chunk * (int64_t)kGBins;
    if (rr.obj < 0 || w0 >= rr.f_hi) return;
    const ObjMeta m = P.meta[rr.obj];
    if (m.status != LSP_OBJ_OK) {
        if (P.n_split == 1) fill_bins(P, rr, m.status, w0, w0 + kGBins, kWave * kSplitW);
        return;
    }
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = threadIdx.x / kWave;
    const int sub = lane & 15, quarter = lane >> 4;
    const double fa =
        (P.f_min + P.df * ((double)(w0 + (int64_t)sub * kBlk) + (kOffs - 0.5))) * P.to_cyc;
    const double hb = P.df * P.to_cyc;
    const double up_w = ldexp(1.0, mx_exp_w(m)), up_y = ldexp(1.0, mx_exp_y(m));

    f4v acc[2][12];
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int q = 0; q < 12; ++q) acc[h][q] = f4v{0.0f, 0.0f, 0.0f, 0.0f};

    int64_t j_lo, j_hi;
    part_range(P, m.n, part, kGSlice, &j_lo, &j_hi);
    for (int64_t jt = j_lo; jt < j_hi; jt += kGSplitObs) {
        const int cnt = (int)(j_hi - jt < kGSplitObs ? j_hi - jt : kGSplitObs);
        const int slices = (cnt + kGSlice - 1) / kGSlice;
        __syncthreads();
        stage_g(P, m, jt, cnt, slices * kGSlice, up_w, up_y, s_tau, s_w, s_wy, kWave * kSplitW);
        __syncthreads();
        for (int s = uniform_i32(wave); s < slices; s += kSplitW) {
            FragG A;
            const int j = s * kGSlice + quarter * 8;
            gen_a_g(A, fa, s_tau + j, s_w + j, s_wy + j);
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                Frag B;
                gen_b(B, hb * ((double)(16 * h + sub) + 0.5), s_tau + j);
                accumulate_g(acc[h], A, B);
            }
        }
    }

    float sum[12];
#pragma unroll
    for (int q = 0; q < 12; ++q) {
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int r = 0; r < 4; ++r) s_sum[q & 1][wave][2 * r + h][lane] = acc[h][q][r];
        __syncthreads();
        float v = s_sum[q & 1][0][wave][lane];
#pragma unroll
        for (int w = 1; w < kSplitW; ++w) v += s_sum[q & 1][w][wave][lane];
        sum[q] = v;
    }
    // wave w: accumulator row w / 2 of the lane's four, offset half w % 2
    const FinishG R = make_finish_g(P, m, rr, w0);
    if (P.n_split > 1) {
        float* const out = P.part + (int64_t)part * 6 * P.n_f + w0;
#pragma unroll
        for (int side = 0; side < 2; ++side) {
            const int bin = tile_bin(4 * quarter + (wave >> 1), 16 * (wave & 1) + sub, side);
            float b6[6];
            bin_sums_g(sum, side, b6);
            if (bin < R.out.left)
#pragma unroll
                for (int q = 0; q < 6; ++q) out[q * P.n_f + bin] = b6[q];
        }
        return;
    }
    LaneBest lb;
    bool ill = false;
#pragma unroll
    for (int side = 0; side < 2; ++side) {
        bool bad;
        const float p = bin_power_g(R, sum, side, bad);
        const int bin = tile_bin(4 * quarter + (wave >> 1), 16 * (wave & 1) + sub, side);
        const bool in = bin < R.out.left;
        ill |= bad & in;
        lb.offer(in ? p : -1.0f, bin);
        if (R.out.pgram) R.out.store(w0, bin, p);
    }
    const uint32_t any = ill_halves(ill);
    if (lane == 0) s_ill[wave] = any;
    __syncthreads();
    uint32_t bad = 0u;
#pragma unroll
    for (int w = 0; w < kSplitW; ++w) bad |= s_ill[w];
    if ((bad >> (lane >> 5)) & 1u) lb.p = -1.0f;
    const unsigned long long key = wave_key(lb, w0);
    if (lane == 0) s_key[wave] = key;
    __syncthreads();
    if (wave != 0) return;
    mark_ill(P, row * P.tiles_per_row + (w0 - rr.f_lo) / kFixG, bad, lane);
    if (lane == 0) {
        unsigned long long best = 0ull;
        for (int w = 0; w < kSplitW; ++w) best = umax64(best, s_key[w]);
        if (best != 0ull) atomicMax(&P.keys[row / P.rows_per_group], best);
    }
}

// Adds the parts' sums of a single series in their order and finishes the bins,
// a workgroup per fix-up tile.
constexpr int kCombThreads = 256;

template <bool GEN>
__global__ __launch_bounds__(kCombThreads) void mx_combine_kernel(const MainParams P) {
    constexpr int kTileBins = GEN ? kFixG : kFix, kPer = kTileBins / kCombThreads;
    constexpr int kSums = GEN ? 6 : 4;
    __shared__ unsigned long long s_key[kCombThreads / kWave];
    const RowRange rr = decode_row(P.row_obj, P.row_band, P.band_bins, P.rows_per_group, P.n_obj,
                                   P.n_f, 0);
    const int64_t w0 = (int64_t)blockIdx.x * kTileBins;
    const ObjMeta m = P.meta[0];
    if (m.status != LSP_OBJ_OK) {
        fill_bins(P, rr, m.status, w0, w0 + kTileBins, kCombThreads);
        return;
    }
    bool ill = false;
    LaneBest lb;
    float p[kPer];
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
        const int bin = k * kCombThreads + (int)threadIdx.x;
        const bool in = w0 + bin < P.n_f;
        const float* at = P.part + w0 + (in ? bin : 0);
        float b[kSums];
#pragma unroll
        for (int q = 0; q < kSums; ++q) b[q] = 0.0f;
#pragma unroll 4
        for (int s = 0; s < P.n_split; ++s, at += kSums * P.n_f)
#pragma unroll
            for (int q = 0; q < kSums; ++q) b[q] += at[q * P.n_f];
        bool bad;
        if constexpr (GEN) {
            p[k] = sums_power_g(make_finish_g(P, m, rr, w0), b, bad);
        } else {
            const Finish R = make_finish(P, m, rr, w0);
            p[k] = power_mx(b[0], b[1], b[2], b[3], R.n4, R.scale4, bad);
        }
        ill |= bad && in;
        lb.offer(in ? p[k] : -1.0f, bin);
    }
    Finish R = make_finish(P, m, rr, w0);
    R.left = (int)(P.n_f - w0 < kTileBins ? P.n_f - w0 : kTileBins);
    if (R.pgram)
#pragma unroll
        for (int k = 0; k < kPer; ++k) R.store(w0, k * kCombThreads + (int)threadIdx.x, p[k]);
    const unsigned long long key = wave_key(lb, w0);
    if ((threadIdx.x & (kWave - 1)) == 0) s_key[threadIdx.x / kWave] = key;
    const bool any = __syncthreads_or(ill);
    if (threadIdx.x != 0) return;
    if (any) {
        atomicOr(&P.ill_bits[blockIdx.x >> 5], 1u << (blockIdx.x & 31));
        return;
    }
    unsigned long long best = 0ull;
    for (int w = 0; w < kCombThreads / kWave; ++w) best = umax64(best, s_key[w]);
    if (best != 0ull) atomicMax(&P.keys[0], best);
}

}  // namespace

int64_t mx_item_bins(int waves, bool split, bool gen) {
    const int64_t tile = gen ? kGBins : kWaveBins;
    return split ? tile : waves * tile;
}

hipError_t launch_mx(const MainParams& p, int waves, bool split, hipStream_t s) {
    if (p.n_items <= 0) return hipSuccess;
    const dim3 grid = grid_for(p.n_items);
    if (p.n_split > 1) {
        // one series, at most a few hundred tiles
        if (!split) return hipErrorInvalidValue;
        if (p.gen)
            hipLaunchKernelGGL(mx_gen_split_kernel, grid, dim3(kWave * kSplitW), 0, s, p);
        else
            hipLaunchKernelGGL(mx_split_kernel, grid, dim3(kWave * kSplitW), 0, s, p);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        const dim3 tiles((unsigned)p.tiles_per_row), threads(kCombThreads);
        if (p.gen)
            hipLaunchKernelGGL(mx_combine_kernel<true>, tiles, threads, 0, s, p);
        else
            hipLaunchKernelGGL(mx_combine_kernel<false>, tiles, threads, 0, s, p);
        return hipGetLastError();
    }
    if (p.gen) {
        if (split)
            hipLaunchKernelGGL(mx_gen_split_kernel, grid, dim3(kWave * kSplitW), 0, s, p);
        else if (waves == kGW)
            hipLaunchKernelGGL(mx_gen_tile_kernel, grid, dim3(kWave * kGW), 0, s, p);
        else
            return hipErrorInvalidValue;
        return hipGetLastError();
    }
    if (split) {
        hipLaunchKernelGGL(mx_split_kernel, grid, dim3(kWave * kSplitW), 0, s, p);
    } else if (waves == 4) {
        hipLaunchKernelGGL(mx_tile_kernel<4>, grid, dim3(kWave * 4), 0, s, p);
    } else if (waves == 2) {
        hipLaunchKernelGGL(mx_tile_kernel<2>, grid, dim3(kWave * 2), 0, s, p);
    } else if (waves == 1) {
        hipLaunchKernelGGL(mx_tile_kernel<1>, grid, dim3(kWave), 0, s, p);
    } else {
        return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

}  // namespace lsp
