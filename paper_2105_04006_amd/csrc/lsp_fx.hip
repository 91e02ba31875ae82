// lsp_fx.hip -- the FP64 form on the matrix cores (lsp_fx.h), and the FP64
// fix-up of the FP32 forms' ill-conditioned tiles.
#include "lsp_fx.h"
#include "lsp_peaks.h"

#include <type_traits>

namespace lsp {
namespace {

// Four waves, each with its own 512-bin tile of one row; or (SPLIT) W waves
// that share one tile and split the observations.
template <bool GEN, int W, bool SPLIT>
__global__ __launch_bounds__(kWave* W, 2) void fx_kernel(const MainParams P) {
    __shared__ FxStage<GEN> S;
    // the split's partial sums, or the shared offset factors
    __shared__ typename std::conditional<SPLIT, double[W][8][kWave], FxOffsets>::type s_buf;
    __shared__ PeakRec s_red[W];
    constexpr int kBins = (SPLIT ? 1 : W) * kFxBins;  // the workgroup's
    __shared__ FxList<kBins> s_list;

    const int64_t b = linear_block();
    if (b >= P.n_items) return;
    const int64_t item = mx_item(P.row_perm, P.row_obj, b, P.n_items);
    const int64_t rank = item / P.chunks_per_row;
    const int64_t chunk = item - rank * P.chunks_per_row;
    const int64_t row = item_row(P.row_perm, rank);
    const RowRange rr =
        decode_row(P.row_obj, P.row_band, P.band_bins, P.rows_per_group, P.n_obj, P.n_f, row);
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = threadIdx.x / kWave;
    const int64_t tile = SPLIT ? chunk : chunk * W + wave;
    const int64_t w0 = rr.f_lo + tile * kFxBins;
    const bool mine = tile < P.tiles_per_row;
    PeakRec* rec = P.rec + row * P.tiles_per_row + tile;
    const int64_t g0 = rr.f_lo + chunk * kBins;
    if (rr.obj < 0 || g0 >= rr.f_hi) {
        if (mine && lane == 0 && (!SPLIT || wave == 0)) *rec = PeakRec{0.0, -1};
        return;
    }
    const ObjMeta m = P.meta[rr.obj];
    if (m.status != LSP_OBJ_OK) {
        if (P.pgram) {
            const double v = fill_value(m.status);
            for (int64_t i = g0 + threadIdx.x; i < g0 + kBins && i < rr.f_hi; i += kWave * W)
                store_pgram(P.pgram, P.pgram_f64, rr.obj * P.n_f + i, v);
        }
        if (mine && lane == 0 && (!SPLIT || wave == 0)) *rec = PeakRec{0.0, -1};
        return;
    }

    PeakRec best{0.0, -1};
    const int64_t out = rr.obj * P.n_f;
    const double f_top = fmax(fabs(P.f_min), fabs(P.f_min + P.df * (double)P.n_f)) * P.to_cyc;
    const bool covered = fx_covers(f_top, m, fx_few(GEN));
    const FxScales sc = fx_scales<GEN>(m);
    if (threadIdx.x == 0) s_list.count = 0;  // (a barrier follows before it is used)
    auto offer = [&](int64_t i, double p) {
        if (P.pgram) store_pgram(P.pgram, P.pgram_f64, out + i, p);
        if (better(p, i, best.p, best.i)) best = PeakRec{p, i};
    };
    if (covered) {
        const double G = fx_centre(P.f_min, P.df, P.to_cyc, w0, lane & 15);
        const double H = fx_offset(P.df, P.to_cyc, lane & 15);
        FxSums<GEN> A;
        fx_zero(A);
        for (int64_t jt = 0; jt < m.n; jt += kFxObs) {
            const int cnt = uniform_i32((int)(m.n - jt < kFxObs ? m.n - jt : kFxObs));
            __syncthreads();
            fx_stage(S, m, P.t, P.y, P.dy, jt, cnt, sc, kWave * W);
            __syncthreads();
            int lo, hi;
            fx_share<SPLIT ? W : 1>(cnt, SPLIT ? uniform_i32(wave) : 0, &lo, &hi);
            if constexpr (SPLIT)
                fx_accumulate(A, S, cnt, lo, hi, G, H, lane);
            else
                fx_accumulate<GEN, W>(A, S, cnt, lo, hi, G, H, lane, &s_buf, uniform_i32(wave),
                                      w0 >= rr.f_hi);
        }
        constexpr int NQ = 4 * FxSums<GEN>::kSums;
        double xs[SPLIT ? NQ : 1];
        float ds[SPLIT ? NQ : 1];
        if constexpr (SPLIT)
            fx_gather<GEN, W>(A, s_buf, wave, lane, xs, ds);
        else
            fx_turn(A);
#pragma unroll
        for (int r = 0; r < (SPLIT ? 1 : 4); ++r) {
            if (SPLIT ? wave >= 4 : w0 >= rr.f_hi) break;
            const int a = fx_row(SPLIT ? wave : r, lane);
            double x[NQ];
            float d[NQ];
#pragma unroll
            for (int q = 0; q < NQ; ++q) {
                if constexpr (SPLIT) {
                    x[q] = xs[q];
                    d[q] = ds[q];
                } else {
                    x[q] = A.x[q][r];
                    d[q] = A.d[q][r];
                }
            }
            const double Ga = fx_centre(P.f_min, P.df, P.to_cyc, w0, a);
            const int64_t i0 = w0 + (int64_t)a * kFxBlk;
            const int c = lane & 15;
#pragma unroll
            for (int side = 0; side < 2; ++side) {
                const int64_t i = side ? i0 + kFxOffs + c : i0 + kFxOffs - 1 - c;
                const bool in = i < rr.f_hi;
                const double f = grid_freq(P.f_min, P.df, i) * P.to_cyc;
                bool ill;
                const double p = fx_power<GEN>(x, d, f, Ga, H, side ? 1.0 : -1.0, m, sc, ill);
                fx_list(s_list, (int)(i - g0), in && ill, lane);
                if (in && !ill) offer(i, p);
            }
        }
    }
    // what is left: the list, or all bins of an object that is not covered
    __syncthreads();
    const int left = (int)(rr.f_hi - g0 < kBins ? rr.f_hi - g0 : kBins);
    const int count = covered ? uniform_i32(s_list.count) : left;
    fx_direct<GEN, kWave * W>(
        S, covered && m.n <= kFxObs, m, P.t, P.y, P.dy, sc, P.f_min, P.df, P.to_cyc, count,
        [&](int q) { return g0 + (covered ? (int)s_list.bin[q] : q); }, offer);
    best = wave_best(best);
    if (SPLIT || count > 0) {  // bins of any tile: one record for all
        if (lane == 0) s_red[wave] = best;
        __syncthreads();
        if (threadIdx.x == 0)
#pragma unroll
            for (int w = 1; w < W; ++w)
                if (better(s_red[w].p, s_red[w].i, best.p, best.i)) best = s_red[w];
        if (wave != 0) best = PeakRec{0.0, -1};
    }
    if (mine && lane == 0 && (!SPLIT || wave == 0)) *rec = best;
}

// FP64 recompute of FP32-form tiles flagged ill-conditioned.  Workgroups stride
// over the tiles' flag bits a span at a time, collect the flagged ones in LDS, and
// recompute every bin of each such tile from the FP64 series, 512 bins at a
// time with the observations shared out over the four waves (rounding the
// power to FP32 so the argmax still compares FP32 values), then rewrite the
// tile's periodogram bins and merge its best bin into the group's peak key.
// K: the peaks to write at the end (of at most kFixThreads groups), or none.
constexpr int kFixThreads = 256;
constexpr int kFixW = kFixThreads / kWave;

// Tiles per workgroup and round.  Flagged tiles come in clumps (an object's low
// frequencies and aliases, or every tile of an object of a few points), so a
// workgroup's share has to be small; but where few are flagged a workgroup costs
// more than its tiles.  The generalized form flags many: 300 objects on 200,000
// bins take 156 us with 1,024-bin tiles 256 at a time, 78 us with 512-bin tiles 64
// at a time (a workgroup's tiles a grid apart: 272 us, the same ones of every
// object).  The standard form flags few: 64 at a time cost 12,000 bands (48,000
// tiles) 7.3 us, 256 at a time 5.0 us; but 2,000 objects of three points (20,000
// tiles, all flagged) 924 and 2,614 us.
static int fix_span(const FixupParams& p) {
    if (p.gen || p.n_tiles < 128 * 256) return 64;
    return p.n_tiles < 256 * 256 ? 128 : kFixThreads;
}

template <bool GEN>
__global__ __launch_bounds__(kFixThreads, 2) void fixup_kernel(const FixupParams P, const PeakParams K,
                                                               const int span) {
    __shared__ int64_t s_list[kFixThreads];
    __shared__ int s_count;
    __shared__ PeakRec s_red[kFixW];
    __shared__ FxStage<GEN> S;
    __shared__ double s_buf[kFixW][8][kWave];
    __shared__ FxList<kFxBins> s_left;
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = threadIdx.x / kWave;
    const double f_top = fmax(fabs(P.f_min), fabs(P.f_min + P.df * (double)P.n_f)) * P.to_cyc;
    for (int64_t base = (int64_t)blockIdx.x * span; base < P.n_tiles;
         base += (int64_t)gridDim.x * span) {
        if (threadIdx.x == 0) s_count = 0;
        __syncthreads();
        const int64_t mine = base + threadIdx.x;
        if ((int)threadIdx.x < span && mine < P.n_tiles &&
            ((P.ill_bits[mine >> 5] >> (mine & 31)) & 1u))
            s_list[atomicAdd(&s_count, 1)] = mine;
        __syncthreads();
        const int count = uniform_i32(s_count);
        for (int q = 0; q < count; ++q) {
            const int64_t tile = uniform_i64(s_list[q]);
            const int64_t row = tile / P.tiles_per_row;
            const RowRange rr =
                decode_row(P.row_obj, P.row_band, P.band_bins, P.rows_per_group, P.n_obj, P.n_f, row);
            const int64_t obj = rr.obj < 0 ? 0 : rr.obj;
            const int64_t f0 = rr.f_lo + (tile - row * P.tiles_per_row) * P.tile_freqs;
            const int64_t f1 = f0 + P.tile_freqs < rr.f_hi ? f0 + P.tile_freqs : rr.f_hi;
            const ObjMeta m = P.meta[obj];
            const int64_t out = obj * P.n_f;
            PeakRec best{0.0, -1};
            auto offer = [&](int64_t i, double power) {
                const double p = (double)(float)power;
                if (P.pgram) store_pgram(P.pgram, P.pgram_f64, out + i, p);
                if (better(p, i, best.p, best.i)) best = PeakRec{p, i};
            };
            const bool covered = fx_covers(f_top, m, fx_few_fix(GEN));
            const FxScales sc = fx_scales<GEN>(m);
            const double H = fx_offset(P.df, P.to_cyc, lane & 15);
            for (int64_t w0 = f0; w0 < f1; w0 += kFxBins) {
                __syncthreads();
                if (threadIdx.x == 0) s_left.count = 0;
                if (covered) {
                    const double G = fx_centre(P.f_min, P.df, P.to_cyc, w0, lane & 15);
                    FxSums<GEN> A;
                    fx_zero(A);
                    for (int64_t jt = 0; jt < m.n; jt += kFxObs) {
                        const int cnt = (int)(m.n - jt < kFxObs ? m.n - jt : kFxObs);
                        __syncthreads();
                        fx_stage(S, m, P.t, P.y, P.dy, jt, cnt, sc, kFixThreads);
                        __syncthreads();
                        int lo, hi;
                        fx_share<kFixW>(cnt, uniform_i32(wave), &lo, &hi);
                        fx_accumulate(A, S, cnt, lo, hi, G, H, lane);
                    }
                    double x[4 * FxSums<GEN>::kSums];
                    float d[4 * FxSums<GEN>::kSums];
                    fx_gather<GEN, kFixW>(A, s_buf, wave, lane, x, d);
                    const int a = fx_row(wave, lane), c = lane & 15;
                    const double Ga = fx_centre(P.f_min, P.df, P.to_cyc, w0, a);
                    const int64_t i0 = w0 + (int64_t)a * kFxBlk;
#pragma unroll
                    for (int side = 0; side < 2; ++side) {
                        const int64_t i = side ? i0 + kFxOffs + c : i0 + kFxOffs - 1 - c;
                        const double f = grid_freq(P.f_min, P.df, i) * P.to_cyc;
                        bool ill;
                        const double p =
                            fx_power<GEN>(x, d, f, Ga, H, side ? 1.0 : -1.0, m, sc, ill);
                        fx_list(s_left, (int)(i - w0), i < f1 && ill, lane);
                        if (i < f1 && !ill) offer(i, p);
                    }
                }
                __syncthreads();
                const int left = (int)(f1 - w0 < kFxBins ? f1 - w0 : kFxBins);
                fx_direct<GEN, kFixThreads>(
                    S, covered && m.n <= kFxObs, m, P.t, P.y, P.dy, sc, P.f_min, P.df, P.to_cyc,
                    covered ? uniform_i32(s_left.count) : left,
                    [&](int q) { return w0 + (covered ? (int)s_left.bin[q] : q); }, offer);
            }
            best = wave_best(best);
            if (lane == 0) s_red[wave] = best;
            __syncthreads();
            if (threadIdx.x == 0) {
                PeakRec b = s_red[0];
                for (int w = 1; w < kFixW; ++w)
                    if (better(s_red[w].p, s_red[w].i, b.p, b.i)) b = s_red[w];
                if (rr.obj >= 0 && b.i >= 0)
                    atomicMax(&P.keys[row / P.rows_per_group], peak_key(b.p, b.i));
            }
            __syncthreads();
        }
        __syncthreads();
    }
    if (K.peaks && last_workgroup(K, gridDim.x) && (int64_t)threadIdx.x < K.n_groups)
        write_key_peak(K, threadIdx.x);
}

}  // namespace

static_assert(kFxBins == kFxTile, "one record per wave tile");

// The fix-up writes the peaks itself where its last workgroup has a thread for
// each group and there are few workgroups to wait for.  With the clearing done
// by the statistics kernel, a series of 256 points on 10,000 bins takes 19 us, 26
// us with kernels of their own for both.  (The FP64 form's last workgroup was no faster
// than a kernel, 23.9 against 24.1 us: it has records to read.)
constexpr int64_t kMaxLastWg = 256;

int64_t fx_item_bins(int waves, bool split) { return split ? kFxBins : waves * kFxBins; }

bool fixup_writes_peaks(const FixupParams& p, const PeakParams& k) {
    return k.n_groups <= kFixThreads && p.n_tiles <= kMaxLastWg * fix_span(p);
}

template <bool GEN>
static hipError_t launch_fx_g(const MainParams& p, int waves, bool split, hipStream_t s) {
    const dim3 grid = grid_for(p.n_items);
    if (split && waves == 8)
        hipLaunchKernelGGL((fx_kernel<GEN, 8, true>), grid, dim3(kWave * 8), 0, s, p);
    else if (!split && waves == 4)
        hipLaunchKernelGGL((fx_kernel<GEN, 4, false>), grid, dim3(kWave * 4), 0, s, p);
    else
        return hipErrorInvalidValue;
    return hipGetLastError();
}

hipError_t launch_fx(const MainParams& p, int waves, bool split, hipStream_t s) {
    if (p.n_items <= 0) return hipSuccess;
    return p.gen ? launch_fx_g<true>(p, waves, split, s) : launch_fx_g<false>(p, waves, split, s);
}

hipError_t launch_fixup(const FixupParams& p, const PeakParams& k, hipStream_t s) {
    if (p.n_tiles <= 0) return hipSuccess;
    const int span = fix_span(p);
    int64_t blocks = (p.n_tiles + span - 1) / span;
    if (blocks > 2048) blocks = 2048;
    const dim3 grid((unsigned)blocks), threads(kFixThreads);
    if (p.gen)
        hipLaunchKernelGGL(fixup_kernel<true>, grid, threads, 0, s, p, k, span);
    else
        hipLaunchKernelGGL(fixup_kernel<false>, grid, threads, 0, s, p, k, span);
    return hipGetLastError();
}

}  // namespace lsp
