// lsp_mlp.hip -- kernels of the learned band proposal: a BF16 matrix-core GEMM
// with FP32 accumulation (forward X.W, backward-data dY.W^T and
// backward-weight X^T.dY all use it through strides), and the small element
// kernels around it (softmax cross-entropy, column sums, Adam, feature
// standardisation, top-k bands, FP32 -> BF16).
//
// GEMM.  A workgroup of four wavefronts owns a BM x BN tile of C and walks K in
// steps of BK.  The operands of the next D steps are in flight to registers
// while the current one's are multiplied out of LDS, and go to the other of two
// LDS buffers, one barrier a step.  An operand whose k is contiguous is kept in
// LDS with k contiguous, one whose rows (m of A, n of B) are contiguous with
// its rows contiguous, so both are written as they come, 16 bytes at a time;
// the latter is turned when it is read, by ds_read_b64_tr_b16 (four k of one
// row per lane from four rows of 16).  Each wavefront then issues
// v_mfma_f32_16x16x32_bf16 on its part of the tile, k in increasing blocks of
// 32 whatever the tile, so that a result does not depend on the tile taken.
// The instruction gets B's fragment first: its result then holds four
// neighbouring columns of one row per lane, which are stored together.
//
// Rows of a ragged last tile are read as the matrix's last row, so that such a
// tile runs at the speed of the others: four of them, taken element by element
// without prefetch, held a whole 20,000-row product up from 54 to 69 us.
//
// What bounds it: at 20,000 x 1,088 x 512 the matrix cores are busy 29 % of the
// time and LDS 43 %; the two waves a SIMD has room for (128 x 128 tiles) wait
// for each other's LDS reads and MFMAs and for the barrier.  In a training step
// (512 rows) every product is a latency chain of K / 64 steps.  Measured (one k
// step of 32 per barrier pair, no prefetch -> here): 20,000 x 1,088 x 512 156 ->
// 44 us (500 TFLOP/s), 20,000 x 512 x 256 54 -> 18 us; a training step of 512
// rows, which was 17 launches, 199 -> 43 us in 8.
#include <math.h>
#include <stdint.h>
#include <string.h>

#include "lsp_common.h"

namespace lsp {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

__host__ __device__ __forceinline__ uint16_t f32_to_bf16_bits(float f) {
    uint32_t u;
    memcpy(&u, &f, sizeof u);
    if ((u & 0x7f800000u) == 0x7f800000u && (u & 0x007fffffu)) return (uint16_t)((u >> 16) | 0x40);
    u += 0x7fffu + ((u >> 16) & 1u);  // round to nearest even
    return (uint16_t)(u >> 16);
}

__device__ __forceinline__ float bf16_bits_to_f32(uint16_t h) {
    return __uint_as_float((uint32_t)h << 16);
}

struct GemmArgs {
    int64_t M, N, K;
    const uint16_t* A;
    int64_t sam, sak;
    const uint16_t* B;
    int64_t sbk, sbn;
    const float* bias;     // [N] or NULL
    const uint16_t* mask;  // BF16 [M x N], leading dimension ldc: keep C where mask > 0
    int32_t relu;
    int32_t pad;
    float* Cf;             // FP32 output or NULL
    uint16_t* Cb;          // BF16 output or NULL
    int64_t ldc;
    int32_t a_mode, b_mode;  // how each operand is staged: kLoad*
    int32_t c_vec;           // four neighbouring results (and mask values) move together
    int32_t pad2;
};

// How an operand tile is read from global memory: 8 consecutive k in one
// 16-byte load, 8 consecutive rows (m of A, n of B) in one 16-byte load, or
// element by element.
enum { kLoadK = 0, kLoadRows = 1, kLoadScalar = 2 };

// Strides (elements) of the 16-byte modes: a tile's places are 32-bit offsets.
constexpr int64_t kMaxStride = 1 << 23;

// One operand's tile of BO rows x BK k: 16-byte chunks per thread in registers
// on the way from global memory to LDS.  MODE: kLoad* (kLoadScalar keeps k
// contiguous in LDS, as kLoadK).
template <int BO, int BK, int MODE, int D = 1>
struct Operand {
    static constexpr int kThreads = 256;
    static constexpr bool kRows = MODE == kLoadRows;
    static constexpr int kChunks = BO * BK / 8;  // 8 elements each
    static constexpr int kPer = kChunks / kThreads;
    static_assert(kChunks % kThreads == 0, "whole chunks per thread");
    // padded pitch (elements) that keeps 16-byte alignment and spreads the
    // fragment reads over the banks
    static constexpr int kPitch = kRows ? BO + 16 : BK + 8;
    static constexpr int kLds = (kRows ? BK : BO) * kPitch;
    // consecutive threads take consecutive chunks of a line (a row's k, or one
    // k's rows), and each thread the same place of kPer lines kStep apart
    static constexpr int kLine = (kRows ? BO : BK) / 8;
    static constexpr int kStep = kThreads / kLine;

    u32x4 v[D][kPer];
    uint32_t off[kPer];
    int line, at;  // this thread's first line, and its element within a line

    __device__ __forceinline__ Operand()
        : line((int)threadIdx.x / kLine), at(((int)threadIdx.x % kLine) * 8) {}

    // Whether fetch() serves a tile of rows from o0: it lies inside the matrix,
    // or its rows past the end can be read as other rows of the matrix (their
    // results are not stored).
    static __device__ __forceinline__ bool plain(int64_t O, int64_t o0) {
        return MODE != kLoadScalar && (o0 + BO <= O || !kRows || O % 8 == 0);
    }

    // This thread's places in a tile of rows from o0, in bytes from the tile's
    // corner (strides are below kMaxStride).
    __device__ __forceinline__ void place(int64_t so, int64_t sk, int64_t O, int64_t o0) {
        const int64_t top = (kRows ? O - 8 : O - 1) - o0;
#pragma unroll
        for (int i = 0; i < kPer; ++i) {
            int64_t o = kRows ? at : line + i * kStep;
            const int64_t k = kRows ? line + i * kStep : at;
            o = o < top ? o : top;
            off[i] = 2u * (uint32_t)(o * so + k * sk);
        }
    }

    // The BK k from the tile's corner (o0, k0) on, into register set d.
    __device__ __forceinline__ void fetch(int d, const uint16_t* corner) {
#pragma unroll
        for (int i = 0; i < kPer; ++i)
            v[d][i] = *reinterpret_cast<const u32x4*>(reinterpret_cast<const char*>(corner) +
                                                      off[i]);
    }

    // The same at the end of k, at a ragged edge of rows and in any mode: zeros
    // outside the matrix.
    __device__ __forceinline__ void fetch_edge(const uint16_t* X, int64_t so, int64_t sk, int64_t O,
                                               int64_t K, int64_t o0, int64_t k0) {
        const int64_t o = o0 + (kRows ? at : line), k = k0 + (kRows ? line : at);
        uint32_t part = 0u;  // chunks partly outside (or scattered)
#pragma unroll
        for (int i = 0; i < kPer; ++i) {
            const int64_t oi = kRows ? o : o + i * kStep, ki = kRows ? k + i * kStep : k;
            v[0][i] = u32x4{0u, 0u, 0u, 0u};
            if (oi < O && ki < K) {
                if (MODE != kLoadScalar && (kRows ? oi + 8 <= O : ki + 8 <= K))
                    v[0][i] = *reinterpret_cast<const u32x4*>(X + oi * so + ki * sk);
                else
                    part |= 1u << i;
            }
        }
        if (!part) return;
#pragma unroll
        for (int i = 0; i < kPer; ++i) {
            if (!((part >> i) & 1u)) continue;
            const int64_t oi = kRows ? o : o + i * kStep, ki = kRows ? k + i * kStep : k;
            uint16_t e[8];
#pragma unroll
            for (int r = 0; r < 8; ++r) {
                const int64_t oe = kRows ? oi + r : oi, ke = kRows ? ki : ki + r;
                e[r] = oe < O && ke < K ? X[oe * so + ke * sk] : 0;
            }
#pragma unroll
            for (int r = 0; r < 4; ++r) v[0][i][r] = e[2 * r] | ((uint32_t)e[2 * r + 1] << 16);
        }
    }

    __device__ __forceinline__ void put(int d, uint16_t* L) const {
#pragma unroll
        for (int i = 0; i < kPer; ++i)
            *reinterpret_cast<u32x4*>(L + (line + i * kStep) * kPitch + at) = v[d][i];
    }

    // The fragment of rows [o, o + 16) and k [kk, kk + 32): row lane % 16,
    // k 8 (lane / 16) + 0..7.
    static __device__ __forceinline__ bf16x8 fragment(const uint16_t* L, int o, int kk, int lane) {
        const int g = lane >> 4, i = lane & 15;
        if (!kRows) return *reinterpret_cast<const bf16x8*>(L + (o + i) * kPitch + kk + 8 * g);
        typedef __attribute__((address_space(3))) s16x4* lds_s16x4;
        const uint16_t* src = L + (kk + 8 * g + (i >> 2)) * kPitch + o + 4 * (i & 3);
        union {
            s16x4 half[2];
            bf16x8 all;
        } f;
        f.half[0] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4)(src));
        f.half[1] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4)(src + 4 * kPitch));
        return f.all;
    }
};

// LDS elements of a BM x BN tile's two buffers of both operands, in any mode.
template <int BM, int BN, int BK>
constexpr int gemm_lds() {
    constexpr int am = Operand<BM, BK, kLoadK>::kLds > Operand<BM, BK, kLoadRows>::kLds
                           ? Operand<BM, BK, kLoadK>::kLds
                           : Operand<BM, BK, kLoadRows>::kLds;
    constexpr int bm = Operand<BN, BK, kLoadK>::kLds > Operand<BN, BK, kLoadRows>::kLds
                           ? Operand<BN, BK, kLoadK>::kLds
                           : Operand<BN, BK, kLoadRows>::kLds;
    return 2 * (am + bm);
}

// Bias, ReLU and mask on a wave's results, and their stores: fragment (i, j)
// of the wave holds columns n + 16 j + 0..3 of row m + 16 i in this lane.
// WHOLE: the tile lies inside C and four neighbouring results move together.
template <int TI, int TJ, bool WHOLE>
__device__ __forceinline__ void gemm_epilogue(const GemmArgs& g, int64_t m, int64_t n,
                                              f32x4 (&acc)[TI][TJ]) {
    auto in = [&](int i, int j, int r) {
        return WHOLE || (m + 16 * i < g.M && n + 16 * j + r < g.N);
    };
    if (g.bias) {
#pragma unroll
        for (int j = 0; j < TJ; ++j) {
            f32x4 bias;
#pragma unroll
            for (int r = 0; r < 4; ++r)
                bias[r] = WHOLE || n + 16 * j + r < g.N ? g.bias[n + 16 * j + r] : 0.0f;
#pragma unroll
            for (int i = 0; i < TI; ++i)
#pragma unroll
                for (int r = 0; r < 4; ++r) acc[i][j][r] += bias[r];
        }
    }
    if (g.relu) {
#pragma unroll
        for (int i = 0; i < TI; ++i)
#pragma unroll
            for (int j = 0; j < TJ; ++j)
#pragma unroll
                for (int r = 0; r < 4; ++r) acc[i][j][r] = acc[i][j][r] > 0.f ? acc[i][j][r] : 0.f;
    }
    if (g.mask) {
#pragma unroll
        for (int i = 0; i < TI; ++i) {
            const uint16_t* const mk = g.mask + (m + 16 * i) * g.ldc + n;
#pragma unroll
            for (int j = 0; j < TJ; ++j) {
                uint16_t e[4];
                if (WHOLE) {
                    const ushort4 q = *reinterpret_cast<const ushort4*>(mk + 16 * j);
                    e[0] = q.x, e[1] = q.y, e[2] = q.z, e[3] = q.w;
                } else {
#pragma unroll
                    for (int r = 0; r < 4; ++r) e[r] = in(i, j, r) ? mk[16 * j + r] : 0;
                }
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    if (!(bf16_bits_to_f32(e[r]) > 0.f)) acc[i][j][r] = 0.f;
            }
        }
    }
    auto each = [&](auto&& store) {
#pragma unroll
        for (int i = 0; i < TI; ++i)
#pragma unroll
            for (int j = 0; j < TJ; ++j) store(i, j, (m + 16 * i) * g.ldc + n + 16 * j);
    };
    if (g.Cf)
        each([&](int i, int j, int64_t at) {
            if (WHOLE)
                *reinterpret_cast<f32x4*>(g.Cf + at) = acc[i][j];
            else
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    if (in(i, j, r)) g.Cf[at + r] = acc[i][j][r];
        });
    if (g.Cb)
        each([&](int i, int j, int64_t at) {
            uint16_t e[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) e[r] = f32_to_bf16_bits(acc[i][j][r]);
            if (WHOLE)
                *reinterpret_cast<ushort4*>(g.Cb + at) = make_ushort4(e[0], e[1], e[2], e[3]);
            else
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    if (in(i, j, r)) g.Cb[at + r] = e[r];
        });
}

// One BM x BN tile of C, by the 256 threads of a workgroup as WM x WN waves.
template <int BM, int BN, int BK, int WM, int WN, int D, int AMODE, int BMODE>
__device__ __forceinline__ void gemm_tile(const GemmArgs& g, int64_t m0, int64_t n0,
                                          uint16_t* lds) {
    typedef Operand<BM, BK, AMODE> OpA;
    typedef Operand<BN, BK, BMODE> OpB;
    constexpr int TI = BM / WM / 16, TJ = BN / WN / 16;  // 16 x 16 fragments per wave
    uint16_t* const As = lds;
    uint16_t* const Bs = lds + 2 * OpA::kLds;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int wm = (wave / WN) * (BM / WM), wn = (wave % WN) * (BN / WN);

    f32x4 acc[TI][TJ];
#pragma unroll
    for (int i = 0; i < TI; ++i)
#pragma unroll
        for (int j = 0; j < TJ; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

    auto multiply = [&](const uint16_t* la, const uint16_t* lb, int kk) {
        bf16x8 af[TI], bf[TJ];
#pragma unroll
        for (int i = 0; i < TI; ++i) af[i] = OpA::fragment(la, wm + 16 * i, kk, lane);
#pragma unroll
        for (int j = 0; j < TJ; ++j) bf[j] = OpB::fragment(lb, wn + 16 * j, kk, lane);
#pragma unroll
        for (int i = 0; i < TI; ++i)
#pragma unroll
            for (int j = 0; j < TJ; ++j)
                acc[i][j] =
                    __builtin_amdgcn_mfma_f32_16x16x32_bf16(bf[j], af[i], acc[i][j], 0, 0, 0);
    };
    int buf = 0;
    int64_t done = 0;  // k handled by the first loop
    if (OpA::plain(g.M, m0) && OpB::plain(g.N, n0) && g.K >= BK) {
        // D steps in flight; loads past the last step repeat it, so that the
        // loop has no branch around a load (the wait for one would be a wait
        // for all)
        Operand<BM, BK, AMODE, D> a;
        Operand<BN, BK, BMODE, D> b;
        a.place(g.sam, g.sak, g.M, m0);
        b.place(g.sbn, g.sbk, g.N, n0);
        const uint16_t* const A0 = g.A + m0 * g.sam;
        const uint16_t* const B0 = g.B + n0 * g.sbn;
        done = g.K / BK * BK;
        const int64_t last = done - BK;
#pragma unroll
        for (int d = 0; d < D; ++d) {
            const int64_t k = (int64_t)d * BK < last ? (int64_t)d * BK : last;
            a.fetch(d, A0 + k * g.sak);
            b.fetch(d, B0 + k * g.sbk);
        }
        auto step = [&](int d, int64_t k0) {
            uint16_t* const la = As + buf * OpA::kLds;
            uint16_t* const lb = Bs + buf * OpB::kLds;
            a.put(d, la);
            b.put(d, lb);
            __syncthreads();
            const int64_t k = k0 + D * BK < last ? k0 + D * BK : last;
            a.fetch(d, A0 + k * g.sak);
            b.fetch(d, B0 + k * g.sbk);
            // the loads stay here, ahead of this step's products
            asm volatile("" ::: "memory");
#pragma unroll
            for (int kk = 0; kk < BK; kk += 32) multiply(la, lb, kk);
            buf ^= 1;
        };
        int64_t k0 = 0;
        for (; k0 + (D - 1) * BK < done; k0 += D * BK)
#pragma unroll
            for (int d = 0; d < D; ++d) step(d, k0 + d * BK);
#pragma unroll
        for (int d = 0; d < D - 1; ++d)
            if (k0 + d * BK < done) step(d, k0 + d * BK);
    }
    for (int64_t k0 = done; k0 < g.K; k0 += BK) {
        OpA a;
        OpB b;
        uint16_t* const la = As + buf * OpA::kLds;
        uint16_t* const lb = Bs + buf * OpB::kLds;
        a.fetch_edge(g.A, g.sam, g.sak, g.M, g.K, m0, k0);
        b.fetch_edge(g.B, g.sbn, g.sbk, g.N, g.K, n0, k0);
        a.put(0, la);
        b.put(0, lb);
        __syncthreads();
#pragma unroll 1
        for (int kk = 0; kk < BK && k0 + kk < g.K; kk += 32) multiply(la, lb, kk);
        buf ^= 1;
    }
    // All of the epilogue's loads come before its first store: a wait for a
    // load also waits for the stores issued before it.
    const int64_t m = m0 + wm + (lane & 15), n = n0 + wn + 4 * (lane >> 4);
    if (m0 + BM <= g.M && n0 + BN <= g.N && g.c_vec) {
        gemm_epilogue<TI, TJ, true>(g, m, n, acc);
    } else {
        gemm_epilogue<TI, TJ, false>(g, m, n, acc);
    }
}

// Column sums of an n x c FP32 matrix, 16 or 64 columns per workgroup of 256
// threads and 16 row phases (row i goes to phase i mod 16): a phase is summed in
// row order by one thread and the 16 phase sums are added in phase order, so the
// result does not depend on scheduling or on the columns per workgroup.
struct ColSums {
    const float* x;
    int64_t n;
    int32_t c;
    int32_t wide;  // 64 columns per workgroup
    float* out;
};

constexpr int kSumCols = 16, kSumWide = 64, kSumPhases = 16;

// 64 columns give whole cache lines of a row, but where there are not as many
// workgroups of them as CUs, 16 columns and a phase a thread keep more rows in
// flight: 100 x 50,000 7.0 us (16 columns 9.5), 1,000 x 20,000 15.0 us (24.7); 100,000
// x 64 271 us with 16 columns.
inline bool sum_wide(int64_t c) { return c >= 256 * kSumWide; }

template <int COLS>
__device__ __forceinline__ void col_sums_block(const ColSums& S, int64_t block, float* lds) {
    constexpr int kRows = 256 / COLS, kPer = kSumPhases / kRows;  // phases per thread
    const int tx = threadIdx.x % COLS, r = threadIdx.x / COLS;
    const int64_t j = block * COLS + tx;
    float s[kPer];
#pragma unroll
    for (int k = 0; k < kPer; ++k) s[k] = 0.f;
    if (j < S.c) {
        // eight rows in flight, each phase's added in order
        constexpr int kTurns = 8 / kPer;
        int64_t i = 0;
        for (; i + kTurns * kSumPhases <= S.n; i += kTurns * kSumPhases) {
            float v[kTurns][kPer];
#pragma unroll
            for (int q = 0; q < kTurns; ++q)
#pragma unroll
                for (int k = 0; k < kPer; ++k)
                    v[q][k] = S.x[(i + q * kSumPhases + k * kRows + r) * S.c + j];
#pragma unroll
            for (int q = 0; q < kTurns; ++q)
#pragma unroll
                for (int k = 0; k < kPer; ++k) s[k] += v[q][k];
        }
        for (; i < S.n; i += kSumPhases)
#pragma unroll
            for (int k = 0; k < kPer; ++k) {
                const int64_t row = i + k * kRows + r;
                if (row < S.n) s[k] += S.x[row * S.c + j];
            }
    }
#pragma unroll
    for (int k = 0; k < kPer; ++k) lds[(k * kRows + r) * COLS + tx] = s[k];
    __syncthreads();
    if (r == 0 && j < S.c) {
        float t = lds[tx];
        for (int q = 1; q < kSumPhases; ++q) t += lds[q * COLS + tx];
        S.out[j] = t;
    }
}

// Up to two independent products and one set of column sums in one launch: the
// blocks below tiles[0] take the first product's tiles, those below
// tiles[0] + tiles[1] the second's, the rest the sums.  (A backward layer's
// weight gradient, input gradient and bias gradient need the same inputs; each
// alone leaves most of the chip idle.)
struct GemmGroup {
    GemmArgs g[2];
    ColSums s;
    int64_t tiles[2];
    int64_t blocks;
};

// GENERAL: any load modes, else those of the network's products (X.W, dY.W^T
// and X^T.dY with 16-byte aligned rows).
template <int BM, int BN, int BK, int WM, int WN, int D, bool GENERAL>
__global__ __launch_bounds__(256, 2) void gemm_group_kernel(const GemmGroup G) {
    __shared__ __attribute__((aligned(16))) uint16_t lds[gemm_lds<BM, BN, BK>()];
    int64_t b = linear_block();
    if (b >= G.blocks) return;
    if (b >= G.tiles[0] + G.tiles[1]) {
        b -= G.tiles[0] + G.tiles[1];
        if (G.s.wide)
            col_sums_block<kSumWide>(G.s, b, reinterpret_cast<float*>(lds));
        else
            col_sums_block<kSumCols>(G.s, b, reinterpret_cast<float*>(lds));
        return;
    }
    const int which = b >= G.tiles[0];
    if (which) b -= G.tiles[0];
    const GemmArgs& g = G.g[which];
    // neighbouring tiles, which share their rows of A, on one XCD
    b = xcd_remap(b, G.tiles[which]);
    const int64_t across = (g.N + BN - 1) / BN;
    const int64_t tm = b / across, m0 = tm * BM, n0 = (b - tm * across) * BN;
    if constexpr (GENERAL) {
        if (g.a_mode == kLoadK && g.b_mode == kLoadScalar)
            gemm_tile<BM, BN, BK, WM, WN, D, kLoadK, kLoadScalar>(g, m0, n0, lds);
        else if (g.a_mode == kLoadRows && g.b_mode == kLoadK)
            gemm_tile<BM, BN, BK, WM, WN, D, kLoadRows, kLoadK>(g, m0, n0, lds);
        else if (g.a_mode == kLoadRows && g.b_mode == kLoadScalar)
            gemm_tile<BM, BN, BK, WM, WN, D, kLoadRows, kLoadScalar>(g, m0, n0, lds);
        else if (g.a_mode == kLoadScalar && g.b_mode == kLoadK)
            gemm_tile<BM, BN, BK, WM, WN, D, kLoadScalar, kLoadK>(g, m0, n0, lds);
        else if (g.a_mode == kLoadScalar && g.b_mode == kLoadRows)
            gemm_tile<BM, BN, BK, WM, WN, D, kLoadScalar, kLoadRows>(g, m0, n0, lds);
        else
            gemm_tile<BM, BN, BK, WM, WN, D, kLoadScalar, kLoadScalar>(g, m0, n0, lds);
    } else {
        if (g.a_mode == kLoadRows)
            gemm_tile<BM, BN, BK, WM, WN, D, kLoadRows, kLoadRows>(g, m0, n0, lds);
        else if (g.b_mode == kLoadRows)
            gemm_tile<BM, BN, BK, WM, WN, D, kLoadK, kLoadRows>(g, m0, n0, lds);
        else
            gemm_tile<BM, BN, BK, WM, WN, D, kLoadK, kLoadK>(g, m0, n0, lds);
    }
}

// One wavefront per row: softmax of the row's logits, cross-entropy against
// the label, and the gradient (softmax - onehot) * scale.
__global__ __launch_bounds__(256) void softmax_xent_kernel(const float* __restrict__ logits,
                                                           const int32_t* __restrict__ labels,
                                                           int64_t n, int32_t c, float scale,
                                                           float* dlogits, uint16_t* dlogits_bf16,
                                                           float* loss_rows) {
    const int64_t row = linear_block() * 4 + (threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    if (row >= n) return;
    const float* z = logits + row * c;
    float mx = -INFINITY;
    for (int j = lane; j < c; j += 64) mx = fmaxf(mx, z[j]);
    for (int off = 32; off >= 1; off >>= 1) mx = fmaxf(mx, __shfl_xor(mx, off, 64));
    float se = 0.f;
    for (int j = lane; j < c; j += 64) se += expf(z[j] - mx);
    for (int off = 32; off >= 1; off >>= 1) se += __shfl_xor(se, off, 64);
    const int32_t lab = labels[row];
    const bool keep = lab >= 0 && lab < c;  // other labels mark rows to ignore
    for (int j = lane; j < c; j += 64) {
        const float p = expf(z[j] - mx) / se;
        const float d = keep ? (p - (j == lab ? 1.f : 0.f)) * scale : 0.f;
        if (dlogits) dlogits[row * c + j] = d;
        if (dlogits_bf16) dlogits_bf16[row * c + j] = f32_to_bf16_bits(d);
    }
    if (lane == 0 && loss_rows)
        loss_rows[row] = keep ? (logf(se) + mx - z[lab]) : 0.f;
}

// Training labels from full-grid peaks: the band holding each peak, or -1 for
// an object without a peak.
__global__ void peak_bands_kernel(const lsp_peak* __restrict__ peaks, int64_t n,
                                  int64_t band_bins, int32_t n_bands, int32_t* labels) {
    const int64_t i = linear_block() * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const lsp_peak pk = peaks[i];
    int32_t b = -1;
    if (pk.status == LSP_OBJ_OK && pk.index >= 0) {
        const int64_t q = pk.index / band_bins;
        b = q < n_bands ? (int32_t)q : -1;
    }
    labels[i] = b;
}

// Objects whose refined peak must be confirmed on the whole grid, listed in
// increasing order: status OK and (proposal mass below mass_min, or refined
// power below power_min or not a number, or no peak found).  One workgroup
// walks the objects 1,024 at a time; each wave compacts its flags with a
// ballot and the waves' counts are prefix-summed in LDS.
constexpr int kSelThreads = 1024;

__global__ __launch_bounds__(kSelThreads) void select_kernel(const lsp_peak* __restrict__ peaks,
                                                           const float* __restrict__ mass,
                                                           int64_t n, float mass_min,
                                                           float power_min, int32_t* out,
                                                           int32_t* count) {
    __shared__ int32_t s_cnt[kSelThreads / 64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    int64_t done = 0;
    for (int64_t base = 0; base < n; base += kSelThreads) {
        const int64_t i = base + threadIdx.x;
        bool need = false;
        if (i < n) {
            const lsp_peak pk = peaks[i];
            if (pk.status == LSP_OBJ_OK)
                need = !(pk.index >= 0) || !(pk.power >= (double)power_min) ||
                       (mass && !(mass[i] >= mass_min));
        }
        const uint64_t m = __ballot(need);
        if (lane == 0) s_cnt[wave] = __popcll(m);
        __syncthreads();
        int64_t off = done;
        int32_t total = 0;
        for (int w = 0; w < kSelThreads / 64; ++w) {
            if (w < wave) off += s_cnt[w];
            total += s_cnt[w];
        }
        if (need) {
            const uint64_t below = lane ? (m & ((~0ull) >> (64 - lane))) : 0ull;
            out[off + __popcll(below)] = (int32_t)i;
        }
        done += total;
        __syncthreads();
    }
    if (threadIdx.x == 0) *count = (int32_t)done;
}

// Column mean and 1/std (population) of an n x d FP32 matrix; a column with no
// spread gets 1/std = 1.  One thread per column, fixed order, FP64 sums.
__global__ void col_stats_kernel(const float* __restrict__ x, int64_t n, int32_t d, float* mean,
                                 float* inv_std) {
    const int32_t j = blockIdx.x * blockDim.x + threadIdx.x;
    if (j >= d) return;
    double s = 0.0;
    for (int64_t i = 0; i < n; ++i) s += (double)x[i * d + j];
    const double mu = n > 0 ? s / (double)n : 0.0;
    double q = 0.0;
    for (int64_t i = 0; i < n; ++i) {
        const double e = (double)x[i * d + j] - mu;
        q += e * e;
    }
    const double sd = n > 0 ? sqrt(q / (double)n) : 0.0;
    mean[j] = (float)mu;
    inv_std[j] = sd > 1e-12 ? (float)(1.0 / sd) : 0.0f;  // a constant column carries nothing
}

// Replace the statistics of columns [start, start + count) by those of the
// pooled block (every entry of those columns taken together):
// mean = mean_j m_j, var = mean_j (var_j + m_j^2) - mean^2.  One workgroup,
// fixed-order sums.
__global__ __launch_bounds__(256) void pool_stats_kernel(float* mean, float* inv_std,
                                                         int32_t start, int32_t count) {
    __shared__ double s_m[256], s_q[256];
    double m = 0.0, q = 0.0;
    for (int32_t j = threadIdx.x; j < count; j += 256) {
        const double mj = mean[start + j];
        const double is = inv_std[start + j];
        m += mj;
        q += (is > 0.0 ? 1.0 / (is * is) : 0.0) + mj * mj;
    }
    s_m[threadIdx.x] = m;
    s_q[threadIdx.x] = q;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) {
            s_m[threadIdx.x] += s_m[threadIdx.x + w];
            s_q[threadIdx.x] += s_q[threadIdx.x + w];
        }
        __syncthreads();
    }
    const double mu = s_m[0] / (double)count;
    const double var = s_q[0] / (double)count - mu * mu;
    const float is = var > 1e-24 ? (float)(1.0 / sqrt(var)) : 0.0f;
    for (int32_t j = threadIdx.x; j < count; j += 256) {
        mean[start + j] = (float)mu;
        inv_std[start + j] = is;
    }
}

// Row standardisation of a column block: in each row of x [n x d], the
// columns [start, start + count) become (x - row mean) / row std over those
// columns (0 where the row is constant).  One wavefront per row, FP64 sums,
// fixed order.  Makes the coarse spectrum's shape, not its overall level,
// what the network sees: a short series has a much higher noise floor than a
// long one, while the band that holds the peak is a property of the shape.
__global__ __launch_bounds__(256) void row_norm_kernel(float* x, int64_t n, int32_t d,
                                                       int32_t start, int32_t count) {
    const int64_t row = linear_block() * 4 + (threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    if (row >= n) return;
    float* r = x + row * d + start;
    double s = 0.0, q = 0.0;
    for (int32_t j = lane; j < count; j += 64) {
        const double v = r[j];
        s += v;
        q += v * v;
    }
    for (int off = 32; off >= 1; off >>= 1) {
        s += __shfl_xor(s, off, 64);
        q += __shfl_xor(q, off, 64);
    }
    const double mu = s / (double)count;
    const double var = q / (double)count - mu * mu;
    const double inv = var > 1e-24 ? 1.0 / sqrt(var) : 0.0;
    for (int32_t j = lane; j < count; j += 64) r[j] = (float)(((double)r[j] - mu) * inv);
}

// Largest value of each band's columns: row i's columns [start + b*group,
// start + (b+1)*group) for b < n_bands.  One thread per (row, band).
__global__ void band_max_kernel(const float* __restrict__ x, int64_t n, int32_t d, int32_t start,
                                int32_t n_bands, int32_t group, float* __restrict__ out) {
    const int64_t e = linear_block() * blockDim.x + threadIdx.x;
    if (e >= n * n_bands) return;
    const int64_t i = e / n_bands;
    const int32_t b = (int32_t)(e - i * n_bands);
    const float* r = x + i * d + start + (int64_t)b * group;
    float m = r[0];
    for (int32_t j = 1; j < group; ++j) m = fmaxf(m, r[j]);
    out[e] = m;
}

// Per row: the entries of a (in order), then those of b not already taken,
// until k_out distinct non-negative bands; -1 fills what is left.
__global__ void merge_bands_kernel(const int32_t* __restrict__ a, int32_t ka,
                                   const int32_t* __restrict__ b, int32_t kb, int64_t n,
                                   int32_t k_out, int32_t* __restrict__ out) {
    const int64_t i = linear_block() * blockDim.x + threadIdx.x;
    if (i >= n) return;
    int32_t* o = out + i * k_out;
    int32_t m = 0;
    for (int32_t src = 0; src < 2; ++src) {
        const int32_t* v = src == 0 ? a + i * ka : b + i * kb;
        const int32_t kv = src == 0 ? ka : kb;
        for (int32_t j = 0; j < kv && m < k_out; ++j) {
            const int32_t band = v[j];
            if (band < 0) continue;
            bool seen = false;
            for (int32_t q = 0; q < m; ++q) seen |= o[q] == band;
            if (!seen) o[m++] = band;
        }
    }
    for (; m < k_out; ++m) o[m] = -1;
}

// Training-time shift augmentation.  Row i's first n_coarse columns hold
// n_bands groups of `group` columns, one group per frequency band; they move
// by shift[i] groups (vacated columns get `fill`), the other columns are
// copied, and the label moves with them (-1 if it leaves [0, n_bands) or was
// already -1).  A signal whose frequency moves by one band width moves its
// coarse spectrum by one group, so this multiplies the labelled examples.
__global__ void shift_bands_kernel(const uint16_t* __restrict__ x,
                                   const int32_t* __restrict__ labels,
                                   const int32_t* __restrict__ shifts, int64_t n, int32_t d,
                                   int32_t n_coarse, int32_t group, int32_t n_bands,
                                   uint16_t fill, uint16_t* __restrict__ out,
                                   int32_t* __restrict__ out_labels) {
    const int64_t e = linear_block() * blockDim.x + threadIdx.x;
    if (e >= n * d) return;
    const int64_t i = e / d;
    const int32_t j = (int32_t)(e - i * d);
    const int32_t sh = shifts[i];
    uint16_t v;
    if (j < n_coarse) {
        const int64_t src = (int64_t)j - (int64_t)sh * group;
        v = (src >= 0 && src < n_coarse) ? x[i * d + src] : fill;
    } else {
        v = x[e];
    }
    out[e] = v;
    if (j == 0) {
        const int32_t lab = labels[i];
        const int32_t nl = lab + sh;
        out_labels[i] = (lab >= 0 && nl >= 0 && nl < n_bands) ? nl : -1;
    }
}

__global__ void standardize_kernel(const float* __restrict__ x, int64_t n, int32_t d,
                                   const float* __restrict__ mean,
                                   const float* __restrict__ inv_std, uint16_t* out) {
    const int64_t i = linear_block() * blockDim.x + threadIdx.x;
    if (i >= n * d) return;
    const int32_t j = (int32_t)(i % d);
    out[i] = f32_to_bf16_bits((x[i] - mean[j]) * inv_std[j]);
}

__global__ void cast_bf16_kernel(const float* __restrict__ x, int64_t count, uint16_t* out) {
    const int64_t i = linear_block() * blockDim.x + threadIdx.x;
    if (i < count) out[i] = f32_to_bf16_bits(x[i]);
}

// Adam with bias correction on FP32 master parameters; optionally refreshes
// the BF16 copy the GEMMs read.  One launch takes up to six parameter arrays,
// each from a block of its own on.
struct AdamArray {
    float* p;
    const float* grad;
    float* m;
    float* v;
    uint16_t* p_bf16;
    int64_t count;
    int64_t first;  // its first block
};

constexpr int kAdamArrays = 6, kAdamThreads = 256;

struct AdamArgs {
    AdamArray a[kAdamArrays];
    int32_t n;
    float lr, b1, b2, eps, c1, c2;
    int64_t blocks;
};

__global__ __launch_bounds__(kAdamThreads) void adam_kernel(const AdamArgs A) {
    const int64_t b = linear_block();
    if (b >= A.blocks) return;
    int k = 0;
#pragma unroll
    for (int q = 1; q < kAdamArrays; ++q)
        if (q < A.n && b >= A.a[q].first) k = q;
    const AdamArray& a = A.a[k];
    const int64_t i = (b - a.first) * kAdamThreads + threadIdx.x;
    if (i >= a.count) return;
    const float gi = a.grad[i];
    const float mi = A.b1 * a.m[i] + (1.f - A.b1) * gi;
    const float vi = A.b2 * a.v[i] + (1.f - A.b2) * gi * gi;
    a.m[i] = mi;
    a.v[i] = vi;
    const float pi = a.p[i] - A.lr * (mi / A.c1) / (sqrtf(vi / A.c2) + A.eps);
    a.p[i] = pi;
    if (a.p_bf16) a.p_bf16[i] = f32_to_bf16_bits(pi);
}

// One wavefront per row: the k largest of c logits (lowest index on ties), in
// decreasing order, and the softmax probability mass they carry.
__global__ __launch_bounds__(256) void top_k_kernel(const float* __restrict__ logits, int64_t n,
                                                    int32_t c, int32_t k, int32_t* idx,
                                                    float* mass) {
    const int64_t row = linear_block() * 4 + (threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    if (row >= n) return;
    const float* z = logits + row * c;
    // each lane holds up to two logits (c <= 128)
    float v0 = lane < c ? z[lane] : -INFINITY;
    float v1 = lane + 64 < c ? z[lane + 64] : -INFINITY;
    float mx = fmaxf(v0, v1);
    for (int off = 32; off >= 1; off >>= 1) mx = fmaxf(mx, __shfl_xor(mx, off, 64));
    float se = (lane < c ? expf(v0 - mx) : 0.f) + (lane + 64 < c ? expf(v1 - mx) : 0.f);
    for (int off = 32; off >= 1; off >>= 1) se += __shfl_xor(se, off, 64);
    float taken = 0.f;
    for (int r = 0; r < k; ++r) {
        float bv = v0;
        int bi = lane < c ? lane : 1 << 30;
        if (v1 > bv || (v1 == bv && lane + 64 < c && lane + 64 < bi)) {
            bv = v1;
            bi = lane + 64 < c ? lane + 64 : 1 << 30;
        }
        for (int off = 32; off >= 1; off >>= 1) {
            const float ov = __shfl_xor(bv, off, 64);
            const int oi = __shfl_xor(bi, off, 64);
            if (ov > bv || (ov == bv && oi < bi)) {
                bv = ov;
                bi = oi;
            }
        }
        if (lane == 0) idx[row * k + r] = bi < c ? bi : -1;
        if (bi < c) taken += expf(bv - mx);
        if (bi == lane) v0 = -INFINITY;
        if (bi == lane + 64) v1 = -INFINITY;
    }
    if (lane == 0 && mass) mass[row] = taken / se;
}

// Adaptive band count, one wavefront per row.  Row i's `top` proposed bands
// idx[i][r] -- slots r < n_net from the network in decreasing probability,
// the rest in decreasing coarse power -- are copied to out[i][r] or replaced
// by -1:
//   a network slot is kept while the softmax mass of the kept network slots
//   before it is below tau (the first is always kept);
//   a coarse slot is kept if its band's score is at least alpha times the
//   row's largest band score (the first slot of a row without network slots
//   is always kept).
// kept_mass[i] (if not NULL) receives the softmax mass of the kept network
// slots, each probability exp(z_b - max z) / sum_j exp(z_j - max z) in FP32.
__global__ __launch_bounds__(256) void trim_bands_kernel(
    const int32_t* __restrict__ idx, int64_t n, int32_t top, int32_t n_net,
    const float* __restrict__ logits, const float* __restrict__ score, int32_t c, float tau,
    float alpha, int32_t* __restrict__ out, float* __restrict__ kept_mass) {
    const int64_t row = linear_block() * 4 + (threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    if (row >= n) return;
    // softmax normaliser of the logits and the largest band score (c <= 128)
    float mx = -INFINITY, se = 0.f, smax = -INFINITY;
    if (logits) {
        const float* z = logits + row * c;
        const float v0 = lane < c ? z[lane] : -INFINITY;
        const float v1 = lane + 64 < c ? z[lane + 64] : -INFINITY;
        mx = fmaxf(v0, v1);
        for (int off = 32; off >= 1; off >>= 1) mx = fmaxf(mx, __shfl_xor(mx, off, 64));
        se = (lane < c ? expf(v0 - mx) : 0.f) + (lane + 64 < c ? expf(v1 - mx) : 0.f);
        for (int off = 32; off >= 1; off >>= 1) se += __shfl_xor(se, off, 64);
    }
    if (score) {
        const float* q = score + row * c;
        smax = fmaxf(lane < c ? q[lane] : -INFINITY, lane + 64 < c ? q[lane + 64] : -INFINITY);
        for (int off = 32; off >= 1; off >>= 1) smax = fmaxf(smax, __shfl_xor(smax, off, 64));
    }
    if (lane != 0) return;
    const int32_t* in = idx + row * top;
    int32_t* o = out + row * top;
    float cum = 0.f;
    bool any_net = false;
    for (int32_t r = 0; r < top; ++r) {
        const int32_t b = in[r];
        bool keep = false;
        if (b >= 0 && b < c) {
            if (r < n_net) {
                keep = !any_net || cum < tau;
                if (keep) {
                    any_net = true;
                    if (logits) cum += expf(logits[row * c + b] - mx) / se;
                }
            } else {
                keep = (n_net == 0 && r == 0) || !score || score[row * c + b] >= alpha * smax;
            }
        }
        o[r] = keep ? b : -1;
    }
    if (kept_mass) kept_mass[row] = cum;
}

}  // namespace
}  // namespace lsp

static lsp::GemmArgs gemm_args(int64_t M, int64_t N, int64_t K, const void* A, int64_t sam,
                               int64_t sak, const void* B, int64_t sbk, int64_t sbn,
                               const float* bias, const void* mask, int32_t relu, float* C,
                               void* C_bf16, int64_t ldc) {
    lsp::GemmArgs g = {};
    g.M = M;
    g.N = N;
    g.K = K;
    g.A = static_cast<const uint16_t*>(A);
    g.sam = sam;
    g.sak = sak;
    g.B = static_cast<const uint16_t*>(B);
    g.sbk = sbk;
    g.sbn = sbn;
    g.bias = bias;
    g.mask = static_cast<const uint16_t*>(mask);
    g.relu = relu;
    g.Cf = C;
    g.Cb = static_cast<uint16_t*>(C_bf16);
    g.ldc = ldc;
    // 16-byte loads where an operand's k (or its rows) are contiguous and
    // every 8-element chunk the tiles read starts on a 16-byte boundary
    auto mode = [](const void* X, int64_t so, int64_t sk) {
        const bool aligned = (reinterpret_cast<uintptr_t>(X) & 15u) == 0;
        auto fits = [](int64_t st) { return st >= 0 && st % 8 == 0 && st < lsp::kMaxStride; };
        if (aligned && sk == 1 && fits(so)) return (int32_t)lsp::kLoadK;
        if (aligned && so == 1 && fits(sk)) return (int32_t)lsp::kLoadRows;
        return (int32_t)lsp::kLoadScalar;
    };
    g.a_mode = mode(A, sam, sak);
    g.b_mode = mode(B, sbn, sbk);
    g.c_vec = ldc % 4 == 0 && (reinterpret_cast<uintptr_t>(C) & 15u) == 0 &&
              (reinterpret_cast<uintptr_t>(C_bf16) & 7u) == 0 &&
              (reinterpret_cast<uintptr_t>(mask) & 7u) == 0;
    return g;
}

// Launches the first n products of G (with G.s where G.s.c > 0) with one tile
// size: 128 x 128 where it gives two workgroups per CU, 64 x 64 where it gives
// one for every other CU, else 32 x 32; neither larger one where half of it would
// lie outside a product.  Measured (us):
//   rows x K x columns     128 tiles    64 tiles    32 tiles
//   20,000 x 1,088 x 512   628:  44   2,504:  52        113
//   20,000 x 512 x 256     314:  18.6 1,252:  18         34
//   20,000 x 256 x 64      157:  11     313:   7.2        9
//   1,088 x 512 x 512                   136:   6.9  544:  8.3
//   512 x 512 x 256 + 512 x 256 x 512    96:   7.1  384:  6.2
//   512 x 1,088 x 512                    64:  10.2  256:  9.2
//   100,000 x 64 x 64      782:  23.6 1,563:  12.0
//   64 x 64 x 200,000    1,563:  39.3 3,125:  19.1
//   100,000 x 64 x 32      782:  15.7 1,563:  13.8  3,125:  10.2
static lsp_status launch_group(lsp::GemmGroup& G, int n, void* stream) {
    for (int q = 0; q < n; ++q)
        if ((G.g[q].M + 63) / 64 > 65535 || (G.g[q].N + 63) / 64 > 65535) return LSP_EUNSUPPORTED;
    auto count = [&](int64_t t) {
        int64_t all = 0;
        for (int q = 0; q < n; ++q) {
            G.tiles[q] = (G.g[q].M + t - 1) / t * ((G.g[q].N + t - 1) / t);
            all += G.tiles[q];
        }
        return all;
    };
    const hipStream_t s = static_cast<hipStream_t>(stream);
    const int64_t cols = G.s.wide ? lsp::kSumWide : lsp::kSumCols;
    const int64_t sums = G.s.c > 0 ? (G.s.c + cols - 1) / cols : 0;
    // other load modes (unaligned or strided operands) take the 64 x 64 tile
    bool general = false;
    for (int q = 0; q < n; ++q) {
        const int32_t am = G.g[q].a_mode, bm = G.g[q].b_mode;
        general |= am == lsp::kLoadScalar || bm == lsp::kLoadScalar ||
                   (am == lsp::kLoadRows && bm == lsp::kLoadK);
    }
    if (general && n > 1) {
        // products of different modes: one launch each, the sums with the last
        for (int q = 0; q < n; ++q) {
            lsp::GemmGroup one = {};
            one.g[0] = G.g[q];
            if (q + 1 == n) one.s = G.s;
            const lsp_status st = launch_group(one, 1, stream);
            if (st != LSP_OK) return st;
        }
        return LSP_OK;
    }
    bool narrow = false, slim = false;
    for (int q = 0; q < n; ++q) {
        narrow |= G.g[q].M <= 64 || G.g[q].N <= 64;
        slim |= G.g[q].M <= 32 || G.g[q].N <= 32;
    }
    const int t = general                          ? 64
                  : !narrow && count(128) >= 512   ? 128
                  : !slim && count(64) >= 128      ? 64
                                                   : 32;
    G.blocks = count(t) + sums;
    const dim3 grid = lsp::grid_for(G.blocks), threads(256);
    if (general)
        hipLaunchKernelGGL((lsp::gemm_group_kernel<64, 64, 64, 2, 2, 1, true>), grid, threads, 0, s, G);
    else if (t == 128)
        hipLaunchKernelGGL((lsp::gemm_group_kernel<128, 128, 64, 2, 2, 1, false>), grid, threads, 0, s,
                           G);
    else if (t == 64)
        hipLaunchKernelGGL((lsp::gemm_group_kernel<64, 64, 64, 2, 2, 3, false>), grid, threads, 0, s,
                           G);
    else
        hipLaunchKernelGGL((lsp::gemm_group_kernel<32, 32, 64, 2, 2, 4, false>), grid, threads, 0, s,
                           G);
    return hipGetLastError() == hipSuccess ? LSP_OK : LSP_EHIP;
}

// Up to six parameter arrays in one launch; arrays of no elements take none.
static lsp_status launch_adam(lsp::AdamArgs& A, int32_t step, float beta1, float beta2,
                              void* stream) {
    A.c1 = 1.f - powf(beta1, (float)step);
    A.c2 = 1.f - powf(beta2, (float)step);
    A.b1 = beta1;
    A.b2 = beta2;
    A.blocks = 0;
    for (int q = 0; q < A.n; ++q) {
        A.a[q].first = A.blocks;
        A.blocks += (A.a[q].count + lsp::kAdamThreads - 1) / lsp::kAdamThreads;
    }
    hipLaunchKernelGGL(lsp::adam_kernel, lsp::grid_for(A.blocks), dim3(lsp::kAdamThreads), 0,
                       static_cast<hipStream_t>(stream), A);
    return hipGetLastError() == hipSuccess ? LSP_OK : LSP_EHIP;
}

extern "C" {

lsp_status lsp_gemm_bf16(int64_t M, int64_t N, int64_t K, const void* A, int64_t sam, int64_t sak,
                         const void* B, int64_t sbk, int64_t sbn, const float* bias,
                         const void* mask, int32_t relu, float* C, void* C_bf16, int64_t ldc,
                         void* stream) {
    if (M < 0 || N < 0 || K < 0 || (M > 0 && N > 0 && (!A || !B)) || (!C && !C_bf16) ||
        ldc < N || (relu != 0 && relu != 1))
        return LSP_EINVAL;
    if ((M + 63) / 64 > 65535 || (N + 63) / 64 > 65535) return LSP_EUNSUPPORTED;
    if (M == 0 || N == 0) return LSP_OK;
    lsp::GemmGroup G = {};
    G.g[0] = gemm_args(M, N, K, A, sam, sak, B, sbk, sbn, bias, mask, relu, C, C_bf16, ldc);
    return launch_group(G, 1, stream);
}

lsp_status lsp_softmax_xent(const float* logits, const int32_t* labels, int64_t n, int32_t c,
                            float scale, float* dlogits, void* dlogits_bf16, float* loss_rows,
                            void* stream) {
    if (n < 0 || c < 1 || (n > 0 && (!logits || !labels))) return LSP_EINVAL;
    if (n == 0) return LSP_OK;
    hipLaunchKernelGGL(lsp::softmax_xent_kernel, lsp::grid_for((n + 3) / 4), dim3(256), 0,
                       static_cast<hipStream_t>(stream), logits, labels, n, c, scale, dlogits,
                       static_cast<uint16_t*>(dlogits_bf16), loss_rows);
    return hipGetLastError() == hipSuccess ? LSP_OK : LSP_EHIP;
}

lsp_status lsp_col_sums(const float* x, int64_t n, int32_t c, float* out, void* stream) {
    if (n < 0 || c < 1 || !out || (n > 0 && !x)) return LSP_EINVAL;
    lsp::GemmGroup G = {};
    G.s = lsp::ColSums{x, n, c, lsp::sum_wide(c), out};
    return launch_group(G, 0, stream);
}

lsp_status lsp_col_stats(const float* x, int64_t n, int32_t d, float* mean, float* inv_std,
                         void* stream) {
    if (n < 0 || d < 1 || !mean || !inv_std || (n > 0 && !x)) return LSP_EINVAL;
    hipLaunchKernelGGL(lsp::col_stats_kernel, dim3((d + 255) / 256), dim3(256), 0,
                       static_cast<hipStream_t>(stream), x, n, d, mean, inv_std);
    return hipGetLastError() == hipSuccess ? LSP_OK : LSP_EHIP;
}

lsp_status lsp_standardize_bf16(const float* x, int64_t n, int32_t d, const float* mean,
                                const float* inv_std, void* out, void* stream) {
    if (n < 0 || d < 1 || !mean || !inv_std || (n > 0 && (!x || !out))) return LSP_EINVAL;
    if (n == 0) return LSP_OK;
    hipLaunchKernelGGL(lsp::standardize_kernel, lsp::grid_for((n * d + 255) / 256), dim3(256), 0,
                       static_cast<hipStream_t>(stream), x, n, d, mean, inv_std,
                       static_cast<uint16_t*>(out));
    return hipGetLastError() == hipSuccess ? LSP_OK : LSP_EHIP;
}

lsp_status lsp_cast_bf16(const float* x, int64_t count, void* out, void* stream) {
    if (count < 0 || (count > 0 && (!x || !out))) return LSP_EINVAL;
    if (count == 0) return LSP_OK;
    hipLaunchKernelGGL(lsp::cast_bf16_kernel, lsp::grid_for((count + 255) / 256), dim3(256), 0,
                       static_cast<hipStream_t>(stream), x, count, static_cast<uint16_t*>(out));
    return hipGetLastError() == hipSuccess ? LSP_OK : LSP_EHIP;
}

lsp_status lsp_adam(float* param, const float* grad, float* m, float* v, int64_t count,
                    int32_t step, float lr, float beta1, float beta2, float eps, void* param_bf16,
                    void* stream) {
    if (count < 0 || step < 1 || (count > 0 && (!param || !grad || !m || !v))) return LSP_EINVAL;
    if (count == 0) return LSP_OK;
    lsp::AdamArgs A = {};
    A.n = 1;
    A.lr = lr;
    A.eps = eps;
    A.a[0] = lsp::AdamArray{param, grad, m, v, static_cast<uint16_t*>(param_bf16), count, 0};
    return launch_adam(A, step, beta1, beta2, stream);
}

// ---- the network as a whole: the layer order of lsp_mlp, from the primitives

static bool mlp_ok(const lsp_mlp* net) {
    if (!net) return false;
    for (int l = 0; l < 4; ++l)
        if (net->dims[l] < 1) return false;
    for (int l = 0; l < 3; ++l)
        if (!net->w[l] || !net->b[l] || !net->w_bf16[l]) return false;
    return true;
}

static bool grads_ok(const lsp_mlp_grads* g) {
    if (!g) return false;
    for (int l = 0; l < 3; ++l)
        if (!g->w[l] || !g->b[l]) return false;
    return true;
}

// Backward scratch: dlogits, dz2, dz1 in FP32 and in BF16, 256-byte aligned.
struct MlpScratch {
    size_t off[6];
    size_t total;
};

static MlpScratch mlp_scratch(const lsp_mlp* net, int64_t n) {
    const int64_t rows[3] = {net->dims[3], net->dims[2], net->dims[1]};
    MlpScratch s{};
    size_t at = 0;
    for (int q = 0; q < 3; ++q) {
        s.off[2 * q] = at;
        at += ((size_t)n * rows[q] * 4 + 255) / 256 * 256;
        s.off[2 * q + 1] = at;
        at += ((size_t)n * rows[q] * 2 + 255) / 256 * 256;
    }
    s.total = at;
    return s;
}

lsp_status lsp_mlp_forward(const lsp_mlp* net, const void* x_bf16, int64_t n, void* h1_bf16,
                           void* h2_bf16, float* logits, void* stream) {
    if (!mlp_ok(net) || n < 0 || (n > 0 && (!x_bf16 || !h1_bf16 || !h2_bf16 || !logits)))
        return LSP_EINVAL;
    if (n == 0) return LSP_OK;
    const int64_t d0 = net->dims[0], d1 = net->dims[1], d2 = net->dims[2], d3 = net->dims[3];
    lsp_status st = lsp_gemm_bf16(n, d1, d0, x_bf16, d0, 1, net->w_bf16[0], d1, 1, net->b[0],
                                  nullptr, 1, nullptr, h1_bf16, d1, stream);
    if (st != LSP_OK) return st;
    st = lsp_gemm_bf16(n, d2, d1, h1_bf16, d1, 1, net->w_bf16[1], d2, 1, net->b[1], nullptr, 1,
                       nullptr, h2_bf16, d2, stream);
    if (st != LSP_OK) return st;
    return lsp_gemm_bf16(n, d3, d2, h2_bf16, d2, 1, net->w_bf16[2], d3, 1, net->b[2], nullptr, 0,
                         logits, nullptr, d3, stream);
}

size_t lsp_mlp_workspace_bytes(const lsp_mlp* net, int64_t n) {
    if (!net || n < 1) return 0;
    for (int l = 0; l < 4; ++l)
        if (net->dims[l] < 1) return 0;
    return mlp_scratch(net, n).total;
}

lsp_status lsp_mlp_backward(const lsp_mlp* net, const void* x_bf16, const int32_t* labels,
                            int64_t n, const void* h1_bf16, const void* h2_bf16,
                            const float* logits, float scale, const lsp_mlp_grads* grads,
                            float* loss_rows, void* workspace, size_t workspace_bytes,
                            void* stream) {
    if (!mlp_ok(net) || !grads_ok(grads) || n < 1 || !x_bf16 || !labels || !h1_bf16 ||
        !h2_bf16 || !logits || !workspace)
        return LSP_EINVAL;
    const MlpScratch sc = mlp_scratch(net, n);
    if (workspace_bytes < sc.total) return LSP_ENOMEM;
    const int64_t d3 = net->dims[3];
    char* ws = static_cast<char*>(workspace);
    float* g3 = reinterpret_cast<float*>(ws + sc.off[0]);
    void* g3b = ws + sc.off[1];
    float* dz2 = reinterpret_cast<float*>(ws + sc.off[2]);
    void* dz2b = ws + sc.off[3];
    float* dz1 = reinterpret_cast<float*>(ws + sc.off[4]);
    void* dz1b = ws + sc.off[5];
    lsp_status st = lsp_softmax_xent(logits, labels, n, (int32_t)d3, scale, g3, g3b, loss_rows,
                                     stream);
    if (st != LSP_OK) return st;
    // Each layer's weight gradient, bias gradient and input gradient in one
    // launch (per call as lsp_gemm_bf16 and lsp_col_sums would compute them).
    // layer 3: dW_2 = h2^T g3, db_2 = column sums of g3, dz2 = (g3 W_2^T) where h2 > 0
    auto layer = [&](int l, const void* in, const float* g, const void* gb, float* dz, void* dzb) {
        const int64_t di = net->dims[l], dn = net->dims[l + 1];
        lsp::GemmGroup G = {};
        G.g[0] = gemm_args(di, dn, n, in, 1, di, gb, dn, 1, nullptr, nullptr, 0, grads->w[l],
                           nullptr, dn);
        if (dz)
            G.g[1] = gemm_args(n, di, dn, gb, dn, 1, net->w_bf16[l], 1, dn, nullptr, in, 0, dz,
                               dzb, di);
        G.s = lsp::ColSums{g, n, (int32_t)dn, lsp::sum_wide(dn), grads->b[l]};
        return launch_group(G, dz ? 2 : 1, stream);
    };
    if ((st = layer(2, h2_bf16, g3, g3b, dz2, dz2b)) != LSP_OK) return st;
    if ((st = layer(1, h1_bf16, dz2, dz2b, dz1, dz1b)) != LSP_OK) return st;
    return layer(0, x_bf16, dz1, dz1b, nullptr, nullptr);
}

lsp_status lsp_mlp_adam(const lsp_mlp* net, const lsp_mlp_grads* grads, const lsp_mlp_grads* m,
                        const lsp_mlp_grads* v, int32_t step, float lr, float beta1, float beta2,
                        float eps, void* stream) {
    if (!mlp_ok(net) || !grads_ok(grads) || !grads_ok(m) || !grads_ok(v) || step < 1)
        return LSP_EINVAL;
    lsp::AdamArgs A = {};
    A.n = 6;
    A.lr = lr;
    A.eps = eps;
    for (int l = 0; l < 3; ++l) {
        const int64_t nw = (int64_t)net->dims[l] * net->dims[l + 1];
        A.a[2 * l] = lsp::AdamArray{net->w[l], grads->w[l], m->w[l], v->w[l],
                                    static_cast<uint16_t*>(net->w_bf16[l]), nw, 0};
        A.a[2 * l + 1] = lsp::AdamArray{net->b[l], grads->b[l], m->b[l], v->b[l], nullptr,
                                        net->dims[l + 1], 0};
    }
    return launch_adam(A, step, beta1, beta2, stream);
}

lsp_status lsp_top_k(const float* logits, int64_t n, int32_t c, int32_t k, int32_t* idx,
                     float* mass, void* stream) {
    if (n < 0 || c < 1 || c > 128 || k < 1 || k > c || (n > 0 && (!logits || !idx)))
        return LSP_EINVAL;
    if (n == 0) return LSP_OK;
    hipLaunchKernelGGL(lsp::top_k_kernel, lsp::grid_for((n + 3) / 4), dim3(256), 0,
                       static_cast<hipStream_t>(stream), logits, n, c, k, idx, mass);
    return hipGetLastError() == hipSuccess ? LSP_OK : LSP_EHIP;
}

lsp_status lsp_row_normalize(float* x, int64_t n, int32_t d, int32_t start, int32_t count,
                             void* stream) {
    if (n < 0 || d < 1 || start < 0 || count < 1 || (int64_t)start + count > d) return LSP_EINVAL;
    if (n > 0 && !x) return LSP_EINVAL;
    if (n == 0) return LSP_OK;
    hipLaunchKernelGGL(lsp::row_norm_kernel, lsp::grid_for((n + 3) / 4), dim3(256), 0,
                       static_cast<hipStream_t>(stream), x, n, d, start, count);
    return hipGetLastError() == hipSuccess ? LSP_OK : LSP_EHIP;
}

lsp_status lsp_band_max(const float* x, int64_t n, int32_t d, int32_t start, int32_t n_bands,
                        int32_t group, float* out, void* stream) {
    if (n < 0 || d < 1 || start < 0 || n_bands < 1 || group < 1 ||
        (int64_t)start + (int64_t)n_bands * group > d)
        return LSP_EINVAL;
    if (n > 0 && (!x || !out)) return LSP_EINVAL;
    if (n == 0) return LSP_OK;
    hipLaunchKernelGGL(lsp::band_max_kernel, lsp::grid_for((n * n_bands + 255) / 256), dim3(256),
                       0, static_cast<hipStream_t>(stream), x, n, d, start, n_bands, group, out);
    return hipGetLastError() == hipSuccess ? LSP_OK : LSP_EHIP;
}

lsp_status lsp_merge_bands(const int32_t* a, int32_t ka, const int32_t* b, int32_t kb, int64_t n,
                           int32_t k_out, int32_t* out, void* stream) {
    if (n < 0 || ka < 0 || kb < 0 || k_out < 1 || k_out > 128) return LSP_EINVAL;
    if (n > 0 && (!out || (ka > 0 && !a) || (kb > 0 && !b))) return LSP_EINVAL;
    if (n == 0) return LSP_OK;
    hipLaunchKernelGGL(lsp::merge_bands_kernel, lsp::grid_for((n + 255) / 256), dim3(256), 0,
                       static_cast<hipStream_t>(stream), a, ka, b, kb, n, k_out, out);
    return hipGetLastError() == hipSuccess ? LSP_OK : LSP_EHIP;
}

lsp_status lsp_trim_bands(const int32_t* idx, int64_t n, int32_t top, int32_t n_net,
                          const float* logits, const float* score, int32_t c, float tau,
                          float alpha, int32_t* out, float* kept_mass, void* stream) {
    if (n < 0 || top < 1 || top > 128 || n_net < 0 || n_net > top || c < 1 || c > 128)
        return LSP_EINVAL;
    if (!(tau == tau) || !(alpha == alpha)) return LSP_EINVAL;
    if (n > 0 && (!idx || !out || (n_net > 0 && !logits))) return LSP_EINVAL;
    if (n == 0) return LSP_OK;
    hipLaunchKernelGGL(lsp::trim_bands_kernel, lsp::grid_for((n + 3) / 4), dim3(256), 0,
                       static_cast<hipStream_t>(stream), idx, n, top, n_net, logits, score, c, tau,
                       alpha, out, kept_mass);
    return hipGetLastError() == hipSuccess ? LSP_OK : LSP_EHIP;
}

lsp_status lsp_pool_stats(float* mean, float* inv_std, int32_t start, int32_t count,
                          void* stream) {
    if (!mean || !inv_std || start < 0 || count < 1) return LSP_EINVAL;
    hipLaunchKernelGGL(lsp::pool_stats_kernel, dim3(1), dim3(256), 0,
                       static_cast<hipStream_t>(stream), mean, inv_std, start, count);
    return hipGetLastError() == hipSuccess ? LSP_OK : LSP_EHIP;
}

lsp_status lsp_shift_bands(const void* x_bf16, const int32_t* labels, const int32_t* shifts,
                           int64_t n, int32_t d, int32_t n_coarse, int32_t group, int32_t n_bands,
                           float fill, void* out_bf16, int32_t* out_labels, void* stream) {
    if (n < 0 || d < 1 || n_coarse < 0 || n_coarse > d || group < 1 || n_bands < 1 ||
        (int64_t)group * n_bands != n_coarse)
        return LSP_EINVAL;
    if (n > 0 && (!x_bf16 || !labels || !shifts || !out_bf16 || !out_labels)) return LSP_EINVAL;
    if (n == 0) return LSP_OK;
    hipLaunchKernelGGL(lsp::shift_bands_kernel, lsp::grid_for((n * d + 255) / 256), dim3(256), 0,
                       static_cast<hipStream_t>(stream), static_cast<const uint16_t*>(x_bf16),
                       labels, shifts, n, d, n_coarse, group, n_bands, lsp::f32_to_bf16_bits(fill),
                       static_cast<uint16_t*>(out_bf16), out_labels);
    return hipGetLastError() == hipSuccess ? LSP_OK : LSP_EHIP;
}

lsp_status lsp_peak_bands(const lsp_peak* peaks, int64_t n, int64_t band_bins, int32_t n_bands,
                          int32_t* labels, void* stream) {
    if (n < 0 || band_bins < 1 || n_bands < 1 || (n > 0 && (!peaks || !labels))) return LSP_EINVAL;
    if (n == 0) return LSP_OK;
    hipLaunchKernelGGL(lsp::peak_bands_kernel, lsp::grid_for((n + 255) / 256), dim3(256), 0,
                       static_cast<hipStream_t>(stream), peaks, n, band_bins, n_bands, labels);
    return hipGetLastError() == hipSuccess ? LSP_OK : LSP_EHIP;
}

lsp_status lsp_select_fallback(const lsp_peak* peaks, const float* mass, int64_t n,
                               float mass_min, float power_min, int32_t* objects, int32_t* count,
                               void* stream) {
    if (n < 0 || n > INT32_MAX || !count || (n > 0 && (!peaks || !objects))) return LSP_EINVAL;
    hipLaunchKernelGGL(lsp::select_kernel, dim3(1), dim3(lsp::kSelThreads), 0,
                       static_cast<hipStream_t>(stream), peaks, mass, n, mass_min, power_min,
                       objects, count);
    return hipGetLastError() == hipSuccess ? LSP_OK : LSP_EHIP;
}

}  // extern "C"
