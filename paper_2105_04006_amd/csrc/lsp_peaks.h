// lsp_peaks.h -- the peak record of an object from its best (power, index), and
// its writing: by kernels of their own (lsp_reduce.hip), or at the end of the
// fix-up (lsp_fx.hip), whose last workgroup does it where there is little to do.
// A launch costs a short call some 4 us of its 20.
#pragma once

#include "lsp_common.h"

namespace lsp {

// The peak record of one object from its best (power, index).
__device__ __forceinline__ lsp_peak make_peak(const PeakParams& P, const ObjMeta& m, PeakRec b) {
    lsp_peak pk;
    pk.status = m.status;
    pk.reserved = 0;
    if (m.status == LSP_OBJ_OK && b.i >= 0) {
        const double f = grid_freq(P.f_min, P.df, b.i);
        pk.index = b.i;
        pk.freq = f;
        pk.period = P.unit == LSP_UNIT_ANGULAR ? kTwoPi / f : 1.0 / f;
        pk.power = b.p;
    } else {
        pk.index = -1;
        pk.freq = __builtin_nan("");
        pk.period = __builtin_nan("");
        pk.power = m.status == LSP_OBJ_OK ? __builtin_nan("") : fill_value(m.status);
    }
    return pk;
}

// Group grp's object, or -1.
// (Without row_obj, row r belongs to object r / rows_per_group, so group g is object g.)
__device__ __forceinline__ int64_t group_object(const PeakParams& P, int64_t grp) {
    const int64_t o = P.row_obj ? (int64_t)P.row_obj[grp * P.rows_per_group] : grp;
    return o >= 0 && o < P.n_obj ? o : -1;
}

// One thread: the peak of a group from its key.  The key is read past the
// caches that this kernel's own atomics bypass.
__device__ __forceinline__ void write_key_peak(const PeakParams& P, int64_t grp) {
    const int64_t o = group_object(P, grp);
    if (o < 0) return;
    const ObjMeta m = P.meta[o];
    const unsigned long long key =
        __hip_atomic_load(&P.keys[grp], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    P.peaks[o] = make_peak(P, m, m.status == LSP_OBJ_OK ? key_peak(key) : PeakRec{0.0, -1});
}

// Whether this workgroup is the last of `blocks` to come here.  All threads
// call it; P.done is zero before the kernel.  What a workgroup hands over must
// have been written, and is to be read, by agent-scope atomics, which go past
// the caches that are not shared (the group keys): they are complete when the
// wait below ends.  (An agent-scope fence writes back and drops a whole
// L2: it cost a 20-workgroup call more than the launch that it saved.)
__device__ __forceinline__ bool last_workgroup(const PeakParams& P, int64_t blocks) {
    __shared__ int s_last;
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (threadIdx.x == 0)
        s_last = blocks == 1 || (int64_t)atomicAdd(P.done, 1u) == blocks - 1;
    __syncthreads();
    return s_last;
}

}  // namespace lsp
