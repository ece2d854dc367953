// Workgroup-level helpers shared by the per-source forms (plain.hip,
// weighted.hip): barriers with device-scope ordering, prefix sums, and the
// LDS-staged, per-arc balanced expansion of a vertex list's adjacency.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace wg {

constexpr int PB = 256; // threads per workgroup, where not given as T

// Workgroup barrier between the phases of a per-source sweep.  The arrays it
// orders (distances, counts, sums, queues in global memory) belong to one
// workgroup, whose waves share a compute unit's L1: workgroup scope, which
// __syncthreads carries, orders them, atomics included.  The wait makes every
// atomic and store of the phase complete before any wave goes on.  With
// agent-scope fences around it every barrier wrote back and invalidated the
// XCD's L2: all sources of G(1024, 8/1023) took 2252 us instead of 578, and
// 1024 sources of RMAT-16 with weights 1..255 304 ms instead of 27.5.
__device__ __forceinline__ void bar() {
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
}

__device__ __forceinline__ int wave_incl_scan(int x) {
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        int y = __shfl_up(x, d, 64);
        if (lane >= d) x += y;
    }
    return x;
}

// Exclusive prefix sum over the workgroup; *total receives the sum.
template <int T = PB>
__device__ __forceinline__ int block_excl_scan(int x, int *wsum, int *total) {
    const int incl = wave_incl_scan(x);
    const int wid = threadIdx.x >> 6, lane = threadIdx.x & 63;
    if (lane == 63) wsum[wid] = incl;
    __syncthreads();
    int off = 0, tot = 0;
#pragma unroll
    for (int i = 0; i < T / 64; ++i) {
        int s = wsum[i];
        if (i < wid) off += s;
        tot += s;
    }
    __syncthreads();
    *total = tot;
    return off + incl - x;
}

// Largest k in [0, T) with off[k] <= e, given off[0] = 0 <= e < off[T].
template <int T = PB>
__device__ __forceinline__ int owner(const int *off, int e) {
    int lo = 0, hi = T;
    while (hi - lo > 1) {
        int mid = (lo + hi) >> 1;
        if (off[mid] <= e) lo = mid;
        else hi = mid;
    }
    return lo;
}

// LDS staging for one chunk of up to T vertices.
template <int T>
struct ChunkOf {
    int32_t v[T];
    int32_t rp[T];
    int32_t off[T + 1];
    int32_t wsum[T / 64];
};
using Chunk = ChunkOf<PB>;

// Stages the vertices list[cb .. min(cb + T, le)) in c (vertex, row offset,
// exclusive degree prefix; c.off[T] = total) and returns their total degree.
// Every thread of the workgroup calls; ends with __syncthreads().
template <int T>
__device__ __forceinline__ int stage_chunk(const int32_t *list, int32_t cb, int32_t le,
                                           const int32_t *__restrict__ rp, ChunkOf<T> &c) {
    const int tid = threadIdx.x;
    const int32_t i = cb + tid;
    int32_t v = -1, r = 0, d = 0;
    if (i < le) {
        v = list[i];
        r = rp[v];
        d = rp[v + 1] - r;
    }
    int tot;
    const int off = block_excl_scan<T>(d, c.wsum, &tot);
    c.v[tid] = v;
    c.rp[tid] = r;
    c.off[tid] = off;
    if (tid == 0) c.off[T] = tot;
    __syncthreads();
    return tot;
}

// Arc positions e0 + j * T (j < U) of a staged chunk of `slots` vertices with
// `tot` arcs: slot k[j] of the owning vertex (the last that starts at or before
// the arc) and arc index a[j] (-1 past the end).  The U searches go step by step
// together, so that their LDS reads overlap, and take log2(slots) steps: with
// each its own search over T slots the plain sweep took 22.4 ms on RMAT-15 with
// 2048 sources, now 19.9.  A chunk that gives a thread one arc needs one search
// (ring of 20000, 1024 sources: 2.40 ms, with all U 2.56).
template <int U, int T>
__device__ __forceinline__ void arc_burst(const ChunkOf<T> &c, int e0, int tot, int slots, int (&k)[U],
                                          int32_t (&a)[U]) {
#pragma unroll
    for (int j = 0; j < U; ++j) k[j] = 0;
    const int h0 = slots > 1 ? 1 << (31 - __builtin_clz((uint32_t)(slots - 1))) : 0;
    if (__builtin_amdgcn_readfirstlane(tot) <= T) { // a narrow level: one arc a thread
        for (int h = h0; h > 0; h >>= 1)
            if (k[0] + h < slots && c.off[k[0] + h] <= e0) k[0] += h;
    } else {
        for (int h = h0; h > 0; h >>= 1) {
            int at[U];
#pragma unroll
            for (int j = 0; j < U; ++j) at[j] = c.off[min(k[j] + h, T)];
#pragma unroll
            for (int j = 0; j < U; ++j)
                if (k[j] + h < slots && at[j] <= e0 + j * T) k[j] += h;
        }
    }
#pragma unroll
    for (int j = 0; j < U; ++j) {
        const int e = e0 + j * T;
        a[j] = -1;
        if (e < tot) a[j] = c.rp[k[j]] + (e - c.off[k[j]]);
        else k[j] = 0;
    }
}

// Arc positions e0 .. e0 + U - 1 of a staged chunk of `slots` vertices, each
// with an arc, and `tot` arcs: slot k[j] of the owning vertex (the last that
// starts at or before the arc) and arc index a[j] (-1 past the end).  One
// search for a thread's U arcs, which mostly share a row: fewer instructions
// than arc_burst, whose neighbouring threads read neighbouring columns.
template <int U, int T>
__device__ __forceinline__ void arc_run(const ChunkOf<T> &c, int e0, int tot, int slots, int (&k)[U],
                                        int32_t (&a)[U]) {
    int lo = 0;
    for (int h = slots > 1 ? 1 << (31 - __builtin_clz((uint32_t)(slots - 1))) : 0; h > 0; h >>= 1)
        if (lo + h < slots && c.off[lo + h] <= e0) lo += h;
    int32_t row = c.rp[lo] - c.off[lo]; // arc index of position 0, were it in this row
    int end = lo + 1 < slots ? c.off[lo + 1] : tot;
#pragma unroll
    for (int j = 0; j < U; ++j) {
        const int e = e0 + j;
        if (e >= end && e < tot) { // the next row
            ++lo;
            row = c.rp[lo] - c.off[lo];
            end = lo + 1 < slots ? c.off[lo + 1] : tot;
        }
        k[j] = lo;
        a[j] = e < tot ? row + e : -1;
    }
}

} // namespace wg
