// Workgroup-level helpers shared by the per-source forms (plain.hip,
// weighted.hip): barriers, prefix sums, and the
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
    int32_t rp[T];  // row offset less off[]: position e of the chunk is arc rp[k] + e
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
    c.rp[tid] = r - off;
    c.off[tid] = off;
    if (tid == 0) c.off[T] = tot;
    __syncthreads();
    return tot;
}

// A staged chunk's arcs are dealt in rounds of T u, 64 u in a row to each wave,
// with u <= U such that a chunk of less than a full round is spread over the
// waves evenly.
template <int U, int T>
__device__ __forceinline__ int arcs_each(int tot) {
    return __builtin_amdgcn_readfirstlane(min(U, max(1, (tot + T - 1) / T)));
}
// The wave's first arc (u > 1), or the thread's (u = 1).
__device__ __forceinline__ int first_arc(int u) { return u > 1 ? (int)(threadIdx.x & ~63u) * u : (int)threadIdx.x; }

// A thread's u arcs of the round at e0 (from first_arc on), of a chunk of `slots`
// vertices, each with an arc, and `tot` arcs: slot k[j] of the owning vertex
// (the last that starts at or before the arc) and arc index a[j] (-1: none).
// Neighbouring threads have neighbouring arcs.  One search serves a wave's
// round, by its 64 lanes in two reads: the rows that start in its 64 u
// positions each set a bit of `run` (2 U words of the wave, zero before and
// after), and a lane counts the bits before its own position.  With a search
// an arc, its steps were most of the sweeps' instructions and LDS reads.  Plain
// form, ms for 1 / 2048 sources, a search an arc in step with a thread's others
// / now: RMAT-15 2.0 / 19.9 and 1.3 / 17.3, RMAT-16 4.0 / 42.4 and 2.5 / 37.4;
// one arc a thread takes its own search (a ring of 20000, 1024 sources: 2.40
// and 2.13).  Weighted form, ms for 1 / 1024 sources, consecutive arcs and one
// search a thread / now: RMAT-16 5.0 / 21.1 and 4.6 / 19.4, G(60000, 10/59999)
// 5.7 / 25.5 and 5.2 / 23.1.
template <int U, int T>
__device__ __forceinline__ void arcs_of(const ChunkOf<T> &c, uint32_t *run, int e0, int u, int tot, int slots,
                                        int (&k)[U], int32_t (&a)[U]) {
    const int lane = threadIdx.x & 63;
    if (u == 1) {
        k[0] = 0;
        for (int h = slots > 1 ? 1 << (31 - __builtin_clz((uint32_t)(slots - 1))) : 0; h > 0; h >>= 1)
            if (k[0] + h < slots && c.off[k[0] + h] <= e0) k[0] += h;
        a[0] = c.rp[k[0]] + e0;
#pragma unroll
        for (int j = 1; j < U; ++j) {
            k[j] = 0;
            a[j] = -1;
        }
        return;
    }
    constexpr int G = T / 64;
    const int r0 = __builtin_amdgcn_readfirstlane(e0);
    const int g = __popcll(__ballot(lane * G < slots && c.off[lane * G] <= r0)) - 1;
    const int f = g * G + (lane & (G - 1));
    const int first = g * G + __popcll(__ballot(lane < G && f < slots && c.off[f] <= r0)) - 1;
    for (int i = first + 1;; i += 64) {
        // a row's bit is one below its start: the count is of starts up to a position
        const int p = i + lane < slots ? c.off[i + lane] - 1 - r0 : 64 * U;
        if (p < 64 * u) atomicOr(&run[p >> 5], 1u << (p & 31));
        if (~__ballot(p < 64 * u) != 0) break;
    }
    __builtin_amdgcn_wave_barrier();
    uint32_t m[2 * U];
#pragma unroll
    for (int i = 0; i < 2 * U; ++i) m[i] = run[i];
    __builtin_amdgcn_wave_barrier();
    if (lane < 2 * U) run[lane] = 0;
    uint32_t base = (uint32_t)first;
#pragma unroll
    for (int j = 0; j < U; ++j) {
        const int e = r0 + 64 * j + lane;
        k[j] = (int)__builtin_amdgcn_mbcnt_hi(m[2 * j + 1], __builtin_amdgcn_mbcnt_lo(m[2 * j], base));
        base += (uint32_t)(__popc(m[2 * j]) + __popc(m[2 * j + 1]));
        a[j] = -1;
        if (j < u && e < tot) a[j] = c.rp[k[j]] + e;
        else k[j] = 0;
    }
}

} // namespace wg
