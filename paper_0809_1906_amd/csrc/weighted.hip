// Weighted graphs (positive integer weights): one workgroup per source,
// bucketed shortest paths with one bucket per distance value (Dial's order).
//
// For each source s (Brandes's algorithm with weights, Sec. 1.1; the weighted
// forward of Sec. 3.2.1 read as path counts summed over P_s in nondecreasing
// distance):
//   forward   phase d = 0, 1, 2, ...: the vertices whose tentative distance is
//             d are final (every weight is >= 1).  They are settled, and one
//             pass over their arcs both pulls their counts over predecessors,
//                 lambda_sw = sum of lambda_sv over v with d(s,v) + w(v,w) = d,
//             and relaxes the arcs, from a single read of each neighbour's
//             distance.  A relaxation that improves x to d + c is listed, then
//             filed in bin c of phase d's slot in a ring of 256 slots (max
//             weight <= 255), so phase d + c finds it again by looking back
//             at most 255 phases: no priority queue.  Each thread keeps eight
//             arcs' loads in flight.
//   backward  distance groups from the farthest down to 1:
//             delta(v) = lambda_sv * sum over successors w
//             (d(s,w) = d(s,v) + w(v,w)) of c(w), c(w) = (1 + delta(w)) / lambda_sw,
//             and BC(v) += delta(v) for v != s (Theorem 1.1, FP64).  The
//             forward's count pull lists every DAG arc (predecessor,
//             successor) by phase, so the backward touches only those arcs (a
//             few percent of all arcs): once a group's c(w) are final, each is
//             added into its predecessors' sums.
//
// Weights above 255 are handled by the same ring with a wider window: the
// ring has W = 256 slots when max weight <= 255 and is refused otherwise
// (BC_ERR_UNSUPPORTED at create).
#include "bc_internal.h"
#include "wg_utils.h"

#include <algorithm>

namespace {

using wg::PB;
constexpr int RING = 256;        // phases kept in the ring (max weight + 1)
constexpr int32_t INF = 0x7FFFFFFF;
constexpr int U = 8;             // arcs per thread with loads in flight together
// Distances of the vertices [0, KH) live in LDS: with degree-ordered internal
// numbering they are the highest-degree vertices, which most arcs point to
// (RMAT-20: 45% of all arcs point into the first 8192), so those random reads
// and minimum updates stay on the compute unit.  The workgroup owns its
// source's distances, so the LDS copy is the only one.  32 KB: four
// workgroups still share a compute unit.
constexpr int32_t KH = 8192;

struct WeightedWork {
    int32_t *dist;   // [groups][n]
    uint64_t *sigma; // [groups][n]
    double *acc;     // [groups][n]
    int32_t *order;  // [groups][n]   settled vertices, nondecreasing distance
    int32_t *gstart; // [groups][n+1] distance groups in order[]
    int32_t *gdist;  // [groups][n]
    int32_t *arena;  // [groups][cap] ring of relaxed vertices, binned per (phase, weight)
    int32_t *bstart; // [groups][RING][RING] unwrapped arena position of each bin
    int32_t *bcount; // [groups][RING][RING]
    int32_t *pstart; // [groups][RING] unwrapped arena position of each phase's bins
    int32_t *imp_x;  // [groups][icap] vertices improved in the current phase
    uint8_t *imp_c;  // [groups][icap] the weight of the improving arc
    int32_t *dag_p;  // [groups][dcap] DAG arcs in phase order: predecessor,
    int32_t *dag_s;  // [groups][dcap]                         successor
    int32_t *dag_a;  // [groups][dcap]                         and arc index
    int32_t *gdag;   // [groups][n+1] first DAG arc of each distance group
    int64_t cap;     // arena entries per workgroup, a power of two
    int64_t icap;    // improvement-list entries per workgroup
    int64_t dcap;    // DAG-arc entries per workgroup
    int32_t *retry;  // rows of the sources to run again: their live bins outgrew the arena, or
                     // the sweep with its distances in LDS does not hold them
    uint32_t *retry_count;
    const int32_t *comp_size; // [n] vertices in each vertex's connected component
};

__global__ __launch_bounds__(PB) void k_weighted_sweep(
    int32_t n, const int32_t *__restrict__ rp, const int32_t *__restrict__ col, const uint8_t *__restrict__ wt,
    const int32_t *__restrict__ sources, const int32_t *__restrict__ slot_of, int64_t count,
    unsigned long long *next_counter, WeightedWork W, double *bc, uint32_t *status, int accumulate,
    double *delta_dump, int32_t *dist_dump, uint64_t *sigma_dump, double *eb) {
    __shared__ wg::Chunk ch;
    __shared__ int32_t s_len[PB + 1];
    __shared__ int32_t s_st[PB];
    __shared__ int32_t s_hist[RING];
    __shared__ int32_t s_cur[RING];
    __shared__ long long s_idx;
    __shared__ int32_t s_nset, s_maxt, s_nimp, s_ndag;
    __shared__ uint32_t s_ovf, s_abort;
    __shared__ int32_t s_top;
    __shared__ int32_t s_hd[KH]; // dist[v] for v < KH
    __shared__ uint32_t s_run[PB / 64 * 2 * U]; // wg::arcs_of's bits, a wave's each

    const int tid = threadIdx.x;
    uint32_t *run = s_run + (tid >> 6) * 2 * U;
    if (tid < PB / 64 * 2 * U) s_run[tid] = 0; // read after a barrier
    const size_t g = blockIdx.x;
    int32_t *dist = W.dist + g * (size_t)n;
    uint64_t *sigma = W.sigma + g * (size_t)n;
    double *acc = W.acc + g * (size_t)n;
    int32_t *order = W.order + g * (size_t)n;
    int32_t *gstart = W.gstart + g * ((size_t)n + 1);
    int32_t *gdist = W.gdist + g * (size_t)n;
    int32_t *arena = W.arena + g * (size_t)W.cap;
    int32_t *bstart = W.bstart + g * (size_t)RING * RING;
    int32_t *bcount = W.bcount + g * (size_t)RING * RING;
    int32_t *pstart = W.pstart + g * (size_t)RING;
    int32_t *imp_x = W.imp_x + g * (size_t)W.icap;
    uint8_t *imp_c = W.imp_c + g * (size_t)W.icap;
    int32_t *dag_p = W.dag_p + g * (size_t)W.dcap;
    int32_t *dag_s = W.dag_s + g * (size_t)W.dcap;
    int32_t *dag_a = W.dag_a + g * (size_t)W.dcap;
    int32_t *gdag = W.gdag + g * ((size_t)n + 1);
    const int32_t cmask = (int32_t)(W.cap - 1);
    auto dget = [&](int32_t v) -> int32_t { return v < KH ? s_hd[v] : dist[v]; };
    auto dmin = [&](int32_t v, int32_t x) -> int32_t { return v < KH ? atomicMin(&s_hd[v], x) : atomicMin(&dist[v], x); };

    for (;;) {
        if (tid == 0) s_idx = (long long)atomicAdd(next_counter, 1ull);
        __syncthreads();
        const long long idx = s_idx;
        if (idx >= count) break;
        const int32_t s = sources[idx];
        const size_t out = slot_of ? (size_t)slot_of[idx] : (size_t)idx; // row of the per-source outputs
        for (int32_t v = tid; v < n; v += PB) {
            if (v < KH) s_hd[v] = INF;
            else dist[v] = INF;
            sigma[v] = 0;
            acc[v] = 0.0;
        }
        wg::bar();
        if (tid == 0) {
            if (s < KH) s_hd[s] = 0;
            else dist[s] = 0;
            sigma[s] = 1;
            s_maxt = 0;
            s_ovf = 0;
            s_abort = 0;
            s_top = 0;
            s_ndag = 0;
        }
        wg::bar();

        // ---- forward: phases in nondecreasing distance ----
        int32_t nsettled = 0, ngroups = 0;
        for (int32_t d = 0; d <= s_maxt; ++d) {
            const int slot = d & (RING - 1);
            // (1) settle: candidates filed for distance d by phases d-255 .. d-1
            if (tid == 0) s_nset = 0;
            int32_t len = 0, st = 0;
            if (tid >= 1 && tid < RING && d - tid >= 0) {
                const int ps = (d - tid) & (RING - 1);
                len = bcount[ps * RING + tid];
                st = bstart[ps * RING + tid];
            }
            int tot;
            const int off = wg::block_excl_scan(len, ch.wsum, &tot);
            s_len[tid] = off;
            s_st[tid] = st;
            if (tid == 0) s_len[PB] = tot;
            __syncthreads();
            if (d == 0) {
                if (tid == 0) {
                    order[0] = s;
                    s_nset = 1;
                }
            } else {
                for (int i = tid; i < tot; i += PB) {
                    const int k = wg::owner(s_len, i);
                    const int32_t w = arena[(s_st[k] + (i - s_len[k])) & cmask];
                    if (dget(w) == d) order[nsettled + atomicAdd(&s_nset, 1)] = w;
                }
            }
            wg::bar();
            const int32_t cnt = s_nset;
            if (cnt == 0) {
                if (tid < RING) bcount[slot * RING + tid] = 0;
                if (tid == 0) pstart[slot] = s_top;
                wg::bar();
                continue;
            }
            const int32_t lb = nsettled, le = nsettled + cnt;
            if (tid == 0) {
                gstart[ngroups] = lb;
                gdist[ngroups] = d;
                gdag[ngroups] = s_ndag;
            }
            nsettled = le;
            ++ngroups;
            // (2) one pass over the settled vertices' arcs: pull each count
            // from its predecessors (all settled at smaller distances) and
            // relax, listing the improvements
            if (tid < RING) s_hist[tid] = 0;
            if (tid == 0) s_nimp = 0;
            __syncthreads();
            for (int32_t cb = lb; cb < le; cb += PB) {
                const int tot = wg::stage_chunk(order, cb, le, rp, ch);
                const int u = wg::arcs_each<U, PB>(tot);
                for (int e0 = wg::first_arc(u); e0 < tot; e0 += PB * u) {
                    int k[U];
                    int32_t a[U], x[U], c[U], dx[U];
                    wg::arcs_of<U, PB>(ch, run, e0, u, tot, min(PB, le - cb), k, a);
#pragma unroll
                    for (int j = 0; j < U; ++j) {
                        x[j] = a[j] >= 0 ? col[a[j]] : 0;
                        c[j] = a[j] >= 0 ? (int32_t)wt[a[j]] : 0;
                    }
#pragma unroll
                    for (int j = 0; j < U; ++j) dx[j] = a[j] >= 0 ? dget(x[j]) : INF;
#pragma unroll
                    for (int j = 0; j < U; ++j) {
                        if (a[j] < 0) continue;
                        if (d > 0 && dx[j] != INF && dx[j] + c[j] == d) { // x in P_s(w)
                            const int32_t w = ch.v[k[j]];
                            const uint64_t sx = sigma[x[j]];
                            const uint64_t old = atomicAdd((unsigned long long *)&sigma[w], (unsigned long long)sx);
                            if (old + sx < old) s_ovf = 1;
                            const int32_t pos = atomicAdd(&s_ndag, 1);
                            if (pos < W.dcap) {
                                dag_p[pos] = x[j];
                                dag_s[pos] = w;
                                dag_a[pos] = a[j];
                            } else {
                                s_abort = 1;
                            }
                        }
                        const int32_t nd = d + c[j];
                        if (nd < dx[j]) {
                            const int32_t old = dmin(x[j], nd);
                            if (nd < old) {
                                const int32_t pos = atomicAdd(&s_nimp, 1);
                                if (pos < W.icap) {
                                    imp_x[pos] = x[j];
                                    imp_c[pos] = (uint8_t)c[j];
                                    atomicAdd(&s_hist[c[j]], 1);
                                    atomicMax(&s_maxt, nd);
                                } else {
                                    s_abort = 1;
                                }
                            }
                        }
                    }
                }
                __syncthreads(); // the chunk's LDS is restaged
            }
            wg::bar();
            if (s_abort) break;
            // Every vertex of the source's component is settled: the bins hold
            // only stale candidates, so no later phase settles anything (each
            // phase writes its ring slot before any phase reads it, so the
            // next source does not see what is left).
            if (nsettled == W.comp_size[s]) break;
            // (3) allocate this phase's bins in the arena ring; the live window
            // (phases d-255 .. d) must fit, else the source is retried later
            {
                const int32_t h = tid < RING ? s_hist[tid] : 0;
                int total;
                const int pre = wg::block_excl_scan(h, ch.wsum, &total);
                const int32_t oldest = d >= RING - 1 ? pstart[(d - (RING - 1)) & (RING - 1)] : 0;
                if ((int64_t)s_top + total - oldest > W.cap) {
                    if (tid == 0) s_abort = 1;
                } else if (tid < RING) {
                    bstart[slot * RING + tid] = s_top + pre;
                    s_cur[tid] = 0;
                }
                __syncthreads();
                if (tid == 0 && !s_abort) {
                    pstart[slot] = s_top;
                    s_top += total;
                }
            }
            wg::bar();
            if (s_abort) break;
            // (4) file the listed improvements in their bins
            const int32_t nimp = s_nimp;
            for (int32_t i = tid; i < nimp; i += PB) {
                const int32_t x = imp_x[i], c = imp_c[i];
                const int kk = atomicAdd(&s_cur[c], 1);
                arena[(bstart[slot * RING + c] + kk) & cmask] = x;
            }
            __syncthreads();
            if (tid < RING) bcount[slot * RING + tid] = s_cur[tid];
            wg::bar();
        }
        if (s_abort) {
            if (tid == 0) W.retry[atomicAdd(W.retry_count, 1u)] = (int32_t)out;
            wg::bar();
            continue;
        }
        if (tid == 0) {
            gstart[ngroups] = nsettled;
            gdag[ngroups] = s_ndag;
        }
        wg::bar();

        // ---- backward: distance groups from the farthest down ----
        const int32_t lowest = accumulate ? 1 : 0;
        for (int32_t gi = ngroups - 1; gi >= lowest; --gi) {
            const int32_t lb = gstart[gi], le = gstart[gi + 1];
            // acc[v] holds the sum of c over v's successors, pushed by the
            // deeper groups
            for (int32_t i = lb + tid; i < le; i += PB) {
                const int32_t v = order[i];
                const double sv = (double)sigma[v];
                const double dl = sv * acc[v];
                if (accumulate && v != s) unsafeAtomicAdd(&bc[v], dl);
                if (delta_dump) delta_dump[out * n + v] = dl;
                acc[v] = (1.0 + dl) / sv;
            }
            wg::bar();
            // c(w) of this group into each predecessor's sum
            const int32_t db = gdag[gi], de = gdag[gi + 1];
            for (int32_t i0 = db + tid; i0 < de; i0 += PB * U) {
                int32_t p[U];
                double cw[U];
#pragma unroll
                for (int j = 0; j < U; ++j) {
                    const int32_t i = i0 + j * PB;
                    p[j] = i < de ? dag_p[i] : -1;
                    cw[j] = i < de ? acc[dag_s[i]] : 0.0;
                }
#pragma unroll
                for (int j = 0; j < U; ++j)
                    if (p[j] >= 0) {
                        unsafeAtomicAdd(&acc[p[j]], cw[j]);
                        // edge term of the DAG arc p -> w: lambda(p) c(w)
                        if (eb) unsafeAtomicAdd(&eb[dag_a[i0 + j * PB]], (double)sigma[p[j]] * cw[j]);
                    }
            }
            wg::bar();
        }
        if (dist_dump) {
            for (int32_t v = tid; v < n; v += PB) {
                const int32_t dv = dget(v);
                dist_dump[out * n + v] = dv == INF ? -1 : dv;
                sigma_dump[out * n + v] = dv == INF ? 0 : sigma[v];
                if (dv == INF) delta_dump[out * n + v] = 0.0;
            }
        }
        if (tid == 0 && s_ovf) atomicOr(status, (uint32_t)BC_DEV_SIGMA_OVERFLOW);
        wg::bar();
    }
}

// The same order with every distance in LDS, 16 bits each.  Measured against
// the sweep above, ms for 1 / 1024 sources: RMAT-16 with weights up to 255 4.6 /
// 19.4 against 12.9 / 25.7, up to 10 2.5 / 13.3 against 10.8 / 23.5; RMAT-13 1.7 /
// 4.2 against 3.2 / 5.7; G(60000, 10/59999) 5.2 / 23.1 against 11.0 / 28.9.
// What bounds the sweep is each phase's chain of dependent accesses and its
// barriers (counters, RMAT-16, weights up to 255, 1024 sources: waves wait 74%
// of their time, vector instructions issue in 32% of it), so:
//   - a phase finds its vertices, and the least distance above its own, by a
//     scan of the distances (two per instruction): no bins to read, search and
//     file in memory, and no phase without a vertex.  The thread that finds a
//     vertex loads its row and takes its place among the phase's arcs by one
//     LDS atomic on (vertices, arcs); then one pass over the arcs.
//   - an add into a count whose result nobody needs does not wait for it:
//     counts up to `safe`, 2^63 over the largest degree, cannot sum past 2^63,
//     and a larger one that brings a sum there hands the source back;
//   - the backward takes c(w) = 1 / lambda_sw + the sum over w's successors
//     straight from the two, one barrier per phase with the next phase's arcs
//     loaded before it; BC is added for all vertices at the end.
// A source is handed to the sweep above when a distance reaches 65535, its
// DAG arcs outgrow W.dcap, or a count comes near 2^64.
__device__ __forceinline__ uint32_t pk_sub16(uint32_t a, uint32_t b) {
    typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));
    return __builtin_bit_cast(uint32_t, (u16x2)(__builtin_bit_cast(u16x2, a) - __builtin_bit_cast(u16x2, b)));
}
__device__ __forceinline__ uint32_t pk_min16(uint32_t a, uint32_t b) {
    typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));
    return __builtin_bit_cast(uint32_t,
                              __builtin_elementwise_min(__builtin_bit_cast(u16x2, a), __builtin_bit_cast(u16x2, b)));
}

constexpr uint32_t FAR16 = 0xFFFF; // not reached

template <int T>
__global__ __launch_bounds__(T, 4) void k_weighted_lds(
    int32_t n, const int32_t *__restrict__ rp, const int32_t *__restrict__ col, const uint8_t *__restrict__ wt,
    const int32_t *__restrict__ sources, int64_t count, unsigned long long *next_counter, WeightedWork W, uint64_t safe,
    double *bc, int accumulate, double *delta_dump, int32_t *dist_dump, uint64_t *sigma_dump, double *eb) {
    constexpr int U = 4; // eight arcs in flight take more than a quarter of the registers
    extern __shared__ uint4 s_dist8[]; // [(n + 7) / 8] eight distances each
    __shared__ wg::ChunkOf<T> ch;
    __shared__ long long s_idx;
    // phase p uses entry p % 3 and clears the next phase's, last used two
    // phases before
    __shared__ unsigned long long s_found[3]; // vertices << 32 | arcs
    __shared__ uint32_t s_next[3];
    __shared__ int32_t s_ndag;
    __shared__ uint32_t s_abort;

    __shared__ uint32_t s_run[T / 64 * 2 * U]; // wg::arcs_of's bits, a wave's each
    const int tid = threadIdx.x;
    uint32_t *run = s_run + (tid >> 6) * 2 * U;
    if (tid < T / 64 * 2 * U) s_run[tid] = 0; // read after a barrier
    const size_t g = blockIdx.x;
    uint32_t *dist2 = reinterpret_cast<uint32_t *>(s_dist8);
    const uint16_t *dist = reinterpret_cast<const uint16_t *>(s_dist8);
    const int32_t n8 = (n + 7) / 8;
    uint64_t *sigma = W.sigma + g * (size_t)n;
    double *acc = W.acc + g * (size_t)n;
    int32_t *order = W.order + g * (size_t)n; // a phase's vertices past the first T
    int32_t *gdag = W.gdag + g * ((size_t)n + 1);
    int32_t *dag_p = W.dag_p + g * (size_t)W.dcap;
    int32_t *dag_s = W.dag_s + g * (size_t)W.dcap;
    int32_t *dag_a = W.dag_a + g * (size_t)W.dcap;

    for (;;) {
        if (tid == 0) {
            s_idx = (long long)atomicAdd(next_counter, 1ull);
            // where most sources so far were handed back, so is the rest
            const uint32_t back = __hip_atomic_load(W.retry_count, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            s_abort = s_idx >= gridDim.x && 2 * (long long)back > s_idx;
        }
        __syncthreads();
        const long long idx = s_idx;
        if (idx >= count) break;
        if (s_abort) {
            if (tid == 0) W.retry[atomicAdd(W.retry_count, 1u)] = (int32_t)idx;
            __syncthreads(); // s_idx and s_abort are read above
            continue;
        }
        const int32_t s = sources[idx];
        for (int32_t i = tid; i < n8; i += T) s_dist8[i] = make_uint4(~0u, ~0u, ~0u, ~0u);
        for (int32_t v = tid; v < n; v += T) {
            sigma[v] = 0;
            acc[v] = 0.0;
        }
        wg::bar();
        if (tid == 0) {
            dist2[s >> 1] = s & 1 ? 0x0000FFFFu : 0xFFFF0000u; // distance 0
            sigma[s] = 1;
            s_ndag = 0;
            gdag[0] = 0;
            s_found[0] = 0;
            s_next[0] = FAR16;
        }
        wg::bar();

        // ---- forward: phases at the distances that occur ----
        int32_t nsettled = 0, ngroups = 0;
        uint32_t d = 0;
        const int32_t all = W.comp_size[s];
        for (int ph = 0;; ph = ph == 2 ? 0 : ph + 1) {
            // the vertices at distance d, and the least distance above it:
            // x - (d + 1) mod 2^16 is largest for the distances up to d
            uint32_t gap = 0xFFFFFFFFu;
            const uint32_t here = d | d << 16, above = (d + 1) | (d + 1) << 16;
            for (int32_t i = tid; i < n8; i += T) {
                const uint4 x4 = s_dist8[i];
                const uint32_t x[4] = {x4.x, x4.y, x4.z, x4.w};
                uint32_t hit = 0;
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    gap = pk_min16(gap, pk_sub16(x[q], above));
                    const uint32_t z = x[q] ^ here;
                    hit |= (z - 0x00010001u) & ~z & 0x80008000u; // some half is zero
                }
                if (hit == 0) continue;
#pragma unroll
                for (int j = 0; j < 8; ++j)
                    if (((x[j >> 1] >> (16 * (j & 1))) & 0xFFFFu) == d) {
                        const int32_t v = 8 * i + j;
                        const int32_t r = rp[v], deg = rp[v + 1] - r;
                        const unsigned long long at = atomicAdd(&s_found[ph], 1ull << 32 | (unsigned long long)deg);
                        const int32_t slot = (int32_t)(at >> 32);
                        if (slot <= T) ch.off[slot] = (int32_t)(uint32_t)at;
                        if (slot < T) {
                            ch.v[slot] = v;
                            ch.rp[slot] = r - (int32_t)(uint32_t)at;
                        } else {
                            order[slot] = v;
                        }
                    }
            }
            gap = min(gap & 0xFFFFu, gap >> 16);
#pragma unroll
            for (int off = 32; off > 0; off >>= 1) gap = min(gap, (uint32_t)__shfl_xor((int)gap, off, 64));
            // with no distance above d, d + 1 + gap = FAR16
            if ((tid & 63) == 0) atomicMin(&s_next[ph], d + 1 + gap);
            __syncthreads();
            const unsigned long long found = s_found[ph];
            const int32_t cnt = (int32_t)(found >> 32);
            if (tid == 0) {
                s_found[ph == 2 ? 0 : ph + 1] = 0;
                s_next[ph == 2 ? 0 : ph + 1] = FAR16;
            }
            nsettled += cnt;
            // one pass over their arcs pulls the counts from the predecessors
            // and relaxes
            uint32_t low = FAR16;
            auto arcs = [&](int slots, int tot) {
                const int u = wg::arcs_each<U, T>(tot);
                for (int e0 = wg::first_arc(u); e0 < tot; e0 += T * u) {
                    int k[U];
                    int32_t a[U], x[U];
                    uint32_t c[U], dx[U], was[U];
                    wg::arcs_of<U, T>(ch, run, e0, u, tot, slots, k, a);
#pragma unroll
                    for (int j = 0; j < U; ++j) {
                        x[j] = a[j] >= 0 ? col[a[j]] : 0;
                        c[j] = a[j] >= 0 ? (uint32_t)wt[a[j]] : 0;
                    }
#pragma unroll
                    for (int j = 0; j < U; ++j) was[j] = dist2[x[j] >> 1];
#pragma unroll
                    for (int j = 0; j < U; ++j) dx[j] = a[j] >= 0 ? (was[j] >> (16 * (x[j] & 1))) & 0xFFFFu : 0u;
                    // the counts of the predecessors (x in P_s(w)), loaded together
                    bool in[U];
                    uint64_t sx[U];
                    bool any = false;
#pragma unroll
                    for (int j = 0; j < U; ++j) {
                        in[j] = a[j] >= 0 && d > 0 && dx[j] + c[j] == d;
                        sx[j] = in[j] ? sigma[x[j]] : 0;
                        any |= in[j];
                    }
                    // lower x's half of its word where the arc improves it: one
                    // attempt each, then those that met another change again
                    uint32_t todo = 0;
#pragma unroll
                    for (int j = 0; j < U; ++j) {
                        const uint32_t nd = d + c[j];
                        if (dx[j] == FAR16 && nd >= FAR16) s_abort = 1; // past 16 bits
                        if (nd >= dx[j]) continue;
                        const int sh = 16 * (x[j] & 1);
                        const uint32_t seen = atomicCAS(&dist2[x[j] >> 1], was[j], (was[j] & ~(0xFFFFu << sh)) | nd << sh);
                        if (seen == was[j]) low = min(low, nd);
                        else todo |= 1u << j;
                        was[j] = seen;
                    }
                    if (todo) {
#pragma unroll
                        for (int j = 0; j < U; ++j) {
                            if (!((todo >> j) & 1)) continue;
                            const uint32_t nd = d + c[j];
                            const int sh = 16 * (x[j] & 1);
                            while (nd < ((was[j] >> sh) & 0xFFFFu)) {
                                const uint32_t seen =
                                    atomicCAS(&dist2[x[j] >> 1], was[j], (was[j] & ~(0xFFFFu << sh)) | nd << sh);
                                if (seen == was[j]) {
                                    low = min(low, nd);
                                    break;
                                }
                                was[j] = seen;
                            }
                        }
                    }
                    if (any) {
                        int mine = 0;
#pragma unroll
                        for (int j = 0; j < U; ++j) mine += in[j];
                        int32_t pos = atomicAdd(&s_ndag, mine);
#pragma unroll
                        for (int j = 0; j < U; ++j) {
                            if (!in[j]) continue;
                            const int32_t w = ch.v[k[j]];
                            if (sx[j] <= safe) {
                                (void)__hip_atomic_fetch_add(&sigma[w], sx[j], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                            } else {
                                const uint64_t old = atomicAdd((unsigned long long *)&sigma[w], (unsigned long long)sx[j]);
                                if (old + sx[j] < old || old + sx[j] >= 1ull << 63) s_abort = 1;
                            }
                            if (pos < W.dcap) {
                                dag_p[pos] = x[j];
                                dag_s[pos] = w;
                                if (eb) dag_a[pos] = a[j];
                            } else {
                                s_abort = 1;
                            }
                            ++pos;
                        }
                    }
                }
            };
            arcs(min(cnt, T), cnt <= T ? (int)(uint32_t)found : ch.off[T]);
            for (int32_t cb = T; cb < cnt; cb += T) {
                __syncthreads(); // the chunk's LDS is restaged
                const int tot = wg::stage_chunk<T>(order, cb, cnt, rp, ch);
                arcs(min(cnt - cb, T), tot);
            }
            if (low < FAR16) atomicMin(&s_next[ph], low);
            __syncthreads();
            ++ngroups;
            if (tid == 0) gdag[ngroups] = s_ndag; // the next arcs are listed a barrier later
            const uint32_t nd = s_next[ph];
            if (s_abort || nsettled == all || nd >= FAR16) break; // uniform
            d = nd;
        }
        wg::bar();
        if (s_abort) {
            if (tid == 0) W.retry[atomicAdd(W.retry_count, 1u)] = (int32_t)idx;
            wg::bar();
            continue;
        }

        // ---- backward: phases from the last down; phase 0 is the source's,
        // phase 1's arcs lead to it (its sum is the readout's only) ----
        {
            int32_t de = gdag[ngroups], db = gdag[ngroups - 1];
            int32_t p = -1, w = 0;
            double inv = 0.0;
            auto fetch = [&](int32_t i) {
                p = -1;
                if (i < de) {
                    p = dag_p[i];
                    w = dag_s[i];
                    inv = 1.0 / (double)sigma[w];
                }
            };
            fetch(db + tid);
            for (int32_t gi = ngroups - 1; gi >= 1; --gi) {
                for (int32_t i = db + tid;;) {
                    if (p >= 0) {
                        const double cw = inv + acc[w];
                        unsafeAtomicAdd(&acc[p], cw);
                        // edge term of the DAG arc p -> w: lambda(p) c(w)
                        if (eb) unsafeAtomicAdd(&eb[dag_a[i]], (double)sigma[p] * cw);
                    }
                    i += T;
                    if (i >= de) break;
                    fetch(i);
                }
                de = db;
                db = gdag[gi - 1];
                fetch(db + tid);
                __syncthreads();
            }
        }
        for (int32_t v = tid; v < n; v += T) {
            const uint32_t dv = dist[v];
            const uint64_t sv = dv == FAR16 ? 0 : sigma[v];
            const double dl = sv ? (double)sv * acc[v] : 0.0;
            if (accumulate && v != s && dl != 0.0) unsafeAtomicAdd(&bc[v], dl);
            if (dist_dump) {
                const size_t at = (size_t)idx * n + v;
                dist_dump[at] = dv == FAR16 ? -1 : (int32_t)dv;
                sigma_dump[at] = sv;
                delta_dump[at] = dl;
            }
        }
        wg::bar();
    }
}

// Main workspaces list a quarter of the ring's size in improvements per phase
// and half of it in DAG arcs, and send a source that needs more to the retry
// workspace; the retry workspace (ring of nnz + 1 entries or more) holds every
// improvement of a phase and every DAG arc, so it never needs a retry itself.
int64_t imp_cap(int64_t cap, bool retry_ws) { return retry_ws ? cap : std::max<int64_t>(cap / 4, 1); }
int64_t dag_cap(int64_t cap) { return std::max<int64_t>(cap / 2, 1); }
// the arena; the improvement list (5 B per entry); the DAG list (12 B per arc)
size_t list_bytes(int64_t cap, bool retry_ws) {
    return (size_t)cap * 4 + (size_t)imp_cap(cap, retry_ws) * 5 + (size_t)dag_cap(cap) * 12;
}

bc_status alloc_work(bc_ctx *ctx, WeightedBuffers &b, int64_t cap, int groups, bool retry_ws) {
    const size_t n = (size_t)std::max(ctx->n, 1);
    const size_t G = (size_t)groups;
    b.groups = groups;
    b.cap = cap;
    b.icap = imp_cap(cap, retry_ws);
    b.dcap = dag_cap(cap);
    b.dist = (int32_t *)bc_dalloc(ctx, G * n * 4);
    b.sigma = (uint64_t *)bc_dalloc(ctx, G * n * 8);
    b.acc = (double *)bc_dalloc(ctx, G * n * 8);
    b.order = (int32_t *)bc_dalloc(ctx, G * n * 4);
    b.gstart = (int32_t *)bc_dalloc(ctx, G * (n + 1) * 4);
    b.gdist = (int32_t *)bc_dalloc(ctx, G * n * 4);
    b.bstart = (int32_t *)bc_dalloc(ctx, G * RING * RING * 4);
    b.bcount = (int32_t *)bc_dalloc(ctx, G * RING * RING * 4);
    b.pstart = (int32_t *)bc_dalloc(ctx, G * RING * 4);
    // the lists, in one piece: the sweep with its distances in LDS divides it
    // otherwise
    b.arena = (int32_t *)bc_dalloc(ctx, G * list_bytes(cap, retry_ws));
    b.dag_p = b.arena + G * (size_t)cap;
    b.dag_s = b.dag_p + G * (size_t)b.dcap;
    b.dag_a = b.dag_s + G * (size_t)b.dcap;
    b.imp_x = b.dag_a + G * (size_t)b.dcap;
    b.imp_c = reinterpret_cast<uint8_t *>(b.imp_x + G * (size_t)b.icap);
    b.gdag = (int32_t *)bc_dalloc(ctx, G * (n + 1) * 4);
    if (!b.dist || !b.sigma || !b.acc || !b.order || !b.gstart || !b.gdist || !b.arena || !b.bstart || !b.bcount ||
        !b.pstart || !b.gdag)
        return bc_fail(ctx, BC_ERR_NOMEM, "weighted form: workspace allocation failed");
    return BC_OK;
}

constexpr size_t LDS_BYTES = 160 << 10;
constexpr int64_t RETRY_CAP = 4096;
template <int T>
constexpr size_t fixed_lds() { return sizeof(wg::ChunkOf<T>) + T / 64 * 2 * 4 * sizeof(uint32_t) + 64; }
size_t dist_lds(int32_t n) { return ((size_t)n + 7) / 8 * 16; }

size_t per_group_bytes(bc_ctx *ctx, int64_t cap, bool retry_ws) {
    const size_t n = (size_t)std::max(ctx->n, 1);
    // per vertex: dist, sigma, acc, order, gstart, gdist, gdag; the lists; the bins
    return n * (4 + 8 + 8 + 4 + 4 + 4 + 4) + 8 + list_bytes(cap, retry_ws) + (2 * (size_t)RING + 1) * RING * 4;
}

int64_t pow2_at_least(int64_t x) {
    int64_t p = 1;
    while (p < x) p <<= 1;
    return p;
}

WeightedWork work_of(bc_ctx *ctx, const WeightedBuffers &b) {
    WeightedState &w = ctx->wt;
    return WeightedWork{b.dist, b.sigma, b.acc, b.order, b.gstart, b.gdist, b.arena, b.bstart, b.bcount,
                        b.pstart, b.imp_x, b.imp_c, b.dag_p, b.dag_s, b.dag_a, b.gdag, b.cap, b.icap, b.dcap, w.retry,
                        w.retry_count, ctx->comp_size};
}

} // namespace

// The sweep with its distances in LDS takes every source first, where it
// applies; what it hands back goes to the main workspace.  Workgroups get an
// arena ring of max(4n, 2^16) entries (rounded up to a power of two); a source
// whose live bins outgrow it is re-run with an arena of nnz entries, which
// always suffices (a vertex settles once, so at most one entry per arc is ever
// filed).
bc_status weighted_prepare(bc_ctx *ctx) {
    WeightedState &w = ctx->wt;
    if (ctx->max_weight > 255)
        return bc_fail(ctx, BC_ERR_UNSUPPORTED, "weighted form: weights above 255 are not supported");
    const int64_t cap = w.arena_log2 > 0 ? (int64_t(1) << w.arena_log2)
                                         : pow2_at_least(std::max<int64_t>(4 * (int64_t)std::max(ctx->n, 1), 1 << 16));
    // workspace budget: 96 GB by default, 192 GB for an explicitly requested grid
    const size_t budget = size_t(w.grid > 0 ? 192 : 96) << 30;
    int groups = w.grid > 0 ? w.grid : 1024;
    while (groups > 1 && per_group_bytes(ctx, cap, false) * (size_t)groups > budget) groups /= 2;
    bc_status st = alloc_work(ctx, w.main, cap, groups, false);
    if (st != BC_OK) return st;
    // The sweep with its distances in LDS, unless a grid or an arena of the
    // other was asked for: 512 threads where two workgroups' distances fit a
    // compute unit, else 1024, and 1024 up to a source per compute unit.  ms
    // with 512 / 1024 threads, before one owner search served a wave: RMAT-15,
    // 1024 sources 10.3 / 13.8, one 4.4 / 3.5; RMAT-13 with weights up to 10,
    // 1024 sources 1.8 / 2.1, one 0.70 / 0.51.
    if (w.grid == 0 && w.arena_log2 == 0 && ctx->n > 0) {
        int cus = 0;
        BC_HIP(ctx, hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, ctx->device));
        const size_t lds = dist_lds(ctx->n);
        const size_t per_cu = std::min<size_t>(LDS_BYTES / (fixed_lds<512>() + lds), 4);
        w.lds_threads = per_cu >= 2 ? 512 : fixed_lds<1024>() + lds <= LDS_BYTES ? 1024 : 0;
        w.lds_few = std::max(cus, 1);
        if (w.lds_threads) {
            // the kernels' limit, the same for every context
            BC_HIP(ctx, hipFuncSetAttribute((const void *)k_weighted_lds<512>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                            (int)(LDS_BYTES - fixed_lds<512>())));
            BC_HIP(ctx, hipFuncSetAttribute((const void *)k_weighted_lds<1024>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                            (int)(LDS_BYTES - fixed_lds<1024>())));
            // The two never run together and share their arrays.  All the
            // lists' bytes go to this one's DAG arcs: with no room for a
            // source's arcs it is handed back, and one with few distinct
            // weights has many (RMAT-14, weights up to 3, 1024 sources:
            // 45 ms handed back, 4.6 with room).
            w.lds = w.main;
            w.lds.groups = std::min(groups, w.lds_few * (w.lds_threads == 512 ? (int)per_cu : 1));
            const size_t bytes = (size_t)groups * list_bytes(cap, false) / (size_t)w.lds.groups;
            w.lds.dcap = std::min<int64_t>((int64_t)(bytes / (ctx->edges ? 12 : 8)), INT32_MAX);
            w.lds.dag_p = w.main.arena;
            w.lds.dag_s = w.lds.dag_p + (size_t)w.lds.groups * (size_t)w.lds.dcap;
            w.lds.dag_a = w.lds.dag_s + (size_t)w.lds.groups * (size_t)w.lds.dcap; // with edge terms only
        }
    }
    w.next = (uint32_t *)bc_dalloc(ctx, 256);
    w.retry_count = (uint32_t *)bc_dalloc(ctx, 256);
    w.retry = (int32_t *)bc_dalloc(ctx, (size_t)RETRY_CAP * 4);
    w.again = (int32_t *)bc_dalloc(ctx, (size_t)RETRY_CAP * 8);
    w.host = (uint32_t *)bc_halloc(256);
    if (!w.next || !w.retry_count || !w.retry || !w.again || !w.host)
        return bc_fail(ctx, BC_ERR_NOMEM, "weighted form: allocation failed");
    return BC_OK;
}

namespace {

struct Outputs {
    bool accumulate;
    double *delta;
    int32_t *dist;
    uint64_t *sigma;
};

// One launch over `count` sources (slot_of: their rows of the outputs); *left
// receives how many it put on the retry list.
bc_status launch(bc_ctx *ctx, const WeightedBuffers &b, const int32_t *d_sources, const int32_t *slot_of,
                 int64_t count, const Outputs &o, uint32_t *left) {
    WeightedState &w = ctx->wt;
    BC_HIP(ctx, hipMemsetAsync(w.next, 0, sizeof(unsigned long long), ctx->stream));
    BC_HIP(ctx, hipMemsetAsync(w.retry_count, 0, sizeof(uint32_t), ctx->stream));
    const int grid = (int)std::min<int64_t>(count, b.groups);
    double *eb = o.accumulate && ctx->edges ? ctx->eb : nullptr;
    LaunchTimer t(ctx, "weighted_sweep");
    if (&b == &w.lds) {
        const int T = count <= w.lds_few ? 1024 : w.lds_threads;
        const auto k = T == 512 ? k_weighted_lds<512> : k_weighted_lds<1024>;
        hipLaunchKernelGGL(k, dim3(grid), dim3(T), dist_lds(ctx->n), ctx->stream, ctx->n, ctx->row_ptr,
                           ctx->col, ctx->weight, d_sources, count, (unsigned long long *)w.next, work_of(ctx, b),
                           (uint64_t(1) << 63) / (uint64_t)std::max(ctx->max_degree, 1), ctx->bc, o.accumulate ? 1 : 0,
                           o.delta, o.dist, o.sigma, eb);
    } else {
        hipLaunchKernelGGL(k_weighted_sweep, dim3(grid), dim3(PB), 0, ctx->stream, ctx->n, ctx->row_ptr, ctx->col,
                           ctx->weight, d_sources, slot_of, count, (unsigned long long *)w.next, work_of(ctx, b),
                           ctx->bc, ctx->status, o.accumulate ? 1 : 0, o.delta, o.dist, o.sigma, eb);
    }
    t.done();
    BC_HIP(ctx, hipGetLastError());
    BC_HIP(ctx, hipMemcpyAsync(w.host, w.retry_count, sizeof(uint32_t), hipMemcpyDeviceToHost, ctx->stream));
    BC_HIP(ctx, hipStreamSynchronize(ctx->stream));
    *left = *w.host;
    return BC_OK;
}

// The `left` sources on the retry list and their rows, into w.again.
bc_status gather_left(bc_ctx *ctx, const int32_t *d_sources, int64_t count, uint32_t left) {
    WeightedState &w = ctx->wt;
    std::vector<int32_t> both(2 * (size_t)left), all((size_t)count);
    BC_HIP(ctx, hipMemcpy(both.data() + left, w.retry, left * sizeof(int32_t), hipMemcpyDeviceToHost));
    BC_HIP(ctx, hipMemcpy(all.data(), d_sources, (size_t)count * sizeof(int32_t), hipMemcpyDeviceToHost));
    for (uint32_t i = 0; i < left; ++i) both[i] = all[(size_t)both[left + i]];
    BC_HIP(ctx, hipMemcpy(w.again, both.data(), both.size() * sizeof(int32_t), hipMemcpyHostToDevice));
    return BC_OK;
}

} // namespace

bc_status weighted_run(bc_ctx *ctx, const int32_t *d_sources, int64_t count, bool accumulate,
                       double *delta_dump, int32_t *dist_dump, uint64_t *sigma_dump) {
    WeightedState &w = ctx->wt;
    // the retry list holds at most one entry per source in flight: run in chunks
    for (int64_t c0 = 0; c0 < count; c0 += RETRY_CAP) {
        const int64_t cnt = std::min<int64_t>(RETRY_CAP, count - c0);
        const int32_t *src = d_sources + c0;
        // per-source output rows are positions in the whole list
        const size_t row = (size_t)c0 * ctx->n;
        const Outputs o{accumulate, delta_dump ? delta_dump + row : nullptr, dist_dump ? dist_dump + row : nullptr,
                        sigma_dump ? sigma_dump + row : nullptr};
        // A graph most of whose sources are handed back goes to the other sweep
        // straight away, once enough of them have said so: one source, or a
        // readout of a far component, tells nothing about the others.
        const bool lds = w.lds_threads && (w.lds_tried < 256 || 2 * w.lds_back <= w.lds_tried);
        uint32_t left = 0;
        bc_status st = launch(ctx, lds ? w.lds : w.main, src, nullptr, cnt, o, &left);
        if (st != BC_OK) return st;
        if (lds) {
            w.lds_tried += cnt;
            w.lds_back += left;
        }
        if (left && lds) {
            if ((st = gather_left(ctx, src, cnt, left)) != BC_OK) return st;
            if ((st = launch(ctx, w.main, w.again, w.again + left, left, o, &left)) != BC_OK) return st;
        }
        if (left == 0) continue;
        if (!w.big.dist) {
            const int64_t cap = pow2_at_least((int64_t)std::max(ctx->nnz, 1) + 1);
            int groups = 64;
            while (groups > 1 && per_group_bytes(ctx, cap, true) * (size_t)groups > (size_t(16) << 30)) groups /= 2;
            st = alloc_work(ctx, w.big, cap, groups, true);
            if (st != BC_OK) return st;
        }
        if ((st = gather_left(ctx, src, cnt, left)) != BC_OK) return st;
        const uint32_t outgrown = left;
        if ((st = launch(ctx, w.big, w.again, w.again + left, left, o, &left)) != BC_OK) return st;
        if (left != 0) // cannot happen: the retry workspace holds any source's lists
            return bc_fail(ctx, BC_ERR_DEVICE, "weighted form: a source outgrew the retry workspace");
        ctx->wt.retried += outgrown;
    }
    return BC_OK;
}
