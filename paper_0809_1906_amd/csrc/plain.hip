// Plain FP64 form: one workgroup per source, the vertices' states in LDS where
// they fit, counts and sums in HBM.  Graphs whose whole state fits the LDS go to
// small.hip instead, unless the caller asks for a grid of workgroups or for edge
// terms.
//
// For each source s (Brandes's algorithm, Sec. 1.1):
//   forward   level-synchronous breadth-first search from s (the parallel BFS
//             of Sec. 4): a vertex w first reached from level l gets
//             d(s,w) = l+1, and every arc (v,w) with d(s,v) = l, d(s,w) = l+1
//             (v in P_s(w)) adds lambda_sv into lambda_sw;
//   backward  levels from the deepest down to 1: for v at level l,
//             delta_s*(v) = lambda_sv * sum over successors w of c(w), with
//             c(w) = (1 + delta_s*(w)) / lambda_sw -- Theorem 1.1 with the
//             factor lambda_sv taken out of the sum (the per-edge term of
//             ParallelCompute, Sec. 4.2.2);
//   score     BC(v) += delta_s*(v) for v != s.
//
// Each level's frontier is expanded in chunks of 256 vertices whose degree
// prefix sums are staged in LDS, so a thread takes arcs, not vertices: hub
// vertices are spread over the whole workgroup.  Each thread keeps up to eight
// arcs' loads in flight.
#include "bc_internal.h"
#include "wg_utils.h"

namespace {

using wg::PB;
constexpr int U = 8; // arcs per thread with loads in flight together

__global__ __launch_bounds__(PB) void k_plain_sweep(
    int32_t n, const int32_t *__restrict__ rp, const int32_t *__restrict__ col,
    const int32_t *__restrict__ sources, int64_t count, unsigned long long *next_counter,
    int32_t *dist_all, uint64_t *sigma_all, double *acc_all, int32_t *queue_all, int32_t *lev_all,
    double *bc, uint32_t *status, int accumulate,
    double *delta_dump, int32_t *dist_dump, uint64_t *sigma_dump, double *eb) {
    __shared__ wg::Chunk ch;
    __shared__ int32_t s_tail;
    __shared__ long long s_idx;
    __shared__ uint32_t s_ovf;
    __shared__ uint32_t s_run[PB / 64 * 2 * U]; // wg::arcs_of's bits, a wave's each

    const int tid = threadIdx.x;
    uint32_t *run = s_run + (tid >> 6) * 2 * U;
    if (tid < PB / 64 * 2 * U) s_run[tid] = 0; // read after a barrier
    const size_t g = blockIdx.x;
    int32_t *dist = dist_all + g * (size_t)n;
    uint64_t *sigma = sigma_all + g * (size_t)n;
    double *acc = acc_all + g * (size_t)n;
    int32_t *queue = queue_all + g * (size_t)n;
    int32_t *lev = lev_all + g * ((size_t)n + 2);

    for (;;) {
        if (tid == 0) s_idx = (long long)atomicAdd(next_counter, 1ull);
        __syncthreads();
        const long long idx = s_idx;
        if (idx >= count) break;
        const int32_t s = sources[idx];

        for (int32_t v = tid; v < n; v += PB) {
            dist[v] = -1;
            sigma[v] = 0;
            acc[v] = 0.0;
        }
        wg::bar();
        if (tid == 0) {
            dist[s] = 0;
            sigma[s] = 1;
            queue[0] = s;
            lev[0] = 0;
            lev[1] = 1;
            s_tail = 1;
            s_ovf = 0;
        }
        wg::bar();

        // ---- forward: level L spans queue[qb, qe) ----
        int32_t qb = 0, qe = 1, L = 0;
        while (qb < qe) {
            for (int32_t cb = qb; cb < qe; cb += PB) {
                const int tot = wg::stage_chunk(queue, cb, qe, rp, ch);
                const int u = wg::arcs_each<U, PB>(tot);
                for (int e0 = wg::first_arc(u); e0 < tot; e0 += PB * u) {
                    int k[U];
                    int32_t a[U], w[U], dw[U];
                    wg::arcs_of<U, PB>(ch, run, e0, u, tot, min(PB, qe - cb), k, a);
#pragma unroll
                    for (int j = 0; j < U; ++j) w[j] = a[j] >= 0 ? col[a[j]] : 0;
#pragma unroll
                    for (int j = 0; j < U; ++j) dw[j] = a[j] >= 0 ? dist[w[j]] : 0;
#pragma unroll
                    for (int j = 0; j < U; ++j) {
                        if (a[j] < 0) continue;
                        int32_t d = dw[j];
                        if (d < 0) {
                            const int32_t old = atomicCAS(&dist[w[j]], -1, L + 1);
                            if (old == -1) {
                                queue[atomicAdd(&s_tail, 1)] = w[j];
                                d = L + 1;
                            } else {
                                d = old;
                            }
                        }
                        if (d == L + 1) { // v in P_s(w)
                            const uint64_t x = sigma[ch.v[k[j]]];
                            const uint64_t old = atomicAdd((unsigned long long *)&sigma[w[j]], (unsigned long long)x);
                            if (old + x < old) s_ovf = 1;
                        }
                    }
                }
                __syncthreads(); // the chunk's LDS is restaged
            }
            wg::bar();
            qb = qe;
            qe = s_tail;
            ++L;
            if (tid == 0) lev[L + 1] = qe;
            wg::bar();
        }
        const int32_t nlev = L; // non-empty levels 0..nlev-1

        // ---- backward: deepest level first ----
        // (level 0 adds nothing to BC, but its arcs carry edge terms)
        const int32_t lowest = accumulate && !eb ? 1 : 0;
        for (int32_t l = nlev - 1; l >= lowest; --l) {
            const int32_t lb = lev[l], le = lev[l + 1];
            if (l < nlev - 1) {
                // acc[v] = sum of c(w) = acc[w] over successors w (level l + 1)
                for (int32_t cb = lb; cb < le; cb += PB) {
                    const int tot = wg::stage_chunk(queue, cb, le, rp, ch);
                    const int u = wg::arcs_each<U, PB>(tot);
                    for (int e0 = wg::first_arc(u); e0 < tot; e0 += PB * u) {
                        int k[U];
                        int32_t a[U], w[U], dw[U];
                        wg::arcs_of<U, PB>(ch, run, e0, u, tot, min(PB, le - cb), k, a);
#pragma unroll
                        for (int j = 0; j < U; ++j) w[j] = a[j] >= 0 ? col[a[j]] : 0;
#pragma unroll
                        for (int j = 0; j < U; ++j) dw[j] = a[j] >= 0 ? dist[w[j]] : -1;
#pragma unroll
                        for (int j = 0; j < U; ++j)
                            if (a[j] >= 0 && dw[j] == l + 1) {
                                const int32_t v = ch.v[k[j]];
                                const double cw = acc[w[j]];
                                unsafeAtomicAdd(&acc[v], cw);
                                // edge term of arc v -> w: lambda(v) c(w)
                                if (eb) unsafeAtomicAdd(&eb[a[j]], (double)sigma[v] * cw);
                            }
                    }
                    __syncthreads();
                }
                wg::bar();
            }
            for (int32_t i = lb + tid; i < le; i += PB) {
                const int32_t v = queue[i];
                const double sv = (double)sigma[v];
                const double dl = sv * acc[v];
                if (accumulate && v != s) unsafeAtomicAdd(&bc[v], dl);
                if (delta_dump) delta_dump[(size_t)idx * n + v] = dl;
                acc[v] = (1.0 + dl) / sv;
            }
            wg::bar();
        }
        if (dist_dump) {
            for (int32_t v = tid; v < n; v += PB) {
                const int32_t d = dist[v];
                dist_dump[(size_t)idx * n + v] = d;
                sigma_dump[(size_t)idx * n + v] = d >= 0 ? sigma[v] : 0;
                if (d < 0) delta_dump[(size_t)idx * n + v] = 0.0;
            }
        }
        if (tid == 0 && s_ovf) atomicOr(status, (uint32_t)BC_DEV_SIGMA_OVERFLOW);
        wg::bar();
    }
}

// The same sweep with every vertex's state in LDS (one byte: its level mod 3 as
// a bit, or UNREACHED, as in lds_sweep.h), for graphs whose bytes fit.  What
// bounds the sweep is random reads and atomics of 8-byte values, a sector each,
// so the two per arc that only ask for a neighbour's level are the ones to
// avoid: now only arcs of the shortest-path DAG leave the compute unit.  A
// vertex's count is replaced by its c in the backward, whose sums form in LDS,
// one accumulator per vertex of the chunk (no atomic in memory), and the
// workgroups are as many as fit the LDS: 12 bytes a vertex each, not 24 times
// 2048.  Up to a source per compute unit a workgroup has 1024 threads.  ms for
// 1 / 2048 sources, against the sweep with the state in memory: RMAT-15 1.3 /
// 17.3 and 9.1 / 61; RMAT-16 2.5 / 37 and 18 / 136; G(30000, 8/29999) 0.8 / 10.2
// and 3.3 / 39.  At n = 90208 one workgroup per unit is left: RMAT-17, 1024
// sources, 39 against 142.
template <int T>
__global__ __launch_bounds__(T) void k_plain_state(
    int32_t n, const int32_t *__restrict__ rp, const int32_t *__restrict__ col,
    const int32_t *__restrict__ sources, int64_t count, unsigned long long *next_counter, uint64_t *sc_all,
    int32_t *queue_all, int32_t *lev_all, double *bc, uint32_t *status, int accumulate,
    double *delta_dump, int32_t *dist_dump, uint64_t *sigma_dump, double *eb) {
    extern __shared__ uint32_t s_state[]; // [(n + 3) / 4] four states each
    __shared__ wg::ChunkOf<T> ch;
    __shared__ double s_sum[T];
    __shared__ int32_t s_tail;
    __shared__ long long s_idx;
    __shared__ uint32_t s_ovf;
    __shared__ uint32_t s_run[T / 64 * 2 * U]; // wg::arcs_of's bits, a wave's each
    constexpr uint32_t UNREACHED = 8;

    const int tid = threadIdx.x;
    const size_t g = blockIdx.x;
    uint8_t *st = reinterpret_cast<uint8_t *>(s_state);
    uint64_t *sc = sc_all + g * (size_t)n; // counts, then c as FP64 bits
    int32_t *queue = queue_all + g * (size_t)n;
    int32_t *lev = lev_all + g * ((size_t)n + 2);

    uint32_t *run = s_run + (tid >> 6) * 2 * U;
    if (tid < T / 64 * 2 * U) s_run[tid] = 0; // read after a barrier
    for (;;) {
        if (tid == 0) s_idx = (long long)atomicAdd(next_counter, 1ull);
        __syncthreads();
        const long long idx = s_idx;
        if (idx >= count) break;
        const int32_t s = sources[idx];
        for (int32_t v = tid; v < n; v += T) sc[v] = 0;
        for (int32_t i = tid; i < (n + 3) / 4; i += T) s_state[i] = 0x01010101u * UNREACHED;
        wg::bar();
        if (tid == 0) {
            st[s] = 1;
            sc[s] = 1;
            queue[0] = s;
            lev[0] = 0;
            lev[1] = 1;
            s_tail = 1;
            s_ovf = 0;
        }
        wg::bar();

        // ---- forward: level L spans queue[qb, qe) ----
        int32_t qb = 0, qe = 1, L = 0;
        while (qb < qe) {
            const uint32_t next = 1u << ((L + 1) % 3), open = UNREACHED | next;
            for (int32_t cb = qb; cb < qe; cb += T) {
                const int tot = wg::stage_chunk<T>(queue, cb, qe, rp, ch);
                const int u = wg::arcs_each<U, T>(tot);
                for (int e0 = wg::first_arc(u); e0 < tot; e0 += T * u) {
                    int k[U];
                    int32_t a[U], w[U];
                    bool in[U];
                    wg::arcs_of<U, T>(ch, run, e0, u, tot, min(T, qe - cb), k, a);
#pragma unroll
                    for (int j = 0; j < U; ++j) w[j] = a[j] >= 0 ? col[a[j]] : 0;
#pragma unroll
                    for (int j = 0; j < U; ++j) in[j] = a[j] >= 0 && (st[w[j]] & open); // v in P_s(w)
                    uint64_t x[U], old[U];
#pragma unroll
                    for (int j = 0; j < U; ++j) x[j] = in[j] ? sc[ch.v[k[j]]] : 0;
#pragma unroll
                    for (int j = 0; j < U; ++j) {
                        old[j] = 1;
                        if (in[j]) old[j] = atomicAdd((unsigned long long *)&sc[w[j]], (unsigned long long)x[j]);
                    }
#pragma unroll
                    for (int j = 0; j < U; ++j) {
                        if (!in[j]) continue;
                        if (old[j] + x[j] < old[j]) s_ovf = 1;
                        if (old[j] == 0) { // the first to reach w
                            st[w[j]] = (uint8_t)next;
                            const int32_t p = atomicAdd(&s_tail, 1);
                            if (p < n) queue[p] = w[j]; // always, unless a count wrapped to zero
                        }
                    }
                }
                __syncthreads(); // the chunk's LDS is restaged
            }
            wg::bar();
            qb = qe;
            qe = min(s_tail, n);
            ++L;
            if (tid == 0) lev[min(L + 1, n + 1)] = qe;
            wg::bar();
        }
        const int32_t nlev = min(L, n); // non-empty levels 0..nlev-1

        if (dist_dump) {
            for (int32_t v = tid; v < n; v += T)
                if (st[v] == UNREACHED) {
                    dist_dump[(size_t)idx * n + v] = -1;
                    sigma_dump[(size_t)idx * n + v] = 0;
                    delta_dump[(size_t)idx * n + v] = 0.0;
                }
            for (int32_t l = 0; l < nlev; ++l)
                for (int32_t i = lev[l] + tid; i < lev[l + 1]; i += T) {
                    const int32_t v = queue[i];
                    dist_dump[(size_t)idx * n + v] = l;
                    sigma_dump[(size_t)idx * n + v] = sc[v];
                }
            wg::bar();
        }

        // ---- backward: deepest level first ----
        // (level 0 adds nothing to BC, but its arcs carry edge terms)
        const int32_t lowest = accumulate && !eb ? 1 : 0;
        for (int32_t l = nlev - 1; l >= lowest; --l) {
            const uint32_t next = 1u << ((l + 1) % 3);
            const int32_t lb = lev[l], le = lev[l + 1];
            for (int32_t cb = lb; cb < le; cb += T) {
                s_sum[tid] = 0.0;
                if (l < nlev - 1) {
                    const int tot = wg::stage_chunk<T>(queue, cb, le, rp, ch);
                    const int u = wg::arcs_each<U, T>(tot);
                    for (int e0 = wg::first_arc(u); e0 < tot; e0 += T * u) {
                        int k[U];
                        int32_t a[U], w[U];
                        bool in[U];
                        wg::arcs_of<U, T>(ch, run, e0, u, tot, min(T, le - cb), k, a);
#pragma unroll
                        for (int j = 0; j < U; ++j) w[j] = a[j] >= 0 ? col[a[j]] : 0;
#pragma unroll
                        for (int j = 0; j < U; ++j) in[j] = a[j] >= 0 && (st[w[j]] & next);
                        double cw[U];
#pragma unroll
                        for (int j = 0; j < U; ++j) cw[j] = in[j] ? __longlong_as_double((long long)sc[w[j]]) : 0.0;
#pragma unroll
                        for (int j = 0; j < U; ++j)
                            if (in[j]) {
                                unsafeAtomicAdd(&s_sum[k[j]], cw[j]);
                                // edge term of arc v -> w: lambda(v) c(w)
                                if (eb) unsafeAtomicAdd(&eb[a[j]], (double)sc[ch.v[k[j]]] * cw[j]);
                            }
                    }
                    __syncthreads();
                }
                if (cb + tid < le) {
                    const int32_t v = queue[cb + tid];
                    const double sv = (double)sc[v];
                    const double dl = sv * s_sum[tid];
                    if (accumulate && v != s) unsafeAtomicAdd(&bc[v], dl);
                    if (delta_dump) delta_dump[(size_t)idx * n + v] = dl;
                    sc[v] = (uint64_t)__double_as_longlong((1.0 + dl) / sv);
                }
                __syncthreads(); // the chunk's LDS is restaged
            }
            wg::bar();
        }
        if (tid == 0 && s_ovf) atomicOr(status, (uint32_t)BC_DEV_SIGMA_OVERFLOW);
        wg::bar();
    }
}

// Threads per workgroup and workgroups per compute unit of the LDS-state sweep.
constexpr int ST_T = 512, WIDE_T = 1024;
constexpr size_t LDS_BYTES = 160 << 10;
template <int T>
constexpr size_t fixed_lds() { return sizeof(wg::ChunkOf<T>) + T * sizeof(double) + T / 64 * 2 * U * sizeof(uint32_t) + 64; }
size_t state_lds(int32_t n) { return ((size_t)n + 3) / 4 * 4; }

} // namespace

bc_status plain_prepare(bc_ctx *ctx) {
    if (ctx->weighted) return weighted_prepare(ctx);
    PlainState &p = ctx->pl;
    if (p.grid == 0 && small_fits(ctx)) return small_prepare(ctx);
    const size_t n = (size_t)std::max(ctx->n, 1);
    // how many workgroups of 512 threads the states of one compute unit allow;
    // one of 1024 where that is less than two
    int cus = 0;
    BC_HIP(ctx, hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, ctx->device));
    cus = std::max(cus, 1);
    const size_t per_cu = std::min<size_t>(LDS_BYTES / (fixed_lds<ST_T>() + state_lds(ctx->n)), 2048 / ST_T);
    p.threads = per_cu >= 2 ? ST_T : fixed_lds<WIDE_T>() + state_lds(ctx->n) <= LDS_BYTES ? WIDE_T : 0;
    // the kernels' limit, the same for every context
    BC_HIP(ctx, hipFuncSetAttribute((const void *)k_plain_state<ST_T>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                    (int)(LDS_BYTES - fixed_lds<ST_T>())));
    BC_HIP(ctx, hipFuncSetAttribute((const void *)k_plain_state<WIDE_T>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                    (int)(LDS_BYTES - fixed_lds<WIDE_T>())));
    p.cus = cus;
    const size_t per_group = (p.threads ? n * (8 + 4) : n * (4 + 8 + 8 + 4)) + (n + 2) * 4;
    const size_t budget = size_t(16) << 30;
    int groups = p.grid > 0 ? p.grid : !p.threads ? 2048 : cus * (p.threads == ST_T ? (int)per_cu : 1);
    while (groups > 1 && per_group * (size_t)groups > budget) groups /= 2;
    p.groups = groups;
    p.sigma = (uint64_t *)bc_dalloc(ctx, n * groups * sizeof(uint64_t));
    p.queue = (int32_t *)bc_dalloc(ctx, n * groups * sizeof(int32_t));
    p.lev = (int32_t *)bc_dalloc(ctx, (n + 2) * groups * sizeof(int32_t));
    p.next = (uint32_t *)bc_dalloc(ctx, 256);
    if (!p.threads) {
        p.dist = (int32_t *)bc_dalloc(ctx, n * groups * sizeof(int32_t));
        p.acc = (double *)bc_dalloc(ctx, n * groups * sizeof(double));
    }
    if (!p.sigma || !p.queue || !p.lev || !p.next || (!p.threads && (!p.dist || !p.acc)))
        return bc_fail(ctx, BC_ERR_NOMEM, "plain form: workspace allocation failed");
    return BC_OK;
}

bc_status plain_run(bc_ctx *ctx, const int32_t *d_sources, int64_t count, bool accumulate,
                    double *delta_dump, int32_t *dist_dump, uint64_t *sigma_dump) {
    if (ctx->weighted) return weighted_run(ctx, d_sources, count, accumulate, delta_dump, dist_dump, sigma_dump);
    if (ctx->sm.on) {
        LaunchTimer t(ctx, "plain_sweep");
        bc_status st = small_run(ctx, d_sources, count, true, accumulate ? nullptr : delta_dump, dist_dump, sigma_dump);
        t.done();
        return st;
    }
    PlainState &p = ctx->pl;
    BC_HIP(ctx, hipMemsetAsync(p.next, 0, sizeof(unsigned long long), ctx->stream));
    const int grid = (int)std::min<int64_t>(count, p.groups);
    double *eb = accumulate && ctx->edges ? ctx->eb : nullptr;
    LaunchTimer t(ctx, "plain_sweep");
    if (p.threads) {
        // up to a source per compute unit: all the threads one can have
        const bool wide = p.threads == WIDE_T ||
                          (count <= p.cus && fixed_lds<WIDE_T>() + state_lds(ctx->n) <= LDS_BYTES);
        hipLaunchKernelGGL(wide ? k_plain_state<WIDE_T> : k_plain_state<ST_T>, dim3(grid),
                           dim3(wide ? WIDE_T : ST_T), state_lds(ctx->n), ctx->stream, ctx->n, ctx->row_ptr,
                           ctx->col, d_sources, count, (unsigned long long *)p.next, p.sigma, p.queue, p.lev, ctx->bc,
                           ctx->status, accumulate ? 1 : 0, delta_dump, dist_dump, sigma_dump, eb);
    } else {
        hipLaunchKernelGGL(k_plain_sweep, dim3(grid), dim3(PB), 0, ctx->stream, ctx->n, ctx->row_ptr, ctx->col,
                           d_sources, count, (unsigned long long *)p.next, p.dist, p.sigma, p.acc, p.queue, p.lev,
                           ctx->bc, ctx->status, accumulate ? 1 : 0, delta_dump, dist_dump, sigma_dump, eb);
    }
    t.done();
    BC_HIP(ctx, hipGetLastError());
    return BC_OK;
}
