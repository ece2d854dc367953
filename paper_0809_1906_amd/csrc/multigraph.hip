// Many small graphs in one persistent launch.
//
// A context built by bc_create_many holds up to millions of small unweighted
// graphs (each with at most MG_MAX_N vertices) concatenated: vertex v of graph
// g has global id voff[g] + v, and BC is returned in that numbering.  bc_run
// computes all-source BC of every graph (Brandes's algorithm, Sec. 1.1, per
// graph).
//
// The work is a device queue of units (graph, [s0, s1) of its sources) sorted
// by n_g descending, largest first (longest-processing-time order).  A grid of
// persistent workgroups pulls units with an atomic counter and exits when the
// queue is drained.  Two sweeps:
//   group sweep  (lds_sweep.h) as many sources at once as the LDS holds, 32-bit
//                counts overwritten by FP32 c(v), at most LEVCAP levels; units
//                it cannot finish again with 64-bit counts and any
//                depth; for graphs of fewer than 65536 bursts of eight columns;
//   full sweep   one source at a time, 64-bit counts, any depth; for the other
//                graphs and the per-source readout.
// In both, each unit's dependencies are summed in an FP64 LDS vector and added
// to BC once per unit.  The full sweep's columns are staged in LDS as 16-bit
// local ids when they fit.  The launches (counter reset, group sweeps, full
// sweep over the remaining graphs, group sweep over the handed-back units) are
// captured once into a HIP graph and replayed.
#include "bc_internal.h"
#include "lds_sweep.h"

#include <algorithm>
#include <type_traits>

namespace {

constexpr int MT = 512;          // threads per workgroup
constexpr int32_t MG_INF = 0x7FFFFFFF;
constexpr int ABURST = 8;        // column reads issued together per vertex
constexpr int32_t COL_CAP = 16320; // 16-bit columns staged in LDS
constexpr int LEVCAP = 1024;       // levels per source in the group sweep
// The group sweep is bound by VALU and LDS issue about equally (counters over
// 256 Watts-Strogatz graphs: each busy half of the time), and gains from
// every source that shares a barrier: one workgroup of 1024 threads with the
// whole LDS (K = 4 at n = 4096).  256 Watts-Strogatz graphs, n = 64..4096:
// 20.0 ms, against 23.0 with two workgroups of 512 and half the LDS each, and
// 67.8 with one source at a time per workgroup, 32-bit columns and a
// compare-and-swap per arc.  Tiny graphs fill a quarter of the LDS with all
// their sources: 5000 graphs of 30 vertices 0.19 ms against 0.33, 3000 of 100
// 0.49 against 0.56; even at 250, and slower from 1000 (8.3 against 6.8 ms).
constexpr int BIG_T = 1024, BIG_BYTES = 163000, SMALL_T = 512, SMALL_BYTES = 40000;
constexpr int32_t SMALL_N = 256;
static_assert(lds_sweep::bytes_for<uint32_t>(MG_MAX_N, 1, LEVCAP) <= BIG_BYTES, "one source of the largest graph");
static_assert(lds_sweep::bytes_for<uint64_t>(MG_MAX_N, 1, MG_MAX_N) <= BIG_BYTES, "the same in 64 bits, any depth");
static_assert(lds_sweep::bytes_for<uint32_t>(SMALL_N, 1, SMALL_N) <= SMALL_BYTES, "one source of a small graph");

struct MultiArgs {
    const int32_t *voff;   // [ngraphs+1] first global vertex of each graph
    const int32_t *rpoff;  // [ngraphs] where graph g's row offsets start in rp
    const int32_t *rp;     // concatenated per-graph row offsets (global arc indices)
    const int32_t *col;    // concatenated arcs, local vertex ids
    const int32_t *units;  // [nunits][3] = (graph, s0, s1), local source ids
    int32_t nunits;
    const unsigned int *nunits_dev; // if set, the unit count is read here instead
    unsigned int *next;    // queue counter
    const uint16_t *brp;   // group sweep: first burst of each row, indexed as rp
    const int64_t *boff;   // [ngraphs] first burst of each graph (-1: not in the group sweep)
    const uint32_t *safe;  // [ngraphs] (2^32 - 1) / largest degree
    const uint4 *bursts;   // columns as 16-bit ids, eight per burst
    int32_t *redo;         // group sweep with 32-bit counts: units to run again in 64 bits
    unsigned int *redo_count;
    double *bc;            // [sum n]
    uint32_t *status;
    // per-source readout (bc_read_sssp): unit u covers one source, row u
    int32_t dump_n;        // sum n (row length); 0 = no readout
    int32_t *dist_dump;
    uint64_t *sigma_dump;
    double *delta_dump;
};

__global__ void k_mg_reset(unsigned int *next) {
    if (threadIdx.x < 5) next[threadIdx.x] = 0;
}

struct MgShared {
    int32_t dist[MG_MAX_N];
    unsigned long long sig[MG_MAX_N];
    float c[MG_MAX_N];
    uint16_t queue[MG_MAX_N];
    uint16_t lev[MG_MAX_N + 2];
    double bc[MG_MAX_N];
    int32_t rp[MG_MAX_N + 1]; // the unit's graph: row offsets relative to its first arc
    uint16_t col[COL_CAP];    // the unit's columns, when they fit
    int32_t unit, cnt[3];
    uint32_t ovf;
};

// The sources [s0, s1) of unit u; columns from LDS (LC) or global memory.
template <bool LC>
__device__ __forceinline__ void mg_unit(const MultiArgs &a, MgShared &sh, int32_t u, int32_t n, int32_t vo,
                                        const int32_t *gcol, int32_t s0, int32_t s1) {
    int32_t *s_dist = sh.dist;
    unsigned long long *s_sig = sh.sig;
    float *s_c = sh.c;
    uint16_t *s_queue = sh.queue, *s_lev = sh.lev;
    double *s_bc = sh.bc;
    const int32_t *s_rp = sh.rp;
    int32_t *s_cnt = sh.cnt;
    const int tid = threadIdx.x;
    auto col = [&](int32_t e) -> int32_t { return LC ? (int32_t)sh.col[e] : gcol[e]; };
        for (int32_t s = s0; s < s1; ++s) {
            for (int32_t v = tid; v < n; v += MT) {
                s_dist[v] = v == s ? 0 : MG_INF;
                s_sig[v] = v == s ? 1ull : 0ull;
            }
            if (tid == 0) {
                s_queue[0] = (uint16_t)s;
                s_lev[0] = 0;
                s_lev[1] = 1;
                s_cnt[0] = 0;
                s_cnt[1] = 0;
                s_cnt[2] = 0;
            }
            __syncthreads();
            // forward: level L spans queue[qb, qe); appends of level L go to
            // queue[qe + s_cnt[L % 3]].  Three counters let one barrier per
            // level suffice: while level L appends to s_cnt[L % 3], thread 0
            // clears s_cnt[(L + 1) % 3], last read before the previous barrier.
            int32_t qb = 0, qe = 1, L = 0;
            while (qb < qe) {
                const int cur = L % 3;
                if (tid == 0) s_cnt[(L + 1) % 3] = 0;
                for (int32_t i = qb + tid; i < qe; i += MT) {
                    const int32_t v = s_queue[i];
                    const unsigned long long sv = s_sig[v];
                    const int32_t rb = s_rp[v], re = s_rp[v + 1];
                    for (int32_t e0 = rb; e0 < re; e0 += ABURST) {
                        int32_t ws[ABURST]; // one burst of column reads in flight
#pragma unroll
                        for (int j = 0; j < ABURST; ++j) ws[j] = e0 + j < re ? col(e0 + j) : -1;
#pragma unroll
                        for (int j = 0; j < ABURST; ++j) {
                            const int32_t w = ws[j];
                            if (w < 0) continue;
                            int32_t dw = s_dist[w];
                            if (dw == MG_INF) {
                                const int32_t old = atomicCAS(&s_dist[w], MG_INF, L + 1);
                                if (old == MG_INF) {
                                    s_queue[qe + atomicAdd(&s_cnt[cur], 1)] = (uint16_t)w;
                                    dw = L + 1;
                                } else {
                                    dw = old;
                                }
                            }
                            if (dw == L + 1) { // v in P_s(w)
                                const unsigned long long old = atomicAdd(&s_sig[w], sv);
                                if (old + sv < old) sh.ovf = 1;
                            }
                        }
                    }
                }
                __syncthreads();
                qb = qe;
                qe += s_cnt[cur];
                ++L;
                if (tid == 0) s_lev[L + 1] = (uint16_t)qe;
            }
            __syncthreads();
            const int32_t nlev = L;
            // backward: deepest level first; one thread per vertex, no atomics
            const int32_t lowest = a.dump_n ? 0 : 1;
            for (int32_t l = nlev - 1; l >= lowest; --l) {
                for (int32_t i = s_lev[l] + tid; i < s_lev[l + 1]; i += MT) {
                    const int32_t v = s_queue[i];
                    double acc = 0.0;
                    if (l + 1 < nlev) {
                        const int32_t rb = s_rp[v], re = s_rp[v + 1];
                        for (int32_t e0 = rb; e0 < re; e0 += ABURST) {
                            int32_t ws[ABURST];
#pragma unroll
                            for (int j = 0; j < ABURST; ++j) ws[j] = e0 + j < re ? col(e0 + j) : -1;
#pragma unroll
                            for (int j = 0; j < ABURST; ++j)
                                if (ws[j] >= 0 && s_dist[ws[j]] == l + 1) acc += (double)s_c[ws[j]];
                        }
                    }
                    const double sv = (double)s_sig[v];
                    const double dl = sv * acc;
                    s_c[v] = (float)((1.0 + dl) / sv);
                    if (v != s) s_bc[v] += dl;
                    if (a.dump_n) a.delta_dump[(size_t)u * a.dump_n + vo + v] = dl;
                }
                __syncthreads();
            }
            if (a.dump_n) {
                for (int32_t v = tid; v < n; v += MT) {
                    const int32_t d = s_dist[v];
                    a.dist_dump[(size_t)u * a.dump_n + vo + v] = d == MG_INF ? -1 : d;
                    a.sigma_dump[(size_t)u * a.dump_n + vo + v] = d == MG_INF ? 0 : s_sig[v];
                    if (d == MG_INF) a.delta_dump[(size_t)u * a.dump_n + vo + v] = 0.0;
                }
            }
            __syncthreads();
        }
}

__global__ __launch_bounds__(MT) void k_mg_sweep(MultiArgs a) {
    __shared__ MgShared sh;
    const int tid = threadIdx.x;
    const int32_t nunits = a.nunits_dev ? (int32_t)*a.nunits_dev : a.nunits;
    for (;;) {
        if (tid == 0) sh.unit = (int32_t)atomicAdd(a.next, 1u);
        __syncthreads();
        const int32_t u = sh.unit;
        if (u >= nunits) break;
        const int32_t g = a.units[3 * u], s0 = a.units[3 * u + 1], s1 = a.units[3 * u + 2];
        const int32_t vo = a.voff[g], n = a.voff[g + 1] - vo;
        const int32_t *grp = a.rp + a.rpoff[g];
        const int32_t *col = a.col + grp[0];
        const int32_t arcs = grp[n] - grp[0];
        const bool lds_col = arcs <= COL_CAP;
        for (int32_t v = tid; v <= n; v += MT) sh.rp[v] = grp[v] - grp[0];
        for (int32_t v = tid; v < n; v += MT) sh.bc[v] = 0.0;
        if (lds_col)
            for (int32_t e = tid; e < arcs; e += MT) sh.col[e] = (uint16_t)col[e];
        if (tid == 0) sh.ovf = 0;
        __syncthreads();
        if (lds_col) mg_unit<true>(a, sh, u, n, vo, col, s0, s1);
        else mg_unit<false>(a, sh, u, n, vo, col, s0, s1);
        if (!a.dump_n)
            for (int32_t v = tid; v < n; v += MT)
                if (sh.bc[v] != 0.0) unsafeAtomicAdd(&a.bc[vo + v], sh.bc[v]);
        if (tid == 0 && sh.ovf) atomicOr(a.status, (uint32_t)BC_DEV_SIGMA_OVERFLOW);
        __syncthreads();
    }
}

// ---- the group sweep --------------------------------------------------------------

// ST = uint32_t hands units it cannot finish to a.redo; ST = uint64_t finishes
// any (it has room for as many levels as vertices).
template <typename ST, int T, int BYTES>
__global__ __launch_bounds__(T) void k_mg_group(MultiArgs a) {
    __shared__ __attribute__((aligned(16))) unsigned char raw[BYTES];
    __shared__ int32_t s_unit, s_cnt[3];
    __shared__ uint32_t s_fail;
    constexpr bool WIDE = sizeof(ST) == 8;
    const int tid = threadIdx.x;
    const int32_t nunits = a.nunits_dev ? (int32_t)*a.nunits_dev : a.nunits;
    for (;;) {
        if (tid == 0) {
            s_unit = (int32_t)atomicAdd(a.next, 1u);
            s_fail = 0;
        }
        __syncthreads();
        const int32_t u = s_unit;
        if (u >= nunits) break;
        const int32_t g = a.units[3 * u], s0 = a.units[3 * u + 1], s1 = a.units[3 * u + 2];
        const int32_t vo = a.voff[g], n = a.voff[g + 1] - vo;
        const int32_t levels = WIDE ? n : min(n, LEVCAP);
        int32_t K = lds_sweep::group_size<ST>(BYTES, n, levels, s1 - s0);
        const int32_t groups = (s1 - s0 + K - 1) / K;
        K = (s1 - s0 + groups - 1) / groups; // even groups
        lds_sweep::Arrays<ST> s(raw, n, K, levels);
        const uint16_t *br = a.brp + a.rpoff[g];
        const uint4 *cols = a.bursts + a.boff[g];
        for (int32_t v = tid; v <= n; v += T) s.rp[v] = br[v];
        for (int32_t v = tid; v < n; v += T) s.bc[v] = 0.0;
        const uint32_t safe = a.safe[g];
        auto sweep = [&](auto heavy) { // false when the unit must be handed back (uniform)
            constexpr bool HV = decltype(heavy)::value;
            for (int32_t k0 = s0; k0 < s1; k0 += K) {
                s.K = min(K, s1 - k0);
                const int32_t nlev = lds_sweep::forward<ST, T, HV>(
                    s, cols, [&](int32_t k) { return k0 + k; }, (ST)safe, s_cnt, &s_fail, lds_sweep::FEW_HEAVY);
                if (nlev < 0 || (!WIDE && s_fail)) return false;
                lds_sweep::backward<ST, T, HV, true>(s, cols, nlev, 1, lds_sweep::FEW_HEAVY,
                                                                      [](int32_t, int32_t, double) {});
            }
            return true;
        };
        // a row of more than HEAVY bursts
        const bool hv = safe < 0xFFFFFFFFu / (lds_sweep::HEAVY * lds_sweep::BURST);
        const bool done = hv ? sweep(std::true_type()) : sweep(std::false_type());
        __syncthreads();
        if (done) {
            for (int32_t v = tid; v < n; v += T)
                if (s.bc[v] != 0.0) unsafeAtomicAdd(&a.bc[vo + v], s.bc[v]);
            if (WIDE && tid == 0 && s_fail) atomicOr(a.status, (uint32_t)BC_DEV_SIGMA_OVERFLOW);
        } else if (tid == 0) {
            const unsigned int k = atomicAdd(a.redo_count, 1u);
            a.redo[3 * k] = g;
            a.redo[3 * k + 1] = s0;
            a.redo[3 * k + 2] = s1;
        }
        __syncthreads();
    }
}

// Fill for the per-source readout rows: vertices of other graphs are
// unreachable (-1, 0, 0).
__global__ __launch_bounds__(256) void k_mg_fill(int64_t cells, int32_t *dist, uint64_t *sigma, double *delta) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= cells) return;
    dist[i] = -1;
    sigma[i] = 0;
    delta[i] = 0.0;
}

MultiArgs args_of(bc_ctx *ctx, const int32_t *units, int32_t nunits) {
    MultiState &m = ctx->mg;
    MultiArgs a{};
    a.voff = m.voff;
    a.rpoff = m.rpoff;
    a.rp = m.rp;
    a.col = ctx->col;
    a.units = units;
    a.nunits = nunits;
    a.brp = m.cols.brp;
    a.boff = m.cols.boff;
    a.safe = m.cols.safe;
    a.bursts = (const uint4 *)m.cols.bursts;
    a.next = m.next;
    a.bc = ctx->bc;
    a.status = ctx->status;
    return a;
}

} // namespace

// Host side of bc_create_many: concatenated arrays and the LPT-ordered queue.
bc_status multigraph_prepare(bc_ctx *ctx, const std::vector<int32_t> &voff, const std::vector<int32_t> &rpoff,
                             const std::vector<int32_t> &rp, int32_t chunk) {
    MultiState &m = ctx->mg;
    const int32_t ng = (int32_t)voff.size() - 1;
    m.ngraphs = ng;
    m.h_voff = voff;
    m.h_arcs.assign((size_t)ng, 0);
    for (int32_t g = 0; g < ng; ++g) {
        const int32_t n = voff[g + 1] - voff[g];
        m.h_arcs[(size_t)g] = rp[(size_t)rpoff[(size_t)g] + n] - rp[(size_t)rpoff[(size_t)g]];
    }
    // graphs by n_g descending (stable: ties keep graph order)
    m.h_order.resize((size_t)ng);
    for (int32_t g = 0; g < ng; ++g) m.h_order[(size_t)g] = g;
    std::stable_sort(m.h_order.begin(), m.h_order.end(), [&](int32_t x, int32_t y) {
        return voff[x + 1] - voff[x] > voff[y + 1] - voff[y];
    });
    m.voff = (int32_t *)bc_dalloc(ctx, voff.size() * sizeof(int32_t));
    m.rpoff = (int32_t *)bc_dalloc(ctx, std::max<size_t>(rpoff.size(), 1) * sizeof(int32_t));
    m.rp = (int32_t *)bc_dalloc(ctx, std::max<size_t>(rp.size(), 1) * sizeof(int32_t));
    m.next = (unsigned int *)bc_dalloc(ctx, 256);
    if (!m.voff || !m.rpoff || !m.rp || !m.next) return bc_fail(ctx, BC_ERR_NOMEM, "many graphs: allocation failed");
    BC_HIP(ctx, hipMemcpy(m.voff, voff.data(), voff.size() * sizeof(int32_t), hipMemcpyHostToDevice));
    if (!rpoff.empty())
        BC_HIP(ctx, hipMemcpy(m.rpoff, rpoff.data(), rpoff.size() * sizeof(int32_t), hipMemcpyHostToDevice));
    if (!rp.empty()) BC_HIP(ctx, hipMemcpy(m.rp, rp.data(), rp.size() * sizeof(int32_t), hipMemcpyHostToDevice));
    bc_status st = lds_columns(ctx, voff, rpoff, rp, m.voff, m.rpoff, m.rp, m.cols, m.h_group);
    if (st != BC_OK) return st;
    return multigraph_set_queue(ctx, nullptr, chunk > 0 ? chunk : 64);
}

// Units (graph, s0, s1) of `chunk` sources: the group sweep's graphs above
// SMALL_N vertices first, then its others, then those for the full sweep, each
// class largest graph first.
bc_status multigraph_set_queue(bc_ctx *ctx, const std::vector<int32_t> *graphs, int32_t chunk) {
    MultiState &m = ctx->mg;
    const std::vector<int32_t> &order = graphs ? *graphs : m.h_order;
    std::vector<int32_t> units;
    int32_t end[3] = {0, 0, 0}; // units through each class
    for (int pass = 0; pass < 3; ++pass) {
        for (int32_t g : order) {
            const int32_t n = m.h_voff[(size_t)g + 1] - m.h_voff[(size_t)g];
            const int cls = !m.h_group[(size_t)g] ? 2 : n > SMALL_N ? 0 : 1;
            if (cls != pass) continue;
            for (int32_t s0 = 0; s0 < n; s0 += chunk) {
                units.push_back(g);
                units.push_back(s0);
                units.push_back(std::min(n, s0 + chunk));
            }
        }
        end[pass] = (int32_t)(units.size() / 3);
    }
    if (m.exec) { // recorded with the old queue's addresses and sizes
        BC_HIP(ctx, hipStreamSynchronize(m.stream));
        BC_HIP(ctx, hipGraphExecDestroy(m.exec));
        m.exec = nullptr;
    }
    BC_HIP(ctx, hipStreamSynchronize(ctx->stream)); // no launch still reads the old queue
    if (m.units) bc_dfree(ctx, m.units);
    if (m.redo) bc_dfree(ctx, m.redo);
    m.units = (int32_t *)bc_dalloc(ctx, std::max<size_t>(units.size(), 3) * sizeof(int32_t));
    m.redo = (int32_t *)bc_dalloc(ctx, (size_t)std::max(end[1], 1) * 3 * sizeof(int32_t));
    if (!m.units || !m.redo) return bc_fail(ctx, BC_ERR_NOMEM, "many graphs: allocation failed");
    if (!units.empty())
        BC_HIP(ctx, hipMemcpy(m.units, units.data(), units.size() * sizeof(int32_t), hipMemcpyHostToDevice));
    m.chunk = chunk;
    m.nbig = end[0];
    m.nsmall = end[1] - end[0];
    m.nunits = (int32_t)(units.size() / 3);
    int cus = 0;
    BC_HIP(ctx, hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, ctx->device));
    m.grid = cus > 0 ? cus : 256; // compute units
    return BC_OK;
}

// All sources of every graph.  The first call records the launch into a HIP
// graph on the context's stream; later calls replay it.
bc_status multigraph_run(bc_ctx *ctx) {
    MultiState &m = ctx->mg;
    if (m.nunits == 0) return BC_OK;
    if (!m.exec) {
        // the group sweep over its two classes, the full sweep over the other
        // graphs, and the group sweep with 64-bit counts over the units handed
        // back (their count read on the device)
        const int32_t ngroup = m.nbig + m.nsmall;
        MultiArgs ab = args_of(ctx, m.units, m.nbig);
        ab.next = m.next;
        ab.redo = m.redo;
        ab.redo_count = m.next + 3;
        MultiArgs as = args_of(ctx, m.units + (size_t)3 * m.nbig, m.nsmall);
        as.next = m.next + 4;
        as.redo = m.redo;
        as.redo_count = m.next + 3;
        MultiArgs af = args_of(ctx, m.units + (size_t)3 * ngroup, m.nunits - ngroup);
        af.next = m.next + 1;
        MultiArgs ar = args_of(ctx, m.redo, 0);
        ar.nunits_dev = m.next + 3;
        ar.next = m.next + 2;
        hipGraph_t graph = nullptr;
        BC_HIP(ctx, hipStreamBeginCapture(m.stream, hipStreamCaptureModeThreadLocal));
        hipLaunchKernelGGL(k_mg_reset, dim3(1), dim3(64), 0, m.stream, m.next);
        if (m.nbig > 0)
            hipLaunchKernelGGL((k_mg_group<uint32_t, BIG_T, BIG_BYTES>), dim3(std::min(m.nbig, m.grid)), dim3(BIG_T), 0, m.stream,
                               ab);
        if (m.nsmall > 0)
            hipLaunchKernelGGL((k_mg_group<uint32_t, SMALL_T, SMALL_BYTES>), dim3(std::min(m.nsmall, 4 * m.grid)), dim3(SMALL_T), 0,
                               m.stream, as);
        if (m.nunits > ngroup)
            hipLaunchKernelGGL(k_mg_sweep, dim3(std::min(m.nunits - ngroup, m.grid)), dim3(MT), 0, m.stream, af);
        if (ngroup > 0)
            hipLaunchKernelGGL((k_mg_group<uint64_t, BIG_T, BIG_BYTES>), dim3(std::min(ngroup, m.grid)), dim3(BIG_T), 0,
                               m.stream, ar);
        BC_HIP(ctx, hipStreamEndCapture(m.stream, &graph));
        const hipError_t e = hipGraphInstantiate(&m.exec, graph, nullptr, nullptr, 0);
        (void)hipGraphDestroy(graph);
        if (e != hipSuccess) return bc_hip(ctx, e, "hipGraphInstantiate");
    }
    // order the private capture stream after prior work on the context stream
    BC_HIP(ctx, hipEventRecord(m.ev, ctx->stream));
    BC_HIP(ctx, hipStreamWaitEvent(m.stream, m.ev, 0));
    LaunchTimer t(ctx, "multigraph_sweep");
    BC_HIP(ctx, hipGraphLaunch(m.exec, m.stream));
    BC_HIP(ctx, hipEventRecord(m.ev, m.stream));
    BC_HIP(ctx, hipStreamWaitEvent(ctx->stream, m.ev, 0));
    t.done();
    return BC_OK;
}

// Per-source readout: global vertex ids of the concatenated numbering.
bc_status multigraph_dump(bc_ctx *ctx, const int32_t *h_sources, int32_t count, int32_t *dist_dump,
                          uint64_t *sigma_dump, double *delta_dump, int32_t *units_buf) {
    MultiState &m = ctx->mg;
    std::vector<int32_t> units((size_t)3 * count);
    for (int32_t i = 0; i < count; ++i) {
        const int32_t s = h_sources[i];
        const int32_t g = (int32_t)(std::upper_bound(m.h_voff.begin(), m.h_voff.end(), s) - m.h_voff.begin()) - 1;
        units[(size_t)3 * i] = g;
        units[(size_t)3 * i + 1] = s - m.h_voff[(size_t)g];
        units[(size_t)3 * i + 2] = s - m.h_voff[(size_t)g] + 1;
    }
    int32_t *du = units_buf ? units_buf : (int32_t *)bc_dalloc(ctx, units.size() * sizeof(int32_t));
    if (!du) return bc_fail(ctx, BC_ERR_NOMEM, "many graphs: readout allocation failed");
    BC_HIP(ctx, hipMemcpy(du, units.data(), units.size() * sizeof(int32_t), hipMemcpyHostToDevice));
    const int64_t cells = (int64_t)count * ctx->n;
    hipLaunchKernelGGL(k_mg_fill, dim3((unsigned)((cells + 255) / 256)), dim3(256), 0, ctx->stream, cells, dist_dump,
                       sigma_dump, delta_dump);
    MultiArgs a = args_of(ctx, du, count);
    a.dump_n = ctx->n;
    a.dist_dump = dist_dump;
    a.sigma_dump = sigma_dump;
    a.delta_dump = delta_dump;
    hipLaunchKernelGGL(k_mg_reset, dim3(1), dim3(64), 0, ctx->stream, m.next);
    hipLaunchKernelGGL(k_mg_sweep, dim3(std::min(count, m.grid)), dim3(MT), 0, ctx->stream, a);
    BC_HIP(ctx, hipGetLastError());
    BC_HIP(ctx, hipStreamSynchronize(ctx->stream));
    if (!units_buf) bc_dfree(ctx, du);
    return BC_OK;
}
