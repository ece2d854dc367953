// Small unweighted graphs: per-source sweeps with all per-source state in LDS
// (lds_sweep.h), for one graph and a list of sources.  The plain form takes
// 64-bit counts and FP64 c(v); the sparse and hybrid forms 32-bit counts and
// FP32 c(v), and the sources whose counts pass 32 bits again with 64-bit ones.
#include "bc_internal.h"
#include "lds_sweep.h"

#include <algorithm>

namespace {

// One workgroup per compute unit with (almost) its whole LDS, as in the
// many-graph group sweep.  The line for the plain form lies where a source's
// 64-bit state still fits (n <= 7084): below it the LDS sweep was faster at
// every size, degree and source count tried, from one source to all.  FP64, ms
// for one source / all, against the sweep with its state in memory: G(1024)
// degree 10 0.049 / 0.051 against 0.175 / 0.53; G(6500) degree 26 0.093 / 1.74
// against 1.86 / 23.4; RMAT-13 (hubs of thousands of arcs) 0.23 / 6.7 against
// 2.2 / 34; a ring lattice of 6001 0.18 / 3.2 against 0.88 / 7.8; a path of
// 1000 1.7 / 1.7 against 5.8 / 6.4.
constexpr int ST_T = 1024, ST_BYTES = 163000;

struct SmallArgs {
    int32_t n;
    const uint16_t *brp;
    const uint4 *bursts;
    const int32_t *sources;
    int64_t count;
    int32_t K, unit;        // sources per group, sources per unit (a multiple of no group: groups split it)
    int64_t nunits;
    const int32_t *list;    // units to run, *list_count of them (null: all nunits)
    const uint32_t *list_count;
    int32_t *redo;          // 32-bit counts: units to run again in 64 bits
    uint32_t *redo_count;
    lds_sweep::Rows rows;   // where the arcs are
    uint64_t safe;          // largest count whose sums need no wrap test
    double *bc;
    uint32_t *status, *depth;
    int32_t *dist_dump;     // per-source readout (DUMP), rows of n
    uint64_t *sigma_dump;
    double *delta_dump;     // may be null: forward only
};

__global__ void k_small_reset(uint32_t *count) {
    if (threadIdx.x == 0) count[0] = count[2] = 0;
}

template <typename ST, bool F32, bool HV, bool DUMP>
__global__ __launch_bounds__(ST_T) void k_small_sweep(SmallArgs a) {
    __shared__ __attribute__((aligned(16))) unsigned char raw[ST_BYTES];
    __shared__ int32_t s_cnt[3];
    __shared__ uint32_t s_fail;
    const int tid = threadIdx.x;
    const int32_t n = a.n, n1 = n + 1;
    lds_sweep::Arrays<ST> s(raw, n, a.K, n);
    for (int32_t v = tid; v <= n; v += ST_T) s.rp[v] = a.brp[v];
    for (int32_t v = tid; v < n; v += ST_T) s.bc[v] = 0.0;
    if (tid == 0) s_fail = 0;
    __syncthreads();
    int32_t depth = 0;
    const int64_t nunits = a.list ? (int64_t)*a.list_count : a.nunits;
    for (int64_t u = blockIdx.x; u < nunits; u += gridDim.x) {
        const int64_t unit = a.list ? a.list[u] : u;
        const int64_t i0 = unit * a.unit, i1 = min(i0 + a.unit, a.count);
        for (int64_t k0 = i0; k0 < i1; k0 += a.K) {
            s.K = (int32_t)min((int64_t)a.K, i1 - k0);
            const int32_t nlev = lds_sweep::forward<ST, ST_T, HV>(
                s, a.bursts, [&](int32_t k) { return a.sources[k0 + k]; }, (ST)a.safe, s_cnt, &s_fail, a.rows);
            if (s_fail) { // uniform: the forward ends with a barrier
                __syncthreads();
                if (tid == 0) {
                    s_fail = 0;
                    if (sizeof(ST) == 4) a.redo[atomicAdd(a.redo_count, 1u)] = (int32_t)unit;
                    else atomicOr(a.status, (uint32_t)BC_DEV_SIGMA_OVERFLOW);
                }
                if (sizeof(ST) == 4) break; // a unit is one group here: nothing of it was added
            }
            depth = max(depth, nlev);
            if constexpr (DUMP) {
                for (int32_t i = tid; i < s.K * n; i += ST_T) {
                    const int32_t k = i / n, v = i - k * n;
                    if (s.st[k * n1 + v] != lds_sweep::UNREACHED) continue;
                    const size_t at = (size_t)(k0 + k) * n + v;
                    a.dist_dump[at] = -1;
                    a.sigma_dump[at] = 0;
                    if (a.delta_dump) a.delta_dump[at] = 0.0;
                }
                for (int32_t l = 0; l < nlev; ++l)
                    for (int32_t i = s.lev[l] + tid; i < s.lev[l + 1]; i += ST_T) {
                        const int32_t id = s.queue[i], k = s.source_of(id);
                        const size_t at = (size_t)(k0 + k) * n + (id - k * n1);
                        a.dist_dump[at] = l;
                        a.sigma_dump[at] = (uint64_t)s.sc[id];
                    }
                __syncthreads(); // the backward overwrites the counts
                if (!a.delta_dump) continue;
                lds_sweep::backward<ST, ST_T, HV, F32>(s, a.bursts, nlev, 0, a.rows,
                                                       [&](int32_t k, int32_t v, double d) {
                    a.delta_dump[(size_t)(k0 + k) * n + v] = d;
                });
            } else {
                lds_sweep::backward<ST, ST_T, HV, F32>(s, a.bursts, nlev, 1, a.rows, [](int32_t, int32_t, double) {});
            }
        }
    }
    __syncthreads();
    if (!DUMP)
        for (int32_t v = tid; v < n; v += ST_T)
            if (s.bc[v] != 0.0) unsafeAtomicAdd(&a.bc[v], s.bc[v]);
    if (tid == 0 && a.depth && depth > 0) atomicMax(a.depth, (uint32_t)depth);
}

template <typename ST, bool F32>
void launch(bc_ctx *ctx, const SmallArgs &a, bool heavy, bool dump, int grid) {
    const auto k = dump ? (heavy ? k_small_sweep<ST, F32, true, true> : k_small_sweep<ST, F32, false, true>)
                        : (heavy ? k_small_sweep<ST, F32, true, false> : k_small_sweep<ST, F32, false, false>);
    hipLaunchKernelGGL(k, dim3(grid), dim3(ST_T), 0, ctx->stream, a);
}

} // namespace

static int64_t bursts_of(const bc_ctx *ctx) {
    int64_t bursts = 0;
    for (int32_t v = 0; v < ctx->n; ++v)
        bursts += (ctx->h_row_ptr[(size_t)v + 1] - ctx->h_row_ptr[(size_t)v] + lds_sweep::BURST - 1) / lds_sweep::BURST;
    return bursts;
}

bool small_fits(const bc_ctx *ctx) {
    if (ctx->weighted || ctx->edges || ctx->n < 1) return false;
    if (lds_sweep::bytes_for<uint64_t>((size_t)ctx->n, 1, (size_t)ctx->n) > ST_BYTES) return false;
    return bursts_of(ctx) < 65536;
}

// The sparse and hybrid forms' line.  A batch pays two launches per level and
// pulls every row at every level; the LDS sweep pays per arc and source.  A run
// and its read, microseconds for one source / milliseconds for all, LDS against
// batches of 256: a path of 1000 1177 / 1.73 against 4968 / 24.6; a ring lattice
// of 6001 220 / 2.3 against 924 / 22.6; G(4000) degree 10 88 / 0.37 against 152 /
// 1.74; RMAT-12 (97 thousand arcs) 135 / 1.02 against 182 / 1.21; G(6500) degree
// 26 (170) 120 / 1.65 against 158 / 3.3; G(2500) degree 75 (194) 130 / 0.61
// against 148 / 0.94.  Past the line the batches catch up: R-MAT of 5960 vertices
// (135) 169 / 2.5 against 185 / 2.2, RMAT-13 (204) 212 / 4.1 against 210 / 2.6,
// and 2.1 at 512.  Hubs cost the LDS sweep more, so the last stretch is for
// graphs without.
// Edge terms, kernel timing, host-driven batches and levels by products ask
// for the batched kernels themselves.
bool small_takes_batches(const bc_ctx *ctx) {
    if (ctx->form != BC_FORM_SPARSE && ctx->form != BC_FORM_HYBRID) return false;
    if (ctx->host_driven || ctx->timing || !small_fits(ctx)) return false;
    if (ctx->hy.products && (ctx->al.every_level || ctx->hy.theta_fwd <= 1.0 || ctx->hy.theta_bwd <= 1.0)) return false;
    return ctx->nnz <= 131072 || (ctx->nnz <= 196608 && ctx->max_degree <= 256);
}

int32_t small_levels(bc_ctx *ctx) {
    if (!ctx->sm.on || ctx->form == BC_FORM_PLAIN_FP64) return 0;
    uint32_t x = 0;
    if (hipMemcpyAsync(&x, ctx->sm.count + 1, sizeof x, hipMemcpyDeviceToHost, ctx->stream) != hipSuccess ||
        hipStreamSynchronize(ctx->stream) != hipSuccess)
        return 0;
    return (int32_t)x;
}

// An allocation-free readout of sources deeper than the frontier levels that
// the batched kernels would hold by now (16, doubled as earlier calls needed
// more) is refused, as it is where those kernels run: whichever route a graph
// takes, a context answers alike.
bc_status small_check_room(bc_ctx *ctx) {
    uint32_t levels[2]; // of ordinary calls, of this one
    BC_HIP(ctx, hipMemcpyAsync(levels, ctx->sm.count + 1, sizeof levels, hipMemcpyDeviceToHost, ctx->stream));
    BC_HIP(ctx, hipStreamSynchronize(ctx->stream));
    const int32_t seen = (int32_t)levels[0], now = (int32_t)levels[1];
    int32_t cap = 16;
    while (cap < seen + 1) cap *= 2;
    if (now > seen && now + 2 > cap)
        return bc_fail(ctx, BC_ERR_NOMEM, "the sources are deeper than any earlier call's: run them by an ordinary call first");
    return BC_OK;
}

bc_status small_prepare(bc_ctx *ctx) {
    SmallState &m = ctx->sm;
    // a small context's preparation is mostly allocations and copies: one
    // allocation (the counts, the columns, the first list, the row starts) and one
    // launch.  Creating a plain context of 300 vertices takes 145 us; with the
    // tables made on the host and uploaded 185.
    const size_t columns = (size_t)bursts_of(ctx) * sizeof(uint4);
    m.redo_cap = std::max(ctx->n, 4096);
    // Heavy rows come next to each other (by degree), a few waves' entries while
    // the others wait, so they are dealt to all waves where they hold a quarter of
    // the arcs.  Microseconds for one source / all, a wave's entries together / as
    // chosen: K(3000,20) 182 / 1204 and 91 / 458, RMAT-12 174 / 1094 and 135 / 1028; of
    // like lengths, G(1700) of degree 75 196 / 682 and 113 / 313, a ring lattice of 1800
    // and degree 72 1137 / 2205 and 271 / 1189.  (All sources of K(1000,60) lose: 304
    // and 342.)  With few arcs in heavy rows the light ones would be mixed by it:
    // G(4000) of degree 40 108 / 650 together, 115 / 717 dealt.
    int64_t heavy = 0;
    for (int32_t v = 0; v < ctx->n; ++v) {
        const int32_t deg = ctx->h_row_ptr[(size_t)v + 1] - ctx->h_row_ptr[(size_t)v];
        if (deg > lds_sweep::HEAVY * lds_sweep::BURST) heavy += deg;
    }
    const bool alike = (int64_t)ctx->max_degree * ctx->n <= 2 * (int64_t)ctx->nnz;
    const bool wide = ctx->nnz >= (int64_t)ctx->n * 2 * lds_sweep::HEAVY * lds_sweep::BURST;
    m.rows = 4 * heavy < ctx->nnz ? lds_sweep::FEW_HEAVY
             : !alike             ? lds_sweep::HUBS
             : wide               ? lds_sweep::ALIKE_LONG
                                  : lds_sweep::ALIKE;
    char *d = (char *)bc_dalloc(ctx, 256 + columns + (size_t)m.redo_cap * sizeof(int32_t) +
                                         ((size_t)ctx->n + 1) * sizeof(uint16_t));
    if (!d) return bc_fail(ctx, BC_ERR_NOMEM, "small graph: allocation failed");
    m.count = (uint32_t *)d;
    m.cols.bursts = d + 256;
    m.redo = m.first_redo = (int32_t *)(d + 256 + columns);
    m.cols.brp = (uint16_t *)(m.redo + m.redo_cap);
    bc_status st = lds_columns_of(ctx, m.cols.brp, m.cols.bursts, m.count, 64);
    if (st != BC_OK) return st;
    BC_HIP(ctx, hipDeviceGetAttribute(&m.cus, hipDeviceAttributeMultiprocessorCount, ctx->device));
    m.on = true;
    return BC_OK;
}

bc_status small_run(bc_ctx *ctx, const int32_t *d_sources, int64_t count, bool wide, double *delta_dump,
                    int32_t *dist_dump, uint64_t *sigma_dump) {
    SmallState &m = ctx->sm;
    const int32_t n = ctx->n, cus = std::max(m.cus, 1);
    const uint64_t deg = (uint64_t)std::max(ctx->max_degree, 1);
    const bool dump = dist_dump != nullptr, heavy = ctx->max_degree > lds_sweep::HEAVY * lds_sweep::BURST;
    SmallArgs a{};
    a.n = n;
    a.brp = m.cols.brp;
    a.bursts = (const uint4 *)m.cols.bursts;
    a.sources = d_sources;
    a.count = count;
    a.rows = (lds_sweep::Rows)m.rows;
    a.bc = ctx->bc;
    a.status = ctx->status;
    a.depth = wide ? nullptr : m.count + (ctx->no_alloc ? 2 : 1);
    a.dist_dump = dist_dump;
    a.sigma_dump = sigma_dump;
    a.delta_dump = delta_dump;
    // As many sources per group as fit, but no fewer groups than compute units,
    // and where they come in several rounds, groups that fill the last one too
    // (G(2500) of degree 75, groups of 8 / of 5: 1860 / 1370 us for all sources).
    const int32_t even = (int32_t)std::min<int64_t>((count + cus - 1) / cus, 65535);
    auto filled = [&](int32_t k) {
        const int64_t rounds = (count + (int64_t)cus * k - 1) / ((int64_t)cus * k);
        return (int32_t)((count + cus * rounds - 1) / (cus * rounds));
    };
    const int32_t k64 = filled(lds_sweep::group_size<uint64_t>(ST_BYTES, n, n, even));
    if (wide) {
        a.K = a.unit = k64;
        a.nunits = (count + a.unit - 1) / a.unit;
        a.safe = ~0ull / deg;
        launch<uint64_t, false>(ctx, a, heavy, dump, (int)std::min<int64_t>(a.nunits, cus));
        BC_HIP(ctx, hipGetLastError());
        return BC_OK;
    }
    a.K = a.unit = filled(lds_sweep::group_size<uint32_t>(ST_BYTES, n, n, even));
    a.nunits = (count + a.unit - 1) / a.unit;
    a.safe = 0xFFFFFFFFull / deg;
    if (a.nunits > m.redo_cap) {
        int32_t *r = (int32_t *)bc_dalloc(ctx, (size_t)a.nunits * sizeof(int32_t));
        if (!r) return bc_fail(ctx, BC_ERR_NOMEM, "small graph: allocation of the handed-back list failed");
        if (m.redo != m.first_redo) bc_dfree(ctx, m.redo);
        m.redo = r;
        m.redo_cap = a.nunits;
    }
    a.redo = m.redo;
    a.redo_count = m.count;
    hipLaunchKernelGGL(k_small_reset, dim3(1), dim3(64), 0, ctx->stream, m.count);
    launch<uint32_t, true>(ctx, a, heavy, dump, (int)std::min<int64_t>(a.nunits, cus));
    SmallArgs r = a;
    r.K = std::min(k64, a.unit);
    r.list = m.redo;
    r.list_count = m.count;
    r.safe = ~0ull / deg;
    launch<uint64_t, true>(ctx, r, heavy, dump, (int)std::min<int64_t>(a.nunits, cus));
    BC_HIP(ctx, hipGetLastError());
    return BC_OK;
}
