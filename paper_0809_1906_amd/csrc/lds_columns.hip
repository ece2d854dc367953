// Columns of small graphs for the LDS sweeps (lds_sweep.h): 16-bit ids in
// bursts of eight, rows padded with the id n.
#include "bc_internal.h"
#include "lds_sweep.h"
#include "wg_utils.h"

#include <algorithm>
#include <cstring>

namespace {

__device__ __forceinline__ uint4 burst_of(const int32_t *__restrict__ col, int32_t e, int32_t end, int32_t n) {
    uint32_t x[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const uint32_t lo = (uint32_t)(e < end ? col[e] : n);
        const uint32_t hi = (uint32_t)(e + 1 < end ? col[e + 1] : n);
        x[q] = lo | hi << 16;
        e += 2;
    }
    return make_uint4(x[0], x[1], x[2], x[3]);
}

// One graph: a block per 256 rows, which adds up the bursts of the rows before
// its own and deals its own bursts to its threads; the first clears `zero`.
__global__ __launch_bounds__(256) void k_pad_graph(int32_t n, const int32_t *__restrict__ rp,
                                                   const int32_t *__restrict__ col, uint16_t *__restrict__ brp,
                                                   uint4 *__restrict__ bursts, uint32_t *__restrict__ zero, int words) {
    __shared__ int s_off[257], s_wave[4];
    const int tid = threadIdx.x;
    const int32_t v0 = blockIdx.x * 256, v = v0 + tid;
    auto bursts_in = [&](int32_t u) { return (rp[u + 1] - rp[u] + lds_sweep::BURST - 1) / lds_sweep::BURST; };
    int before = 0, base, total;
    for (int32_t u = tid; u < v0; u += 256) before += bursts_in(u);
    (void)wg::block_excl_scan(before, s_wave, &base);
    const int mine = v < n ? bursts_in(v) : 0;
    const int off = wg::block_excl_scan(mine, s_wave, &total);
    s_off[tid] = off;
    if (tid == 0) s_off[256] = total;
    if (v < n) brp[v] = (uint16_t)(base + off);
    if (v == n - 1) brp[n] = (uint16_t)(base + off + mine);
    if (blockIdx.x == 0 && tid < words) zero[tid] = 0;
    __syncthreads();
    for (int i = tid; i < total; i += 256) {
        const int k = wg::owner(s_off, i);
        const int32_t r = rp[v0 + k];
        bursts[base + i] = burst_of(col, r + (i - s_off[k]) * lds_sweep::BURST, rp[v0 + k + 1], n);
    }
}

// One block per graph.
__global__ __launch_bounds__(256) void k_pad_columns(const int32_t *__restrict__ voff, const int32_t *__restrict__ rpoff,
                                                     const int32_t *__restrict__ rp, const int32_t *__restrict__ col,
                                                     const uint16_t *__restrict__ brp, const int64_t *__restrict__ boff,
                                                     uint4 *__restrict__ bursts) {
    const int32_t g = blockIdx.x;
    if (boff[g] < 0) return;
    const int32_t n = voff[g + 1] - voff[g];
    const int32_t *r = rp + rpoff[g];
    const uint16_t *br = brp + rpoff[g];
    uint4 *out = bursts + boff[g];
    for (int32_t v = threadIdx.x; v < n; v += 256) {
        int32_t e = r[v];
        for (int32_t b = br[v]; b < br[v + 1]; ++b, e += lds_sweep::BURST) out[b] = burst_of(col, e, r[v + 1], n);
    }
}

} // namespace

bc_status lds_columns(bc_ctx *ctx, const std::vector<int32_t> &voff, const std::vector<int32_t> &rpoff,
                      const std::vector<int32_t> &rp, const int32_t *d_voff, const int32_t *d_rpoff,
                      const int32_t *d_rp, LdsColumns &out, std::vector<uint8_t> &taken) {
    const int32_t ng = (int32_t)voff.size() - 1;
    std::vector<uint16_t> brp(std::max<size_t>(rp.size(), 1));
    std::vector<int64_t> boff((size_t)std::max(ng, 1));
    std::vector<uint32_t> safe((size_t)std::max(ng, 1));
    taken.assign((size_t)ng, 0);
    int64_t total = 0;
    for (int32_t g = 0; g < ng; ++g) {
        const int32_t *r = rp.data() + rpoff[(size_t)g];
        uint16_t *b = brp.data() + rpoff[(size_t)g];
        const int32_t n = voff[(size_t)g + 1] - voff[(size_t)g];
        int64_t at = 0;
        int32_t deg = 1;
        for (int32_t v = 0; v < n && at < 65536; ++v) {
            b[v] = (uint16_t)at;
            deg = std::max(deg, r[v + 1] - r[v]);
            at += (r[v + 1] - r[v] + lds_sweep::BURST - 1) / lds_sweep::BURST;
        }
        taken[(size_t)g] = at < 65536; // 16-bit burst indices
        safe[(size_t)g] = 0xFFFFFFFFu / (uint32_t)deg;
        boff[(size_t)g] = at < 65536 ? total : -1;
        if (at < 65536) {
            b[n] = (uint16_t)at;
            total += at;
        }
    }
    // the tables in one piece, one copy: a small context's preparation is mostly
    // allocations and copies
    auto rounded = [](size_t bytes) { return (bytes + 255) / 256 * 256; };
    const size_t safe_at = rounded(boff.size() * sizeof(int64_t));
    const size_t brp_at = safe_at + rounded(safe.size() * sizeof(uint32_t));
    std::vector<char> host(brp_at + brp.size() * sizeof(uint16_t));
    char *d = (char *)bc_dalloc(ctx, host.size());
    out.bursts = bc_dalloc(ctx, (size_t)std::max<int64_t>(total, 1) * sizeof(uint4));
    if (!d || !out.bursts) return bc_fail(ctx, BC_ERR_NOMEM, "padded columns: allocation failed");
    out.boff = (int64_t *)d;
    out.safe = (uint32_t *)(d + safe_at);
    out.brp = (uint16_t *)(d + brp_at);
    if (ng == 0) return BC_OK;
    std::memcpy(host.data(), boff.data(), boff.size() * sizeof(int64_t));
    std::memcpy(host.data() + safe_at, safe.data(), safe.size() * sizeof(uint32_t));
    std::memcpy(host.data() + brp_at, brp.data(), brp.size() * sizeof(uint16_t));
    BC_HIP(ctx, hipMemcpy(d, host.data(), host.size(), hipMemcpyHostToDevice));
    hipLaunchKernelGGL(k_pad_columns, dim3(ng), dim3(256), 0, ctx->stream, d_voff, d_rpoff, d_rp, ctx->col, out.brp,
                       out.boff, (uint4 *)out.bursts);
    BC_HIP(ctx, hipGetLastError());
    return BC_OK;
}

bc_status lds_columns_of(bc_ctx *ctx, uint16_t *brp, void *bursts, uint32_t *zero, int words) {
    hipLaunchKernelGGL(k_pad_graph, dim3((ctx->n + 255) / 256), dim3(256), 0, ctx->stream, ctx->n, ctx->row_ptr,
                       ctx->col, brp, (uint4 *)bursts, zero, words);
    BC_HIP(ctx, hipGetLastError());
    return BC_OK;
}
