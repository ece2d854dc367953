// Per-source sweeps of a small graph with all per-source state in LDS, K
// sources at once in one workgroup (multigraph.hip, small.hip).
//
// Brandes's algorithm (Sec. 1.1) for the sources of a group together: an entry
// id = k (n + 1) + v stands for vertex v of the group's k-th source, and one
// queue holds the entries of every source in nondecreasing level, so that a
// level step (one barrier) expands that level of all K sources.
//   - A row's columns come in bursts of eight 16-bit ids, one 16-byte load per
//     lane; rows are padded to whole bursts with the id n, an entry whose
//     state matches nothing, so the padding takes no test.
//   - A vertex's state is one bit: which of the levels mod 3 it is at, or
//     UNREACHED.  Neighbours' levels differ by at most one, so that tells
//     predecessor, same level and successor apart, by one mask.  A vertex
//     unreached or already at the next level takes the count of the vertex
//     that found it by an atomic add; the add that finds zero (counts are at
//     least 1) claims it: it writes the state and appends the entry.
//   - A wave appends all it found in a burst at once, one LDS atomic.
//   - Counts are ST = uint32_t, then replaced by c(v) = (1 + delta(v)) /
//     lambda(v) as FP32; or uint64_t, and c(v) in FP64 or (F32) rounded to FP32,
//     so that a source whose counts need 64 bits gets the same result as the
//     other batched forms'.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace lds_sweep {

constexpr int BURST = 8; // columns per 16-byte load
// Rows of more bursts than this are taken a burst per lane: by 16 lanes each,
// four rows at once, where a wave holds four or more of them, else by the
// whole wave; the other rows by one lane each.  HV = false compiles that out,
// for graphs without such a row.
constexpr int HEAVY = 8;
constexpr uint32_t UNREACHED = 8, NOBODY = 16; // states; levels are 1 << (l % 3)

__host__ __device__ inline uint32_t level_bit(int32_t l) { return 1u << (l % 3); }

// Bytes of one workgroup's arrays for n vertices, K sources and `levels`
// levels: BC sums, row starts, level starts, alignment, and per entry a count,
// a queue slot and a state.
template <typename ST>
constexpr size_t bytes_for(size_t n, size_t K, size_t levels) {
    return 8 * n + 2 * (n + 1) + 2 * (levels + 2) + 32 + (sizeof(ST) + 3) * K * (n + 1);
}

// Sources a group takes: what fits, at most `want`, ids below 2^16 - 1.
template <typename ST>
__host__ __device__ inline int32_t group_size(int64_t bytes, int32_t n, int32_t levels, int32_t want) {
    const int64_t k = (bytes - (int64_t)bytes_for<ST>((size_t)n, 0, (size_t)levels)) / (int64_t)((sizeof(ST) + 3) * (n + 1));
    const int64_t ids = 65535 / (n + 1);
    const int64_t m = k < ids ? k : ids;
    return (int32_t)(m < want ? m : want);
}

template <typename ST>
struct Arrays {
    double *bc;      // [n] the unit's sums
    ST *sc;          // [K (n + 1)] counts, then c
    uint8_t *st;     // [K (n + 1)]
    uint16_t *queue; // [K (n + 1)]
    uint16_t *rp;    // [n + 1] first burst of each row
    uint16_t *lev;   // [levels + 2] level starts in the queue
    int32_t n, K, levels;
    uint32_t magic;  // id / (n + 1) = umulhi(id, magic) for id < 2^16

    __device__ Arrays(unsigned char *raw, int32_t n_, int32_t K_, int32_t levels_) : n(n_), K(K_), levels(levels_) {
        const int32_t e = K * (n + 1);
        int32_t at = 8 * n;
        bc = reinterpret_cast<double *>(raw);
        sc = reinterpret_cast<ST *>(raw + at);
        at = (at + (int32_t)sizeof(ST) * e + 15) & ~15;
        st = reinterpret_cast<uint8_t *>(raw + at);
        at = (at + e + 1) & ~1;
        queue = reinterpret_cast<uint16_t *>(raw + at);
        at += 2 * e;
        rp = reinterpret_cast<uint16_t *>(raw + at);
        at += 2 * (n + 1);
        lev = reinterpret_cast<uint16_t *>(raw + at);
        magic = 0xFFFFFFFFu / (uint32_t)(n + 1) + 1;
    }
    __device__ __forceinline__ int32_t source_of(int32_t id) const { return (int32_t)__umulhi((uint32_t)id, magic); }
};

__device__ __forceinline__ double coef(uint32_t bits) { return (double)__uint_as_float(bits); }
__device__ __forceinline__ double coef(uint64_t bits) { return __longlong_as_double((long long)bits); }
__device__ __forceinline__ void set_coef(uint32_t *p, double c) { *p = __float_as_uint((float)c); }
__device__ __forceinline__ void set_coef(uint64_t *p, double c) { *p = (uint64_t)__double_as_longlong(c); }
__device__ __forceinline__ uint32_t add_count(uint32_t *p, uint32_t x) { return atomicAdd(p, x); }
__device__ __forceinline__ uint64_t add_count(uint64_t *p, uint64_t x) {
    return atomicAdd((unsigned long long *)p, (unsigned long long)x);
}

__device__ __forceinline__ int lanes_below(uint64_t m) {
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0));
}

__device__ __forceinline__ void unpack(const uint4 c, uint32_t (&w)[BURST]) {
    const uint32_t x[4] = {c.x, c.y, c.z, c.w};
#pragma unroll
    for (int j = 0; j < BURST; ++j) w[j] = j & 1 ? x[j >> 1] >> 16 : x[j >> 1] & 0xFFFFu;
}

// The next heavy rows of a wave (bits of `heavy`, taken out), and this lane's
// part: row is the lane that holds it, at the lane's first burst in it.
struct HeavyRows {
    int rows[4], lanes, at, row;
    bool live;
    __device__ HeavyRows(uint64_t &heavy, int lane) {
        const bool many = __popcll(heavy) >= 4;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            rows[q] = -1;
            if (q == 0 || many) {
                if (heavy) rows[q] = __ffsll((unsigned long long)heavy) - 1;
                heavy &= heavy - 1;
            }
        }
        lanes = many ? 16 : 64;
        at = lane & (lanes - 1);
        const int q = many ? lane >> 4 : 0;
        row = q == 0 ? rows[0] : q == 1 ? rows[1] : q == 2 ? rows[2] : rows[3];
        live = row >= 0;
        if (!live) row = 0;
    }
};

// Where a graph's arcs are (small.hip): few in heavy rows; many, in rows far
// longer than others (hubs); many, in rows of like lengths, of twice HEAVY bursts
// or more on average (long).
enum Rows { FEW_HEAVY, HUBS, ALIKE_LONG, ALIKE };

// The entries of a level that a wave takes: its first, the step from lane to
// lane, and so on every T-th; and the bursts up to which a row is one lane's.  A
// wave's lanes have entries next to each other, whose rows are of like lengths.
// Or the workgroup's waves take turns, so that the heavy rows, which come
// together too, are dealt to all of them: where there are hubs, and at levels
// that leave waves without entries.  At other levels rows of like lengths, not
// long ones, keep a wave's lanes busy up to twice the bursts.
template <int T, bool HV>
struct Deal {
    int32_t first, step, limit;
    __device__ Deal(Rows rows, int32_t entries) {
        const bool turns = HV && (rows == HUBS || (rows >= ALIKE_LONG && entries < T / 2));
        first = turns ? threadIdx.x >> 6 : threadIdx.x & ~63u;
        step = turns ? T / 64 : 1;
        limit = HV && rows == ALIKE && entries >= T / 2 ? 2 * HEAVY : HEAVY;
    }
};

// Forward sweep of the group from sources src(0) .. src(K - 1) by the T
// threads of the workgroup; cnt[0..2] is LDS scratch.  Returns the number of
// levels, or -1 when there were more than a.levels.  *ovf in LDS is set when a
// count may have passed the range of ST.  64-bit counts: every add is tested,
// so it is set exactly when a sum wrapped.  32-bit counts: it is set when a
// vertex with a count above `safe`, that range over the largest degree, is
// expanded; no sum of smaller counts can wrap.  (Testing only the adds of
// such vertices would not do: a small count can be the one that wraps.)
template <typename ST, int T, bool HV, typename Src>
__device__ __forceinline__ int32_t forward(const Arrays<ST> &a, const uint4 *__restrict__ cols, Src src, ST safe,
                                           int32_t *cnt, uint32_t *ovf, Rows rows) {
    const int tid = threadIdx.x, lane = tid & 63;
    const int32_t n1 = a.n + 1, E = a.K * n1;
    {
        uint32_t *st4 = reinterpret_cast<uint32_t *>(a.st);
        for (int32_t i = tid; i < (E >> 2); i += T) st4[i] = 0x01010101u * UNREACHED;
        if (tid < (E & 3)) a.st[(E & ~3) + tid] = UNREACHED;
        for (int32_t i = tid; i < E; i += T) a.sc[i] = 0;
    }
    __syncthreads();
    for (int32_t k = tid; k < a.K; k += T) {
        const int32_t id = k * n1 + src(k);
        a.st[id] = 1;
        a.sc[id] = 1;
        a.queue[k] = (uint16_t)id;
        a.st[k * n1 + a.n] = NOBODY;
    }
    if (tid == 0) {
        a.lev[0] = 0;
        a.lev[1] = (uint16_t)a.K;
        cnt[0] = cnt[1] = cnt[2] = 0;
    }
    __syncthreads();
    // level L spans queue[qb, qe); its finds go to queue[qe + cnt[L % 3]].
    // Three counters let one barrier per level suffice: while level L appends
    // to cnt[L % 3], thread 0 clears cnt[(L + 1) % 3], last read before the
    // previous barrier.
    int32_t qb = 0, qe = a.K, L = 0, c0 = 0;
    while (qb < qe) {
        const int32_t c1 = c0 == 2 ? 0 : c0 + 1; // (L + 1) % 3
        const uint32_t next = 1u << c1;
        if (tid == 0) cnt[c1] = 0;
        // one burst per lane (every lane of the wave calls): the arcs to
        // `mask` states take sv, the vertices found first are appended
        auto burst = [&](const uint4 c, uint32_t mask, ST sv, int32_t base) {
            ST *sc = a.sc + base;
            uint8_t *st = a.st + base;
            uint32_t w[BURST], t[BURST];
            unpack(c, w);
#pragma unroll
            for (int j = 0; j < BURST; ++j) t[j] = st[w[j]];
            ST old[BURST];
#pragma unroll
            for (int j = 0; j < BURST; ++j) {
                old[j] = 1; // an arc not added claims nothing
                if (t[j] & mask) old[j] = add_count(&sc[w[j]], sv); // v in P_s(w)
            }
            // every add is issued before the first result is looked at
            // (256 graphs of 64..4096 vertices: 20.6 against 22.7 ms)
            __asm__ volatile("" ::: "memory");
#pragma unroll
            for (int j = 0; j < BURST; ++j) __asm__ volatile("" : "+v"(old[j]));
            if (sizeof(ST) == 8) {
                bool wrap = false;
#pragma unroll
                for (int j = 0; j < BURST; ++j) wrap |= (t[j] & mask) && (ST)(old[j] + sv) < sv;
                if (wrap) *ovf = 1;
            }
            uint64_t claim[BURST];
            int total = 0;
#pragma unroll
            for (int j = 0; j < BURST; ++j) {
                claim[j] = __ballot(old[j] == 0);
                total += __popcll(claim[j]);
            }
            if (total == 0) return;
            int32_t at = 0;
            if (lane == 0) at = atomicAdd(cnt + c0, total);
            at = qe + __builtin_amdgcn_readfirstlane(at);
            // at most one claim per entry, unless a count wrapped to zero
            // (then *ovf is set and the queue's contents do not matter)
#pragma unroll
            for (int j = 0; j < BURST; ++j) {
                if (old[j] == 0) {
                    st[w[j]] = (uint8_t)next;
                    const int32_t p = at + lanes_below(claim[j]);
                    if (p < E) a.queue[p] = (uint16_t)(base + (int32_t)w[j]);
                }
                at += __popcll(claim[j]);
            }
        };
        bool large = false;
        const Deal<T, HV> deal(rows, qe - qb);
        for (int32_t i0 = qb + deal.first; i0 < qe; i0 += T) {
            const int32_t i = i0 + lane * deal.step;
            const bool act = i < qe;
            const int32_t id = act ? (int32_t)a.queue[i] : 0;
            const int32_t base = a.source_of(id) * n1;
            const int32_t v = id - base;
            const ST sv = a.sc[id];
            int32_t b = act ? (int32_t)a.rp[v] : 0;
            const int32_t e = act ? (int32_t)a.rp[v + 1] : 0;
            large |= act && sv > safe;
            uint64_t heavy = HV ? __ballot(e - b > deal.limit) : 0;
            const bool light = !HV || e - b <= deal.limit;
            while (__any(light && b < e)) {
                const bool more = light && b < e;
                uint4 c = make_uint4(0, 0, 0, 0);
                if (more) c = cols[b++]; // a heavy row keeps its first burst
                burst(c, more ? UNREACHED | next : 0u, sv, base);
            }
            while (HV && heavy) {
                const HeavyRows r(heavy, lane);
                const int32_t hbase = __shfl(base, r.row, 64), he = r.live ? __shfl(e, r.row, 64) : 0;
                const ST hsv = __shfl(sv, r.row, 64);
                int32_t hb = __shfl(b, r.row, 64) + r.at;
                while (__any(hb < he)) {
                    const bool more = hb < he;
                    uint4 c = make_uint4(0, 0, 0, 0);
                    if (more) c = cols[hb];
                    hb += r.lanes;
                    burst(c, more ? UNREACHED | next : 0u, hsv, hbase);
                }
            }
        }
        if (sizeof(ST) == 4 && large) *ovf = 1;
        __syncthreads();
        qb = qe;
        qe = min(qe + cnt[c0], E);
        c0 = c1;
        ++L;
        if (L > a.levels) return -1;
        if (tid == 0) a.lev[L + 1] = (uint16_t)qe;
    }
    __syncthreads();
    return L;
}

// Backward sweep, deepest level first, down to level `lowest`: delta(v) =
// lambda_sv * sum of c(w) over successors w (Theorem 1.1), BC sums in LDS for
// every level but 0.  put(k, v, delta) receives every dependency.
template <typename ST, int T, bool HV, bool F32, typename Put>
__device__ __forceinline__ void backward(const Arrays<ST> &a, const uint4 *__restrict__ cols, int32_t nlev,
                                         int32_t lowest, Rows rows, Put put) {
    const int lane = threadIdx.x & 63;
    const int32_t n1 = a.n + 1;
    for (int32_t l = nlev - 1; l >= lowest; --l) {
        const uint32_t next = level_bit(l + 1);
        const int32_t lb = a.lev[l], le = a.lev[l + 1];
        // sum += c over the successors among one burst's columns
        auto burst = [&](const uint4 c, int32_t base, double &sum) {
            const ST *sc = a.sc + base;
            const uint8_t *st = a.st + base;
            uint32_t w[BURST], t[BURST];
            unpack(c, w);
#pragma unroll
            for (int j = 0; j < BURST; ++j) t[j] = st[w[j]];
            // straight-line reads, the successors selected afterwards: the
            // reads of a burst are in flight together
            ST x[BURST];
#pragma unroll
            for (int j = 0; j < BURST; ++j) x[j] = sc[w[j]];
#pragma unroll
            for (int j = 0; j < BURST; ++j) sum += coef(t[j] & next ? x[j] : (ST)0);
        };
        const Deal<T, HV> deal(rows, le - lb);
        for (int32_t i0 = lb + deal.first; i0 < le; i0 += T) {
            const int32_t i = i0 + lane * deal.step;
            const bool act = i < le;
            const int32_t id = act ? (int32_t)a.queue[i] : 0;
            const int32_t k = a.source_of(id), base = k * n1;
            const int32_t v = id - base;
            double acc = 0.0;
            if (l + 1 < nlev) {
                int32_t b = act ? (int32_t)a.rp[v] : 0;
                const int32_t e = act ? (int32_t)a.rp[v + 1] : 0;
                uint64_t heavy = HV ? __ballot(e - b > deal.limit) : 0;
                if (!HV || e - b <= deal.limit)
                    for (; b < e; ++b) burst(cols[b], base, acc);
                while (HV && heavy) {
                    const HeavyRows r(heavy, lane);
                    const int32_t hbase = __shfl(base, r.row, 64), he = r.live ? __shfl(e, r.row, 64) : 0;
                    double sum = 0.0;
                    for (int32_t hb = __shfl(b, r.row, 64) + r.at; hb < he; hb += r.lanes) burst(cols[hb], hbase, sum);
                    for (int off = r.lanes >> 1; off > 0; off >>= 1) sum += __shfl_xor(sum, off, 64);
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const double x = __shfl(sum, 16 * q, 64);
                        if (lane == r.rows[q]) acc = x;
                    }
                }
            }
            if (!act) continue;
            const double sv = (double)a.sc[id];
            const double dl = sv * acc;
            const double c = (1.0 + dl) / sv;
            set_coef(&a.sc[id], F32 ? (double)(float)c : c);
            if (l > 0 && dl != 0.0) unsafeAtomicAdd(&a.bc[v], dl);
            put(k, v, dl);
        }
        __syncthreads();
    }
}

} // namespace lds_sweep
