// Graph plan: degrees, the transposed (by-source) structure as a stable radix sort, and the
// degree-binned work lists of both aggregation directions.  Integer work only; every output
// is exactly defined, so it can be compared bit for bit.
//
// The paper keeps CSR for the forward pass and observes that CSC suits the backward pass
// ("Training for GNNs") and that per-batch format translation is pure overhead ("Graph
// simulation approach" and the kernel breakdown of its evaluation); here the translation is
// done once per graph and reused by every layer and epoch.
#include <stdarg.h>
#include <stdio.h>
#include <new>

#include "gt_internal.h"
#include "gt_prims.h"

// ---------------------------------------------------------------------------------------------
// status / error plumbing
// ---------------------------------------------------------------------------------------------
static thread_local char g_err[512] = "";

void gt_set_error(const char *fmt, ...) {
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(g_err, sizeof(g_err), fmt, ap);
    va_end(ap);
}

gt_status gt_fail(gt_status s, const char *fmt, ...) {
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(g_err, sizeof(g_err), fmt, ap);
    va_end(ap);
    return s;
}

gt_status gt_hip_fail(hipError_t e, const char *what) {
    snprintf(g_err, sizeof(g_err), "HIP error %d (%s) at %s", (int)e, hipGetErrorString(e), what);
    return GT_ERR_HIP;
}

extern "C" const char *gt_last_error(void) { return g_err; }

extern "C" const char *gt_status_string(gt_status s) {
    switch (s) {
        case GT_OK: return "GT_OK";
        case GT_ERR_INVALID_ARG: return "GT_ERR_INVALID_ARG";
        case GT_ERR_UNSUPPORTED: return "GT_ERR_UNSUPPORTED";
        case GT_ERR_WORKSPACE: return "GT_ERR_WORKSPACE";
        case GT_ERR_HIP: return "GT_ERR_HIP";
        case GT_ERR_INTERNAL: return "GT_ERR_INTERNAL";
    }
    return "GT_ERR_UNKNOWN";
}

extern "C" const char *gt_version(void) { return "gt 0.1 (gfx950)"; }

namespace {

// ---------------------------------------------------------------------------------------------
// plan kernels
// ---------------------------------------------------------------------------------------------
constexpr int PT = 256;
inline unsigned nblocks(int64_t n, int per = PT) { return (unsigned)((n + per - 1) / per); }

// Row of every entry of a CSR, written coalesced, and (square graphs) the symmetric-norm coefficient
// w_e / sqrt(d(src) d(dst)) of every entry in the given order.  A workgroup takes ROWS_TILE consecutive entries: it finds the
// row of its first entry by a 64-way search, marks in LDS where the rows of its range begin, and fills in between with a running
// maximum.  (Looking up the row of each transposed entry by binary search over rowptr instead, 20 dependent loads
// per entry, took 1.70 ms on 1 M vertices and 25 M entries; this takes 0.16 and the pass below 0.16.)  Both passes are bound by one random read of a
// vertex's degree per entry: what they stream goes past the caches, which keeps the degrees in the L2s (188 -> 157 us and 198 -> 161).  Where a tile spans more
// than ROWS_WALK rows, almost all of them empty, walking them would be one workgroup's work of the whole launch
// (16 M rows, 100,000 entries in the first and last 200: plan 24.7 ms walked, 1.2 searched): its entries are searched for instead, a thread's eight at a time.
constexpr int ROWS_PER = 8, ROWS_TILE = PT * ROWS_PER, ROWS_WALK = 32768;
__global__ void __launch_bounds__(PT) k_entry_rows(const int32_t *rowptr, int64_t n_rows, int64_t E, const int32_t *colidx,
                                                   const float *ew, const float *dinv, int32_t *row_of, float *coef_sym) {
    __shared__ int32_t mark[ROWS_TILE];
    __shared__ int32_t wmax[PT / 64];
    __shared__ int64_t bound_row[2];
    const int64_t base = (int64_t)blockIdx.x * ROWS_TILE;
    const int64_t end = base + ROWS_TILE < E ? base + ROWS_TILE : E;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
    for (int i = 0; i < ROWS_PER; ++i) mark[i * PT + threadIdx.x] = -1;
    if (wave < 2) {   // the last row r with rowptr[r] <= at, for the first and the last entry of the tile
        const int64_t at = wave == 0 ? base : end - 1;
        int64_t lo = 0, hi = n_rows;
        while (hi - lo > 1) {
            const int64_t step = (hi - lo + 63) / 64;
            const int64_t r = lo + (lane + 1) * step;          // 64 ascending probes, the last at or past hi
            const bool le = r < hi && (int64_t)rowptr[r] <= at;
            const int k = __popcll(__ballot(le));              // probes 1..k are <= at
            const int64_t nlo = lo + k * step, nhi = lo + (k + 1) * step;
            lo = nlo;
            hi = nhi < hi ? nhi : hi;
        }
        if (lane == 0) bound_row[wave] = lo;
    }
    __syncthreads();
    const int64_t r0 = bound_row[0], r1 = bound_row[1];
    if (r1 - r0 > ROWS_WALK) {   // uniform over the workgroup
        int64_t lo[ROWS_PER];
#pragma unroll
        for (int i = 0; i < ROWS_PER; ++i) lo[i] = r0;
        for (int64_t len = r1 - r0 + 1; len > 1;) {   // the row is among lo .. lo + len - 1
            const int64_t half = len / 2;
#pragma unroll
            for (int i = 0; i < ROWS_PER; ++i)
                if ((int64_t)rowptr[lo[i] + half] <= base + i * PT + threadIdx.x) lo[i] += half;
            len -= half;
        }
#pragma unroll
        for (int i = 0; i < ROWS_PER; ++i) mark[i * PT + threadIdx.x] = (int32_t)lo[i];   // read back by this thread only
    } else {
        if (threadIdx.x == 0) mark[0] = (int32_t)r0;
        __syncthreads();
        // rows that begin inside the tile; of several rows beginning at one entry (empty ones) the last owns it
#pragma unroll 4
        for (int64_t r = r0 + 1 + threadIdx.x; r <= r1; r += PT) {
            const int64_t s = rowptr[r];
            if (s >= base && s < end) atomicMax(&mark[s - base], (int32_t)r);
        }
        __syncthreads();
        int32_t v[ROWS_PER], mx = -1;
#pragma unroll
        for (int i = 0; i < ROWS_PER; ++i) {
            mx = max(mx, mark[threadIdx.x * ROWS_PER + i]);
            v[i] = mx;
        }
        int32_t inc = mx;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const int32_t x = __shfl_up(inc, o, 64);
            if (lane >= o) inc = max(inc, x);
        }
        if (lane == 63) wmax[wave] = inc;
        int32_t pre = __shfl_up(inc, 1, 64);
        if (lane == 0) pre = -1;
        __syncthreads();
        for (int w = 0; w < wave; ++w) pre = max(pre, wmax[w]);
#pragma unroll
        for (int i = 0; i < ROWS_PER; ++i) mark[threadIdx.x * ROWS_PER + i] = max(v[i], pre);
        __syncthreads();
    }
#pragma unroll
    for (int i = 0; i < ROWS_PER; ++i) {
        const int64_t e = base + i * PT + threadIdx.x;
        if (e >= end) continue;
        const int32_t r = mark[i * PT + threadIdx.x];
        __builtin_nontemporal_store(r, row_of + e);
        if (dinv) __builtin_nontemporal_store(((ew ? ew[e] : 1.0f) * dinv[__builtin_nontemporal_load(colidx + e)]) * dinv[r], coef_sym + e);
    }
}

// rowptr_t from the sorted source keys (rowptr_t[u] = first position whose key >= u), and per transposed entry k (position e = perm[k] in
// the given CSR, source u = skeys[k]): its destination, its weight, and the per-entry coefficients of the normalised reduce modes in this order:
//   symmetric norm  w_e / sqrt(d(src) d(dst))   (coef_sym_b[k]; square graphs)
//   mean, backward  w_e / indeg(dst)            (coef_mean_b[k])
// row_of null: the destinations have travelled through the sort and are in colidx_t already (looking each one up by its
// entry is a random 4-byte read from an array of E: 25 M entries 0.51 ms, carried along 0.28 ms more in the sort).
// A thread has four consecutive entries (25 M entries, with the row ends, which had a launch of their own, 212 -> 186 us).
__global__ void __launch_bounds__(PT) k_transposed_entries(const int32_t *perm, const uint32_t *skeys, const int32_t *row_of, int64_t E, int64_t n_src,
                                                           const float *ew, const int32_t *in_deg, int square, int32_t *rowptr_t, int32_t *colidx_t,
                                                           float *ew_t, float *coef_sym_b, float *coef_mean_b) {
    const int lane = threadIdx.x & 63;
    const int64_t k0 = ((int64_t)blockIdx.x * PT + threadIdx.x) * 4;
    const bool whole = k0 + 4 <= E;   // (all arrays are aligned)
    uint32_t u[4];
    if (whole) {
        typedef uint32_t u4 __attribute__((ext_vector_type(4)));
        const u4 x = __builtin_nontemporal_load(reinterpret_cast<const u4 *>(skeys + k0));
        u[0] = x.x; u[1] = x.y; u[2] = x.z; u[3] = x.w;
    } else {
#pragma unroll
        for (int i = 0; i < 4; ++i) u[i] = k0 + i < E ? skeys[k0 + i] : 0u;
    }
    // position k closes the gap (key[k-1], key[k]]; k == E closes (key[E-1], n_src].  Short gaps by their own thread, long ones (runs of
    // vertices without out-edges) by the whole wavefront; lanes past E stay for the exchanges
    int64_t lo = (int64_t)(uint32_t)__shfl_up((int)u[3], 1, 64);
    if (k0 == 0) lo = -1;
    else if (lane == 0 && k0 <= E) lo = skeys[k0 - 1];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int64_t k = k0 + i, hi = k < E ? (int64_t)u[i] : k == E ? n_src : lo;   // (past E: no gap)
        if (hi - lo <= 4)
            for (int64_t r = lo + 1; r <= hi; ++r) rowptr_t[r] = (int32_t)k;
        for (uint64_t m = __ballot(hi - lo > 4); m; m &= m - 1) {
            const int l = __ffsll((unsigned long long)m) - 1;
            const int64_t a = __shfl(lo, l), b = __shfl(hi, l), kk = __shfl(k, l);
            for (int64_t r = a + 1 + lane; r <= b; r += 64) rowptr_t[r] = (int32_t)kk;
        }
        lo = hi;
    }
    if (k0 >= E) return;
    int32_t v[4];
    float w[4] = {1.0f, 1.0f, 1.0f, 1.0f}, cs[4], cm[4];
    if (!row_of && whole) {
        typedef int32_t i4 __attribute__((ext_vector_type(4)));
        const i4 x = __builtin_nontemporal_load(reinterpret_cast<const i4 *>(colidx_t + k0));
        v[0] = x.x; v[1] = x.y; v[2] = x.z; v[3] = x.w;
    } else {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            v[i] = 0;
            if (k0 + i >= E) continue;
            v[i] = row_of ? row_of[perm[k0 + i]] : colidx_t[k0 + i];
            if (row_of) colidx_t[k0 + i] = v[i];
        }
    }
    if (ew_t) {
#pragma unroll
        for (int i = 0; i < 4; ++i)
            if (k0 + i < E) ew_t[k0 + i] = w[i] = ew[perm[k0 + i]];
    }
    // (the reciprocals from the degree, as k_row_counts forms them: one gather per vertex instead of two)
    int32_t d[4], du[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        d[i] = in_deg[v[i]];
        du[i] = square ? in_deg[u[i]] : 0;
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const float iu = du[i] > 0 ? 1.0f / sqrtf((float)du[i]) : 0.0f, iv = d[i] > 0 ? 1.0f / sqrtf((float)d[i]) : 0.0f;
        cs[i] = (w[i] * iu) * iv;
        cm[i] = w[i] * (d[i] > 0 ? 1.0f / (float)d[i] : 0.0f);
    }
    if (whole) {
        typedef float f4 __attribute__((ext_vector_type(4)));
        if (square) __builtin_nontemporal_store(f4{cs[0], cs[1], cs[2], cs[3]}, reinterpret_cast<f4 *>(coef_sym_b + k0));
        __builtin_nontemporal_store(f4{cm[0], cm[1], cm[2], cm[3]}, reinterpret_cast<f4 *>(coef_mean_b + k0));
    } else {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            if (k0 + i >= E) continue;
            if (square) coef_sym_b[k0 + i] = cs[i];
            coef_mean_b[k0 + i] = cm[i];
        }
    }
}

// per row: degree (with its reciprocal and reciprocal square root where wanted) and item / partial / split / long-item counts.  The call for
// the given CSR (other null) clears max_len[0..1]; the one for the transposed structure finds the longest split row of both directions
// (other: the given CSR's n_other degrees), the given one's first, where asked (else both stay 0).  (An integer maximum: its value does not depend on the order.)
__global__ void k_row_counts(const int32_t *rowptr, int64_t n_rows, int chunk, int long_min, int32_t *deg, float *rdeg, float *dinv,
                             int32_t *c_items, int32_t *c_parts, int32_t *c_splits, int32_t *c_long, int32_t *max_len, const int32_t *other,
                             int64_t n_other) {
    const int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (!other) {
        if (r < 2) max_len[r] = 0;   // (again by the second call where nobody asks)
    } else {
        int32_t mx[2] = {r < n_other ? other[r] : 0, r < n_rows ? rowptr[r + 1] - rowptr[r] : 0};
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            if (__ballot(mx[k] > chunk + chunk / 2) == 0) continue;
#pragma unroll
            for (int o = 1; o < 64; o <<= 1) mx[k] = max(mx[k], __shfl_xor(mx[k], o, 64));
            // (most wavefronts find a longer one there already)
            if ((threadIdx.x & 63) == 0 && mx[k] > __hip_atomic_load(&max_len[k], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
                atomicMax(&max_len[k], mx[k]);
        }
    }
    if (r > n_rows) return;
    if (r == n_rows) {   // the extra entry makes the exclusive scans end with the totals
        c_items[r] = 0; c_parts[r] = 0; c_splits[r] = 0; c_long[r] = 0;
        return;
    }
    const int32_t d = rowptr[r + 1] - rowptr[r];
    deg[r] = d;
    if (rdeg) rdeg[r] = d > 0 ? 1.0f / (float)d : 0.0f;
    if (dinv) dinv[r] = d > 0 ? 1.0f / sqrtf((float)d) : 0.0f;
    const bool split = d > chunk + chunk / 2;
    const int32_t chunks = (d + chunk - 1) / chunk;
    c_items[r] = split ? chunks : 1;
    c_parts[r] = split ? chunks : 0;
    c_splits[r] = split ? 1 : 0;
    // a split row's chunks are whole (long) except possibly the last
    c_long[r] = split ? chunks - (d - (chunks - 1) * chunk < long_min ? 1 : 0) : (d >= long_min ? 1 : 0);
}

struct CountArrays { const int32_t *c[8]; };   // forward: items, partials, splits, long items; transposed: the same
__global__ void k_collect_counts(const CountArrays a, int64_t n_dst, int64_t n_src, int32_t *cnt8) {
    if (threadIdx.x < 8) cnt8[threadIdx.x] = a.c[threadIdx.x][threadIdx.x < 4 ? n_dst : n_src];
}

__device__ inline uint32_t length_key(int32_t len) {
    // Descending-length sort key, half-octave resolution (exact below 4).  Measured on MI355X with
    // quarter-octave, half-octave and octave classes: coarser classes leave more of the order to
    // the locality key (better L2 reuse), finer ones balance the groups of a wavefront better;
    // half an octave was the best or within 2 % of it on every width of configs 2 and 3.
    uint32_t k;
    if (len < 4) {
        k = (uint32_t)len;
    } else {
        const int lg = 31 - __clz(len);
        k = 4u + (uint32_t)(lg - 2) * 2u + (((uint32_t)len >> (lg - 1)) & 1u);
    }
    return 255u - k;
}

// Sort key of an item: length class (longest first) in bits 8-15, then the range its MEDIAN
// neighbour id falls in (256 ranges) in bits 0-7, so that items running at the same time gather
// from the same region of the table and reuse each other's rows in the L2.  (Rows are sorted by
// neighbour id; on power-law graphs the first neighbour is a hub for almost every row and tells
// little, the median separates rows much better: config 3, width 256, 3.47 -> 3.27 ms.)
__device__ inline uint32_t item_key(int32_t len, const int32_t *nbr, int32_t e0, int64_t n_in) {
    uint32_t loc = 0;
    if (len > 0 && n_in > 0) loc = (uint32_t)(((int64_t)nbr[e0 + len / 2] << 8) / n_in) & 255u;
    return (length_key(len) << 8) | loc;
}

__device__ inline void fill_items(const int32_t *rowptr, const int32_t *nbr, int64_t n_in, int64_t n_rows, int chunk,
                                  const int32_t *o_items, const int32_t *o_parts, const int32_t *o_splits, const int32_t *o_long,
                                  int long_min, int64_t n_long, gt_item *items, uint32_t *keys, gt_split *splits) {
    const int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const bool in = r < n_rows;   // (all lanes stay for the exchanges below)
    const int32_t b = in ? rowptr[r] : 0, e = in ? rowptr[r + 1] : 0, d = e - b;
    // long items first (their order among themselves and that of the others stays the row order)
    const int32_t it_long = in ? o_long[r] : 0, it_short = in ? (int32_t)n_long + o_items[r] - it_long : 0;
    const bool split = d > chunk + chunk / 2;
    const int32_t chunks = split ? (d + chunk - 1) / chunk : 0, p0 = split ? o_parts[r] : 0;
    // The chunks of all split rows of a wavefront are shared out over its lanes, whatever rows they belong to: a hub row has
    // hundreds, each with a dependent read of its median neighbour (one thread alone was the kernel's whole time), and 64 rows of
    // a few chunks each would be 64 turns if taken one after the other (255 rows, 50,000 edges: plan 164 us that way, 97 this way).
    const int lane = threadIdx.x & 63;
    int32_t upto = chunks;   // chunks of the rows up to this lane's
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int32_t x = __shfl_up(upto, o, 64);
        if (lane >= o) upto += x;
    }
    const int32_t total = __shfl(upto, 63, 64);
    for (int32_t i0 = 0; i0 < total; i0 += 64) {
        const int32_t i = i0 + lane;
        int l = 0;   // the first lane with upto > i
#pragma unroll
        for (int step = 32; step > 0; step >>= 1)
            if (__shfl(upto, l + step - 1, 64) <= i) l += step;
        const int32_t row = __shfl((int32_t)r, l), rb = __shfl(b, l), re = __shfl(e, l), rp = __shfl(p0, l);
        const int32_t al = __shfl(it_long, l), as = __shfl(it_short, l), c = i - (__shfl(upto, l) - __shfl(chunks, l));
        if (i < total) {
            gt_item x;
            x.row = row;
            x.e0 = rb + c * chunk;
            x.e1 = min(re, x.e0 + chunk);
            x.slot = rp + c;
            const int32_t at = x.e1 - x.e0 >= long_min ? al + c : as;   // (only the last chunk may be short)
            items[at] = x;
            if (keys) keys[at] = item_key(x.e1 - x.e0, nbr, x.e0, n_in);
        }
    }
    if (!in) return;
    if (split) {
        gt_split s;
        s.row = (int32_t)r; s.first = p0; s.count = chunks; s.pad = 0;
        splits[o_splits[r]] = s;
    } else {
        gt_item x;
        x.row = (int32_t)r; x.e0 = b; x.e1 = e; x.slot = -1;
        const int32_t at = d >= long_min ? it_long : it_short;
        items[at] = x;
        if (keys) keys[at] = item_key(d, nbr, b, n_in);
    }
}

__global__ void k_fill_items(const int32_t *rowptr, const int32_t *nbr, int64_t n_in, int64_t n_rows, int chunk,
                             const int32_t *o_items, const int32_t *o_parts, const int32_t *o_splits, const int32_t *o_long,
                             int long_min, int64_t n_long, gt_item *items, uint32_t *keys, gt_split *splits) {
    fill_items(rowptr, nbr, n_in, n_rows, chunk, o_items, o_parts, o_splits, o_long, long_min, n_long, items, keys, splits);
}

// Both directions of a plan whose lists stay in row order (see build_direction), before the host has read their sizes: the number of long items
// comes from the counts, lists past their bound are not written (the host then refuses the graph), and the first workgroup leaves the
// sizes for the read-back.  One launch and one synchronisation instead of three and two (a batch of 300 seeds, two plans, 589 us with those, 555 this way).
struct FillDirection {
    const int32_t *rowptr;
    int64_t n_rows, max_items;
    const int32_t *o_items, *o_parts, *o_splits, *o_long;
    gt_item *items;
    gt_split *splits;
};
__global__ void k_fill_both(const FillDirection f, const FillDirection b, int chunk, int long_min, int64_t max_splits, int32_t *cnt8) {
    if (blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x < 8) {
        const FillDirection &d = threadIdx.x < 4 ? f : b;
        const int k = threadIdx.x & 3;
        cnt8[threadIdx.x] = (k == 0 ? d.o_items : k == 1 ? d.o_parts : k == 2 ? d.o_splits : d.o_long)[d.n_rows];
    }
    const FillDirection &d = blockIdx.y ? b : f;
    if (d.o_items[d.n_rows] > d.max_items || d.o_splits[d.n_rows] > max_splits) return;   // whole grid rows
    fill_items(d.rowptr, nullptr, 0, d.n_rows, chunk, d.o_items, d.o_parts, d.o_splits, d.o_long, long_min, d.o_long[d.n_rows], d.items, nullptr, d.splits);
}

__global__ void k_gather_items(const gt_item *src, const uint32_t *idx, int64_t n, gt_item *dst) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) dst[i] = src[idx[i]];
}

__global__ void k_validate(const int32_t *rowptr, const int32_t *colidx, int64_t n_dst, int64_t n_src, int64_t E,
                           unsigned long long *bad) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    unsigned long long v = 0;
    if (i < n_dst && rowptr[i + 1] < rowptr[i]) v++;
    if (i == 0 && rowptr[0] != 0) v++;
    if (i == 0 && (int64_t)rowptr[n_dst] != E) v++;
    if (i < E && (colidx[i] < 0 || (int64_t)colidx[i] >= n_src)) v++;
    if (v) atomicAdd(bad, v);   // integer atomic: the count does not depend on the order
}

// ---------------------------------------------------------------------------------------------
// workspace layout
// ---------------------------------------------------------------------------------------------
struct PlanLayout {
    size_t in_deg, out_deg, rowptr_t, colidx_t, perm, ew_t, dinv, rdeg;
    size_t items_f, splits_f, items_b, splits_b;
    size_t counts;                       // 10 int32 read back by the host
    size_t ca, cb, cc, cd;               // per-row count arrays (max(n_dst, n_src) + 1 each), forward direction
    size_t ca2, cb2, cc2, cd2;           // the same for the transposed direction
    size_t items_tmp, item_keys, item_keys2, item_idx, item_idx2;   // unsorted items, sort keys / indices
    size_t k0, k1, v1, e1;               // sort ping-pong (E each), with perm and colidx_t as the other halves of v1 and e1;
                                         // one of k0 / k1 (not the sorted keys), and v1, hold coefficients afterwards
    size_t coef_f;                       // symmetric-norm coefficients of the given order
    size_t hist, scan_tmp;
    size_t total;
};

int64_t max_items(int64_t n_rows, int64_t E) { return n_rows + E / gt_chunk_for(E) + 1; }
int64_t max_splits(int64_t E) { return E / gt_split_min(gt_chunk_for(E)) + 1; }

PlanLayout plan_layout(int64_t n_dst, int64_t n_src, int64_t E, bool has_ew) {
    PlanLayout L{};
    size_t off = 0;
    auto take = [&](size_t bytes) { size_t o = off; off += gt_align_up(bytes ? bytes : 4); return o; };
    const int64_t nmax = (n_dst > n_src ? n_dst : n_src);
    const int64_t imax = max_items(nmax, E);
    L.in_deg = take((size_t)n_dst * 4);
    L.out_deg = take((size_t)n_src * 4);
    L.rowptr_t = take((size_t)(n_src + 1) * 4);
    L.colidx_t = take((size_t)E * 4);
    L.perm = take((size_t)E * 4);
    L.ew_t = take(has_ew ? (size_t)E * 4 : 0);
    L.dinv = take((size_t)nmax * 4);
    L.rdeg = take((size_t)n_dst * 4);
    L.items_f = take((size_t)max_items(n_dst, E) * sizeof(gt_item));
    L.splits_f = take((size_t)max_splits(E) * sizeof(gt_split));
    L.items_b = take((size_t)max_items(n_src, E) * sizeof(gt_item));
    L.splits_b = take((size_t)max_splits(E) * sizeof(gt_split));
    L.counts = take(128);
    L.ca = take((size_t)(nmax + 1) * 4);
    L.cb = take((size_t)(nmax + 1) * 4);
    L.cc = take((size_t)(nmax + 1) * 4);
    L.cd = take((size_t)(nmax + 1) * 4);
    L.ca2 = take((size_t)(nmax + 1) * 4);
    L.cb2 = take((size_t)(nmax + 1) * 4);
    L.cc2 = take((size_t)(nmax + 1) * 4);
    L.cd2 = take((size_t)(nmax + 1) * 4);
    L.items_tmp = take((size_t)imax * sizeof(gt_item));
    L.item_keys = take((size_t)imax * 4);
    L.item_keys2 = take((size_t)imax * 4);
    L.item_idx = take((size_t)imax * 4);
    L.item_idx2 = take((size_t)imax * 4);
    L.k0 = take((size_t)E * 4);
    L.k1 = take((size_t)E * 4);
    L.v1 = take((size_t)E * 4);
    L.e1 = take((size_t)E * 4);
    L.coef_f = take(n_dst == n_src ? (size_t)E * 4 : 0);
    const int64_t nsort = E > imax ? E : imax;
    const int64_t hist_n = (int64_t)rs_hist_ints(nsort);
    L.hist = take((size_t)hist_n * 4);
    const size_t scan_h = scan_tmp_ints(hist_n), scan_c = 8 * scan_tmp_ints(nmax + 1);
    L.scan_tmp = take((scan_h > scan_c ? scan_h : scan_c) * 4);
    L.total = off;
    return L;
}

template <typename T>
T *at(void *ws, size_t off) { return reinterpret_cast<T *>(static_cast<char *>(ws) + off); }

// items of one direction, sorted longest first (stable, so equal lengths keep row order).
constexpr int64_t GT_SORT_ITEMS_MIN = 16384;
constexpr int64_t GT_ASK_MAX_EDGES = (int64_t)4 << 20;   // larger graphs do not ask for their longest split row (25 M edges: 30 us)
gt_status build_direction(const int32_t *rowptr, const int32_t *nbr, int64_t n_in, int64_t n_rows, int chunk,
                          int64_t n_items, int64_t n_long, void *ws, const PlanLayout &L, bool transposed, gt_item *items_out,
                          gt_split *splits_out, hipStream_t st) {
    if (n_rows <= 0 || n_items <= 0) return GT_OK;
    int32_t *ca = at<int32_t>(ws, transposed ? L.ca2 : L.ca), *cb = at<int32_t>(ws, transposed ? L.cb2 : L.cb);
    int32_t *cc = at<int32_t>(ws, transposed ? L.cc2 : L.cc), *cd = at<int32_t>(ws, transposed ? L.cd2 : L.cd);
    gt_item *tmp = at<gt_item>(ws, L.items_tmp);
    uint32_t *keys = at<uint32_t>(ws, L.item_keys), *keys2 = at<uint32_t>(ws, L.item_keys2);
    uint32_t *idx = at<uint32_t>(ws, L.item_idx), *idx2 = at<uint32_t>(ws, L.item_idx2);
    // A small graph is bound by launch latency, not by load balance or locality: its items stay in
    // row order (long ones first) and the two sort passes and the gather are saved.
    const bool sorted = n_items > GT_SORT_ITEMS_MIN;
    k_fill_items<<<nblocks(n_rows), PT, 0, st>>>(rowptr, nbr, n_in, n_rows, chunk, ca, cb, cc, cd, gt_long_min(chunk), n_long,
                                                 sorted ? tmp : items_out, keys, splits_out);
    GT_LAUNCH_CHECK("k_fill_items");
    if (!sorted) return GT_OK;
    SortTmp t{at<int32_t>(ws, L.hist), at<int32_t>(ws, L.scan_tmp)};
    gt_status s = radix_pass(keys, nullptr, keys2, idx, n_items, 0, 8, t, st);      // neighbour range
    if (s != GT_OK) return s;
    s = radix_pass(keys2, idx, keys, idx2, n_items, 8, 8, t, st);                   // length class (stable)
    if (s != GT_OK) return s;
    k_gather_items<<<nblocks(n_items), PT, 0, st>>>(tmp, idx2, n_items, items_out);
    GT_LAUNCH_CHECK("k_gather_items");
    return GT_OK;
}

}  // namespace

// ---------------------------------------------------------------------------------------------
// C ABI
// ---------------------------------------------------------------------------------------------
extern "C" gt_status gt_graph_plan_size(int64_t n_dst, int64_t n_src, int64_t n_edges, int has_edge_weight,
                                        size_t *ws_bytes) {
    if (!ws_bytes) return gt_fail(GT_ERR_INVALID_ARG, "gt_graph_plan_size: ws_bytes is null");
    if (n_dst < 0 || n_src < 0 || n_edges < 0) return gt_fail(GT_ERR_INVALID_ARG, "gt_graph_plan_size: negative size");
    // int32 indices everywhere; the kernels step through an entry list in strides of up to 512 and
    // look one stride ahead, so the largest entry index plus two strides must still fit an int32
    const int64_t lim = 2147483648LL - 1024;
    if (n_dst >= lim || n_src >= lim || n_edges >= lim)
        return gt_fail(GT_ERR_UNSUPPORTED, "gt_graph_plan_size: sizes must be below 2^31 - 1024 (int32 indices)");
    *ws_bytes = plan_layout(n_dst, n_src, n_edges, has_edge_weight != 0).total;
    return GT_OK;
}

extern "C" gt_status gt_graph_create(gt_graph **out, int64_t n_dst, int64_t n_src, int64_t E, const int32_t *rowptr,
                                     const int32_t *colidx, const float *ew, void *ws, size_t ws_bytes, void *stream) {
    if (!out) return gt_fail(GT_ERR_INVALID_ARG, "gt_graph_create: g is null");
    *out = nullptr;
    size_t need = 0;
    gt_status s = gt_graph_plan_size(n_dst, n_src, E, ew != nullptr, &need);
    if (s != GT_OK) return s;
    if (!rowptr) return gt_fail(GT_ERR_INVALID_ARG, "gt_graph_create: rowptr is null");
    if (E > 0 && !colidx) return gt_fail(GT_ERR_INVALID_ARG, "gt_graph_create: colidx is null with n_edges > 0");
    if (E > 0 && n_src == 0) return gt_fail(GT_ERR_INVALID_ARG, "gt_graph_create: edges but n_src == 0");
    if (E > 0 && n_dst == 0) return gt_fail(GT_ERR_INVALID_ARG, "gt_graph_create: edges but n_dst == 0");
    if (!ws || ((uintptr_t)ws & 255)) return gt_fail(GT_ERR_WORKSPACE, "gt_graph_create: ws null or not 256-byte aligned");
    if (ws_bytes < need) return gt_fail(GT_ERR_WORKSPACE, "gt_graph_create: ws_bytes %zu < required %zu", ws_bytes, need);
    hipStream_t st = (hipStream_t)stream;
    const PlanLayout L = plan_layout(n_dst, n_src, E, ew != nullptr);

    gt_graph *g = new (std::nothrow) gt_graph();
    if (!g) return gt_fail(GT_ERR_INTERNAL, "gt_graph_create: out of host memory");
    g->n_dst = n_dst; g->n_src = n_src; g->n_edges = E;
    g->rowptr = rowptr; g->colidx = colidx; g->ew = ew;
    g->in_deg = at<int32_t>(ws, L.in_deg);
    g->out_deg = at<int32_t>(ws, L.out_deg);
    g->rowptr_t = at<int32_t>(ws, L.rowptr_t);
    g->colidx_t = at<int32_t>(ws, L.colidx_t);
    g->perm = at<int32_t>(ws, L.perm);
    g->ew_t = ew ? at<float>(ws, L.ew_t) : nullptr;
    g->dinv = (n_dst == n_src) ? at<float>(ws, L.dinv) : nullptr;
    g->rdeg = at<float>(ws, L.rdeg);
    g->vcount = at<unsigned long long>(ws, L.counts + 64);

    auto fail = [&](gt_status rc) { delete g; return rc; };
#define PLAN_HIP(call) do { hipError_t e__ = (call); if (e__ != hipSuccess) return fail(gt_hip_fail(e__, #call)); } while (0)
#define PLAN_LAUNCH(what) do { hipError_t e__ = hipGetLastError(); if (e__ != hipSuccess) return fail(gt_hip_fail(e__, what)); } while (0)

    const int chunk = gt_chunk_for(E), long_min = gt_long_min(chunk);
    g->chunk = chunk;
    int32_t *ca = at<int32_t>(ws, L.ca), *cb = at<int32_t>(ws, L.cb), *cc = at<int32_t>(ws, L.cc), *cd = at<int32_t>(ws, L.cd);
    int32_t *ca2 = at<int32_t>(ws, L.ca2), *cb2 = at<int32_t>(ws, L.cb2), *cc2 = at<int32_t>(ws, L.cc2), *cd2 = at<int32_t>(ws, L.cd2);
    int32_t *d_counts = at<int32_t>(ws, L.counts);
    // degrees and work-list counts of the given CSR
    k_row_counts<<<nblocks(n_dst + 1), PT, 0, st>>>(rowptr, n_dst, chunk, long_min, g->in_deg, g->rdeg, g->dinv, ca, cb, cc, cd, d_counts + 8,
                                                nullptr, 0);
    PLAN_LAUNCH("k_row_counts");
    // transposed structure: stable sort of (source, position) pairs by source.  A sort that runs pass by pass carries the
    // entries' destinations along; the one-launch sort of a short list has its LDS full with the pairs.
    SortTmp t{at<int32_t>(ws, L.hist), at<int32_t>(ws, L.scan_tmp)};
    uint32_t *k0 = at<uint32_t>(ws, L.k0), *k1 = at<uint32_t>(ws, L.k1);
    uint32_t *v1 = at<uint32_t>(ws, L.v1), *e1 = at<uint32_t>(ws, L.e1);
    const bool carry = E > RS_ONE_MAX;
    int32_t *row_of = reinterpret_cast<int32_t *>(e1);
    uint32_t *sorted_keys = nullptr;
    if (E > 0) {
        g->coef_sym_f = g->dinv ? at<float>(ws, L.coef_f) : nullptr;
        int bits = 1;
        while (bits < 32 && ((int64_t)1 << bits) < n_src) ++bits;
        const int passes = (bits + 7) / 8;
        // values go back and forth between perm and v1, destinations between colidx_t and e1, so that the last pass writes perm and
        // colidx_t; the first pass reads the destinations from the buffer that it does not write
        uint32_t *const pv[2] = {reinterpret_cast<uint32_t *>(g->perm), v1}, *const pe[2] = {reinterpret_cast<uint32_t *>(g->colidx_t), e1};
        if (carry) row_of = reinterpret_cast<int32_t *>(pe[passes & 1]);
        k_entry_rows<<<nblocks(E, ROWS_TILE), PT, 0, st>>>(rowptr, n_dst, E, colidx, ew, g->dinv, row_of, g->coef_sym_f);
        PLAN_LAUNCH("k_entry_rows");
        const uint32_t *kin = reinterpret_cast<const uint32_t *>(colidx);
        const uint32_t *vin = nullptr, *ein = carry ? reinterpret_cast<const uint32_t *>(row_of) : nullptr;
        SortPasses sp{};
        sp.passes = passes;
        sp.bits = bits;
        for (int p = 0; p < passes; ++p) {
            const int other = (passes - 1 - p) & 1;
            sp.kin[p] = kin; sp.vin[p] = vin; sp.ein[p] = ein;
            sorted_keys = sp.kout[p] = (p & 1) ? k1 : k0;
            sp.vout[p] = pv[other];
            sp.eout[p] = carry ? pe[other] : nullptr;
            kin = sp.kout[p]; vin = sp.vout[p]; ein = sp.eout[p];
        }
        if ((s = radix_sort(sp, E, t, st)) != GT_OK) return fail(s);
    }
    // the sort's ping-pong buffers are dead from here on, except the sorted keys: v1 and the other key buffer hold coefficients
    g->coef_sym_b = g->dinv && E > 0 ? reinterpret_cast<float *>(v1) : nullptr;
    g->coef_mean_b = E > 0 ? reinterpret_cast<float *>(sorted_keys == k0 ? k1 : k0) : nullptr;
    k_transposed_entries<<<nblocks(E + 1, 4 * PT), PT, 0, st>>>(g->perm, sorted_keys, carry ? nullptr : row_of, E, n_src, ew, g->in_deg, g->dinv ? 1 : 0,
                                                                g->rowptr_t, g->colidx_t, g->ew_t, g->coef_sym_b, g->coef_mean_b);
    PLAN_LAUNCH("k_transposed_entries");
    k_row_counts<<<nblocks((n_src > n_dst ? n_src : n_dst) + 1), PT, 0, st>>>(g->rowptr_t, n_src, chunk, long_min, g->out_deg, nullptr, nullptr, ca2, cb2, cc2,
                                                                              cd2, d_counts + 8, E <= GT_ASK_MAX_EDGES ? g->in_deg : nullptr, n_dst);
    PLAN_LAUNCH("k_row_counts(out)");
    // work-list sizes of both directions: the exclusive scans over n_rows + 1 entries (last input 0) leave the totals in element
    // n_rows; read back once
    const bool in_row_order = max_items(n_dst, E) <= GT_SORT_ITEMS_MIN && max_items(n_src, E) <= GT_SORT_ITEMS_MIN;
    int32_t h_counts[10] = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0};   // forward: items, partials, splits, long items; transposed; longest split rows
    {
        int32_t *const arr[8] = {ca, cb, cc, cd, ca2, cb2, cc2, cd2};
        const int64_t len[8] = {n_dst + 1, n_dst + 1, n_dst + 1, n_dst + 1, n_src + 1, n_src + 1, n_src + 1, n_src + 1};
        if ((s = scan_exclusive_batch(8, arr, arr, len, t.scan_tmp, st)) != GT_OK) return fail(s);
        if (in_row_order) {
            const FillDirection f{rowptr, n_dst, max_items(n_dst, E), ca, cb, cc, cd, at<gt_item>(ws, L.items_f), at<gt_split>(ws, L.splits_f)};
            const FillDirection b{g->rowptr_t, n_src, max_items(n_src, E), ca2, cb2, cc2, cd2, at<gt_item>(ws, L.items_b), at<gt_split>(ws, L.splits_b)};
            k_fill_both<<<dim3(nblocks((n_src > n_dst ? n_src : n_dst) + 1), 2), PT, 0, st>>>(f, b, chunk, long_min, max_splits(E), d_counts);
            PLAN_LAUNCH("k_fill_both");
        } else {
            CountArrays counts;
            for (int k = 0; k < 8; ++k) counts.c[k] = arr[k];
            k_collect_counts<<<1, 64, 0, st>>>(counts, n_dst, n_src, d_counts);
            PLAN_LAUNCH("k_collect_counts");
        }
    }
    PLAN_HIP(hipMemcpyAsync(h_counts, d_counts, 10 * 4, hipMemcpyDeviceToHost, st));
    PLAN_HIP(hipStreamSynchronize(st));
    g->fwd.rowptr = rowptr; g->fwd.nbr = colidx; g->fwd.wt = ew; g->fwd.n_rows = n_dst;
    g->fwd.coef_sym = g->coef_sym_f;
    g->fwd.n_items = h_counts[0]; g->fwd.n_partials = h_counts[1]; g->fwd.n_splits = h_counts[2];
    g->fwd.n_long = h_counts[3]; g->fwd.max_len = h_counts[8];
    g->fwd.items = at<gt_item>(ws, L.items_f); g->fwd.splits = at<gt_split>(ws, L.splits_f);
    if (g->fwd.n_items > max_items(n_dst, E) || g->fwd.n_splits > max_splits(E))
        return fail(gt_fail(GT_ERR_INTERNAL, "gt_graph_create: forward work list exceeds its bound (is rowptr valid?)"));
    g->bwd.rowptr = g->rowptr_t; g->bwd.nbr = g->colidx_t; g->bwd.wt = g->ew_t; g->bwd.n_rows = n_src;
    g->bwd.coef_sym = g->coef_sym_b; g->bwd.coef_mean = g->coef_mean_b;
    g->bwd.n_items = h_counts[4]; g->bwd.n_partials = h_counts[5]; g->bwd.n_splits = h_counts[6];
    g->bwd.n_long = h_counts[7]; g->bwd.max_len = h_counts[9];
    g->bwd.items = at<gt_item>(ws, L.items_b); g->bwd.splits = at<gt_split>(ws, L.splits_b);
    if (g->bwd.n_items > max_items(n_src, E) || g->bwd.n_splits > max_splits(E))
        return fail(gt_fail(GT_ERR_INTERNAL, "gt_graph_create: transposed work list exceeds its bound"));
    if (in_row_order) { *out = g; return GT_OK; }
    if ((s = build_direction(rowptr, colidx, n_src, n_dst, g->chunk, g->fwd.n_items, g->fwd.n_long, ws, L, false,
                             at<gt_item>(ws, L.items_f), at<gt_split>(ws, L.splits_f), st)) != GT_OK) return fail(s);
    if ((s = build_direction(g->rowptr_t, g->colidx_t, n_dst, n_src, g->chunk, g->bwd.n_items, g->bwd.n_long, ws, L, true,
                             at<gt_item>(ws, L.items_b), at<gt_split>(ws, L.splits_b), st)) != GT_OK) return fail(s);
    PLAN_HIP(hipStreamSynchronize(st));
#undef PLAN_HIP
#undef PLAN_LAUNCH
    *out = g;
    return GT_OK;
}

extern "C" gt_status gt_graph_destroy(gt_graph *g) {
    delete g;
    return GT_OK;
}

extern "C" gt_status gt_graph_outputs(const gt_graph *g, const int32_t **in_deg, const int32_t **out_deg,
                                      const int32_t **rowptr_t, const int32_t **colidx_t, const int32_t **perm) {
    if (!g) return gt_fail(GT_ERR_INVALID_ARG, "gt_graph_outputs: g is null");
    if (in_deg) *in_deg = g->in_deg;
    if (out_deg) *out_deg = g->out_deg;
    if (rowptr_t) *rowptr_t = g->rowptr_t;
    if (colidx_t) *colidx_t = g->colidx_t;
    if (perm) *perm = g->perm;
    return GT_OK;
}

extern "C" gt_status gt_graph_info(const gt_graph *g, int64_t *n_dst, int64_t *n_src, int64_t *n_edges,
                                   int64_t *fwd_items, int64_t *fwd_split_rows, int64_t *bwd_items,
                                   int64_t *bwd_split_rows) {
    if (!g) return gt_fail(GT_ERR_INVALID_ARG, "gt_graph_info: g is null");
    if (n_dst) *n_dst = g->n_dst;
    if (n_src) *n_src = g->n_src;
    if (n_edges) *n_edges = g->n_edges;
    if (fwd_items) *fwd_items = g->fwd.n_items;
    if (fwd_split_rows) *fwd_split_rows = g->fwd.n_splits;
    if (bwd_items) *bwd_items = g->bwd.n_items;
    if (bwd_split_rows) *bwd_split_rows = g->bwd.n_splits;
    return GT_OK;
}

extern "C" gt_status gt_graph_validate(const gt_graph *g, int64_t *n_violations, void *stream) {
    if (!g || !n_violations) return gt_fail(GT_ERR_INVALID_ARG, "gt_graph_validate: null argument");
    hipStream_t st = (hipStream_t)stream;
    GT_HIP(hipMemsetAsync(g->vcount, 0, 8, st));
    const int64_t n = (g->n_edges > g->n_dst ? g->n_edges : g->n_dst);
    k_validate<<<nblocks(n > 0 ? n : 1), PT, 0, st>>>(g->rowptr, g->colidx, g->n_dst, g->n_src, g->n_edges, g->vcount);
    GT_LAUNCH_CHECK("k_validate");
    unsigned long long h = 0;
    GT_HIP(hipMemcpyAsync(&h, g->vcount, 8, hipMemcpyDeviceToHost, st));
    GT_HIP(hipStreamSynchronize(st));
    *n_violations = (int64_t)h;
    return GT_OK;
}
