// Neighbour aggregation (the paper's Pull primitive without per-call weights) and its derivative:
// host side of gt_aggregate_fwd / gt_aggregate_bwd.  The kernels live in gt_aggregate_kernel.h.
#include "gt_aggregate_kernel.h"

size_t gt_aggregate_ws_bytes(const gt_graph *g, int64_t F) {
    const int64_t ldp = (F + 7) / 8 * 8;
    const int64_t parts = g->fwd.n_partials > g->bwd.n_partials ? g->fwd.n_partials : g->bwd.n_partials;
    return gt_align_up((size_t)parts * (size_t)ldp * 4);
}

// ---------------------------------------------------------------------------------------------
// Rows gathered from whole lines.  A gather beyond the L2s costs what it has of lines: a row of 94 bytes at a stride of 94 lies in
// 1.73 of them on average, at 96 in 1.5, at 128 in one.  Where a uniform graph reads every row often enough, the table is copied
// to such a stride (64 bytes for rows of up to 64, 128 for up to 128) into the caller's workspace before it is gathered.
// ---------------------------------------------------------------------------------------------
namespace {

// Lines that a row of `rb` bytes lies in, on average over the rows of a table
double mean_lines(uintptr_t base, int64_t stride, int64_t rb) {
    int64_t step = 128;
    for (int64_t b = stride % 128; b;) { const int64_t r = step % b; step = b; b = r; }   // gcd(stride, 128)
    int64_t lines = 0, n = 0;
    for (int64_t o = (int64_t)(base % (uintptr_t)step); o < 128; o += step, ++n) lines += (o % 128 + rb + 127) / 128;
    return (double)lines / (double)n;
}

// Stride (bytes) of the copy that a gather of rows of `rb` bytes from `lines` lines each would be made from, or 0.  What the copy saves is lines of
// misses (10 TB/s of them), what it costs are its bytes (4.5 TB/s); it has to be clearly ahead, and the table well past the L2s.  us, both
// directions of the gather as it is / copied: 1 M rows of degree 16, 47 bf16 columns 1026 / 822, of degree 8 601 / 531, 61 columns 1175 / 845, 25 columns 840 /
// 765; 300 K rows of degree 20, 47 columns 295 / 268; 1 M rows of degree 4, 47 columns 365 / 369; 65 K rows of degree 25 (6 MB) 68 / 70.
// On power-law graphs, whose rows read most are hits, it saves what it costs (1 M rows of degree 16, 47 bf16 columns 633 / 640).
int64_t repack_stride(const gt_sched &sc, int64_t n_in, int64_t n_edges, int64_t rb, double lines) {
    if (rb <= 32 || rb > 128 || n_in * rb < ((int64_t)24 << 20) || agg_skewed(sc.n_splits, sc.n_long, sc.n_items)) return 0;
    const int64_t stride = rb <= 64 ? 64 : 128;
    return (double)n_edges * (lines - 1.0) * 30.0 > (double)n_in * (double)(rb + stride) ? stride : 0;
}

// That of a table as it is given
int64_t table_copy_stride(const gt_sched &sc, int64_t n_in, int64_t n_edges, int64_t rb, const void *X, int64_t stride) {
    return repack_stride(sc, n_in, n_edges, rb, mean_lines((uintptr_t)X, stride, rb));
}

// out[row] (stride `stride`) = in[row] (stride `ld`), rb bytes each; L lanes per row, each 16 bytes, the last that the row needs ending with it (no
// alignment past the elements').  Bound by memory.
template <int L>
__global__ void __launch_bounds__(256) k_repack(const unsigned char *in, int64_t ld, int rb, int64_t rows, unsigned char *out) {
    const int l = threadIdx.x % L;
    const int off = l * 16 + 16 <= rb ? l * 16 : rb - 16, to = l * 16 < rb ? off : l * 16;
    constexpr int RPB = 256 / L;
    const int64_t r0 = (int64_t)blockIdx.x * RPB * 4 + threadIdx.x / L;
    typedef uint32_t vec __attribute__((ext_vector_type(4), aligned(2)));
    vec v[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int64_t r = r0 + i * RPB < rows ? r0 + i * RPB : rows - 1;
        v[i] = *reinterpret_cast<const vec *>(in + r * ld + off);
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int64_t r = r0 + i * RPB;
        if (r < rows) *reinterpret_cast<vec *>(out + r * (L * 16) + to) = v[i];
    }
}

}  // namespace

// Room for such a copy at width F, of whichever direction it may serve and at whichever stride the table is given; 0 where no stride could make
// it pay.  The most lines that a row lies in are those of one that begins with a line's last element, and at a stride of whole lines all rows may.
size_t gt_aggregate_repack_bytes(const gt_graph *g, int64_t F, gt_dtype t) {
    const int64_t rb = F * (int64_t)gt_dtype_size(t);
    const double most = (double)((128 - (int64_t)gt_dtype_size(t) + rb + 127) / 128);
    const int64_t f = repack_stride(g->fwd, g->n_src, g->n_edges, rb, most) * g->n_src, b = repack_stride(g->bwd, g->n_dst, g->n_edges, rb, most) * g->n_dst;
    return (size_t)(f > b ? f : b);
}

// Row stride (elements) of a table that the library writes itself and then gathers, `transposed` or not: 16-byte padding, or the next multiple of 64 or 128 bytes where
// a uniform graph's rows then lie in fewer lines (1 M rows of degree 16, one direction, 47 bf16 columns at 96 bytes 467 us, at 128 364; 41 fp32 columns at 176
// bytes 683, at 192 621; 101 bf16 columns at 208 bytes 755, at 256 623).  On power-law graphs fewer lines are not always ahead, because the table grows in the L2s
// and a power of two maps the rows read most to few channels: 262 K rows, 12 M edges, one direction, 41 fp32 columns at 176 bytes 171 us, at 192 161; 47 bf16
// columns at 96 bytes 120, at 128 112; 101 bf16 columns at 208 bytes 227, at 256 277; 70 bf16 columns at 144 bytes 188, at 256 245: they keep 16-byte padding.
int64_t gt_aggregate_table_ld(const gt_graph *g, bool transposed, int64_t F, gt_dtype t) {
    const int64_t es = (int64_t)gt_dtype_size(t), rb = F * es, pad = (rb + 15) / 16 * 16;
    const gt_sched &sc = transposed ? g->bwd : g->fwd;
    if (rb <= 32 || agg_skewed(sc.n_splits, sc.n_long, sc.n_items)) return pad / es;
    int64_t best = pad;
    for (const int64_t to : {64, 128}) {
        const int64_t s = (pad + to - 1) / to * to;
        if (mean_lines(0, s, rb) < mean_lines(0, best, rb) - 0.01) best = s;
    }
    return best / es;
}

gt_status gt_agg_launch(const AggArgs &a, gt_dtype t, bool vec, hipStream_t st, bool by_element) {
    if (by_element) return t == GT_F32 ? dispatch<float, 1>(a, st) : dispatch<bf16_t, 1>(a, st);
    return t == GT_F32 ? agg_dispatch<float>(a, vec, st) : agg_dispatch<bf16_t>(a, vec, st);
}

gt_status gt_aggregate_run(const gt_graph *g, bool transposed, gt_reduce reduce, gt_dtype in_dtype, gt_dtype out_dtype,
                           int64_t F, const void *X, int64_t ldx, void *Y, int64_t ldy, const float *bias, gt_act act,
                           void *ws, size_t ws_bytes, hipStream_t st, bool traced, const void *mask, int64_t ldmask, bool pad_out) {
    const char *fn = transposed ? "gt_aggregate_bwd" : "gt_aggregate_fwd";
    if (!g) return gt_fail(GT_ERR_INVALID_ARG, "%s: g is null", fn);
    if (F < 0) return gt_fail(GT_ERR_INVALID_ARG, "%s: F < 0", fn);
    if (reduce != GT_SUM && reduce != GT_MEAN && reduce != GT_SYMNORM)
        return gt_fail(GT_ERR_INVALID_ARG, "%s: unknown reduce %d", fn, (int)reduce);
    if (in_dtype != GT_F32 && in_dtype != GT_BF16) return gt_fail(GT_ERR_INVALID_ARG, "%s: unknown dtype", fn);
    if (in_dtype != out_dtype) return gt_fail(GT_ERR_UNSUPPORTED, "%s: input and output dtype must match", fn);
    if (reduce == GT_SYMNORM && g->n_dst != g->n_src)
        return gt_fail(GT_ERR_UNSUPPORTED, "%s: GT_SYMNORM needs a square graph (n_src == n_dst)", fn);
    const gt_sched &sc = transposed ? g->bwd : g->fwd;
    const int64_t n_in = transposed ? g->n_dst : g->n_src;
    const int64_t n_out = sc.n_rows;
    if (F == 0 || n_out == 0) return GT_OK;
    if (!Y) return gt_fail(GT_ERR_INVALID_ARG, "%s: output pointer is null", fn);
    if (!X && n_in > 0) return gt_fail(GT_ERR_INVALID_ARG, "%s: input pointer is null", fn);
    if (ldx < F || ldy < F) return gt_fail(GT_ERR_INVALID_ARG, "%s: leading dimension smaller than F", fn);
    const size_t es = gt_dtype_size(in_dtype);
    if (((uintptr_t)X % es) || ((uintptr_t)Y % es)) return gt_fail(GT_ERR_INVALID_ARG, "%s: pointer misaligned for dtype", fn);
    {
        const char *xb = (const char *)X, *xe = xb + (size_t)n_in * ldx * es;
        const char *yb = (const char *)Y, *ye = yb + (size_t)n_out * ldy * es;
        if (X && xb < ye && yb < xe) return gt_fail(GT_ERR_INVALID_ARG, "%s: input and output overlap", fn);
    }
    const size_t need = sc.n_partials > 0 ? gt_aggregate_ws_bytes(g, F) : 0;
    if (need > 0) {
        if (!ws || ((uintptr_t)ws & 255)) return gt_fail(GT_ERR_WORKSPACE, "%s: ws null or not 256-byte aligned", fn);
        if (ws_bytes < need) return gt_fail(GT_ERR_WORKSPACE, "%s: ws_bytes %zu < required %zu", fn, ws_bytes, need);
    }
    if (mask && ldmask < F) return gt_fail(GT_ERR_INVALID_ARG, "%s: mask leading dimension smaller than F", fn);

    AggArgs a{};
    a.trace_kind = !traced ? -1 : transposed ? GT_TRACE_AGG_BWD : GT_TRACE_AGG_FWD;
    a.n_rows = n_out; a.n_edges = g->n_edges;
    const int64_t rb = F * (int64_t)es, stride = table_copy_stride(sc, n_in, g->n_edges, rb, X, ldx * (int64_t)es);
    if (stride && ws && ((uintptr_t)ws & 255) == 0 && ws_bytes >= need + (size_t)(n_in * stride)) {
        unsigned char *copy = static_cast<unsigned char *>(ws) + need;
        const unsigned blocks = (unsigned)((n_in + 1024 / (stride / 16) - 1) / (1024 / (stride / 16)));
        a.trace_open = 1 + gt_trace_open(a.trace_kind, F, n_out, g->n_edges, st);   // (the gather's time has the copy in it)
        if (stride == 64) k_repack<4><<<blocks, 256, 0, st>>>(static_cast<const unsigned char *>(X), ldx * (int64_t)es, (int)rb, n_in, copy);
        else k_repack<8><<<blocks, 256, 0, st>>>(static_cast<const unsigned char *>(X), ldx * (int64_t)es, (int)rb, n_in, copy);
        if (const hipError_t e = hipGetLastError(); e != hipSuccess) {
            gt_trace_close(a.trace_open - 1, st);
            return gt_hip_fail(e, "k_repack");
        }
        X = copy;
        ldx = stride / (int64_t)es;
    }
    a.items = sc.items; a.n_items = sc.n_items; a.n_long = sc.n_long; a.max_len = sc.max_len;
    a.rowptr = sc.rowptr; a.nbr = sc.nbr;
    a.coef = sc.wt; a.post_mode = 0;
    if (reduce == GT_MEAN) {
        if (!transposed) a.post_mode = 2;   // divide by the destination's in-degree (exact for ones)
        else a.coef = sc.coef_mean;         // w_e / indeg(dst), stored per transposed entry
    } else if (reduce == GT_SYMNORM) {
        a.coef = sc.coef_sym;               // w_e / sqrt(d(u) d(v)), stored per entry
    }
    a.bias = bias; a.relu = (act == GT_ACT_RELU);
    a.mask = mask; a.ldmask = ldmask;
    a.pad_out = pad_out ? 1 : 0;
    a.X = X; a.ldx = ldx; a.Y = Y; a.ldy = ldy; a.F = F;
    a.partials = static_cast<float *>(ws); a.ldp = (F + 7) / 8 * 8;
    a.splits = sc.splits; a.n_splits = sc.n_splits;
    a.table_bytes = n_in * ldx * (int64_t)es;

    const int ve = in_dtype == GT_F32 ? 4 : 8;
    const bool vec = aligned16(X) && aligned16(Y) && (ldx % ve == 0) && (ldy % ve == 0) &&
                     (!mask || (aligned16(mask) && ldmask % ve == 0));
    return gt_agg_launch(a, in_dtype, vec, st);
}

extern "C" gt_status gt_aggregate_ws_size(const gt_graph *g, int64_t F, size_t *ws_bytes) {
    if (!g || !ws_bytes) return gt_fail(GT_ERR_INVALID_ARG, "gt_aggregate_ws_size: null argument");
    if (F < 0) return gt_fail(GT_ERR_INVALID_ARG, "gt_aggregate_ws_size: F < 0");
    const bool any = g->fwd.n_partials > 0 || g->bwd.n_partials > 0;
    *ws_bytes = any ? gt_aggregate_ws_bytes(g, F) : 0;
    return GT_OK;
}

extern "C" gt_status gt_aggregate_best_ws_size(const gt_graph *g, int transposed, gt_dtype dtype, int64_t F, const void *X, int64_t ldx,
                                               size_t *ws_bytes) {
    const char *fn = "gt_aggregate_best_ws_size";
    size_t least = 0;
    const gt_status s = gt_aggregate_ws_size(g, F, &least);
    if (s != GT_OK) return s;
    if (!ws_bytes) return gt_fail(GT_ERR_INVALID_ARG, "%s: null argument", fn);
    if (dtype != GT_F32 && dtype != GT_BF16) return gt_fail(GT_ERR_INVALID_ARG, "%s: unknown dtype", fn);
    const gt_sched &sc = transposed ? g->bwd : g->fwd;
    const int64_t es = (int64_t)gt_dtype_size(dtype), rb = F * es, n_in = transposed ? g->n_dst : g->n_src;
    const size_t copy = ldx < F ? 0 : (size_t)(n_in * table_copy_stride(sc, n_in, g->n_edges, rb, X, ldx * es));   // (the call refuses such a table)
    const size_t best = copy ? copy + (sc.n_partials > 0 ? gt_aggregate_ws_bytes(g, F) : 0) : 0;
    *ws_bytes = best > least ? best : least;
    return GT_OK;
}

extern "C" gt_status gt_aggregate_fwd(const gt_graph *g, gt_reduce reduce, gt_dtype dtype, int64_t F, const void *X,
                                      int64_t ldx, void *Y, int64_t ldy, void *ws, size_t ws_bytes, void *stream) {
    return gt_aggregate_run(g, false, reduce, dtype, dtype, F, X, ldx, Y, ldy, nullptr, GT_ACT_NONE, ws, ws_bytes,
                            (hipStream_t)stream);
}

extern "C" gt_status gt_aggregate_bwd(const gt_graph *g, gt_reduce reduce, gt_dtype dtype, int64_t F, const void *dY,
                                      int64_t lddy, void *dX, int64_t lddx, void *ws, size_t ws_bytes, void *stream) {
    return gt_aggregate_run(g, true, reduce, dtype, dtype, F, dY, lddy, dX, lddx, nullptr, GT_ACT_NONE, ws, ws_bytes,
                            (hipStream_t)stream);
}

// ---------------------------------------------------------------------------------------------
// gt_aggregate_fwd for callers that cannot allocate: the fp32 partial rows of the split long rows
// live in a fixed array inside the library instead of a caller workspace.
// ---------------------------------------------------------------------------------------------
#include <mutex>

#define GT_STATIC_SCRATCH_BYTES ((size_t)32 << 20)
// No kernel names the array (they receive its address as an argument); the host-side reference in
// static_scratch() below is what makes the compiler keep it and export its device symbol.  (Marking
// it `used` as well leaves the device symbol with local binding, and the runtime's lookup fails.)
static __device__ __align__(256) unsigned char scratch[GT_STATIC_SCRATCH_BYTES];

namespace {
constexpr int GT_MAX_DEVICES = 64;
std::mutex g_scratch_lock;
void *g_scratch_ptr[GT_MAX_DEVICES] = {};   // device address of `scratch` on each device, looked up once

// `scratch` names a host-side stand-in here; its device address is different on every GPU and
// comes from hipGetSymbolAddress with that GPU current.
gt_status static_scratch(void **ptr) {
    int dev = -1;
    GT_HIP(hipGetDevice(&dev));
    if (dev < 0 || dev >= GT_MAX_DEVICES) return gt_fail(GT_ERR_UNSUPPORTED, "gt_aggregate_fwd_static: device index %d", dev);
    std::lock_guard<std::mutex> hold(g_scratch_lock);
    if (!g_scratch_ptr[dev]) {
        void *p = nullptr;
        GT_HIP(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
        if (!p || ((uintptr_t)p & 255)) return gt_fail(GT_ERR_INTERNAL, "gt_aggregate_fwd_static: bad address of the static scratch");
        g_scratch_ptr[dev] = p;
    }
    *ptr = g_scratch_ptr[dev];
    return GT_OK;
}
}  // namespace

extern "C" gt_status gt_aggregate_static_capacity(size_t *bytes) {
    if (!bytes) return gt_fail(GT_ERR_INVALID_ARG, "gt_aggregate_static_capacity: null");
    *bytes = GT_STATIC_SCRATCH_BYTES;
    return GT_OK;
}

extern "C" gt_status gt_aggregate_fwd_static(const gt_graph *g, gt_reduce reduce, gt_dtype dtype, int64_t F, const void *X,
                                             int64_t ldx, void *Y, int64_t ldy, void *stream) {
    if (!g) return gt_fail(GT_ERR_INVALID_ARG, "gt_aggregate_fwd_static: g is null");
    if (F < 0) return gt_fail(GT_ERR_INVALID_ARG, "gt_aggregate_fwd_static: F < 0");
    const size_t need = g->fwd.n_partials > 0 ? gt_aggregate_ws_bytes(g, F) : 0;
    if (need > GT_STATIC_SCRATCH_BYTES)
        return gt_fail(GT_ERR_WORKSPACE, "gt_aggregate_fwd_static: %zu bytes of partial rows exceed the built-in %zu; "
                       "use gt_aggregate_fwd with a caller workspace", need, (size_t)GT_STATIC_SCRATCH_BYTES);
    void *ws = nullptr;
    if (need > 0) {
        const gt_status s = static_scratch(&ws);
        if (s != GT_OK) return s;
    }
    // every partial slot is written by its work item before the second kernel reads it: nothing in
    // the array has to start at zero; kernel timing is off for this call (it would create events)
    return gt_aggregate_run(g, false, reduce, dtype, dtype, F, X, ldx, Y, ldy, nullptr, GT_ACT_NONE, ws,
                            need, (hipStream_t)stream, false);
}
