// Edge weighting: the paper's NeighborApply primitive (the edge-weight function g of the source
// and destination embeddings, i.e. SDDMM) and Pull with per-call edge weights (the function h that
// transforms the source embedding with g's output before the aggregation f), forward and backward.
//
// Kept from the paper (Frontend section, NeighborApply / Pull): traversal is destination-centric
// and feature-wise; the destination's row is loaded once per work item and reused for all of its
// in-edges; the edge tensor produced by NeighborApply is what Pull consumes.  As for the plain
// aggregation, a group of G lanes of a 64-lane wavefront owns a work item and long rows are cut
// into chunk-sized items.  Three kernel shapes cover every call:
//   gather     out[r]  = sum_e c_e * h(X[nbr e], W_e)           (k_aggregate with vector weights)
//   edge-out   W_e     = s_r * (R[r] (.) X[nbr e])  or  s_r * R[r]        (k_edge_out)
//   edge-dot   w_e     = s_r * <R[r], X[nbr e]>                           (k_edge_dot)
// Derivatives with outputs on the source vertices run over the transposed structure and reach the
// per-edge data through its permutation (no atomics; results are reproducible).
#include "gt_aggregate_kernel.h"

namespace {

struct EdgeArgs {
    const gt_item *items;
    int64_t n_items;
    const int32_t *nbr;
    const void *R;        // row operand [n_rows][ldr]
    int64_t ldr;
    const float *rscale;  // per-row scale or null
    const void *X;        // gathered operand [n_in][ldx] (unused for broadcast)
    int64_t ldx;
    void *W;              // output: [E][ldw] of T (edge-out) or float[E] (edge-dot)
    int64_t ldw;
    int64_t F;
    int xcd_run;          // item blocks per XCD run (set at launch)
    int skewed;           // host-side: see agg_skewed
    int stream;           // host-side: see edge_streams
    int64_t n_long;       // host-side: the first n_long items are long ones
    int64_t n_cut;        // set at launch: the first n_cut items are cut into EDGE_CUT work items each
};

enum { EO_MUL = 0, EO_BCAST = 1 };

// SH: rows without 16-byte alignment, see agg_col
template <bool SH, int V>
__device__ inline int64_t edge_col(const EdgeArgs &a, int64_t own) { return agg_col<SH, V>(a.F, own); }

// The row and the entries of this group's work item.  An entry's result depends on no other entry, so long items may be cut into
// EDGE_CUT parts (whole batches of G entries), each of them a work item: on skewed graphs the longest items' chains outlast the
// rest (dot product and scaled aggregation, both derivatives, power law, 900 K edges, 24 bf16 columns 248 -> 150 us; 1.5 M edges, 60 columns 331 -> 253).
constexpr int EDGE_CUT = 4;
template <int G>
__device__ inline bool edge_item(const EdgeArgs &a, int run, int grp, int wave, int &row, int &e0, int &e1) {
    const int64_t v = ((int64_t)agg_item_block(run, blockIdx.x, gridDim.x, 3) * 4 + wave) * (64 / G) + grp;
    const bool cut = v < a.n_cut * EDGE_CUT;
    const int64_t id = cut ? v / EDGE_CUT : v - a.n_cut * (EDGE_CUT - 1);
    if (id >= a.n_items) return false;
    const int4 raw = reinterpret_cast<const int4 *>(a.items)[id];
    row = raw.x; e0 = raw.y; e1 = raw.z;
    if (cut) {
        const int per = ((e1 - e0 + EDGE_CUT - 1) / EDGE_CUT + G - 1) / G * G, part = (int)(v % EDGE_CUT);
        e0 += part * per;
        e1 = e0 + per < e1 ? e0 + per : e1;
    }
    return e0 < e1;
}

// W[e, :] = s_r * R[r, :] (.) X[nbr[e], :]   (EO_MUL)   or   s_r * R[r, :]   (EO_BCAST).  NT: W is streamed past the caches
template <typename T, int V, int G, int NP, int MODE, bool SH, bool NT>
__global__ void __launch_bounds__(256) k_edge_out(const EdgeArgs a) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int gl = lane & (G - 1), grp = lane / G;
    int row, e0, e1;
    if (!edge_item<G>(a, gridDim.y == 1 ? a.xcd_run : 1, grp, wave, row, e0, e1)) return;
    const int64_t col0 = (int64_t)blockIdx.y * (G * V * NP);
    const T *X = static_cast<const T *>(a.X);
    const T *R = static_cast<const T *>(a.R) + (int64_t)row * a.ldr;
    T *W = static_cast<T *>(a.W);
    typedef typename Raw<T, V>::type raw_t;

    float r[NP][V];
    const float s = a.rscale ? a.rscale[row] : 1.0f;
#pragma unroll
    for (int p = 0; p < NP; ++p) {
        const int64_t own = col0 + (int64_t)(p * G + gl) * V;
        raw_t rv = raw_t{};
        if (own < a.F && e0 < e1) rv = load_raw<T, V>(R + edge_col<SH, V>(a, own));
        unpack_raw(rv, r[p]);
#pragma unroll
        for (int i = 0; i < V; ++i) r[p][i] *= s;
    }
    // U edges at a time; the rows of the next U are requested before the current ones are stored, so that a wait for
    // rows never includes the stores just issued (loads and stores share one in-order counter).  Measured on MI355X,
    // 4.2 M edges x 64 fp32 (1.07 GB written): 432 -> 330 us.
    constexpr int U = NP == 1 ? (G >= 8 && V > 1 ? 8 : 4) : 2;
    int idx = 0, idx_next = 0;
    auto fetch = [&](int e) { return MODE == EO_MUL && e < e1 ? a.nbr[e] : 0; };
    // entries j .. j + U - 1 of the current ids (branch free: one past the end stands for row 0 and is not stored)
    auto load = [&](raw_t (&v)[U][NP], int j) {
        int src[U];
#pragma unroll
        for (int u = 0; u < U; ++u) src[u] = __shfl(idx, (j + u) & (G - 1), G);
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const T *xr = X + (int64_t)src[u] * a.ldx;
#pragma unroll
            for (int p = 0; p < NP; ++p) v[u][p] = load_raw<T, V>(xr + edge_col<SH, V>(a, col0 + (int64_t)(p * G + gl) * V));
        }
    };
    raw_t v[U][NP];
    if constexpr (MODE == EO_MUL) {
        idx = fetch(e0 + gl);
        idx_next = fetch(e0 + G + gl);
        load(v, 0);
    }
    for (int e = e0; e < e1; e += U) {
        raw_t nx[U][NP];
        if constexpr (MODE == EO_MUL) {
            if (e + U < e1) {
                const int jn = (e + U - e0) & (G - 1);
                if (jn == 0) {
                    idx = idx_next;
                    idx_next = fetch(e + U + G + gl);
                }
                load(nx, jn);
            }
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (e + u >= e1) continue;
            T *wr = W + (int64_t)(e + u) * a.ldw;
#pragma unroll
            for (int p = 0; p < NP; ++p) {
                const int64_t own = col0 + (int64_t)(p * G + gl) * V;
                if (own >= a.F) continue;
                const int64_t col = edge_col<SH, V>(a, own);
                const int n = (int)((a.F - col) < V ? (a.F - col) : V);
                float o[V];
                if constexpr (MODE == EO_MUL) {
                    float x[V];
                    unpack_raw(v[u][p], x);
#pragma unroll
                    for (int i = 0; i < V; ++i) o[i] = r[p][i] * x[i];
                } else {
#pragma unroll
                    for (int i = 0; i < V; ++i) o[i] = r[p][i];
                }
                if constexpr (NT) store_vec_nt<T, V>(wr + col, o, n);
                else store_vec<T, V>(wr + col, o, n);
            }
        }
        if constexpr (MODE == EO_MUL) {
#pragma unroll
            for (int u = 0; u < U; ++u)
#pragma unroll
                for (int p = 0; p < NP; ++p) v[u][p] = nx[u][p];
        }
    }
}

// Sum over the G lanes of a group, in every lane, in a fixed order: exchanges inside 16 lanes ride on the addition itself
// (data-parallel primitives: neighbour, pair, mirrored four, mirrored eight); only wider groups need a trip
// through the LDS permute unit, of which the plain butterfly made log2 G per edge.
template <int CTRL>
__device__ inline float dpp_add(float x) {
    return x + __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), CTRL, 0xf, 0xf, true));
}
template <int G>
__device__ inline float group_sum(float x) {
    x = dpp_add<0xB1>(x);                    // quad_perm [1, 0, 3, 2]
    x = dpp_add<0x4E>(x);                    // quad_perm [2, 3, 0, 1]
    if constexpr (G >= 8) x = dpp_add<0x141>(x);    // mirror inside 8 lanes
    if constexpr (G >= 16) x = dpp_add<0x140>(x);   // mirror inside 16 lanes
    if constexpr (G >= 32) x += __shfl_xor(x, 16, G);
    if constexpr (G >= 64) x += __shfl_xor(x, 32, G);
    return x;
}

// The elements of a raw vector that take part in a dot product: all ones or all zeros per element, so that a masked vector adds exact
// zeros whatever the row's padding holds
template <int V>
__device__ inline uint4 dot_mask(int64_t col, int64_t own, int64_t F) {
    uint32_t m[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        if constexpr (V == 4) {
            m[q] = col + q >= own && col + q < F ? ~0u : 0u;
        } else {
            m[q] = (col + 2 * q >= own && col + 2 * q < F ? 0xffffu : 0u) | (col + 2 * q + 1 >= own && col + 2 * q + 1 < F ? 0xffff0000u : 0u);
        }
    }
    return make_uint4(m[0], m[1], m[2], m[3]);
}
__device__ inline float4 mask_raw(const float4 &v, const uint4 &m) {
    return make_float4(__uint_as_float(__float_as_uint(v.x) & m.x), __uint_as_float(__float_as_uint(v.y) & m.y),
                       __uint_as_float(__float_as_uint(v.z) & m.z), __uint_as_float(__float_as_uint(v.w) & m.w));
}
__device__ inline uint4 mask_raw(const uint4 &v, const uint4 &m) { return make_uint4(v.x & m.x, v.y & m.y, v.z & m.z, v.w & m.w); }
__device__ inline float mask_raw(const float &v, const uint4 &m) { return __uint_as_float(__float_as_uint(v) & m.x); }
__device__ inline bf16_t mask_raw(const bf16_t &v, const uint4 &m) { return v & (bf16_t)m.x; }

// w[e] = s_r * <R[r, :], X[nbr[e], :]>   (all columns inside one column tile).  U: row loads in flight per lane.  WIDE: rows of more
// than one column tile are walked tile by tile, the row operand read again per tile and batch; otherwise it stays in registers
// (read per batch, it was a round trip in front of every batch's rows; power law, 8.4 M edges, 128 bf16 columns 216 -> 177 us).
template <typename T, int V, int G, int NP, bool SH, int U, bool WIDE>
__global__ void __launch_bounds__(256) k_edge_dot(const EdgeArgs a) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int gl = lane & (G - 1), grp = lane / G;
    int row, e0, e1;
    if (!edge_item<G>(a, a.xcd_run, grp, wave, row, e0, e1)) return;
    const T *X = static_cast<const T *>(a.X);
    const T *R = static_cast<const T *>(a.R) + (int64_t)row * a.ldr;
    float *W = static_cast<float *>(a.W);
    typedef typename Raw<T, V>::type raw_t;

    const float s = a.rscale ? a.rscale[row] : 1.0f;
    constexpr int TILE = G * V * NP;
    raw_t r[NP];
    uint4 m[NP];
    int64_t col[NP];
    auto tile = [&](int64_t c0) {   // this lane's columns of the tile at c0: which of them count, and the row operand
#pragma unroll
        for (int p = 0; p < NP; ++p) {
            const int64_t own = c0 + (int64_t)(p * G + gl) * V;
            col[p] = edge_col<SH, V>(a, own);
            if constexpr (V == 1) m[p].x = own < a.F ? ~0u : 0u;
            else m[p] = dot_mask<V>(col[p], own, a.F);
            r[p] = mask_raw(load_raw<T, V>(R + col[p]), m[p]);
        }
    };
    if (!WIDE && a.F > 0) tile(0);
    int idx_next = e0 + gl < e1 ? a.nbr[e0 + gl] : 0;
    for (int base = e0; base < e1; base += G) {
        const int idx = idx_next;
        idx_next = base + G + gl < e1 ? a.nbr[base + G + gl] : 0;   // requested before this batch's rows are used
        const int cnt = (e1 - base) < G ? (e1 - base) : G;
        float mine = 0.0f;   // lane gl keeps the result of edge base + gl
        for (int64_t c0 = 0; c0 < (WIDE ? a.F : a.F > 0 ? 1 : 0); c0 += TILE) {
            if constexpr (WIDE) tile(c0);
            for (int j = 0; j < cnt; j += U) {
                // (branch free: an entry past the end stands for row 0 and its product is not kept)
                int src[U];
                raw_t v[U][NP];
#pragma unroll
                for (int u = 0; u < U; ++u) src[u] = __shfl(idx, (j + u) & (G - 1), G);
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const T *xr = X + (int64_t)src[u] * a.ldx;
#pragma unroll
                    for (int p = 0; p < NP; ++p) v[u][p] = load_raw<T, V>(xr + col[p]);
                }
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    float part = 0.0f;
#pragma unroll
                    for (int p = 0; p < NP; ++p) {
                        float x[V], y[V];
                        unpack_raw(mask_raw(v[u][p], m[p]), x);
                        unpack_raw(r[p], y);
#pragma unroll
                        for (int i = 0; i < V; ++i) part = fmaf(y[i], x[i], part);
                    }
                    part = group_sum<G>(part);
                    if (gl == ((j + u) & (G - 1))) mine += part;
                }
            }
        }
        if (base + gl < e1) W[base + gl] = s * mine;   // one coalesced store of up to G results
    }
}

// Both derivatives of the scaled aggregation from one gather, over the transposed structure:  Y[u] = sum_e c_e X[v],
// dW[perm e] = f_e <X[v], R[u]>  (X: the upstream gradient, R: the source embeddings; c_e = W[perm e] f_e).  The same rows of X that the sum reads give the
// products, which otherwise take a pass of their own that gathers R for every edge; what it costs is that they leave by the permutation, a line each.
// One entry's product is formed as in k_edge_dot (same lanes, same order).  Long items may be shared out as in k_aggregate, whose items, partial rows and
// row ends these are.  Power law, 8.4 M edges, 128 bf16 columns: 268 + 187 us apart (a gather, a product).
template <typename T, int V, int G, bool SH, int U>
__global__ void __launch_bounds__(256) k_scale_bwd(const AggArgs a, const void *R, int64_t ldr, float *dW) {
    constexpr int NG = 64 / G;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int gl = lane & (G - 1), grp = lane / G;
    const int bx = blockIdx.x;
    const bool coop = bx < a.n_coop, one_wave = a.coop_waves == 1;   // uniform over the workgroup
    const int64_t item_id = coop ? (one_wave ? (int64_t)bx * 4 + wave : (int64_t)bx)
                                 : (int64_t)a.n_coop * (one_wave ? 4 : 1) + ((int64_t)agg_item_block(a.xcd_run, bx - a.n_coop, a.n_blocks - a.n_coop, 3) * 4 + wave) * NG + grp;
    if (item_id >= a.n_items) return;   // whole groups (in a cooperative workgroup: all, or whole wavefronts that meet no barrier)
    const int4 raw = reinterpret_cast<const int4 *>(a.items)[item_id];
    const int row = raw.x, slot = raw.w;
    int e0 = raw.y, e1 = raw.z;
    if (coop) {   // this group's slice
        const int ng = one_wave ? NG : 4 * NG, per = (e1 - e0 + ng - 1) / ng;
        e0 += (one_wave ? grp : wave * NG + grp) * per;
        e1 = e0 + per < e1 ? e0 + per : e1;   // (may lie before e0: an empty slice)
    }
    typedef typename Raw<T, V>::type raw_t;
    const T *X = static_cast<const T *>(a.X);
    const int64_t own = (int64_t)gl * V, col = agg_col<SH, V>(a, own);
    const uint4 m = dot_mask<V>(col, own, a.F);
    const raw_t r = mask_raw(load_raw<T, V>(static_cast<const T *>(R) + (int64_t)row * ldr + col), m);
    float acc[1][V], msk[1][V];
#pragma unroll
    for (int i = 0; i < V; ++i) { acc[0][i] = 0.0f; msk[0][i] = 1.0f; }
    int idx_next, ei_next = 0, ei_later;   // places of the next batch and of the one after: the scores are not waited for between the row loads
    float c_next, f_next;
    if (e0 + gl < e1) ei_next = a.eidx[e0 + gl];
    auto place = [&](int base, int ahead) {
        ei_later = 0;
        if (ahead + gl < e1 - base) ei_later = a.eidx[base + ahead + gl];
    };
    auto fetch = [&](int e) {   // this lane's entry of a batch
        idx_next = 0; c_next = 0.0f; f_next = 1.0f;
        if (e < e1) {
            idx_next = a.nbr[e];
            if (a.coef2) f_next = a.coef2[e];
            c_next = a.coef[ei_next];
        }
    };
    if constexpr (G < 64) place(e0, G);
    fetch(e0 + gl);
    for (int base = e0; base < e1; base += G) {
        const int idx = idx_next, ei = ei_next;
        const float f = f_next, c = c_next * f;
        if constexpr (G == 64) place(base, G);   // (long batches hide the places' latency, and the register costs: 150 fp32 columns, power law, 4 M edges 459 / 464 us)
        ei_next = ei_later;
        fetch(base + G + gl);   // requested before this batch's rows are used
        if constexpr (G < 64) place(base, 2 * G);
        const int cnt = (e1 - base) < G ? (e1 - base) : G;
        float mine = 0.0f;   // lane gl keeps the product of entry base + gl
        for (int j = 0; j < cnt; j += U) {
            // (branch free: an entry past the end stands for row 0, with a coefficient of zero on a vector of zeros)
            raw_t v[U];
            float cj[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                cj[u] = __shfl(c, (j + u) & (G - 1), G);
                v[u] = load_raw<T, V>(X + (int64_t)__shfl(idx, (j + u) & (G - 1), G) * a.ldx + col);
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                if (j + u >= cnt) { v[u] = raw_t{}; cj[u] = 0.0f; }
                fma_raw(acc[0], cj[u], v[u]);
                float x[V], y[V], part = 0.0f;
                unpack_raw(mask_raw(v[u], m), x);
                unpack_raw(r, y);
#pragma unroll
                for (int i = 0; i < V; ++i) part = fmaf(y[i], x[i], part);
                part = group_sum<G>(part);
                if (gl == ((j + u) & (G - 1))) mine += part;
            }
        }
        if (base + gl < e1) dW[ei] = f * mine;
    }
    if (coop) {
        __shared__ float red[4][G * V];
        // groups of a wavefront: exchanged pairwise; wavefronts: through LDS, in order
#pragma unroll
        for (int o = G; o < 64; o <<= 1)
#pragma unroll
            for (int i = 0; i < V; ++i) acc[0][i] += __shfl_xor(acc[0][i], o, 64);
        if (!one_wave) {   // uniform over the workgroup
            if (grp == 0) {
#pragma unroll
                for (int i = 0; i < V; ++i) red[wave][i * G + gl] = acc[0][i];
            }
            __syncthreads();
            if (wave != 0) return;
        }
        if (grp != 0) return;
        if (!one_wave)
#pragma unroll
            for (int i = 0; i < V; ++i) acc[0][i] = ((red[0][i * G + gl] + red[1][i * G + gl]) + red[2][i * G + gl]) + red[3][i * G + gl];
    }
    if (slot < 0) {
        finish_row<T, V, G, 1, SH>(a, row, gl, 0, acc, msk);
    } else if (own < a.F) {   // (partial rows are padded to 8 floats: a whole vector always fits)
        float *P = a.partials + (int64_t)slot * a.ldp + col;
#pragma unroll
        for (int q = 0; q < V / 4; ++q) {
            const float4 x = make_float4(acc[0][4 * q], acc[0][4 * q + 1], acc[0][4 * q + 2], acc[0][4 * q + 3]);
            __builtin_memcpy(P + 4 * q, &x, 16);
        }
    }
}

template <typename T, int V, int G, bool SH, int U>
gt_status launch_scale_bwd(const AggArgs &a, const void *R, int64_t ldr, float *dW, hipStream_t st) {
    constexpr int NG = 64 / G;
    AggArgs b = a;
    const double bytes = agg_bytes<T>(a);
    b.coop_waves = G == 64 || (U == 2 && G >= 8) || (G == 16 && bytes > 1.0e9) ? 4 : 1;   // (as in the plain gather)
    const int64_t ipc = b.coop_waves == 1 ? 4 : 1;   // items per cooperative workgroup
    b.n_coop = agg_share_out(a, G, U, bytes) ? (int)((a.n_long + ipc - 1) / ipc) : 0;
    const int64_t left = a.n_items > b.n_coop * ipc ? a.n_items - b.n_coop * ipc : 0, gi = (left + 4 * NG - 1) / (4 * NG);
    b.n_blocks = (int)(b.n_coop + gi);
    b.xcd_run = agg_xcd_run(gi);
    const int tr = gt_trace_open(a.trace_kind, a.F, a.n_rows, a.n_edges, st);
    gt_trace_variant(tr, V, G, 1, U, false);
    if (b.n_blocks > 0) k_scale_bwd<T, V, G, SH, U><<<(unsigned)b.n_blocks, 256, 0, st>>>(b, R, ldr, dW);
    gt_trace_close(tr, st);
    GT_LAUNCH_CHECK("k_scale_bwd");
    if (a.n_splits > 0) {
        k_reduce_partials<T, V, G, 1, SH><<<(unsigned)((a.n_splits + 3) / 4), 256, 0, st>>>(a);
        GT_LAUNCH_CHECK("k_reduce_partials");
    }
    return GT_OK;
}

template <typename T, bool SH>
gt_status dispatch_scale_bwd(const AggArgs &a, const void *R, int64_t ldr, float *dW, hipStream_t st) {
    constexpr int V = 16 / (int)sizeof(T);
    const int64_t nvec = (a.F + V - 1) / V;
    const bool many = agg_skewed(a);   // rows in flight as in the edge product (see launch_edge)
#define GT_SCALE_BWD(G_, U_) (many ? launch_scale_bwd<T, V, G_, SH, U_>(a, R, ldr, dW, st) : launch_scale_bwd<T, V, G_, SH, 2>(a, R, ldr, dW, st))
    if (nvec <= 4) return GT_SCALE_BWD(4, 4);
    if (nvec <= 8) return GT_SCALE_BWD(8, 8);
    if (nvec <= 16) return GT_SCALE_BWD(16, 8);
    if (a.n_edges < 8 * a.n_items) return nvec <= 32 ? launch_scale_bwd<T, V, 32, SH, 2>(a, R, ldr, dW, st) : launch_scale_bwd<T, V, 64, SH, 2>(a, R, ldr, dW, st);
    if (nvec <= 32) return GT_SCALE_BWD(32, 4);
    return GT_SCALE_BWD(64, 4);
#undef GT_SCALE_BWD
}

template <typename T, int V, int G, int NP, bool SH>
gt_status launch_edge(const EdgeArgs &a, int kind, hipStream_t st) {
    constexpr int NG = 64 / G;
    if (a.n_items <= 0) return GT_OK;
    const int64_t tile = (int64_t)G * V * NP;
    const unsigned gy = kind == 2 ? 1u : (unsigned)((a.F + tile - 1) / tile);
    EdgeArgs b = a;
    b.n_cut = a.skewed ? a.n_long : 0;
    const int64_t gx = (a.n_items + b.n_cut * (EDGE_CUT - 1) + 4 * NG - 1) / (4 * NG);
    const dim3 grid((unsigned)gx, gy);
    b.xcd_run = agg_xcd_run(gx);
    if constexpr (V > 1 && !SH) {
        if (kind < 2 && a.stream) {
            if (kind == 0) k_edge_out<T, V, G, NP, EO_MUL, SH, true><<<grid, 256, 0, st>>>(b);
            else k_edge_out<T, V, G, NP, EO_BCAST, SH, true><<<grid, 256, 0, st>>>(b);
            GT_LAUNCH_CHECK("k_edge");
            return GT_OK;
        }
    }
    if (kind == 0) k_edge_out<T, V, G, NP, EO_MUL, SH, false><<<grid, 256, 0, st>>>(b);
    else if (kind == 1) k_edge_out<T, V, G, NP, EO_BCAST, SH, false><<<grid, 256, 0, st>>>(b);
    else {
        // Many rows in flight hide the chain of a long row; where there is none, two do, and keep the rows that are read at a time
        // in the L2s (us, two / eight: power law, 4 M edges, 64 fp32 columns 153 / 108; uniform, 2 M edges of degree 6, 128 bf16
        // columns 81 / 86, 7.5 M edges, 40 bf16 columns 203 / 217).  Rows of a whole or half a wavefront need fewer (both derivatives too,
        // four / eight: 1.5 M edges, 151 fp32 columns 566 / 584; 2.4 M edges, 128 columns 868 / 900).
        constexpr int MANY = NP == 1 ? (G == 8 || G == 16 ? 8 : 4) : 2;
        if constexpr (NP == 4) {   // (the widest shape also walks what is wider still)
            if (a.F > tile) {
                k_edge_dot<T, V, G, NP, SH, 2, true><<<grid, 256, 0, st>>>(b);
                GT_LAUNCH_CHECK("k_edge");
                return GT_OK;
            }
        }
        if (a.skewed) k_edge_dot<T, V, G, NP, SH, MANY, false><<<grid, 256, 0, st>>>(b);
        else k_edge_dot<T, V, G, NP, SH, 2, false><<<grid, 256, 0, st>>>(b);
    }
    GT_LAUNCH_CHECK("k_edge");
    return GT_OK;
}

template <typename T, int V, bool SH = false>
gt_status dispatch_edge(const EdgeArgs &a, int kind, hipStream_t st) {
    const int64_t nvec = (a.F + V - 1) / V;
    if (nvec <= 4) return launch_edge<T, V, 4, 1, SH>(a, kind, st);
    if (nvec <= 8) return launch_edge<T, V, 8, 1, SH>(a, kind, st);
    if constexpr (V == 1) return launch_edge<T, V, 16, 1, SH>(a, kind, st);   // narrow rows only (see run_edge)
    if (nvec <= 16) return launch_edge<T, V, 16, 1, SH>(a, kind, st);
    if (nvec <= 32) return launch_edge<T, V, 32, 1, SH>(a, kind, st);
    if (nvec <= 64) return launch_edge<T, V, 64, 1, SH>(a, kind, st);
    if (nvec <= 128) return launch_edge<T, V, 64, 2, SH>(a, kind, st);
    if (nvec <= 192) return launch_edge<T, V, 64, 3, SH>(a, kind, st);
    return launch_edge<T, V, 64, 4, SH>(a, kind, st);
}

bool vec_ok(gt_dtype t, const void *p, int64_t ld) {
    const int64_t ve = t == GT_BF16 ? 8 : 4;
    return p == nullptr || (aligned16(p) && ld % ve == 0);
}

// Whether a tensor of one row per edge is streamed past the caches, which keeps the vertices' rows in them (us, element-wise product and
// aggregation with all derivatives; the reader alone is the tensor's next one and finds a small tensor in the last-level cache).
//  * Rows of whole lines: read so from about 100 MB on (nowhere / reader / both: power law, 64 fp32 columns, 122 MB 180 / 175 / 191, 244 MB 375 / 370 / 347,
//    1.07 GB 1435 / 1349 / 1208), written so from 224 MB on.
//  * Other rows: read so from 224 MB on, if they are a line or more (100 columns, 191 MB 261 / 286 / 331, 305 MB 636 / 610 / 617; 33 columns and 304-byte
//    rows, reader, 508 / 548 and 1022 / 985); written so where the part of a line at a row's end, which is then written twice, is little of the row
//    and the tensor large (400-byte rows, 381 MB 711 / 682 / 690, 687 MB 918 / 924 / 1027; 480-byte rows 229 MB 330 / 334 / 361, 458 MB 822 / 774 / 744,
//    1.1 GB 2308 / 2254 / 2196).
bool edge_streams(int64_t E, const void *W, int64_t ldw, gt_dtype t, bool vec, bool write) {
    const int64_t row = ldw * (int64_t)gt_dtype_size(t), MB = (int64_t)1 << 20;
    if (!vec || row < 128) return false;
    if (row % 128 == 0 && ((uintptr_t)W & 127) == 0) return E * row >= (write ? 224 : 96) * MB;
    return (!write || row >= 440) && E * row >= (write ? 320 : 224) * MB;
}

// kind: 0 edge-out product, 1 edge-out broadcast, 2 edge-dot
gt_status run_edge(const gt_graph *g, int kind, gt_dtype t, int64_t F, const void *R, int64_t ldr, const float *rscale,
                   const void *X, int64_t ldx, void *W, int64_t ldw, hipStream_t st) {
    EdgeArgs a{};
    a.items = g->fwd.items; a.n_items = g->fwd.n_items; a.nbr = g->colidx;
    a.R = R; a.ldr = ldr; a.rscale = rscale; a.X = X; a.ldx = ldx; a.W = W; a.ldw = ldw; a.F = F;
    const bool vec = vec_ok(t, R, ldr) && vec_ok(t, X, ldx) && (kind == 2 || vec_ok(t, W, ldw));
    a.stream = kind < 2 && edge_streams(g->n_edges, W, ldw, t, vec, true);
    const int ve = t == GT_F32 ? 4 : 8;
    a.n_long = g->fwd.n_long;
    a.skewed = agg_skewed(g->fwd.n_splits, g->fwd.n_long, g->fwd.n_items);
    // Narrow rows without alignment: element by element, whose neighbouring lanes share a line, where two to four lanes with shifted
    // vectors per edge leave most of a wavefront's loads idle (us, vectors / elements: 7.5 M uniform edges, 13 fp32 columns, product 301 / 245,
    // dot product 237 / 152; 13 bf16 columns 213 / 157, 189 / 136; from 17 columns on vectors, 313 / 309 and below).  Broadcasts gain nothing.
    if (!vec && (F < ve || (F <= 16 && kind != 1))) return t == GT_F32 ? dispatch_edge<float, 1>(a, kind, st) : dispatch_edge<bf16_t, 1>(a, kind, st);
    if (t == GT_F32) return vec ? dispatch_edge<float, 4>(a, kind, st) : dispatch_edge<float, 4, true>(a, kind, st);
    return vec ? dispatch_edge<bf16_t, 8>(a, kind, st) : dispatch_edge<bf16_t, 8, true>(a, kind, st);
}

// gather: Y[r] = post( sum_e coef[ei] * coef2[e] * h(X[nbr e], VW[ei]) ), over the given or the
// transposed structure
gt_status run_gather(const gt_graph *g, bool transposed, gt_dtype t, int64_t F, const void *X, int64_t ldx, void *Y,
                     int64_t ldy, const float *coef, bool via_perm, const float *coef2, const void *VW, int64_t ldvw,
                     int vwm, int post_mode, void *ws, hipStream_t st) {
    const gt_sched &sc = transposed ? g->bwd : g->fwd;
    if (sc.n_rows == 0) return GT_OK;
    AggArgs a{};
    a.items = sc.items; a.n_items = sc.n_items; a.n_long = sc.n_long; a.max_len = sc.max_len; a.rowptr = sc.rowptr; a.nbr = sc.nbr;
    a.coef = coef; a.eidx = via_perm ? g->perm : nullptr; a.coef2 = coef2;
    if (!coef && vwm == VWM_NONE) { a.coef = coef2; a.coef2 = nullptr; }   // (one factor per entry)
    a.VW = VW; a.ldvw = ldvw; a.post_mode = post_mode;
    a.bias = nullptr; a.relu = 0;
    a.X = X; a.ldx = ldx; a.Y = Y; a.ldy = ldy; a.F = F;
    a.partials = static_cast<float *>(ws); a.ldp = (F + 7) / 8 * 8;
    a.splits = sc.splits; a.n_splits = sc.n_splits;
    // (with per-entry factors beside the rows, eight of them in flight pay only where they hide the chains of long rows: us, two / eight,
    // power law, 1 M edges, 28 fp32 columns 49 / 34; uniform, 4.8 M edges, 28 fp32 columns 137 / 157, 2 M edges of degree 6, 8 columns 41 / 43)
    a.table_bytes = agg_skewed(a) ? (transposed ? g->n_dst : g->n_src) * ldx * (int64_t)gt_dtype_size(t) : (int64_t)1 << 40;
    a.trace_kind = transposed ? GT_TRACE_AGG_BWD : GT_TRACE_AGG_FWD;
    a.n_rows = sc.n_rows; a.n_edges = g->n_edges;
    const bool vec = vec_ok(t, X, ldx) && vec_ok(t, Y, ldy) && vec_ok(t, VW, ldvw);
    // Narrow rows without alignment go element by element (as in agg_dispatch) also in bf16 and also where ids come in long batches if
    // an entry's factor or vector is looked up through the permutation: sixteen lanes per row keep four times as many wavefronts for
    // those random reads (us, vectors / elements: 7.5 M uniform edges, 13 bf16 columns, scaled aggregation backward 498 / 426).
    const bool el = !vec && F <= 16 && !agg_skewed(a) &&
                    (via_perm || (vwm == VWM_NONE && !agg_vectors_pay(a, (double)a.n_edges * (double)F * gt_dtype_size(t))));
    if (vwm == VWM_NONE && !via_perm) return gt_agg_launch(a, t, vec, st, el);
#define GT_SCORE(T_) (el ? dispatch<T_, 1, VWM_SCORE>(a, st) : agg_dispatch<T_, VWM_SCORE>(a, vec, st))
    if (vwm == VWM_NONE) return t == GT_F32 ? GT_SCORE(float) : GT_SCORE(bf16_t);
#undef GT_SCORE
#define GT_GATHER_EL(T_) (vwm == VWM_ADD ? dispatch<T_, 1, VWM_ADD>(a, st) : dispatch<T_, 1, VWM_MUL>(a, st))
#define GT_GATHER_NT(T_)                                                                                                         \
    (vwm == VWM_ADD ? dispatch<T_, 16 / (int)sizeof(T_), VWM_ADD | VWM_NT>(a, st) : dispatch<T_, 16 / (int)sizeof(T_), VWM_MUL | VWM_NT>(a, st))
    if (edge_streams(g->n_edges, VW, ldvw, t, vec, false)) return t == GT_F32 ? GT_GATHER_NT(float) : GT_GATHER_NT(bf16_t);
#define GT_GATHER(T_) (vwm == VWM_ADD ? agg_dispatch<T_, VWM_ADD>(a, vec, st) : agg_dispatch<T_, VWM_MUL>(a, vec, st))
    if (el) return t == GT_F32 ? GT_GATHER_EL(float) : GT_GATHER_EL(bf16_t);
    return t == GT_F32 ? GT_GATHER(float) : GT_GATHER(bf16_t);
#undef GT_GATHER_EL
#undef GT_GATHER_NT
#undef GT_GATHER
}

// Whether both derivatives of the scaled aggregation come from one gather: rows of at most a wavefront's vectors.  Narrow ones without alignment
// stay with the element-wise kernels.  Where the L2s hold the rows but not the scores, the rows are found there and the places of the products
// are not, and two passes are ahead: rows of up to 128 bytes, on skewed graphs from 2.25 Mi edges on, on uniform graphs of tables up to 10 MB from 1.5 Mi
// on (us, two passes / one: power law, 8.4 M edges, 32 bf16 columns 410 / 435, 128 columns 507 / 455; 4 M edges, 32 columns
// 209 / 227; uniform, 131 K rows, 8.4 M edges, 8 fp32 columns 319 / 437, 32 bf16 columns 375 / 462, 24 fp32 columns 387 / 481; 90 K rows, 2.3 M edges, 20 fp32 columns 104 / 119;
// 262 K rows, 5 M edges, 47 bf16 columns 381 / 326; 262 K rows, 8.4 M edges, 128 columns 772 / 567; 1 M edges, 150 fp32 columns 220 / 143; 60 K edges 14.0 / 9.0.  One over two passes in
// the geometric mean of 2,080 random shapes: power law, rows of 65 to 128 bytes, 1.4 to 2 Mi edges 0.94, 2 to 2.8 Mi 1.01, 2.8 to 4 Mi 1.04; uniform, 2 to 4 Mi edges, tables up to
// 4 MB 1.07 to 1.2, 4 to 8 MB 1.03, 8 to 16 MB 0.96, larger 0.82; under 1 Mi edges 0.6 to 0.86).
bool scale_bwd_joined(const gt_graph *g, gt_dtype t, int64_t F, const void *dY, int64_t lddy, const void *Xs, int64_t ldxs, const void *dXs, int64_t lddxs) {
    const int ve = t == GT_F32 ? 4 : 8;
    const bool vec = vec_ok(t, dY, lddy) && vec_ok(t, Xs, ldxs) && vec_ok(t, dXs, lddxs);
    const int64_t rb = F * (int64_t)gt_dtype_size(t), Mi = (int64_t)1 << 20;
    if (rb <= 128 && (agg_skewed(g->bwd.n_splits, g->bwd.n_long, g->bwd.n_items) ? 4 * g->n_edges > 9 * Mi : 2 * g->n_edges > 3 * Mi && g->n_dst * rb <= 10 * Mi)) return false;
    return g->n_edges > 0 && F <= 64 * ve && (vec || F > 16);
}

gt_status run_scale_bwd(const gt_graph *g, gt_dtype t, int64_t F, const void *dY, int64_t lddy, const void *Xs, int64_t ldxs, const float *W,
                        const float *cmean, void *dXs, int64_t lddxs, float *dW, void *ws, hipStream_t st) {
    const gt_sched &sc = g->bwd;
    AggArgs a{};
    a.items = sc.items; a.n_items = sc.n_items; a.n_long = sc.n_long; a.max_len = sc.max_len; a.rowptr = sc.rowptr; a.nbr = sc.nbr;
    a.coef = W; a.eidx = g->perm; a.coef2 = cmean;
    a.X = dY; a.ldx = lddy; a.Y = dXs; a.ldy = lddxs; a.F = F;
    a.partials = static_cast<float *>(ws); a.ldp = (F + 7) / 8 * 8;
    a.splits = sc.splits; a.n_splits = sc.n_splits;
    a.table_bytes = g->n_dst * lddy * (int64_t)gt_dtype_size(t);
    a.trace_kind = GT_TRACE_AGG_BWD;
    a.n_rows = sc.n_rows; a.n_edges = g->n_edges;
    const bool vec = vec_ok(t, dY, lddy) && vec_ok(t, Xs, ldxs) && vec_ok(t, dXs, lddxs);
    if (t == GT_F32) return vec ? dispatch_scale_bwd<float, false>(a, Xs, ldxs, dW, st) : dispatch_scale_bwd<float, true>(a, Xs, ldxs, dW, st);
    return vec ? dispatch_scale_bwd<bf16_t, false>(a, Xs, ldxs, dW, st) : dispatch_scale_bwd<bf16_t, true>(a, Xs, ldxs, dW, st);
}

gt_status check_common(const char *fn, const gt_graph *g, gt_dtype t, int64_t F, void *ws, size_t ws_bytes,
                       bool needs_ws) {
    if (!g) return gt_fail(GT_ERR_INVALID_ARG, "%s: g is null", fn);
    if (t != GT_F32 && t != GT_BF16) return gt_fail(GT_ERR_INVALID_ARG, "%s: unknown dtype", fn);
    if (F < 0) return gt_fail(GT_ERR_INVALID_ARG, "%s: F < 0", fn);
    if (g->ew) return gt_fail(GT_ERR_UNSUPPORTED, "%s: the graph carries static edge weights; per-call edge weights "
                                                  "need a plan built without them", fn);
    if (needs_ws && (g->fwd.n_partials > 0 || g->bwd.n_partials > 0)) {
        const size_t need = gt_aggregate_ws_bytes(g, F);
        if (!ws || ((uintptr_t)ws & 255)) return gt_fail(GT_ERR_WORKSPACE, "%s: ws null or not 256-byte aligned", fn);
        if (ws_bytes < need) return gt_fail(GT_ERR_WORKSPACE, "%s: ws_bytes %zu < required %zu", fn, ws_bytes, need);
    }
    return GT_OK;
}

}  // namespace

extern "C" gt_status gt_neighbor_apply_fwd(const gt_graph *g, gt_edge_fn fn_g, gt_dtype t, int64_t F, const void *Xs,
                                           int64_t ldxs, const void *Xd, int64_t ldxd, void *W, int64_t ldw,
                                           void *stream) {
    const char *fn = "gt_neighbor_apply_fwd";
    gt_status s = check_common(fn, g, t, F, nullptr, 0, false);
    if (s != GT_OK) return s;
    if (fn_g != GT_G_DOT && fn_g != GT_G_MUL) return gt_fail(GT_ERR_INVALID_ARG, "%s: unknown edge function", fn);
    if (g->n_edges == 0) return GT_OK;
    if (!W) return gt_fail(GT_ERR_INVALID_ARG, "%s: W is null", fn);
    if (F > 0 && (!Xs || !Xd)) return gt_fail(GT_ERR_INVALID_ARG, "%s: Xs or Xd is null", fn);
    if (ldxs < F || ldxd < F || (fn_g == GT_G_MUL && ldw < F))
        return gt_fail(GT_ERR_INVALID_ARG, "%s: leading dimension smaller than F", fn);
    if (F == 0 && fn_g == GT_G_MUL) return GT_OK;
    return run_edge(g, fn_g == GT_G_DOT ? 2 : 0, t, F, Xd, ldxd, nullptr, Xs, ldxs, W, ldw, (hipStream_t)stream);
}

extern "C" gt_status gt_neighbor_apply_bwd(const gt_graph *g, gt_edge_fn fn_g, gt_dtype t, int64_t F, const void *dW,
                                           int64_t lddw, const void *Xs, int64_t ldxs, const void *Xd, int64_t ldxd,
                                           void *dXs, int64_t lddxs, void *dXd, int64_t lddxd, void *ws,
                                           size_t ws_bytes, void *stream) {
    const char *fn = "gt_neighbor_apply_bwd";
    gt_status s = check_common(fn, g, t, F, ws, ws_bytes, true);
    if (s != GT_OK) return s;
    if (fn_g != GT_G_DOT && fn_g != GT_G_MUL) return gt_fail(GT_ERR_INVALID_ARG, "%s: unknown edge function", fn);
    if (F == 0) return GT_OK;
    if (!Xs || !Xd || !dXs || !dXd || (g->n_edges > 0 && !dW)) return gt_fail(GT_ERR_INVALID_ARG, "%s: null pointer", fn);
    if (ldxs < F || ldxd < F || lddxs < F || lddxd < F || (fn_g == GT_G_MUL && lddw < F))
        return gt_fail(GT_ERR_INVALID_ARG, "%s: leading dimension smaller than F", fn);
    hipStream_t st = (hipStream_t)stream;
    if (fn_g == GT_G_DOT) {
        // dXd[v] = sum_{e in in(v)} dw_e Xs[u];   dXs[u] = sum_{e in out(u)} dw_e Xd[v]
        s = run_gather(g, false, t, F, Xs, ldxs, dXd, lddxd, static_cast<const float *>(dW), false, nullptr, nullptr, 0,
                       VWM_NONE, 0, ws, st);
        if (s != GT_OK) return s;
        return run_gather(g, true, t, F, Xd, ldxd, dXs, lddxs, static_cast<const float *>(dW), true, nullptr, nullptr, 0,
                          VWM_NONE, 0, ws, st);
    }
    // dXd[v] = sum_e dW_e (.) Xs[u];   dXs[u] = sum_e dW_e (.) Xd[v]
    s = run_gather(g, false, t, F, Xs, ldxs, dXd, lddxd, nullptr, false, nullptr, dW, lddw, VWM_MUL, 0, ws, st);
    if (s != GT_OK) return s;
    return run_gather(g, true, t, F, Xd, ldxd, dXs, lddxs, nullptr, true, nullptr, dW, lddw, VWM_MUL, 0, ws, st);
}

extern "C" gt_status gt_pull_fwd(const gt_graph *g, gt_reduce reduce, gt_weight_fn h, gt_dtype t, int64_t F,
                                 const void *Xs, int64_t ldxs, const void *W, int64_t ldw, void *Y, int64_t ldy,
                                 void *ws, size_t ws_bytes, void *stream) {
    const char *fn = "gt_pull_fwd";
    gt_status s = check_common(fn, g, t, F, ws, ws_bytes, true);
    if (s != GT_OK) return s;
    if (reduce != GT_SUM && reduce != GT_MEAN) return gt_fail(GT_ERR_UNSUPPORTED, "%s: reduce must be GT_SUM or GT_MEAN", fn);
    if (h != GT_H_SCALE && h != GT_H_ADD && h != GT_H_MUL) return gt_fail(GT_ERR_INVALID_ARG, "%s: unknown weight function", fn);
    if (F == 0 || g->n_dst == 0) return GT_OK;
    if (!Y || (g->n_src > 0 && !Xs) || (g->n_edges > 0 && !W)) return gt_fail(GT_ERR_INVALID_ARG, "%s: null pointer", fn);
    if (ldxs < F || ldy < F || (h != GT_H_SCALE && ldw < F)) return gt_fail(GT_ERR_INVALID_ARG, "%s: leading dimension smaller than F", fn);
    const int post = reduce == GT_MEAN ? 2 : 0;
    hipStream_t st = (hipStream_t)stream;
    if (h == GT_H_SCALE)
        return run_gather(g, false, t, F, Xs, ldxs, Y, ldy, static_cast<const float *>(W), false, nullptr, nullptr, 0,
                          VWM_NONE, post, ws, st);
    return run_gather(g, false, t, F, Xs, ldxs, Y, ldy, nullptr, false, nullptr, W, ldw, h == GT_H_ADD ? VWM_ADD : VWM_MUL,
                      post, ws, st);
}

extern "C" gt_status gt_pull_bwd(const gt_graph *g, gt_reduce reduce, gt_weight_fn h, gt_dtype t, int64_t F,
                                 const void *dY, int64_t lddy, const void *Xs, int64_t ldxs, const void *W, int64_t ldw,
                                 void *dXs, int64_t lddxs, void *dW, int64_t lddw, void *ws, size_t ws_bytes,
                                 void *stream) {
    const char *fn = "gt_pull_bwd";
    gt_status s = check_common(fn, g, t, F, ws, ws_bytes, true);
    if (s != GT_OK) return s;
    if (reduce != GT_SUM && reduce != GT_MEAN) return gt_fail(GT_ERR_UNSUPPORTED, "%s: reduce must be GT_SUM or GT_MEAN", fn);
    if (h != GT_H_SCALE && h != GT_H_ADD && h != GT_H_MUL) return gt_fail(GT_ERR_INVALID_ARG, "%s: unknown weight function", fn);
    if (F == 0) return GT_OK;
    if (!dY && g->n_dst > 0) return gt_fail(GT_ERR_INVALID_ARG, "%s: dY is null", fn);
    if ((g->n_src > 0 && (!Xs || !dXs)) || (g->n_edges > 0 && (!W || !dW))) return gt_fail(GT_ERR_INVALID_ARG, "%s: null pointer", fn);
    if (lddy < F || ldxs < F || lddxs < F || (h != GT_H_SCALE && (ldw < F || lddw < F)))
        return gt_fail(GT_ERR_INVALID_ARG, "%s: leading dimension smaller than F", fn);
    hipStream_t st = (hipStream_t)stream;
    const bool mean = reduce == GT_MEAN;
    const float *cmean = (mean && g->n_edges > 0) ? g->coef_mean_b : nullptr;   // 1 / indeg(dst) per transposed entry
    const float *rdeg = mean ? g->rdeg : nullptr;                                // 1 / indeg per destination row
    // gradient of the source embeddings: outputs on the source vertices, transposed structure
    if (h == GT_H_SCALE && scale_bwd_joined(g, t, F, dY, lddy, Xs, ldxs, dXs, lddxs))
        return run_scale_bwd(g, t, F, dY, lddy, Xs, ldxs, static_cast<const float *>(W), cmean, dXs, lddxs, static_cast<float *>(dW), ws, st);
    if (h == GT_H_SCALE) {
        s = run_gather(g, true, t, F, dY, lddy, dXs, lddxs, static_cast<const float *>(W), true, cmean, nullptr, 0,
                       VWM_NONE, 0, ws, st);
    } else if (h == GT_H_ADD) {
        s = run_gather(g, true, t, F, dY, lddy, dXs, lddxs, nullptr, false, cmean, nullptr, 0, VWM_NONE, 0, ws, st);
    } else {
        s = run_gather(g, true, t, F, dY, lddy, dXs, lddxs, nullptr, true, cmean, W, ldw, VWM_MUL, 0, ws, st);
    }
    if (s != GT_OK || g->n_edges == 0) return s;
    // gradient of the edge weights: one value (or row) per edge, destination-centric
    if (h == GT_H_SCALE) return run_edge(g, 2, t, F, dY, lddy, rdeg, Xs, ldxs, dW, 0, st);
    if (h == GT_H_ADD) return run_edge(g, 1, t, F, dY, lddy, rdeg, nullptr, 0, dW, lddw, st);
    return run_edge(g, 0, t, F, dY, lddy, rdeg, Xs, ldxs, dW, lddw, st);
}
