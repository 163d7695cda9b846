// Kernel templates of the neighbour aggregation (included by gt_aggregate.hip and gt_edge.hip).
//
// Neighbour aggregation (the paper's Pull primitive) and its derivative, as one gather-reduce
// kernel family over a work list.
//
// Prior art kept from the paper (Frontend section, "GNN graph aware scheduling" and the Pull
// description): traversal is destination-centric, all features of one output row are handled by
// one group of lanes spread over the feature columns, the running sum stays in registers and the
// row is written once, so no atomics or locks are needed.  What differs for CDNA4 and for full
// power-law graphs: a "group" is G = 4..64 lanes of a 64-wide wavefront, each lane moving
// 16 bytes per gathered row, so narrow rows still issue full-width memory instructions; rows
// longer than 1.5 chunks (a chunk is 512 entries, fewer on small graphs) are cut into chunk-sized work items whose fp32 partial rows
// are added by a second kernel in a fixed order (every n-th one per group of lanes, the groups then in pairs: deterministic, no
// floating-point atomics); work items are ordered longest first so the groups of a wavefront see similar trip counts.
//
// The same kernels serve the backward pass on the transposed structure: the derivative of the
// aggregation is an aggregation whose outputs are the source vertices (paper, "Training for
// GNNs").
#pragma once
#include "gt_internal.h"
#include "gt_trace.h"

#include <type_traits>

struct AggArgs {
    const gt_item *items;
    int64_t n_items;
    const int32_t *rowptr;   // of the output rows (for the mean's divisor)
    const int32_t *nbr;
    const float *coef;       // per-entry coefficient (edge weight x normalisation) or null (= 1)
    const int32_t *eidx;     // entry -> position in coef / VW (the transposed structure's perm), or null (= entry)
    const float *coef2;      // per-entry factor, indexed by the entry itself, or null (= 1): beside coef with VWM_SCORE, instead of it with vector weights
    const void *VW;          // per-entry vector weights [E][ldvw] (type T) for the VWM modes, or null
    int64_t ldvw;
    int post_mode;           // 0 none, 2 divide by the row's entry count (mean, forward)
    const float *bias;       // per-column bias added after scaling, or null
    int relu;
    const void *mask;        // [n_rows][ldmask] of type T or null: outputs are zeroed where mask <= 0 (the
    int64_t ldmask;          // derivative of the ReLU that produced `mask`, applied as the row is written)
    int pad_out;             // a row's last vector may be stored whole, with zeros past F, where it fits below ldy:
                             // a row end written in 2-byte pieces leaves a hole in its 32-byte sector, and memory
                             // has to read the sector back to merge it (2^21 rows of 47 bf16: 0.977 -> 0.918 ms)
    const void *X;
    int64_t ldx;
    void *Y;
    int64_t ldy;
    int64_t F;
    float *partials;         // [n_partials][ldp]
    int64_t ldp;
    const gt_split *splits;
    int64_t n_splits;
    int64_t table_bytes;     // host-side: size of the gathered table (picks the unroll)
    int64_t n_long;          // host-side: the first n_long items are long ones (gt_long_min)
    int n_coop;              // set at launch: the first n_coop workgroups give their items a whole workgroup each
    int coop_waves;          // (4) or a whole wavefront each (1)
    int n_whole;             // set at launch: before those, one workgroup per split row, which sums the whole row (see agg_whole_rows)
    int64_t max_len;         // host-side: entries of the longest split row
    int xcd_run;             // item blocks per XCD run (0 or 1: plain order)
    int slices_lg;           // set at launch: 1 << slices_lg column tiles are shared out over the XCDs (see launch)
    int n_blocks;            // set at launch: workgroups per column tile
    int only_split;          // run only the chunk items of split rows (the whole-row items are someone else's)
    int no_reduce;           // host-side: do not launch the kernel that adds the partial rows
    int64_t chunk_entries;   // host-side: entries of the chunk items where these are all that the launch gathers and they set its form (see launch_u), or 0
    int trace_kind;          // host-side bookkeeping of the optional kernel timing
    int trace_open;          // 1 + the record that the caller has opened for this launch, or 0
    int64_t n_rows, n_edges;
};

// Launches a plain gather (no per-entry vector weights) of `t`: vec as in agg_dispatch; by_element: one element per lane, whatever the
// alignment.  Defined in gt_aggregate.hip, so that the kernel's instances exist once in the library.
gt_status gt_agg_launch(const AggArgs &a, gt_dtype t, bool vec, hipStream_t st, bool by_element = false);

namespace {

typedef uint16_t bf16_t;

__device__ inline float bf16_to_f32(uint32_t h) { return __uint_as_float(h << 16); }

__device__ inline uint32_t f32_to_bf16(float f) { return gt_to_bf16(f); }   // round to nearest even; NaN stays NaN

// Raw (unconverted) V consecutive elements, as they travel from memory: 16 bytes when V > 1.
template <typename T, int V> struct Raw;
template <> struct Raw<float, 4> { typedef float4 type; };
template <> struct Raw<float, 1> { typedef float type; };
template <> struct Raw<bf16_t, 8> { typedef uint4 type; };
template <> struct Raw<bf16_t, 1> { typedef bf16_t type; };

// Rows need only the alignment of their element type (gfx950 takes 16-byte global accesses at any such
// address): the copies below compile to one 16-byte load or store whatever the row stride is.
template <typename T, int V>
__device__ inline typename Raw<T, V>::type load_raw(const T *p) {
    typename Raw<T, V>::type r;
    __builtin_memcpy(&r, p, sizeof(r));
    return r;
}

// acc += c * raw  (fp32 accumulation)
__device__ inline void fma_raw(float (&acc)[4], float c, const float4 &v) {
    acc[0] = fmaf(c, v.x, acc[0]); acc[1] = fmaf(c, v.y, acc[1]);
    acc[2] = fmaf(c, v.z, acc[2]); acc[3] = fmaf(c, v.w, acc[3]);
}
__device__ inline void fma_raw(float (&acc)[1], float c, const float &v) { acc[0] = fmaf(c, v, acc[0]); }
__device__ inline void fma_raw(float (&acc)[8], float c, const uint4 &v) {
    acc[0] = fmaf(c, __uint_as_float(v.x << 16), acc[0]); acc[1] = fmaf(c, __uint_as_float(v.x & 0xffff0000u), acc[1]);
    acc[2] = fmaf(c, __uint_as_float(v.y << 16), acc[2]); acc[3] = fmaf(c, __uint_as_float(v.y & 0xffff0000u), acc[3]);
    acc[4] = fmaf(c, __uint_as_float(v.z << 16), acc[4]); acc[5] = fmaf(c, __uint_as_float(v.z & 0xffff0000u), acc[5]);
    acc[6] = fmaf(c, __uint_as_float(v.w << 16), acc[6]); acc[7] = fmaf(c, __uint_as_float(v.w & 0xffff0000u), acc[7]);
}
__device__ inline void fma_raw(float (&acc)[1], float c, const bf16_t &v) {
    acc[0] = fmaf(c, __uint_as_float((uint32_t)v << 16), acc[0]);
}

// raw -> fp32 values
__device__ inline void unpack_raw(const float4 &v, float (&o)[4]) { o[0] = v.x; o[1] = v.y; o[2] = v.z; o[3] = v.w; }
__device__ inline void unpack_raw(const float &v, float (&o)[1]) { o[0] = v; }
__device__ inline void unpack_raw(const uint4 &v, float (&o)[8]) {
    o[0] = __uint_as_float(v.x << 16); o[1] = __uint_as_float(v.x & 0xffff0000u);
    o[2] = __uint_as_float(v.y << 16); o[3] = __uint_as_float(v.y & 0xffff0000u);
    o[4] = __uint_as_float(v.z << 16); o[5] = __uint_as_float(v.z & 0xffff0000u);
    o[6] = __uint_as_float(v.w << 16); o[7] = __uint_as_float(v.w & 0xffff0000u);
}
__device__ inline void unpack_raw(const bf16_t &v, float (&o)[1]) { o[0] = __uint_as_float((uint32_t)v << 16); }

// Vector-weight modes of the gather (paper: the function h that transforms the source embedding
// with the edge weight before the aggregation): 1: acc += c * (x + w),  2: acc += c * (x * w); VWM_NT beside either: the weights are
// streamed past the caches (see edge_streams).  VWM_SCORE: no vectors, one coefficient per entry, found through the permutation.
enum { VWM_NONE = 0, VWM_ADD = 1, VWM_MUL = 2, VWM_NT = 4, VWM_SCORE = 8 };
constexpr bool agg_plain(int vwm) { return (vwm & 3) == 0; }   // no vectors beside the rows
template <int VWM, int V, typename RawT>
__device__ inline void fma_vw(float (&acc)[V], float c, const RawT &x, const RawT &w) {
    float xf[V], wf[V];
    unpack_raw(x, xf);
    unpack_raw(w, wf);
#pragma unroll
    for (int i = 0; i < V; ++i) {
        const float t = ((VWM & 3) == VWM_ADD) ? xf[i] + wf[i] : xf[i] * wf[i];
        acc[i] = fmaf(c, t, acc[i]);
    }
}

// V consecutive elements starting at p -> fp32
template <typename T, int V>
__device__ inline void load_vec(const T *p, float (&out)[V]) { unpack_raw(load_raw<T, V>(p), out); }

// store the first `n` (<= V) of V values; full vectors go out as 16-byte stores
template <typename T, int V>
__device__ inline void store_vec(T *p, const float (&v)[V], int n);

template <>
__device__ inline void store_vec<float, 4>(float *p, const float (&v)[4], int n) {
    if (n >= 4) {
        const float4 o = make_float4(v[0], v[1], v[2], v[3]);
        __builtin_memcpy(p, &o, 16);
    } else {
        for (int i = 0; i < n; ++i) p[i] = v[i];
    }
}
template <>
__device__ inline void store_vec<float, 1>(float *p, const float (&v)[1], int n) { if (n > 0) p[0] = v[0]; }
template <>
__device__ inline void store_vec<bf16_t, 8>(bf16_t *p, const float (&v)[8], int n) {
    if (n >= 8) {
        uint4 o;
        o.x = gt_pack_bf16(v[0], v[1]);
        o.y = gt_pack_bf16(v[2], v[3]);
        o.z = gt_pack_bf16(v[4], v[5]);
        o.w = gt_pack_bf16(v[6], v[7]);
        __builtin_memcpy(p, &o, 16);
    } else {
        for (int i = 0; i < n; ++i) p[i] = (bf16_t)f32_to_bf16(v[i]);
    }
}
template <>
__device__ inline void store_vec<bf16_t, 1>(bf16_t *p, const float (&v)[1], int n) {
    if (n > 0) p[0] = (bf16_t)f32_to_bf16(v[0]);
}

// The same for data that is read or written once per launch and is larger than the caches (see edge_streams): it leaves the rows
// that are gathered beside it in them.  Aligned whole vectors.
typedef uint32_t nt_vec __attribute__((ext_vector_type(4)));
template <typename T, int V>
__device__ inline void store_vec_nt(T *p, const float (&v)[V], int n) {
    if (n < V) {
        store_vec<T, V>(p, v, n);
        return;
    }
    nt_vec o;
    if constexpr (V == 4) o = {__float_as_uint(v[0]), __float_as_uint(v[1]), __float_as_uint(v[2]), __float_as_uint(v[3])};
    else o = {gt_pack_bf16(v[0], v[1]), gt_pack_bf16(v[2], v[3]), gt_pack_bf16(v[4], v[5]), gt_pack_bf16(v[6], v[7])};
    __builtin_nontemporal_store(o, reinterpret_cast<nt_vec *>(p));
}
template <typename T, int V>
__device__ inline typename Raw<T, V>::type load_raw_nt(const T *p) {
    const nt_vec o = __builtin_nontemporal_load(reinterpret_cast<const nt_vec *>(p));
    typename Raw<T, V>::type r;
    __builtin_memcpy(&r, &o, sizeof(r));
    return r;
}

// SH: rows without 16-byte alignment.  The lane that holds a row's ragged end takes the row's last V columns instead of
// starting at its own column: it repeats some of its neighbour's (and stores the same values there), and every
// access is a whole vector inside the row.  Needs F >= V.
// Lanes past the row's end get its last vector (see the row loads of k_aggregate).
template <bool SH, int V>
__device__ inline int64_t agg_col(int64_t F, int64_t own) {
    const int64_t last = SH ? F - V : (F - 1) / V * V;
    return own > last ? last : own;
}
template <bool SH, int V>
__device__ inline int64_t agg_col(const AggArgs &a, int64_t own) { return agg_col<SH, V>(a.F, own); }

// the mask values of this lane's segments of output row `row` (16-byte loads where the segment is whole);
// issued early by the callers so that the load is not a dependent round trip at the end of the item
template <typename T, int V, int G, int NP, bool SH>
__device__ inline void load_mask_row(const AggArgs &a, int row, int gl, int64_t col0, float (&m)[NP][V]) {
#pragma unroll
    for (int p = 0; p < NP; ++p) {
        const int64_t own = col0 + (int64_t)(p * G + gl) * V;
#pragma unroll
        for (int i = 0; i < V; ++i) m[p][i] = 1.0f;
        if (own >= a.F) continue;
        const int64_t col = agg_col<SH, V>(a, own);
        const int n = (int)((a.F - col) < V ? (a.F - col) : V);
        const T *mp = static_cast<const T *>(a.mask) + (int64_t)row * a.ldmask + col;
        if (n >= V) {
            load_vec<T, V>(mp, m[p]);
        } else {
#pragma unroll
            for (int i = 0; i < V; ++i) {
                float one[1] = {1.0f};
                if (i < n) load_vec<T, 1>(mp + i, one);
                m[p][i] = one[0];
            }
        }
    }
}

// scale, bias, activation and store of one finished output row segment
template <typename T, int V, int G, int NP, bool SH>
__device__ inline void finish_row(const AggArgs &a, int row, int gl, int64_t col0, float (&acc)[NP][V],
                                  const float (&msk)[NP][V]) {
    bool zero = false;
    float div = 1.0f;
    if (a.post_mode == 2) {
        const int d = a.rowptr[row + 1] - a.rowptr[row];
        zero = d <= 0;
        div = (float)(d > 0 ? d : 1);
    }
    T *y = static_cast<T *>(a.Y) + (int64_t)row * a.ldy;
#pragma unroll
    for (int p = 0; p < NP; ++p) {
        const int64_t own = col0 + (int64_t)(p * G + gl) * V;
        if (own >= a.F) continue;
        const int64_t col = agg_col<SH, V>(a, own);
        const int n = (int)((a.F - col) < V ? (a.F - col) : V);
        float o[V];
#pragma unroll
        for (int i = 0; i < V; ++i) {
            float x = acc[p][i];
            if (a.post_mode == 2) x = zero ? 0.0f : x / div;
            if (a.bias && i < n) x += a.bias[col + i];
            if (a.relu) x = x > 0.0f ? x : 0.0f;
            if (a.mask) x = msk[p][i] > 0.0f ? x : 0.0f;
            o[i] = x;
        }
        int nst = n;
        if (V > 1 && a.pad_out && n < V && col + V <= a.ldy) {
#pragma unroll
            for (int i = 0; i < V; ++i) o[i] = i < n ? o[i] : 0.0f;
            nst = V;
        }
        store_vec<T, V>(y + col, o, nst);
    }
}

// Item block of workgroup `bx` of `n` under the XCD-run order (run: a power of two, 1: plain order), where consecutive workgroups go
// to 1 << xcds_lg XCDs in turn.  The remapping is a bijection on the blocks of every complete group of run blocks per XCD; the
// ragged end of the grid keeps the plain order.
__device__ inline int agg_item_block(int run, int bx, int n, int xcds_lg) {
    const int super = run << xcds_lg, w = bx & (super - 1);
    if (run > 1 && bx < (n & ~(super - 1))) bx = bx - w + (w & ((1 << xcds_lg) - 1)) * run + (w >> xcds_lg);
    return bx;
}

// Run length for a grid of gx item blocks: as long as possible for L2 reuse, but at least 64 turns
// over the 8 XCDs so that the longest-first order stays balanced (measured on MI355X: 2^18-vertex
// graph, 512-byte rows, 0.58 -> 0.50 ms at 64; narrow rows and small grids prefer 16-32; 256 was
// slower than 64 on a 2^21-vertex graph).
static inline int agg_xcd_run(int64_t gx) {
    int run = 1;
    while (run < 64 && (int64_t)run * 2 * 512 <= gx) run *= 2;
    return run;
}

// Instances with cooperative workgroups for the long items
template <int NP, int VWM>
constexpr bool agg_coop() { return NP == 1 && agg_plain(VWM); }

// Whether a launch that shares its long items out gives each split row a workgroup instead of cutting it into chunks: the row is finished there,
// and the launch that adds the partial rows is saved.  Up to rows of 64 entries per group, whose sum takes about as long as that
// launch (us, partial rows / whole rows: 5 K rows, 50 K power-law edges, 16 fp32 columns, both directions 31.7 / 24.6; a training step on 4 K rows,
// 61 K edges 77 / 68; with 256 entries per group 50 K rows, 500 K edges, 100 bf16 columns 41 / 78).
static inline bool agg_whole_rows(const AggArgs &a, int G) { return a.n_splits > 0 && !a.only_split && !a.no_reduce && a.max_len > 0 && a.max_len * G <= 16384; }

// Ids that a lane of a narrow group may hold per batch: sixteen per group
constexpr int agg_many_ids(int G) { return G >= 16 ? 1 : 16 / G; }

// Wavefronts per SIMD that the registers have to leave room for: eight where one register past 64 cost one (41 fp32 columns without
// alignment, 262 K rows, 12 M edges, in a training step 190 us with 64, 192.5 with 65; rows of up to 64 bytes gain nothing by it, 2 M rows, 52 M edges, 8
// columns, backward 644 with five wavefronts, 697 with six)
template <typename T, int V, int G, int NP, int U, int VWM, bool MK>
constexpr int agg_waves() { return V == 4 && (G == 16 || G == 32) && NP == 1 && U == 8 && VWM == VWM_NONE && !MK ? 8 : 1; }

// One group of G lanes per work item; 64/G items per wavefront; 4 wavefronts per workgroup.
// blockIdx.y selects a column tile of G*V*NP columns.
// MK: an output mask is present (its values are fetched when the item starts; a separate instance so
// that the registers they occupy during the gather cost the unmasked kernel nothing)
// COOP: 1: long items are shared out; 2: and split rows are summed whole (separate instances for the same reason)
// IPL: neighbour ids per lane and batch
template <typename T, int V, int G, int NP, int U, int VWM, bool MK, bool SH, int COOP, int IPL>
__global__ void __launch_bounds__(256, (agg_waves<T, V, G, NP, U, VWM, MK>())) k_aggregate(const AggArgs a) {
    constexpr int NG = 64 / G;
    const int lane = threadIdx.x & 63;
    const int wave = threadIdx.x >> 6;
    const int gl = lane & (G - 1);
    const int grp = lane / G;
    // Workgroups go to the 8 XCDs round-robin by index, and every XCD has its own L2.  Items are
    // sorted so that neighbours in the list gather from the same slice of the table; runs of
    // xcd_run consecutive item blocks are therefore handed to ONE XCD (the runs themselves still
    // rotate over the XCDs, which keeps the longest-first order balanced).
    // Cooperative items: a long item walked by one group of lanes is a chain of len / U round trips, and narrow rows pack
    // 64 / G such chains into one wavefront; a graph of a few million edges has nothing to hide them behind
    // (100 K vertices, 3 M edges, 15 fp32 columns, both directions: 247 -> 101 us).  The first n_coop workgroups therefore
    // give each of their items all groups of the workgroup or of one wavefront (coop_waves, see launch): every group sums a slice,
    // and the slices are added in a fixed order.
    // Column tiles may be shared out over the XCDs (slices_lg, see launch): the XCDs of one tile then walk the whole list.
    int bx = blockIdx.x, slice = 0;
    if (a.slices_lg > 0) {
        const int xcd = bx & 7;
        slice = xcd & ((1 << a.slices_lg) - 1);
        bx = ((bx >> 3) << (3 - a.slices_lg)) + (xcd >> a.slices_lg);
    }
    const int whole = COOP == 2 ? a.n_whole : 0;
    const bool all_row = COOP == 2 && bx < whole;   // uniform over the workgroup, as the next two
    bx -= whole;
    const bool coop = COOP && bx < a.n_coop;
    const bool one_wave = COOP && a.coop_waves == 1 && !all_row;
    const int first = COOP ? a.n_coop : 0;
    const int64_t item_id = coop ? (one_wave ? (int64_t)bx * 4 + wave : (int64_t)bx)
                                 : (int64_t)first * (one_wave ? 4 : 1) +
                                       ((int64_t)agg_item_block(a.xcd_run, bx - first, a.n_blocks - whole - first, 3 - a.slices_lg) * 4 + wave) * NG + grp;
    int row, e0, e1, slot;
    if (all_row) {
        row = a.splits[bx + whole].row;
        e0 = a.rowptr[row];
        e1 = a.rowptr[row + 1];
        slot = -1;
    } else {
        if (item_id >= a.n_items) return;   // whole groups leave together; the only barrier below is the cooperative one
        const int4 raw = reinterpret_cast<const int4 *>(a.items)[item_id];
        row = raw.x; e0 = raw.y; e1 = raw.z; slot = raw.w;
        if (a.only_split && slot < 0) return;   // uniform within the group
        if (COOP == 2 && slot >= 0) return;   // (summed with its row)
    }
    if (coop) {   // this group's slice
        const int ng = one_wave ? NG : 4 * NG;
        const int per = (e1 - e0 + ng - 1) / ng;
        const int s0 = e0 + (one_wave ? grp : wave * NG + grp) * per;
        e1 = s0 + per < e1 ? s0 + per : e1;
        e0 = s0;   // (may lie past e1: an empty slice)
    }
    if constexpr (G == 64) {   // one item per wavefront: keep its bounds in scalar registers
        row = __builtin_amdgcn_readfirstlane(row);
        e0 = __builtin_amdgcn_readfirstlane(e0);
        e1 = __builtin_amdgcn_readfirstlane(e1);
        slot = __builtin_amdgcn_readfirstlane(slot);
    }
    const int64_t col0 = ((int64_t)blockIdx.y * (1 << a.slices_lg) + slice) * (G * V * NP);
    const T *X = static_cast<const T *>(a.X);

    float acc[NP][V];
#pragma unroll
    for (int p = 0; p < NP; ++p)
#pragma unroll
        for (int i = 0; i < V; ++i) acc[p][i] = 0.0f;
    float msk[NP][V];
#pragma unroll
    for (int p = 0; p < NP; ++p)
#pragma unroll
        for (int i = 0; i < V; ++i) msk[p][i] = 1.0f;
    if constexpr (MK) {
        if (slot < 0) load_mask_row<T, V, G, NP, SH>(a, row, gl, col0, msk);   // needed only when the row is finished here
    }

    typedef typename Raw<T, V>::type raw_t;
    // The group fetches GB neighbour ids and coefficients with coalesced loads and walks them; the next GB are requested
    // before the current ones are used, so the id fetch of the next batch overlaps the row gathers of this one.
    constexpr int GB = G * IPL;
    // A coefficient that is looked up through the permutation (VWM_SCORE) waits for its place there.  EARLY: the places are requested a batch
    // earlier still, and the two factors of an entry are multiplied when they are used, so that no load waits for another between the row loads.  That is
    // ahead in groups of four lanes, and of eight and sixteen with eight rows in flight.  The others have rows in flight without it, and wait for every score
    // before the next place is asked for, which leaves the L2s to the rows.  The transposed gather alone, us, places early / waited for: power law, 262 K rows, 8.4 M edges,
    // 4 to 16 fp32 columns 0.84, 32 fp32 columns 0.96, 128 bf16 columns 0.98 of the time; uniform, 500 K rows, 8 M edges, 16 fp32 columns 304 / 328, 60 K rows, 2.2 M edges 49 / 55 (with exactly 36 entries
    // each 44 / 41); 131 K rows, 8.4 M edges, 47 bf16 columns without alignment 264 / 238; 64 bf16 columns and more, 32 fp32 columns and more, uniform: 1.00 to 1.21
    // of the time.
    constexpr bool SCORE = VWM == VWM_SCORE, EARLY = SCORE && (G == 4 || (G <= 16 && U == 8 && IPL == 1));
    int idx_next[IPL], ei_next[IPL];
    float c_next[IPL], f_next[IPL];
    if constexpr (EARLY) {
#pragma unroll
        for (int k = 0; k < IPL; ++k) {   // the first batch's places; the second's follow
            const int e = e0 + k * G + gl;
            ei_next[k] = 0;
            if (e < e1) ei_next[k] = a.eidx[e];
        }
    }
    int ei_later[IPL];
    auto places = [&](int base, int ahead) {
#pragma unroll
        for (int k = 0; k < IPL; ++k) {
            const int d = ahead + k * G + gl;
            ei_later[k] = 0;
            if (d < e1 - base) ei_later[k] = a.eidx[base + d];
        }
    };
    auto fetch = [&](int e_first) {
#pragma unroll
        for (int k = 0; k < IPL; ++k) {
            const int e = e_first + k * G + gl;
            idx_next[k] = 0;
            c_next[k] = 0.0f;
            f_next[k] = 1.0f;
            if constexpr (!EARLY) ei_next[k] = 0;
            if (e < e1) {
                idx_next[k] = a.nbr[e];
                if constexpr (EARLY) {
                    c_next[k] = a.coef[ei_next[k]];
                    if (a.coef2) f_next[k] = a.coef2[e];
                } else if constexpr (SCORE) {
                    ei_next[k] = a.eidx[e];
                    c_next[k] = a.coef[ei_next[k]];
                    if (a.coef2) c_next[k] *= a.coef2[e];
                    __builtin_amdgcn_s_waitcnt(0x0f70);   // vmcnt(0)
                } else if constexpr (VWM == VWM_NONE) {
                    // Groups of four lanes ask for the next batch's coefficients when its ids are there, which leaves the L2s to the rows in the same way (uniform
                    // graphs, derivative of the mean, 264 shapes of one row in flight 0.905 of the time waiting for nothing 0.935; at most 1.13 and 1.36 of it).
                    if constexpr (G == 4 && IPL > 1)
                        if (a.coef) __builtin_amdgcn_s_waitcnt(0x0f70);   // vmcnt(0)
                    c_next[k] = a.coef ? a.coef[e] : 1.0f;
                } else {
                    ei_next[k] = a.eidx ? a.eidx[e] : e;
                    c_next[k] = a.coef2 ? a.coef2[e] : 1.0f;
                }
            }
        }
    };
    if constexpr (EARLY) places(e0, GB);
    fetch(e0);
    const T *VWp = static_cast<const T *>(a.VW);
    // This lane's columns, counted from the tile's first one.  Lanes past the row's end repeat its last vector, in sums that nobody stores: a line
    // that is read anyway, and no branch around the load.  Where rows are not aligned that vector mostly lies in two lines, and these
    // lanes load nothing (IDLE; power law, 6.5 M edges, 161 bf16 columns of 32 lanes 239 us without it, 214 with it; 100 K rows, 2 M edges, 81 / 72),
    // except where what counts is how soon the loads leave (eight in flight or wide tiles; power law, 61 K edges, 602 fp32 columns 25 / 29).
    constexpr bool IDLE = SH && (U == 1 || (U == 2 && NP == 1) || G == 32);
    const T *Xt = X + col0, *VWt = VWp + col0;
    constexpr int TILE = G * V * NP;
    const int64_t left = a.F - col0, at = SH ? left - V : (left - 1) / V * V;
    const int width = left < TILE ? (int)left : TILE, last = at < TILE ? (int)at : TILE;
    int col[NP];
#pragma unroll
    for (int p = 0; p < NP; ++p) col[p] = (p * G + gl) * V > last ? last : (p * G + gl) * V;
    for (int base = e0; base < e1; base += GB) {
        int idx[IPL], ei[IPL];
        float c[IPL];
#pragma unroll
        for (int k = 0; k < IPL; ++k) {
            idx[k] = idx_next[k];
            ei[k] = ei_next[k];
            c[k] = EARLY ? c_next[k] * f_next[k] : c_next[k];
            if constexpr (EARLY) ei_next[k] = ei_later[k];
        }
        fetch(base + GB);
        if constexpr (EARLY) places(base, 2 * GB);
        const int cnt = (e1 - base) < GB ? (e1 - base) : GB;
        // entries j .. j + N - 1 of the batch (j is a constant where IPL > 1); ALL: every one of them is there, and the loads are
        // branch free (with a branch around each, the exchange that brings its id and the load wait for one another)
        auto step = [&](int j, auto n, auto all) {
            constexpr int N = decltype(n)::value;
            constexpr bool ALL = decltype(all)::value;
            raw_t v[N][NP];
            raw_t w[agg_plain(VWM) ? 1 : N][agg_plain(VWM) ? 1 : NP];
            float cj[N];
            int src[N], we[N];
#pragma unroll
            for (int u = 0; u < N; ++u) {
                const int jj = j + u, k = IPL > 1 ? jj / G : 0;
                we[u] = 0;
                if constexpr (G == 64) {   // wave-uniform: scalar broadcast, scalar row base
                    src[u] = __builtin_amdgcn_readlane(idx[0], jj & 63);
                    cj[u] = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(c[0]), jj & 63));
                    if constexpr (!agg_plain(VWM)) we[u] = __builtin_amdgcn_readlane(ei[0], jj & 63);
                } else {
                    src[u] = __shfl(idx[k], jj & (G - 1), G);
                    cj[u] = __shfl(c[k], jj & (G - 1), G);
                    if constexpr (!agg_plain(VWM)) we[u] = __shfl(ei[k], jj & (G - 1), G);
                }
                if (!ALL && jj >= cnt) cj[u] = 0.0f;
            }
            auto load = [&](int u, int p, const T *xr) {
                v[u][p] = load_raw<T, V>(xr + col[p]);
                if constexpr (!agg_plain(VWM)) {
                    const T *wr = VWt + (int64_t)we[u] * a.ldvw + col[p];
                    if constexpr ((VWM & VWM_NT) != 0) w[u][p] = load_raw_nt<T, V>(wr);
                    else w[u][p] = load_raw<T, V>(wr);
                }
            };
            if constexpr (ALL && IDLE) {
#pragma unroll
                for (int u = 0; u < N; ++u)   // (ahead of all loads: a register that is zeroed between them waits for those in flight)
#pragma unroll
                    for (int p = 0; p < NP; ++p) {
                        v[u][p] = raw_t{};
                        if constexpr (!agg_plain(VWM)) w[u][p] = raw_t{};
                    }
#pragma unroll
                for (int p = 0; p < NP; ++p)
                    if ((p * G + gl) * V < width)
#pragma unroll
                        for (int u = 0; u < N; ++u) load(u, p, Xt + (int64_t)src[u] * a.ldx);
            } else {
#pragma unroll
                for (int u = 0; u < N; ++u) {
                    const T *xr = Xt + (int64_t)src[u] * a.ldx;
#pragma unroll
                    for (int p = 0; p < NP; ++p) {
                        if constexpr (!ALL) {
                            v[u][p] = raw_t{};
                            if constexpr (!agg_plain(VWM)) w[u][p] = raw_t{};
                        }
                        if (ALL || (j + u < cnt && (!IDLE || (p * G + gl) * V < width))) load(u, p, xr);
                    }
                }
            }
#pragma unroll
            for (int u = 0; u < N; ++u)
#pragma unroll
                for (int p = 0; p < NP; ++p) {
                    if constexpr (agg_plain(VWM)) fma_raw(acc[p], cj[u], v[u][p]);
                    else fma_vw<VWM, V>(acc[p], cj[u], v[u][p], w[u][p]);
                }
        };
        // At most two rows in flight: a last entry of an odd number by itself.  With eight, a remainder step of its own is a round trip more for
        // every batch that is no multiple of eight (power law, 1.5 M edges, 280 bf16 columns shared out, 99 us without it, 126 with it); with
        // weights' vectors beside the rows it pays all the same (4.2 M edges, 64 fp32 columns, 1254 and 1220).
        constexpr std::integral_constant<int, U> some{};
        constexpr std::integral_constant<int, 1> single{};
        if constexpr (IPL == 1) {
            int j = 0;
            if constexpr (U <= 2 || !agg_plain(VWM))
                for (; j + U <= cnt; j += U) step(j, some, std::true_type{});
            if constexpr (U <= 2) {
                if (U == 2 && j < cnt) step(j, single, std::true_type{});
            } else {
                for (; j < cnt; j += U) step(j, some, std::false_type{});
            }
        } else {
#pragma unroll
            for (int j = 0; j < GB; j += U) {
                if (j + U <= cnt) step(j, some, std::true_type{});
                else if constexpr (U > 2) {
                    if (j < cnt) step(j, some, std::false_type{});
                } else if constexpr (U == 2) {
                    if (j < cnt) step(j, single, std::true_type{});
                }
            }
        }
    }

    if constexpr (COOP != 0) {
        __shared__ float red[4][G * V];
        if (coop) {
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
                for (int i = 0; i < V; ++i)
                    acc[0][i] = ((red[0][i * G + gl] + red[1][i * G + gl]) + red[2][i * G + gl]) + red[3][i * G + gl];
        }
    }
    if (slot >= 0) {
        float *P = a.partials + (int64_t)slot * a.ldp;
#pragma unroll
        for (int p = 0; p < NP; ++p) {
            const int64_t own = col0 + (int64_t)(p * G + gl) * V;
            if (own >= a.F) continue;
            const int64_t col = agg_col<SH, V>(a, own);   // (partial rows are padded to 8 floats: a whole vector always fits)
            if constexpr (V == 1) {
                P[col] = acc[p][0];
            } else {
#pragma unroll
                for (int q = 0; q < V / 4; ++q) {
                    const float4 x = make_float4(acc[p][4 * q], acc[p][4 * q + 1], acc[p][4 * q + 2], acc[p][4 * q + 3]);
                    __builtin_memcpy(P + col + 4 * q, &x, 16);
                }
            }
        }
    } else {
        finish_row<T, V, G, NP, SH>(a, row, gl, col0, acc, msk);
    }
}

// Second pass for split rows: add the row's partial rows.  One wavefront per row: its 64 / G groups take every (64 / G)-th
// partial row each, in order, and their sums are added pairwise (a fixed order).  The kernel lasts as long as its
// longest row, which one group alone walked 16 partial rows at a time (2^21 vertices, 170 partial rows on the longest: 22 -> 12 us).
template <typename T, int V, int G, int NP, bool SH>
__global__ void __launch_bounds__(256) k_reduce_partials(const AggArgs a) {
    constexpr int NG = 64 / G;
    const int lane = threadIdx.x & 63;
    const int wave = threadIdx.x >> 6;
    const int gl = lane & (G - 1);
    const int grp = lane / G;
    const int64_t sid = (int64_t)blockIdx.x * 4 + wave;
    if (sid >= a.n_splits) return;
    const gt_split s = a.splits[sid];
    const int64_t col0 = (int64_t)blockIdx.y * (G * V * NP);
    float acc[NP][V];
#pragma unroll
    for (int p = 0; p < NP; ++p)
#pragma unroll
        for (int i = 0; i < V; ++i) acc[p][i] = 0.0f;
    float msk[NP][V];
#pragma unroll
    for (int p = 0; p < NP; ++p)
#pragma unroll
        for (int i = 0; i < V; ++i) msk[p][i] = 1.0f;
    if (a.mask) load_mask_row<T, V, G, NP, SH>(a, s.row, gl, col0, msk);
    // UR partial rows per group are requested at a time (branch free: a request past the end re-reads the last row
    // and is discarded).  Partial rows are padded to a multiple of 8 floats, so whole vectors can be read;
    // padding lanes are never stored.
    constexpr int UR = NP * V <= 4 ? 16 : (NP * V <= 16 ? 8 : 4);
    for (int k = grp; k < s.count; k += UR * NG) {
        float t[UR][NP][V];
#pragma unroll
        for (int u = 0; u < UR; ++u) {
            const int kk = (k + u * NG < s.count) ? k + u * NG : s.count - 1;
            const float *P = a.partials + (int64_t)(s.first + kk) * a.ldp;
#pragma unroll
            for (int p = 0; p < NP; ++p) {
                const int64_t own = col0 + (int64_t)(p * G + gl) * V;
                const int64_t c = own < a.F ? agg_col<SH, V>(a, own) : 0;
                if constexpr (V == 1) {
                    t[u][p][0] = P[c];
                } else {
#pragma unroll
                    for (int q = 0; q < V / 4; ++q) {
                        const float4 x = load_raw<float, 4>(P + c + 4 * q);
                        t[u][p][4 * q + 0] = x.x; t[u][p][4 * q + 1] = x.y;
                        t[u][p][4 * q + 2] = x.z; t[u][p][4 * q + 3] = x.w;
                    }
                }
            }
        }
#pragma unroll
        for (int u = 0; u < UR; ++u) {
            const bool live = k + u * NG < s.count;
#pragma unroll
            for (int p = 0; p < NP; ++p)
#pragma unroll
                for (int i = 0; i < V; ++i) acc[p][i] += live ? t[u][p][i] : 0.0f;
        }
    }
#pragma unroll
    for (int o = G; o < 64; o <<= 1)
#pragma unroll
        for (int p = 0; p < NP; ++p)
#pragma unroll
            for (int i = 0; i < V; ++i) acc[p][i] += __shfl_xor(acc[p][i], o, 64);
    if (grp == 0) finish_row<T, V, G, NP, SH>(a, s.row, gl, col0, acc, msk);
}

// What a launch gathers
static inline int64_t agg_entries(const AggArgs &a) { return a.chunk_entries > 0 ? a.chunk_entries : a.n_edges; }
template <typename T>
static inline double agg_bytes(const AggArgs &a) { return (double)agg_entries(a) * (double)a.F * sizeof(T); }

// Skewed: rows longer than 1.5 chunks exist, and most items are not long.  A long item is then a chain of up to 1.5 chunk / U round
// trips while the other items of the launch are soon done; where every row is long (and about as long as the next one), no
// chain outlasts the others and sharing them out only cuts the work into small pieces (uniform graph, degree 130, 4 M edges,
// 8 fp32 columns: 27 us, shared out 55; 128 bf16 columns 59 and 94).  Power-law graphs with chunks of 64 reach 0.3 long items to an item
// (20,000 vertices, 500 K edges, 128 fp32 columns, both directions 56 us alone, 40 shared out).
static inline bool agg_skewed(int64_t n_splits, int64_t n_long, int64_t n_items) { return n_splits > 0 && n_long * 5 <= n_items * 2; }
static inline bool agg_skewed(const AggArgs &a) { return agg_skewed(a.n_splits, a.n_long, a.n_items); }

// Whether a launch shares its long items out.  Either it has too few items to fill the chip (less than about two wavefronts per SIMD):
// uniform graph, degree 600, 4 M edges, 41 fp32 columns 63 us alone, 43 shared out.  Or it is skewed, and gathers so little that the
// rest does not hide the chains.  A chain's time goes with the chunk, the rest's with the bytes: with two rows in flight (U == 2; rows of
// more than 256 bytes, which take eight only where they are shared out) the line lies at 5 MB per entry of the chunk, at 8 MB where the
// table fits the L2s and the rest is faster; with eight in flight and a table past 64 MB at a quarter of that.  us, both directions, alone / shared out, power-law graphs: chunk 128, 128 fp32 columns
// 0.33 GB 112 / 88, 230 columns 0.60 GB 163 / 168; chunk 256, 128 columns 0.61 GB 195 / 125, 500 bf16 columns 1.35 GB 213 / 223; chunk 512,
// 230 columns 2.5 GB 554 / 422, 128 columns 2.9 GB 616 / 710; a 29 MB table, chunk 512, 128 columns 3.1 GB 401 / 295; eight in flight, a 67 MB
// table, chunk 512, 41 columns 0.5 GB 204 / 168, 0.9 GB 220 / 238.
// Smaller tables of narrow rows, one direction: 41 fp32 columns 1.9 GB 172 / 162, 2.7 GB 396 / 403; 128 bf16 columns 1.1 GB 92 / 71, 2.1 GB
// 154 / 165; 64 bf16 columns 1.5 GB 104 / 97; U == 2: 64 bf16 columns 2.1 GB 312 / 243, 3.4 GB 306 / 330.
static inline bool agg_share_out(const AggArgs &a, int G, int U, double bytes) {
    if (a.n_long > 0 && a.n_items * G <= 1792 * 64) return true;
    if (!agg_skewed(a)) return false;
    if (a.chunk_entries > 0) return bytes <= 2.0e9;   // (nothing else in the launch hides them, whatever the table)
    const double chunk = gt_chunk_for(a.n_edges);
    if (G >= 32) return bytes <= chunk * (a.table_bytes <= ((int64_t)32 << 20) ? 8.0e6 : 5.0e6);
    if (U == 8 && G >= 8 && a.table_bytes > ((int64_t)64 << 20)) return bytes <= chunk * 1.25e6;
    return bytes <= (U <= 2 && G <= 8 ? 3.0e9 : 2.0e9);
}

// Whether a narrow group holds several ids per lane (batches of 16 ids instead of 4 or 8, at the price of registers).  It pays on
// launches of millions of edges whose rows are not uniformly long: with four lanes from about four entries per row (us, one id / several, uniform
// graphs, mean backward, 16 fp32 columns: 1 M rows of degree 6 182 / 167, of degree 11 325 / 278, of degree 4 128 / 123; degree 3, forward, 15 bf16 columns 84 / 86;
// 1 M edges 13.0 / 13.6); with eight lanes, where rows fill a batch (64 bf16 columns: 1 M rows of degree 8 192 / 201, of degree 14, backward,
// 339 / 329) and no chain of a long row is lengthened by it: next to no long rows, or a launch that hides them (power law, 47 bf16
// columns 52 M edges 798 / 777, 64 bf16 columns 26 M edges 306 / 327; degree 130, 12 M edges, 32 bf16 columns 77 / 89).
static inline bool agg_long_batches(const AggArgs &a, int G, double bytes) {
    return agg_entries(a) >= ((int64_t)2 << 20) && agg_entries(a) >= (G == 4 ? 4 : 12) * a.n_items && a.n_long * 4 <= a.n_items &&
           (G == 4 || a.n_long * 1024 <= a.n_rows || bytes > 4.0e9);
}
// ... and with rows long enough that vectors and long batches outdo elements on narrow fp32 rows without alignment (see agg_dispatch)
static inline bool agg_vectors_pay(const AggArgs &a, double bytes) {
    return a.n_edges >= 12 * a.n_items && agg_long_batches(a, 4, bytes);
}

// Whether rows of more than 256 bytes keep eight loads in flight (see launch_u)
static inline bool agg_wide_eight(const AggArgs &a, int G, double bytes) { return agg_share_out(a, G, 8, bytes) && a.table_bytes <= ((int64_t)32 << 20); }

// Rows of more than 256 bytes may be cut into column tiles of 256 bytes (G = 16) or 512 (G = 32): the groups read shorter pieces of more
// rows at a time, and what an L2 has to hold of a popular row is one tile of it.  The tiles of a launch either follow one another
// (grid.y), or, in pairs, share out the XCDs (slices_lg = 1): four XCDs walk the list for one tile, four for the other, so each L2
// holds twice as many rows and no tile has to wait for the long items of the one before.  us, whole rows / tiles, one direction:
// power law, 262 K rows, 12 M edges, 128 fp32 columns 415 / 367, 256 columns 1067 / 776; 524 K rows, 13 M edges, 256 bf16 columns 687 / 582;
// 66 K rows, 1 M edges, 256 fp32 columns 103 / 73; uniform, 66 K rows, 1.6 M edges, 128 fp32 columns 94 / 75, 512 columns 455 / 296;
// 1 M rows, 17 M edges, 128 columns 1240 / 1263.
//  * Only where a tile begins and ends with a line: otherwise each end costs a line more (uniform, 200 K rows, 3 M edges, 300 fp32
//    columns 545 / 728; power law, 262 K rows, 6.5 M edges, 200 columns 451 / 501).  Such power-law rows of more than two vectors per lane of
//    a wavefront lose more by that width: 512-byte tiles there (602 fp32 columns, 12 M edges 2869 / 2146, 1.6 M edges 327 / 285) and, in tables past
//    256 MB, from one on (304 MB, 602 bf16 columns 787 / 696); 256-byte ones on aligned rows past 512 MB, where only the L2s are left to hit (638 MB, 602
//    bf16 columns 889 / 753, in 512-byte tiles 833).
//  * Uniform graphs of few entries per row lose by tiles of whole wavefronts' rows as long as the table is beyond the L2s and not far beyond the
//    last-level cache (degree 4, 66 K rows, 1024 fp32 columns 192 / 219, 131 K rows, 640 columns 237 / 264; 16 K rows, 1024 columns 51 / 41 and 1 M rows, 512 columns 1.00 / 0.84 gain
//    all the same; 128 columns 0.99 / 1.03), others by three or four tiles of such a table (262 K rows of degree 10, 224 columns
//    350 / 377, 300 K rows of degree 20, 192 columns 628 / 665).  So do gathers that look their coefficients up by entry, once per tile (200 K rows of
//    degree 10, 160 columns, backward 433 / 516).
//  * The two tiles of the first pair have to be nearly full (96 fp32 columns, power law, 262 K rows 267 / 278); a half empty last one of
//    four still pays (224 columns, 21 power-law graphs, geometric mean: paired 0.90 of the rows whole, one after the other 0.93).
//  * Pairs share out the XCDs on skewed graphs of tables up to 600 MB (537 MB, 256 bf16 columns 1229, one after the other 1250; 1.07 GB
//    3384 and 3193) and in small launches of uniform ones (16 K rows, 262 K edges 13.7 and 15.1; 131 K rows, 3.3 M edges 201 and 193).
//  * Skewed launches keep whole rows below half a gigabyte (33 K rows, 0.8 M edges, 128 fp32 columns 29 / 32) and where those have eight loads in
//    flight (20 K rows, 0.5 M edges, 256 columns 36 / 58, 0.9 M edges 50 / 64).
//  * Uniform tiles keep two rows in flight; one where rows are long and the table beyond the L2s (131 K rows of degree 25, 256 columns 402 / 374, 1 M rows
//    of degree 16, 1024 columns 10.5 / 10.1 ms; degree 8, 256 columns 1320 / 1340).
//  * Eight rows in flight and long items shared out where the chains of long items matter: tiles that gather at most 2.9 GB one after the
//    other from at most 450 MB (us, that / two rows in flight alone: 131 K rows, 3.3 M edges, 128 columns 103 / 120; 262 K rows, 12 M edges, 160 columns
//    464 / 504; 262 K rows, 2.6 M edges, 320 columns 310 / 449; 6.5 M edges, 128 columns, 3.4 GB 260 / 224).  Chunks of graphs below a million edges
//    make no chains (512 columns, 0.5 M edges 114 / 72, 0.66 M edges 123 / 116).  Beyond, two in flight, shared out from 32 entries per item on
//    (12 M edges, degree 45, symmetric norm 429 / 449) and where a tile gathers up to 1.7 GB (524 K rows, 5.2 M edges, 160 columns, backward 476 alone,
//    381; 10 M edges 725 and 775).
struct AggTiles { int G, U, slices_lg; bool share; };   // G 0: the row whole
static inline AggTiles agg_tiles(const AggArgs &a, bool shifted, int64_t nvec, size_t es, double bytes) {
    const bool lines = (a.ldx * (int64_t)es) % 128 == 0 && ((uintptr_t)a.X & 127) == 0;
    const int64_t tiles = (nvec + 15) / 16, MB = (int64_t)1 << 20;
    const AggTiles whole = {0, 0, 0, false};
    if (nvec < 28) return whole;
    if (!agg_skewed(a)) {
        if (!lines || a.eidx) return whole;
        if (a.n_edges < 10 * a.n_items ? a.table_bytes < 600 * MB && (nvec <= 32 || (nvec >= 56 && a.table_bytes > 80 * MB))
                                      : nvec > 32 && nvec < 64 && a.table_bytes > (a.n_edges < 16 * a.n_items ? 80 : 140) * MB && a.table_bytes < 300 * MB)
            return whole;
        const bool few = a.n_long > 0 && a.n_items * 16 <= 1792 * 64;
        return {16, a.n_edges >= 12 * a.n_items && a.table_bytes > 80 * MB ? 1 : 2, tiles % 2 == 0 && bytes < 0.3e9 ? 1 : 0, few};
    }
    if (bytes < 0.5e9) return whole;
    const int lg = tiles % 2 == 0 && a.table_bytes <= 600 * MB ? 1 : 0;
    const bool share = a.n_long > 0 && (a.n_edges >= 32 * a.n_items || (double)a.n_edges * 256 <= 1.7e9);
    if (!lines) {
        if (nvec < 64 || (nvec <= 128 && a.table_bytes <= 256 * MB)) return whole;
        return nvec <= 128 && !shifted && a.table_bytes > 512 * MB ? AggTiles{16, 2, 0, share} : AggTiles{32, 2, 0, false};
    }
    if (nvec <= 64 && agg_wide_eight(a, nvec <= 32 ? 32 : 64, bytes)) return whole;
    if (a.n_edges < ((int64_t)1 << 20)) return {16, 2, lg, false};
    if (bytes * (1 << lg) <= 2.9e9 * (double)tiles && a.table_bytes <= 450 * MB) return {16, 8, lg, true};
    return {16, 2, lg, share};
}

// tiled: the row is cut into several column tiles of this launch (see agg_tiles); share: whether its long items are shared out
template <typename T, int V, int G, int NP, int U, int VWM, bool SH>
gt_status launch(const AggArgs &a, hipStream_t st, bool tiled = false, int slices_lg = 0, bool share = false) {
    constexpr int NG = 64 / G;
    const int64_t tile = (int64_t)G * V * NP;
    const unsigned tiles = (unsigned)((a.F + tile - 1) / tile);
    if (a.n_edges > 0 && (VWM == VWM_NONE ? a.eidx || a.coef2 : VWM == VWM_SCORE ? !a.eidx || !a.coef || a.mask : a.coef != nullptr))
        return gt_fail(GT_ERR_INTERNAL, "k_aggregate: coefficients that this mode does not read");
    if (a.n_items > 0) {
        AggArgs b = a;
        b.slices_lg = slices_lg;
        const double bytes = agg_bytes<T>(a);
        // A whole wavefront per long item where its groups then sum a few dozen entries each; a whole workgroup where a row has only
        // a group or two per wavefront's width to share it, or the chains are four times as long (U == 2).  us, one wavefront / a workgroup
        // per item, power-law graphs: 4 M edges, 64 bf16 columns 47 / 58, 32 columns 54 / 67, 41 fp32 columns 62 / 65; 12 M edges,
        // 41 fp32 columns 173 / 162; 17 M edges, 64 bf16 columns (U == 2) 270 / 247.
        b.coop_waves = tiled || G == 64 || (U == 2 && G >= 8) || (G == 16 && bytes > 1.0e9) ? 4 : 1;
        bool coop = agg_coop<NP, VWM>() && (tiled ? share : agg_share_out(a, G, U, bytes));
        const int64_t ipc = b.coop_waves == 1 ? 4 : 1;   // items per cooperative workgroup
        b.n_coop = coop ? (int)((a.n_long + ipc - 1) / ipc) : 0;
        b.n_whole = coop && agg_whole_rows(a, G) ? (int)a.n_splits : 0;
        const int64_t left = a.n_items > b.n_coop * ipc ? a.n_items - b.n_coop * ipc : 0;
        const int64_t gi = (left + 4 * NG - 1) / (4 * NG), gb = b.n_whole + b.n_coop + gi;
        b.n_blocks = (int)gb;
        b.xcd_run = agg_xcd_run(gi);
        const int S = 1 << b.slices_lg;
        const int64_t gx = S > 1 ? (gb + 8 / S - 1) / (8 / S) * 8 : gb;
        const int tr = a.trace_open > 0 ? a.trace_open - 1 : gt_trace_open(a.trace_kind, a.F, a.n_rows, a.n_edges, st);
        gt_trace_variant(tr, V, G, NP, U, agg_plain(VWM) && a.mask != nullptr);
        const dim3 grid((unsigned)gx, (tiles + S - 1) / S);
        // (narrow groups hold several ids per lane where items are shared out to 64 / G groups of four lanes)
        constexpr int MANY = NP == 1 && agg_plain(VWM) && U != 2 ? agg_many_ids(G) : 1, MANY_COOP = G == 4 ? MANY : 1;
        constexpr bool MASKED = VWM == VWM_NONE;   // (a score comes with no mask)
        if constexpr (agg_plain(VWM)) {
            if (b.n_coop > 0) {
                if constexpr (agg_coop<NP, VWM>()) {
                    if (b.n_whole > 0) {
                        if (b.mask) k_aggregate<T, V, G, NP, U, VWM, MASKED, SH, 2, MANY_COOP><<<grid, 256, 0, st>>>(b);
                        else k_aggregate<T, V, G, NP, U, VWM, false, SH, 2, MANY_COOP><<<grid, 256, 0, st>>>(b);
                    } else if (b.mask) k_aggregate<T, V, G, NP, U, VWM, MASKED, SH, 1, MANY_COOP><<<grid, 256, 0, st>>>(b);
                    else k_aggregate<T, V, G, NP, U, VWM, false, SH, 1, MANY_COOP><<<grid, 256, 0, st>>>(b);
                }
            } else if (MANY > 1 && agg_long_batches(a, G, bytes)) {
                if (b.mask) k_aggregate<T, V, G, NP, U, VWM, MASKED, SH, 0, MANY><<<grid, 256, 0, st>>>(b);
                else k_aggregate<T, V, G, NP, U, VWM, false, SH, 0, MANY><<<grid, 256, 0, st>>>(b);
            } else {
                if (b.mask) k_aggregate<T, V, G, NP, U, VWM, MASKED, SH, 0, 1><<<grid, 256, 0, st>>>(b);
                else k_aggregate<T, V, G, NP, U, VWM, false, SH, 0, 1><<<grid, 256, 0, st>>>(b);
            }
        } else {
            k_aggregate<T, V, G, NP, U, VWM, false, SH, 0, 1><<<grid, 256, 0, st>>>(b);
        }
        gt_trace_close(tr, st);
        GT_LAUNCH_CHECK("k_aggregate");
        if (b.n_whole > 0) return GT_OK;   // no partial rows
    }
    if (a.n_splits > 0 && !a.no_reduce) {
        const int64_t gx = (a.n_splits + 3) / 4;
        k_reduce_partials<T, V, G, NP, SH><<<dim3((unsigned)gx, tiles), 256, 0, st>>>(a);
        GT_LAUNCH_CHECK("k_reduce_partials");
    }
    return GT_OK;
}

// Row loads kept in flight per lane.  What they hide are the chains of long rows, on skewed graphs, and latency where the launch has few wavefronts;
// what they cost is reuse: the more rows the resident groups read at a time, the fewer of them the caches still hold when they are wanted again.
// us, one / two / eight (s.o.: several ids per lane):
//  * Rows of up to 256 bytes: eight where the table fits the last-level cache (power law, 131 K rows, 1.3 M edges, 16 fp32 columns 58 / 44 / 30), and on
//    uniform graphs where it fits the L2s (20 K rows of degree 25, 64 columns 17.6 / 12.9 / 11.2; 131 K rows of degree 25, 4 columns, backward s.o. 40 / 38 / 32) or the launch
//    does not fill the chip (a sampled block of 300 rows, 64 columns - / 9.3 / 7.5).  Beyond the L2s, uniform rows of up to 128 bytes take one where
//    a group has a batch of ids to walk (s.o.; 300 K rows of degree 20, 8 columns 55 / 61 / 75, backward 77 / 85 / 91; 1 M rows of degree 16, 4 columns
//    196 / 229 / 243; 300 K rows, 32 columns 100 / 104 / 113; just past the L2s a direction may lose by it, 131 K rows of degree 25, 16 columns 31 / 30 / 37, backward
//    47 / 44 / 44); those of 129 to 256 bytes two from eight entries on (131 K rows of degree 25, 64 columns 92 / 97 / 112; degree 4 27.7 / 27.7 / 26.1).
//  * The same past the last-level cache: one for rows of up to 64 bytes that are shared out (2 M power-law rows, 52 M edges, 13 columns, backward 715 / 787 / 743)
//    and for launches with several ids per lane (47 bf16 columns without padding 890 / 917 / 925), else two (1 M power-law rows, 16 M edges,
//    64 bf16 columns, one row in flight takes 1.7 times as long).
//  * Wider rows: eight only where chains are the launch's time, i.e. where long items would be shared out (power law, 1 M edges,
//    128 fp32 columns: two 95, eight 42 with items shared out); elsewhere two.  Uniform graphs of whole-wavefront rows take one from ten entries on,
//    if there are wavefronts enough (30 K rows of degree 130, 300 columns 360 / 557; 131 K rows of degree 25, 200 columns, one vector per lane 386 / 405;
//    degree 6, 300 K rows 276 / 261; 130 columns, 33 of 64 lanes, 1 M rows of degree 8 1100 / 913; 6 K rows of 600 entries, 602 bf16 columns 342 / 255),
//    and four vectors per lane take one wherever rows are short (degree 5, 66 K rows, 1030 columns 275 / 283).
//  * The chunks of long rows alone (chunk_entries, the launch before a fused layer): eight, whatever the table (see gt_fused_run).
template <typename T, int V, int G, int NP, int VWM, bool SH>
gt_status launch_u(const AggArgs &a, hipStream_t st) {
    if constexpr (NP == 1 && agg_plain(VWM) && G <= 16) {
        if (a.chunk_entries > 0) return launch<T, V, G, NP, 8, VWM, SH>(a, st);
        const double bytes = agg_bytes<T>(a);
        const bool fits = a.table_bytes <= ((int64_t)96 << 20);   // the last-level cache
        const bool fills = !agg_skewed(a) && a.n_items * G > 1792 * 64 && a.table_bytes > ((int64_t)6 << 20);
        if constexpr (G < 16)
            if (agg_share_out(a, G, 1, bytes) ? G == 4 && !fits : (fills || !fits) && agg_long_batches(a, G, bytes)) return launch<T, V, G, NP, 1, VWM, SH>(a, st);
        if (fits && !(V > 1 && G == 16 && fills && a.n_edges >= 8 * a.n_items)) return launch<T, V, G, NP, 8, VWM, SH>(a, st);
    } else if constexpr (NP == 1 && agg_plain(VWM)) {
        if (agg_wide_eight(a, G, agg_bytes<T>(a))) return launch<T, V, G, NP, 8, VWM, SH>(a, st);
    }
    if constexpr (G == 64 && V > 1 && agg_plain(VWM)) {
        bool one = agg_skewed(a) ? NP == 4 && a.n_edges < 4 * a.n_items : NP == 4 || (a.n_edges >= 10 * a.n_items && a.n_items >= 16384);
        if constexpr (NP == 1) one = one && !SH && a.F >= 40 * V && a.table_bytes > ((int64_t)40 << 20) && a.table_bytes < ((int64_t)300 << 20);
        if (one) return launch<T, V, G, NP, 1, VWM, SH>(a, st);
    }
    // per-entry vector weights stream from memory, each row once, and the gathered table beside them is smaller than they
    // are: eight in flight (4.2 M edges x 64 fp32: two 333 us, four 301, eight 296), four of the widest (1.8 M edges of degree 6,
    // 130 fp32 columns: two 344 us, four 339, eight 368)
    if constexpr (NP == 1 && !agg_plain(VWM)) return launch<T, V, G, NP, (G == 64 ? 4 : 8), VWM, SH>(a, st);
    else return launch<T, V, G, NP, 2, VWM, SH>(a, st);
}

template <typename T, int V, int VWM = VWM_NONE, bool SH = false>
gt_status dispatch(const AggArgs &a, hipStream_t st) {
    const int64_t nvec = (a.F + V - 1) / V;   // lanes needed to cover one row
    if (nvec <= 4) return launch_u<T, V, 4, 1, VWM, SH>(a, st);
    if (nvec <= 8) return launch_u<T, V, 8, 1, VWM, SH>(a, st);
    if constexpr (V == 1 && sizeof(T) == 4 && agg_plain(VWM)) {   // (see agg_dispatch)
        if (nvec > 16) return launch_u<T, V, 64, 3, VWM, SH>(a, st);
    }
    if constexpr (V == 1) return launch_u<T, V, 16, 1, VWM, SH>(a, st);
    if (nvec <= 16) return launch_u<T, V, 16, 1, VWM, SH>(a, st);
    if constexpr (agg_plain(VWM)) {
        const AggTiles t = agg_tiles(a, SH, nvec, sizeof(T), agg_bytes<T>(a));
        if (t.G == 32) return launch<T, V, 32, 1, 2, VWM, SH>(a, st, true, t.slices_lg, t.share);
        if (t.G == 16 && t.U == 8) return launch<T, V, 16, 1, 8, VWM, SH>(a, st, true, t.slices_lg, t.share);
        if (t.G == 16 && t.U == 1) return launch<T, V, 16, 1, 1, VWM, SH>(a, st, true, t.slices_lg, t.share);
        if (t.G == 16) return launch<T, V, 16, 1, 2, VWM, SH>(a, st, true, t.slices_lg, t.share);
    }
    if (nvec <= 32) return launch_u<T, V, 32, 1, VWM, SH>(a, st);
    if (nvec <= 64) return launch_u<T, V, 64, 1, VWM, SH>(a, st);
    if (nvec <= 128) return launch_u<T, V, 64, 2, VWM, SH>(a, st);
    if (nvec <= 192) return launch_u<T, V, 64, 3, VWM, SH>(a, st);
    return launch_u<T, V, 64, 4, VWM, SH>(a, st);   // wider rows take several column tiles (grid.y)
}

// Picks the access width.  `vec`: every row involved is 16-byte aligned and padded to 16 bytes.  Rows that are not take
// whole vectors all the same, the last one shifted to the row's end (element-wise lanes moved 4 or 2 bytes each and
// took twice as long: 16 M gathered rows of 47 bf16 columns without padding, two directions 2.29 -> 1.08 ms).  Element by element go
// rows shorter than one vector, and the fp32 rows of which vectors leave most lanes idle: up to 16 columns where neither long
// rows are shared out nor long batches of ids used to the full (us, vectors / elements, uniform graphs: 1.8 M edges, 5 columns 15.6 / 13.4;
// 5.6 M edges of degree 8, 13 columns 172 / 165), and, without shared-out rows, 129 to 176, which a wavefront of vectors covers little more than half of (130
// columns: 1 M edges of degree 10 100 / 94, 4 M power-law edges 253 / 238; at 200 they are even).
template <typename T, int VWM = VWM_NONE>
gt_status agg_dispatch(const AggArgs &a, bool vec, hipStream_t st) {
    constexpr int V = 16 / (int)sizeof(T);
    if (vec) return dispatch<T, V, VWM>(a, st);
    if (a.F < V) return dispatch<T, 1, VWM>(a, st);
    if constexpr (sizeof(T) == 4 && agg_plain(VWM)) {
        if (a.F <= 16 && !agg_skewed(a) && !agg_vectors_pay(a, agg_bytes<T>(a))) return dispatch<T, 1, VWM>(a, st);
        if (a.F > 128 && a.F <= 176 && !agg_share_out(a, 64, 2, agg_bytes<T>(a))) return dispatch<T, 1, VWM>(a, st);
    }
    return dispatch<T, V, VWM, true>(a, st);
}

bool aligned16(const void *p) { return ((uintptr_t)p & 15) == 0; }

}  // namespace
