// Device-wide primitives shared by the plan builder and the batch-preparation kernels: an
// exclusive int32 scan and a stable LSD radix sort of (key, value) pairs.  Header-only with
// internal linkage: every translation unit that includes it gets its own copy of the kernels.
#pragma once
#include "gt_internal.h"

namespace {

// ---------------------------------------------------------------------------------------------
// exclusive scan of int32, several arrays at a time
// ---------------------------------------------------------------------------------------------

constexpr int SCAN_THREADS = 256;
constexpr int SCAN_PER_THREAD = 16;
constexpr int SCAN_TILE = SCAN_THREADS * SCAN_PER_THREAD;   // 4096
constexpr int SCAN_BATCH = 8;
constexpr int64_t SCAN_DIRECT_TILES = 1024;   // up to here every workgroup adds the tile sums before its own itself

struct ScanBatch {
    const int32_t *in[SCAN_BATCH];
    int32_t *out[SCAN_BATCH];
    int64_t n[SCAN_BATCH];
    int32_t *sums[SCAN_BATCH];   // tile sums (or, scanned, tile offsets) of each array
};

// Exclusive prefix of v over a workgroup of 64 * W threads; *total = its sum.  Leaves with the staging free for reuse.
template <int W>
__device__ inline int32_t block_exclusive_scan(int32_t v, int32_t *total) {
    __shared__ int32_t wave_sums[W];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    int32_t inc = v;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const int32_t o = __shfl_up(inc, d, 64);
        if (lane >= d) inc += o;
    }
    if (lane == 63) wave_sums[wave] = inc;
    __syncthreads();
    int32_t base = 0, tot = 0;
#pragma unroll
    for (int w = 0; w < W; ++w) {
        const int32_t s = wave_sums[w];
        if (w < wave) base += s;
        tot += s;
    }
    __syncthreads();
    *total = tot;
    return base + inc - v;
}

// SCAN_PER_THREAD consecutive elements from p0 on, zeros from n on (16-byte accesses where the array is aligned and they are all there:
// element by element a wavefront's sixteen loads each touched 32 lines; the 3 x 1.5 M counts and 4 M row counts of a plan over 25 M entries 94 -> 31 us)
__device__ inline void scan_load(const int32_t *in, int64_t p0, int64_t n, int32_t (&v)[SCAN_PER_THREAD]) {
    if (((uintptr_t)in & 15) == 0 && p0 + SCAN_PER_THREAD <= n) {
#pragma unroll
        for (int i = 0; i < SCAN_PER_THREAD; i += 4) {
            const int4 x = *reinterpret_cast<const int4 *>(in + p0 + i);
            v[i] = x.x; v[i + 1] = x.y; v[i + 2] = x.z; v[i + 3] = x.w;
        }
    } else {
#pragma unroll
        for (int i = 0; i < SCAN_PER_THREAD; ++i) v[i] = p0 + i < n ? in[p0 + i] : 0;
    }
}
__device__ inline void scan_store(int32_t *out, int64_t p0, int64_t n, int32_t ex, const int32_t (&v)[SCAN_PER_THREAD]) {
    int32_t o[SCAN_PER_THREAD];
#pragma unroll
    for (int i = 0; i < SCAN_PER_THREAD; ++i) {
        o[i] = ex;
        ex += v[i];
    }
    if (((uintptr_t)out & 15) == 0 && p0 + SCAN_PER_THREAD <= n) {
#pragma unroll
        for (int i = 0; i < SCAN_PER_THREAD; i += 4) *reinterpret_cast<int4 *>(out + p0 + i) = make_int4(o[i], o[i + 1], o[i + 2], o[i + 3]);
    } else {
#pragma unroll
        for (int i = 0; i < SCAN_PER_THREAD; ++i)
            if (p0 + i < n) out[p0 + i] = o[i];
    }
}

// sums[tile] of array blockIdx.y
__global__ void __launch_bounds__(SCAN_THREADS) k_tile_sums(const ScanBatch b) {
    const int k = blockIdx.y;
    const int64_t n = b.n[k], base = (int64_t)blockIdx.x * SCAN_TILE;
    if (base >= n) return;
    int32_t v[SCAN_PER_THREAD], s = 0;
    scan_load(b.in[k], base + (int64_t)threadIdx.x * SCAN_PER_THREAD, n, v);
#pragma unroll
    for (int i = 0; i < SCAN_PER_THREAD; ++i) s += v[i];
    int32_t total;
    block_exclusive_scan<SCAN_THREADS / 64>(s, &total);
    if (threadIdx.x == 0) b.sums[k][blockIdx.x] = total;
}

// out of one tile of array blockIdx.y: the tile's offset is the sum of the tile sums before it (added up here, or
// already scanned), the rest a scan inside the workgroup.  Two launches for all arrays, and every element is written
// once (scanning tiles, then adding offsets in place, took three launches per array and wrote twice: the
// eight count arrays of a plan over 1 M rows 190 -> 40 us).
__global__ void __launch_bounds__(SCAN_THREADS) k_scan_apply(const ScanBatch b, int scanned) {
    const int k = blockIdx.y;
    const int64_t n = b.n[k], base = (int64_t)blockIdx.x * SCAN_TILE;
    if (base >= n) return;
    int32_t off = 0;
    if (scanned) {
        off = b.sums[k][blockIdx.x];
    } else {
        int32_t s = 0;
        for (int t = threadIdx.x; t < (int)blockIdx.x; t += SCAN_THREADS) s += b.sums[k][t];
        block_exclusive_scan<SCAN_THREADS / 64>(s, &off);
    }
    const int64_t p0 = base + (int64_t)threadIdx.x * SCAN_PER_THREAD;
    int32_t v[SCAN_PER_THREAD];
    int32_t s = 0;
    scan_load(b.in[k], p0, n, v);
#pragma unroll
    for (int i = 0; i < SCAN_PER_THREAD; ++i) s += v[i];
    int32_t total;
    const int32_t ex = off + block_exclusive_scan<SCAN_THREADS / 64>(s, &total);
    scan_store(b.out[k], p0, n, ex, v);
}

// int32 of scratch one array of n elements takes (a batch: the sum over its arrays)
size_t scan_tmp_ints(int64_t n) {
    size_t t = 64;
    while (n > SCAN_TILE) {
        n = (n + SCAN_TILE - 1) / SCAN_TILE;
        t += gt_align_up((size_t)n * 4) / 4;
    }
    return t;
}

// Short arrays in one launch: one workgroup of 1,024 threads per array walks it in steps of 16,384 elements and
// carries the running total.  A sampled batch's scans (a few thousand rows) are bound by launch latency.
// Only up to one step: beyond that the serial walk costs more than the launch it saves.
constexpr int SCAN_SMALL_THREADS = 1024;
constexpr int64_t SCAN_SMALL_MAX = 16384;

__global__ void __launch_bounds__(SCAN_SMALL_THREADS) k_scan_small(const ScanBatch b) {
    const int k = blockIdx.x;
    const int64_t n = b.n[k];
    int32_t carry = 0;
    for (int64_t t0 = 0; t0 < n; t0 += (int64_t)SCAN_SMALL_THREADS * SCAN_PER_THREAD) {
        const int64_t p0 = t0 + (int64_t)threadIdx.x * SCAN_PER_THREAD;
        int32_t v[SCAN_PER_THREAD];
        int32_t s = 0;
        scan_load(b.in[k], p0, n, v);
#pragma unroll
        for (int i = 0; i < SCAN_PER_THREAD; ++i) s += v[i];
        int32_t total;
        const int32_t ex = carry + block_exclusive_scan<SCAN_SMALL_THREADS / 64>(s, &total);
        scan_store(b.out[k], p0, n, ex, v);
        carry += total;
    }
}

// out[k][i] = sum_{j<i} in[k][j] for `count` (1..8) arrays of n[k] elements (in == out allowed).
// tmp: the sum of scan_tmp_ints(n[k]) int32.
gt_status scan_exclusive_batch(int count, const int32_t *const *in, int32_t *const *out, const int64_t *n, int32_t *tmp,
                               hipStream_t st) {
    if (count <= 0) return GT_OK;
    if (count > SCAN_BATCH) return gt_fail(GT_ERR_INTERNAL, "scan_exclusive_batch: too many arrays");
    ScanBatch b{};
    int64_t most = 0;
    for (int k = 0; k < count; ++k) {
        b.in[k] = in[k]; b.out[k] = out[k]; b.n[k] = n[k];
        if (n[k] > most) most = n[k];
    }
    if (most <= 0) return GT_OK;
    if (most <= SCAN_SMALL_MAX) {
        k_scan_small<<<count, SCAN_SMALL_THREADS, 0, st>>>(b);
        GT_LAUNCH_CHECK("k_scan_small");
        return GT_OK;
    }
    int64_t tiles[SCAN_BATCH] = {};
    for (int k = 0; k < count; ++k) {
        tiles[k] = (n[k] + SCAN_TILE - 1) / SCAN_TILE;
        b.sums[k] = tmp;
        tmp += gt_align_up((size_t)tiles[k] * 4) / 4;
    }
    const int64_t mt = (most + SCAN_TILE - 1) / SCAN_TILE;
    k_tile_sums<<<dim3((unsigned)mt, count), SCAN_THREADS, 0, st>>>(b);
    GT_LAUNCH_CHECK("k_tile_sums");
    const int scanned = mt > SCAN_DIRECT_TILES;
    if (scanned) {
        const gt_status s = scan_exclusive_batch(count, b.sums, b.sums, tiles, tmp, st);
        if (s != GT_OK) return s;
    }
    k_scan_apply<<<dim3((unsigned)mt, count), SCAN_THREADS, 0, st>>>(b, scanned);
    GT_LAUNCH_CHECK("k_scan_apply");
    return GT_OK;
}

// out[i] = sum_{j<i} in[j] for i < n (in == out allowed).  tmp: scan_tmp_ints(n) int32.
gt_status scan_exclusive(const int32_t *in, int32_t *out, int64_t n, int32_t *tmp, hipStream_t st) {
    return scan_exclusive_batch(1, &in, &out, &n, tmp, st);
}

// ---------------------------------------------------------------------------------------------
// stable LSD radix sort of (key, value) pairs, at most 8 bits per pass
// ---------------------------------------------------------------------------------------------
// A pass = per-tile digit counts, their offsets, and a scatter that ranks a tile's items (wavefront by wavefront, 64 items at a
// time, in order, so equal digits keep their order), sorts the tile in LDS and writes it out from there: the runs of a
// digit leave as consecutive stores (scattering from registers wrote 4-byte pieces: 25 M pairs 149 us per pass,
// 58 us average over a plan with this).  Tiles: 8,192 pairs (8 wavefronts) on long inputs, where an XCD takes consecutive tiles so that
// neighbouring runs of a digit meet in its L2; 4,096 and 1,024 pairs (4 wavefronts) on shorter ones, so that a few hundred thousand or
// thousand pairs still spread over the compute units.  The bits of a key are shared out evenly over the passes: 20 bits in 6, 7 and 7
// leave a tile's digits in runs twice as long as 8, 8 and 4 do, and half the counts to scan.  With at most RS_DIRECT tiles the scatter adds up the counts of the
// tiles before its own itself: two launches per pass instead of four.
template <int WAVES, int CH> constexpr int rs_tile() { return WAVES * CH * 64; }
constexpr int RS_DIRECT = 128;

__device__ inline int64_t rs_tile_of_block(int nblk) {   // consecutive tiles on one XCD (workgroups go round-robin over 8)
    const int per = (nblk + 7) / 8;
    return (int64_t)(blockIdx.x & 7) * per + (blockIdx.x >> 3);
}
static inline unsigned rs_grid(int nblk) { return (unsigned)((nblk + 7) / 8 * 8); }

// counts of one tile, nb bits: hist[tile][256] (direct) or hist[1 << nb][nblk] (to be scanned)
template <int WAVES, int CH>
__global__ void __launch_bounds__(WAVES * 64) k_rs_hist(const uint32_t *keys, int64_t n, int shift, int nb, int32_t *hist, int nblk,
                                                        int direct) {
    constexpr int NT = WAVES * 64, TILE = rs_tile<WAVES, CH>();
    // eight counters per digit, by lane: the lanes of a wavefront that meet on one (most, in the upper digits of a power-law graph's ids) take
    // turns (25 M keys 30 us a pass with one counter per digit, 22 with eight)
    constexpr int COPIES = 8, HSTR = 257;
    __shared__ int32_t h[COPIES * HSTR];
    const int64_t tile = rs_tile_of_block(nblk);
    if (tile >= nblk) return;
    for (int i = threadIdx.x; i < COPIES * HSTR; i += NT) h[i] = 0;
    __syncthreads();
    const int64_t base = tile * TILE + threadIdx.x;
    uint32_t k[CH];
#pragma unroll
    for (int i = 0; i < CH; ++i) {
        const int64_t p = base + (int64_t)i * NT;
        k[i] = p < n ? keys[p] : 0u;
    }
    int32_t *mine = h + (threadIdx.x % COPIES) * HSTR;
#pragma unroll
    for (int i = 0; i < CH; ++i)
        if (base + (int64_t)i * NT < n) atomicAdd(&mine[(k[i] >> shift) & ((1u << nb) - 1u)], 1);
    __syncthreads();
    const int d = threadIdx.x;
    if (d < (direct ? 256 : 1 << nb)) {
        int32_t sum = 0;
#pragma unroll
        for (int c = 0; c < COPIES; ++c) sum += h[c * HSTR + d];
        hist[direct ? tile * 256 + d : (int64_t)d * nblk + tile] = sum;
    }
}

template <int WAVES, int CH>
constexpr size_t rs_lds_bytes() { return (size_t)rs_tile<WAVES, CH>() * 4 + (size_t)WAVES * 256 * 4 + 256 * 4; }

// vals_in == nullptr means value = position (iota).  EXTRA: a second value travels along.
template <int WAVES, int CH, bool EXTRA>
__global__ void __launch_bounds__(WAVES * 64) k_rs_scatter(const uint32_t *keys_in, const uint32_t *vals_in, const uint32_t *ext_in,
                                                           uint32_t *keys_out, uint32_t *vals_out, uint32_t *ext_out, int64_t n,
                                                           int shift, int nb, const int32_t *hist, int nblk, int direct) {
    constexpr int NT = WAVES * 64, TILE = rs_tile<WAVES, CH>();
    extern __shared__ __align__(16) unsigned char rs_smem[];
    uint32_t *lx = reinterpret_cast<uint32_t *>(rs_smem);        // the tile's keys, sorted; then its values; then the second ones
    int32_t *cnt = reinterpret_cast<int32_t *>(lx + TILE);       // [WAVES][256] counts, then bases
    int32_t *gdelta = cnt + WAVES * 256;                         // output position minus tile position, per digit
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, d = threadIdx.x;
    const int64_t tile = rs_tile_of_block(nblk);
    if (tile >= nblk) return;   // whole workgroups leave
    for (int i = threadIdx.x; i < WAVES * 256; i += NT) cnt[i] = 0;
    const int64_t t0 = tile * TILE, wstart = t0 + (int64_t)wave * CH * 64;
    const uint32_t dmask = (1u << nb) - 1u;
    uint32_t key[CH], val[CH], ext[EXTRA ? CH : 1];
    int32_t rank[CH];
    const uint64_t lt_mask = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
    // all loads first, so that their latencies overlap instead of adding up chunk by chunk; past the caches, which keeps the lines there that
    // the tiles' runs are filling (25 M triples 128 us a pass, 122 so)
#pragma unroll
    for (int c = 0; c < CH; ++c) {
        const int64_t p = wstart + (int64_t)c * 64 + lane;
        key[c] = p < n ? __builtin_nontemporal_load(keys_in + p) : 0u;
        val[c] = vals_in ? (p < n ? __builtin_nontemporal_load(vals_in + p) : 0u) : (uint32_t)p;
        if constexpr (EXTRA) ext[c] = p < n ? __builtin_nontemporal_load(ext_in + p) : 0u;
    }
    // digit d (threads 0..255): output position of the tile's first item with it
    int32_t goff = 0, before = 0, all = 0;
    if (d < 256) {
        if (direct) {
            // 32 counts in flight, none of them in a remainder loop (each of whose rounds waits for its load: 300 K pairs, 75 tiles,
            // eight in flight and a remainder 18.4 us a pass, 12.6 this way with eight wavefronts of eight
            // chunks instead of four of sixteen)
            for (int t0 = 0; t0 < nblk; t0 += 32) {
                int32_t x[32];
#pragma unroll
                for (int u = 0; u < 32; ++u) x[u] = hist[(t0 + u < nblk ? t0 + u : 0) * 256 + d];
#pragma unroll
                for (int u = 0; u < 32; ++u) {
                    before += t0 + u < (int)tile ? x[u] : 0;
                    all += t0 + u < nblk ? x[u] : 0;
                }
            }
        } else {
            goff = d < (1 << nb) ? hist[(int64_t)d * nblk + tile] : 0;
        }
    }
    int32_t unused;
    if (direct) goff = block_exclusive_scan<WAVES>(all, &unused) + before;   // uniform branch; threads past 255 add 0
    else __syncthreads();                                                    // the counters are zero from here on
#pragma unroll
    for (int c = 0; c < CH; ++c) {
        rank[c] = 0;
        if (wstart + (int64_t)c * 64 >= n) continue;   // wavefront-uniform: the chunk is empty
        const bool valid = wstart + (int64_t)c * 64 + lane < n;
        const uint32_t digit = (key[c] >> shift) & dmask;
        uint64_t m = __ballot(valid);
#pragma unroll
        for (int b = 0; b < 8; ++b) {
            const bool bit = (digit >> b) & 1u;
            const uint64_t bal = __ballot(valid && bit);
            m &= bit ? bal : ~bal;
        }
        // m: valid lanes of this chunk with the same digit (meaningful on valid lanes)
        const int ahead = __popcll(m & lt_mask);
        int32_t prev = 0;
        if (valid) prev = cnt[wave * 256 + digit];
        rank[c] = prev + ahead;
        if (valid && ahead == 0) cnt[wave * 256 + digit] = prev + __popcll(m);
    }
    __syncthreads();
    int32_t tot = 0;
    int32_t wb[WAVES];
    if (d < 256) {
#pragma unroll
        for (int w = 0; w < WAVES; ++w) {
            wb[w] = tot;
            tot += cnt[w * 256 + d];
        }
    }
    const int32_t start = block_exclusive_scan<WAVES>(tot, &unused);   // tile position of the digit's first item
    if (d < 256) {
        gdelta[d] = goff - start;
#pragma unroll
        for (int w = 0; w < WAVES; ++w) cnt[w * 256 + d] = start + wb[w];
    }
    __syncthreads();
    // One array at a time goes through LDS: with room for all of them a CU held two workgroups (25 M triples 198 us a pass,
    // 130 this way; 16 items per thread 135, and more where the tiles are few)
#pragma unroll
    for (int c = 0; c < CH; ++c) {
        if (wstart + (int64_t)c * 64 + lane < n) {
            rank[c] += cnt[wave * 256 + ((key[c] >> shift) & dmask)];
            lx[rank[c]] = key[c];
        }
    }
    __syncthreads();
    const int m = n - t0 < TILE ? (int)(n - t0) : TILE;
    int32_t dst[CH];
#pragma unroll
    for (int j = 0; j < CH; ++j) {
        const int i = j * NT + threadIdx.x;
        dst[j] = 0;
        if (i < m) {
            const uint32_t k = lx[i];
            dst[j] = gdelta[(k >> shift) & dmask] + i;
            keys_out[dst[j]] = k;
        }
    }
    auto carry = [&](const uint32_t *x, uint32_t *out) {
        __syncthreads();
#pragma unroll
        for (int c = 0; c < CH; ++c)
            if (wstart + (int64_t)c * 64 + lane < n) lx[rank[c]] = x[c];
        __syncthreads();
#pragma unroll
        for (int j = 0; j < CH; ++j)
            if (j * NT + (int)threadIdx.x < m) out[dst[j]] = lx[j * NT + threadIdx.x];
    };
    carry(val, vals_out);
    if constexpr (EXTRA) carry(ext, ext_out);
}

// All passes of a sort of at most 16,384 pairs in one launch: a single workgroup of 16 wavefronts,
// each owning a sixteenth of the items (up to 1,024 consecutive ones), keeps keys and values in LDS (128 KB) between the passes:
// a pass reads its items from LDS in order, ranks them exactly as k_rs_scatter does (so the
// order is the same stable one) and writes them back to LDS at their sorted positions; the last
// pass is followed by one coalesced copy to the caller's output.  A sampled batch sorts a few
// thousand keys in 2-3 passes: one launch instead of one per pass, and no scattered 4-byte stores
// to memory, which a single compute unit retires at about one cache line per clock (measured on
// MI355X, 15 K pairs, 3 passes: 54 us as three launches, 47 us as one launch through memory).
constexpr int RS_CHUNKS = 16;                       // 64-item chunks per wave
constexpr int RS_WAVE_ITEMS = RS_CHUNKS * 64;       // 1024
constexpr int RS_ONE_THREADS = 1024;
constexpr int RS_ONE_WAVES = RS_ONE_THREADS / 64;
constexpr int64_t RS_ONE_MAX = (int64_t)RS_ONE_WAVES * RS_WAVE_ITEMS;
constexpr int RS_MAX_PASSES = 4;
constexpr size_t RS_ONE_LDS = (size_t)RS_ONE_MAX * 8 + (size_t)RS_ONE_WAVES * 256 * 2 * 2;

struct SortPasses {
    const uint32_t *kin[RS_MAX_PASSES];
    const uint32_t *vin[RS_MAX_PASSES];   // null: value = position
    uint32_t *kout[RS_MAX_PASSES];
    uint32_t *vout[RS_MAX_PASSES];
    const uint32_t *ein[RS_MAX_PASSES];   // second value, or null (multi-launch sorts only: n > RS_ONE_MAX)
    uint32_t *eout[RS_MAX_PASSES];
    int passes;                           // at least bits / 8
    int bits;                             // of a key, shared out over the passes (see sort_shift)
};

__host__ __device__ inline int sort_shift(int bits, int passes, int p) { return p * bits / passes; }   // pass p sorts by the bits from here on

__global__ void __launch_bounds__(RS_ONE_THREADS) k_rs_sort_one(const uint32_t *keys_in, const uint32_t *vals_in,
                                                                uint32_t *keys_out, uint32_t *vals_out, int64_t n,
                                                                int passes, int bits) {
    extern __shared__ __align__(16) unsigned char rs_one_smem[];
    uint32_t *lk = reinterpret_cast<uint32_t *>(rs_one_smem);       // [RS_ONE_MAX]
    uint32_t *lv = lk + RS_ONE_MAX;                                  // [RS_ONE_MAX]
    uint16_t *cnt = reinterpret_cast<uint16_t *>(lv + RS_ONE_MAX);   // [RS_ONE_WAVES][256], at most 1,024 each
    uint16_t *wbase = cnt + RS_ONE_WAVES * 256;                      // [RS_ONE_WAVES][256], below 16,384
    __shared__ int32_t wsum[4];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const uint64_t lt_mask = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
    const int nn = (int)n;
    const int per = ((nn + RS_ONE_WAVES - 1) / RS_ONE_WAVES + 63) / 64 * 64, wstart = wave * per;   // a wavefront's items (at most RS_WAVE_ITEMS)
    const int wend = wstart + per < nn ? wstart + per : nn;
    uint32_t key[RS_CHUNKS], val[RS_CHUNKS];
#pragma unroll
    for (int c = 0; c < RS_CHUNKS; ++c) {
        const int q = wstart + c * 64 + lane;
        key[c] = q < wend ? keys_in[q] : 0u;
        val[c] = (q < wend && vals_in) ? vals_in[q] : (uint32_t)q;
    }
    for (int p = 0; p < passes; ++p) {
        const int shift = sort_shift(bits, passes, p), nb = sort_shift(bits, passes, p + 1) - shift;
        const uint32_t dmask = (1u << nb) - 1u;
        for (int i = threadIdx.x; i < RS_ONE_WAVES * 256; i += RS_ONE_THREADS) cnt[i] = 0;
        if (p > 0) {
#pragma unroll
            for (int c = 0; c < RS_CHUNKS; ++c) {
                const int q = wstart + c * 64 + lane;
                key[c] = q < wend ? lk[q] : 0u;
                val[c] = q < wend ? lv[q] : 0u;
            }
        }
        __syncthreads();
        int rank[RS_CHUNKS];
#pragma unroll
        for (int c = 0; c < RS_CHUNKS; ++c) {
            rank[c] = 0;
            if (wstart + c * 64 >= wend) continue;   // wavefront-uniform: the chunk is empty
            const bool valid = wstart + c * 64 + lane < wend;
            const uint32_t digit = (key[c] >> shift) & dmask;
            uint64_t m = __ballot(valid);
#pragma unroll
            for (int b = 0; b < 8; ++b) {
                const bool bit = (digit >> b) & 1u;
                const uint64_t bal = __ballot(valid && bit);
                m &= bit ? bal : ~bal;
            }
            const int before = __popcll(m & lt_mask);
            int prev = 0;
            if (valid) prev = cnt[wave * 256 + digit];
            rank[c] = prev + before;
            if (valid && before == 0) cnt[wave * 256 + digit] = (uint16_t)(prev + __popcll(m));
        }
        __syncthreads();
        // threads 0..255 <-> digits: per-wavefront bases within the digit, then the digits' starts
        const int d = threadIdx.x & 255;
        int tot = 0;
        int wb[RS_ONE_WAVES];
        if (threadIdx.x < 256) {
#pragma unroll
            for (int w = 0; w < RS_ONE_WAVES; ++w) {
                wb[w] = tot;
                tot += cnt[w * 256 + d];
            }
        }
        int inc = tot;
#pragma unroll
        for (int s = 1; s < 64; s <<= 1) {
            const int o = __shfl_up(inc, s, 64);
            if (lane >= s) inc += o;
        }
        if (threadIdx.x < 256 && lane == 63) wsum[wave] = inc;
        __syncthreads();
        if (threadIdx.x < 256) {
            int start = inc - tot;
            for (int w = 0; w < wave; ++w) start += wsum[w];
#pragma unroll
            for (int w = 0; w < RS_ONE_WAVES; ++w) wbase[w * 256 + d] = (uint16_t)(start + wb[w]);
        }
        __syncthreads();
        // every wavefront has its items in registers: the LDS copies may be overwritten
#pragma unroll
        for (int c = 0; c < RS_CHUNKS; ++c) {
            const int q = wstart + c * 64 + lane;
            if (q < wend) {
                const uint32_t digit = (key[c] >> shift) & dmask;
                const int dst = (int)wbase[wave * 256 + digit] + rank[c];
                lk[dst] = key[c];
                lv[dst] = val[c];
            }
        }
        __syncthreads();
    }
    if (passes <= 0) {   // nothing sorted: the registers still hold the input
#pragma unroll
        for (int c = 0; c < RS_CHUNKS; ++c) {
            const int q = wstart + c * 64 + lane;
            if (q < wend) { keys_out[q] = key[c]; vals_out[q] = val[c]; }
        }
        return;
    }
    for (int q = threadIdx.x; q < nn; q += RS_ONE_THREADS) {
        keys_out[q] = lk[q];
        vals_out[q] = lv[q];
    }
}

struct SortTmp {
    int32_t *hist;      // rs_hist_ints(n)
    int32_t *scan_tmp;  // scan_tmp_ints(rs_hist_ints(n))
};

// tile of a pass over n pairs: each larger one from where the smaller would give more than RS_DIRECT tiles (the passes just above
// have few: 131,073 pairs 33 tiles of 4,096, 524,289 pairs 65 of 8,192; plans of such graphs, 175 and 250 us, grow evenly)
constexpr int64_t RS_T1 = rs_tile<4, 4>(), RS_T2 = rs_tile<4, 16>(), RS_T3 = rs_tile<8, 16>();   // 1,024 / 4,096 / 8,192
int64_t rs_tile_for(int64_t n) { return n <= RS_T1 * RS_DIRECT ? RS_T1 : (n <= RS_T2 * RS_DIRECT ? RS_T2 : RS_T3); }
// entries of `hist` for any input of at most n pairs
size_t rs_hist_ints(int64_t n) { return (size_t)256 * (size_t)((n + RS_T2 - 1) / RS_T2 > RS_DIRECT ? (n + RS_T2 - 1) / RS_T2 : RS_DIRECT); }

template <int WAVES, int CH, bool EXTRA>
gt_status radix_pass_t(const uint32_t *kin, const uint32_t *vin, const uint32_t *ein, uint32_t *kout, uint32_t *vout, uint32_t *eout,
                       int64_t n, int shift, int nb, const SortTmp &t, hipStream_t st) {
    constexpr int64_t TILE = rs_tile<WAVES, CH>();
    constexpr size_t lds = rs_lds_bytes<WAVES, CH>();
    static_assert(lds <= 64 * 1024, "more needs the kernel's attribute set");
    const int nblk = (int)((n + TILE - 1) / TILE);
    const int direct = nblk <= RS_DIRECT;
    const unsigned grid = rs_grid(nblk);
    k_rs_hist<WAVES, CH><<<grid, WAVES * 64, 0, st>>>(kin, n, shift, nb, t.hist, nblk, direct);
    GT_LAUNCH_CHECK("k_rs_hist");
    if (!direct) {
        const gt_status s = scan_exclusive(t.hist, t.hist, (int64_t)nblk << nb, t.scan_tmp, st);
        if (s != GT_OK) return s;
    }
    k_rs_scatter<WAVES, CH, EXTRA><<<grid, WAVES * 64, lds, st>>>(kin, vin, ein, kout, vout, eout, n, shift, nb, t.hist, nblk, direct);
    GT_LAUNCH_CHECK("k_rs_scatter");
    return GT_OK;
}

gt_status radix_pass(const uint32_t *kin, const uint32_t *vin, uint32_t *kout, uint32_t *vout, int64_t n,
                     int shift, int nb, const SortTmp &t, hipStream_t st, const uint32_t *ein = nullptr, uint32_t *eout = nullptr) {
    if (n <= 0) return GT_OK;
    const int64_t tile = rs_tile_for(n);
    if (ein) {
        if (tile == RS_T1) return radix_pass_t<4, 4, true>(kin, vin, ein, kout, vout, eout, n, shift, nb, t, st);
        return radix_pass_t<8, 8, true>(kin, vin, ein, kout, vout, eout, n, shift, nb, t, st);
    }
    if (tile == RS_T1) return radix_pass_t<4, 4, false>(kin, vin, nullptr, kout, vout, nullptr, n, shift, nb, t, st);
    if (tile == RS_T2) return radix_pass_t<8, 8, false>(kin, vin, nullptr, kout, vout, nullptr, n, shift, nb, t, st);
    return radix_pass_t<8, 16, false>(kin, vin, nullptr, kout, vout, nullptr, n, shift, nb, t, st);
}

// Runs the passes of `a` in order: one launch when the input is short, one pass at a time otherwise.
gt_status radix_sort(const SortPasses &a, int64_t n, const SortTmp &t, hipStream_t st) {
    if (n <= 0 || a.passes <= 0) return GT_OK;
    if (a.passes > RS_MAX_PASSES || a.bits > 8 * a.passes || a.bits < a.passes) return gt_fail(GT_ERR_INTERNAL, "radix_sort: too many passes");
    if (n <= RS_ONE_MAX) {
        if (a.ein[0]) return gt_fail(GT_ERR_INTERNAL, "radix_sort: a second value on a one-launch sort");
        const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(k_rs_sort_one),
                                                 hipFuncAttributeMaxDynamicSharedMemorySize, (int)RS_ONE_LDS);
        if (e != hipSuccess) return gt_hip_fail(e, "hipFuncSetAttribute(k_rs_sort_one)");
        k_rs_sort_one<<<1, RS_ONE_THREADS, RS_ONE_LDS, st>>>(a.kin[0], a.vin[0], a.kout[a.passes - 1],
                                                              a.vout[a.passes - 1], n, a.passes, a.bits);
        GT_LAUNCH_CHECK("k_rs_sort_one");
        return GT_OK;
    }
    for (int p = 0; p < a.passes; ++p) {
        const int shift = sort_shift(a.bits, a.passes, p), nb = sort_shift(a.bits, a.passes, p + 1) - shift;
        const gt_status s = radix_pass(a.kin[p], a.vin[p], a.kout[p], a.vout[p], n, shift, nb, t, st, a.ein[p], a.eout[p]);
        if (s != GT_OK) return s;
    }
    return GT_OK;
}

}  // namespace
