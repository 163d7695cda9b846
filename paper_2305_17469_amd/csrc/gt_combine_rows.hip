// Tall bf16 products  C[M, N] = act(A op(B) + bias)  whose weights do not fit the LDS at once (K beyond the weight-stationary
// kernels) or are several of their column slices wide.
#include "gt_combine.h"

namespace {

typedef gemm_bf16_t bf16_t;

__device__ inline uint32_t lo16(uint32_t a, uint32_t b) { return __builtin_amdgcn_perm(b, a, 0x05040100u); }   // lo16(a) | lo16(b) << 16
__device__ inline uint32_t hi16(uint32_t a, uint32_t b) { return __builtin_amdgcn_perm(b, a, 0x07060302u); }   // hi16(a) | hi16(b) << 16

// 128 x 256 tile, eight wavefronts of 64 x 64, k-tile 64, two workgroups per CU: one multiplies while the other waits for its loads or
// writes its rows.  A goes to LDS as it is; B, where it is stored [K][N], is transposed on the way (a thread's 4 (k) x 8 (n) patch),
// so that every fragment is one 16-byte LDS read.  The MFMA operands are swapped (weights first): a lane ends up with four
// consecutive columns of one row, which go through LDS in bf16 and leave as whole rows of the tile, 512 bytes each (through the
// fp32 stages of the general epilogue, 64 columns at a time, 2^19 x 256 -> 602 took 490 us instead of 364).  What bounds it is LDS
// traffic beside the loads: 2^19 x 602 -> 256 runs at 520 TFLOP/s and 2.9 TB/s, 233 us without the epilogue.
// Rows past M and columns past N repeat valid ones (their results are not stored); k past K is zero in both operands.
constexpr int KT = 64, STR = KT + 8, BM = 128, BN = 256, CSTR = BN + 8;
constexpr size_t ROWS_LDS_BYTES = (size_t)BM * CSTR * 2 > (size_t)(BM + BN) * STR * 2 ? (size_t)BM * CSTR * 2 : (size_t)(BM + BN) * STR * 2;

template <bool TB, bool MASK>
__global__ void __launch_bounds__(512, 4) k_gemm_rows_bf16(const GemmArgs g) {
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    bf16_t *As = reinterpret_cast<bf16_t *>(smem);
    bf16_t *Bs = As + BM * STR;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int l32 = lane & 31, h = lane >> 5;
    const int wm = wave >> 2, wn = wave & 3;
    int tile_m, tile_n, split;
    if (!gemm_tile_of_block(g, tile_m, tile_n, split)) return;   // whole workgroup leaves before any barrier
    const int64_t m0 = (int64_t)tile_m * BM, n0 = (int64_t)tile_n * BN;
    const bf16_t *A = static_cast<const bf16_t *>(g.A), *B = static_cast<const bf16_t *>(g.B);
    const int K = (int)g.K;

    // A: 16-byte vectors of rows r and r + 64, eight lanes per row and k-tile
    const int av = (threadIdx.x & 7) * 8, ar = threadIdx.x >> 3;
    const bf16_t *pa[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int64_t row = m0 + ar + 64 * i;
        pa[i] = A + (row < g.M ? row : g.M - 1) * g.lda;
    }
    // B: (TB) vectors of rows n, n + 64, ...; else a patch of four k and eight n
    const int kq = threadIdx.x & 15, rq = threadIdx.x >> 4;
    const bf16_t *pb[TB ? 4 : 1];
    if constexpr (TB) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int64_t n = n0 + ar + 64 * i;
            pb[i] = B + (n < g.N ? n : g.N - 1) * g.ldb;
        }
    } else {
        const int64_t n = n0 + rq * 8;
        pb[0] = B + (n < g.N ? n : (g.N - 1) / 8 * 8);   // (a row's last vector may be read whole: vecB)
    }
    uint4 ra[2], rb[4];
    auto fetch = [&](int k0) {
        const int ka = k0 + av < K ? k0 + av : 0;   // (what lies past K is zeroed when it is stored)
#pragma unroll
        for (int i = 0; i < 2; ++i) ra[i] = *reinterpret_cast<const uint4 *>(pa[i] + ka);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            if constexpr (TB) {
                rb[i] = *reinterpret_cast<const uint4 *>(pb[i] + ka);
            } else {
                const int k = k0 + kq * 4 + i;
                rb[i] = *reinterpret_cast<const uint4 *>(pb[0] + (int64_t)(k < K ? k : 0) * g.ldb);
            }
        }
    };
    auto head = [](uint4 v, int n) {   // the first n elements (n may be negative or past 8), zeros after them
        v.x &= n >= 2 ? ~0u : n == 1 ? 0xffffu : 0u;
        v.y &= n >= 4 ? ~0u : n == 3 ? 0xffffu : 0u;
        v.z &= n >= 6 ? ~0u : n == 5 ? 0xffffu : 0u;
        v.w &= n >= 8 ? ~0u : n == 7 ? 0xffffu : 0u;
        return v;
    };
    auto put = [&](int k0) {
        if (k0 + KT > K) {   // uniform: the last k-tile
#pragma unroll
            for (int i = 0; i < 2; ++i) ra[i] = head(ra[i], K - k0 - av);
#pragma unroll
            for (int i = 0; i < 4; ++i) rb[i] = head(rb[i], TB ? K - k0 - av : k0 + kq * 4 + i < K ? 8 : 0);
        }
#pragma unroll
        for (int i = 0; i < 2; ++i) *reinterpret_cast<uint4 *>(As + (ar + 64 * i) * STR + av) = ra[i];
        if constexpr (TB) {
#pragma unroll
            for (int i = 0; i < 4; ++i) *reinterpret_cast<uint4 *>(Bs + (ar + 64 * i) * STR + av) = rb[i];
        } else {
            bf16_t *dst = Bs + rq * 8 * STR + kq * 4;
            const uint32_t w[4][4] = {{rb[0].x, rb[0].y, rb[0].z, rb[0].w}, {rb[1].x, rb[1].y, rb[1].z, rb[1].w},
                                      {rb[2].x, rb[2].y, rb[2].z, rb[2].w}, {rb[3].x, rb[3].y, rb[3].z, rb[3].w}};
#pragma unroll
            for (int c = 0; c < 4; ++c) {   // columns 2c and 2c + 1 of the patch: their four k as one 8-byte run each
                *reinterpret_cast<uint2 *>(dst + (2 * c) * STR) = make_uint2(lo16(w[0][c], w[1][c]), lo16(w[2][c], w[3][c]));
                *reinterpret_cast<uint2 *>(dst + (2 * c + 1) * STR) = make_uint2(hi16(w[0][c], w[1][c]), hi16(w[2][c], w[3][c]));
            }
        }
    };
    // acc[a][b], register 4 q + i: row (wm * 2 + a) * 32 + l32, column (wn * 2 + b) * 32 + 8 q + 4 h + i of the tile
    floatx16 acc[2][2];
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int64_t n = n0 + (wn * 2 + b) * 32 + 8 * q + 4 * h + i;
                const float x = g.bias && n < g.N ? g.bias[n] : 0.0f;
                acc[0][b][4 * q + i] = x;
                acc[1][b][4 * q + i] = x;
            }
    fetch(0);
    for (int k0 = 0; k0 < K; k0 += KT) {
        __syncthreads();   // previous tile fully consumed
        put(k0);
        __syncthreads();
        if (k0 + KT < K) fetch(k0 + KT);
#pragma unroll
        for (int s = 0; s < KT / 16; ++s) {
            const int kk = s * 16 + h * 8;   // lane half h supplies k = kk .. kk + 7 of this step
            bf16x8 af[2], bf[2];
#pragma unroll
            for (int a = 0; a < 2; ++a) af[a] = *reinterpret_cast<const bf16x8 *>(&As[((wm * 2 + a) * 32 + l32) * STR + kk]);
#pragma unroll
            for (int b = 0; b < 2; ++b) bf[b] = *reinterpret_cast<const bf16x8 *>(&Bs[((wn * 2 + b) * 32 + l32) * STR + kk]);
#pragma unroll
            for (int a = 0; a < 2; ++a)
#pragma unroll
                for (int b = 0; b < 2; ++b) acc[a][b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bf[b], af[a], acc[a][b], 0, 0, 0);
        }
    }
    __syncthreads();   // every wavefront is done reading the operand tiles
    bf16_t *Cs = reinterpret_cast<bf16_t *>(smem);   // [BM][CSTR]
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                float v[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    v[i] = acc[a][b][4 * q + i];
                    if (g.relu) v[i] = v[i] > 0.0f ? v[i] : 0.0f;
                }
                *reinterpret_cast<uint2 *>(Cs + ((wm * 2 + a) * 32 + l32) * CSTR + (wn * 2 + b) * 32 + 8 * q + 4 * h) =
                    make_uint2(gt_pack_bf16(v[0], v[1]), gt_pack_bf16(v[2], v[3]));
            }
    __syncthreads();
    const int64_t col = n0 + l32 * 8;
    const int left = (int)(g.N - col < 8 ? g.N - col : 8);   // this lane's columns of a row
    if (left <= 0) return;
    // whole vectors: inside N, or (padded rows whose padding may be written) the row's last one, zeros past N
    const bool whole = left == 8 || (g.pad_c && col + 8 <= g.ldc);
#pragma unroll
    for (int it = 0; it < BM / 16; ++it) {   // two rows at a time, 16 per wavefront
        const int r = wave * 16 + it * 2 + h;
        const int64_t row = m0 + r;
        if (row >= g.M) break;
        uint4 v = head(*reinterpret_cast<const uint4 *>(Cs + r * CSTR + l32 * 8), left);
        bf16_t *c = static_cast<bf16_t *>(g.C) + row * g.ldc + col;
        if constexpr (MASK) {   // zero where the mask is not positive (NaN included): sign set, zero, or above infinity
            const bf16_t *m = static_cast<const bf16_t *>(g.mask) + row * g.ldmask + col;
            bf16_t mk[8], *o = reinterpret_cast<bf16_t *>(&v);
            if (left == 8) __builtin_memcpy(mk, m, 16);
            else
                for (int i = 0; i < 8; ++i) mk[i] = i < left ? m[i] : 0;
#pragma unroll
            for (int i = 0; i < 8; ++i)
                if (!(gemm_bf16_to_f32(mk[i]) > 0.0f)) o[i] = 0;
        }
        if (whole) __builtin_memcpy(c, &v, 16);
        else {
            const bf16_t *o = reinterpret_cast<const bf16_t *>(&v);
#pragma unroll
            for (int i = 0; i < 7; ++i)
                if (i < left) c[i] = o[i];
        }
    }
}

template <bool TB>
gt_status launch_rows(const GemmArgs &g, hipStream_t st) {
    const void *f = g.mask ? reinterpret_cast<const void *>(&k_gemm_rows_bf16<TB, true>) : reinterpret_cast<const void *>(&k_gemm_rows_bf16<TB, false>);
    GT_HIP(hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)ROWS_LDS_BYTES));
    const dim3 grid(gemm_grid_x(g.ntm, g.ntn));
    if (g.mask) k_gemm_rows_bf16<TB, true><<<grid, 512, ROWS_LDS_BYTES, st>>>(g);
    else k_gemm_rows_bf16<TB, false><<<grid, 512, ROWS_LDS_BYTES, st>>>(g);
    GT_LAUNCH_CHECK("k_gemm_rows_bf16");
    return GT_OK;
}

}  // namespace

// Which products come here (vecA and vecB: rows of both operands aligned and padded to 16 bytes; vecC: those of C).  us, the kernel that
// would take it otherwise / this one:
//  * K past 256 (tiled kernels): more than 128 columns (2^19 x 602 -> 256 435 / 310, transposed weights 1000 columns, 200 K rows -> 256 265 / 183,
//    2 K rows, 602 -> 130 29 / 21); up to 128 columns, where half of the tile is padding, up to 50,000 rows (30 K rows, 602 -> 65
//    29 / 22, 200 K rows 88 / 97).
//  * Smaller K and fewer than 8,192 rows (tiled): from 4,096 rows on 0.53 to 0.74 of the time at any width; more than 128 columns from 2,000
//    rows on, or where the output has as many elements (2 K rows, 100 -> 130 0.58 of the time, 1.5 K rows 1.30, -> 300 0.71; 1 K rows -> 300
//    1.44, -> 602 0.61): below, the tiled kernel has more workgroups.
//  * Smaller K, more rows (weight-stationary, which holds 256 columns at a time and reads A once for each), more than 256 columns:
//    - more than 128 terms up to 65,536 rows (30 K rows, 256 -> 300 28 / 19; 70 K rows 1.07 of the time), unless the tiles are a round of
//      workgroups and a part of the next (16 K rows, 200 -> 602, 375 tiles 16.3 / 17.6; -> 1001, 500 tiles 0.71 of the time);
//    - large outputs whose rows are not aligned, since rows leave this kernel 512 bytes at a time: with up to 128 terms from 250 Mi elements
//      on (2^19 rows, 128 -> 602 0.87 of the time, -> 402 1.00; 1 M rows -> 300 1.01, -> 402 0.90; 350 K rows, 128 -> 602, 201 Mi, 1.05), transposed
//      weights from 200 Mi (2^19 rows, 128 -> 402 0.80, -> 602 0.67; 200 K rows, 100 -> 1001, 191 Mi, 1.03); with more terms
//      transposed weights of more than 384 columns (2^19 rows, 256 -> 602 0.79 of the time, 200 -> 402 1.00; 1 M rows, 200 -> 300 1.09; weights as they are
//      256 -> 402 1.10, -> 602 1.00).
bool gt_gemm_rows_applicable(gt_dtype dtype, gt_dtype c_dtype, int transA, int transB, int64_t M, int64_t N, int64_t K, int vecA, int vecB, int vecC) {
    if (dtype != GT_BF16 || c_dtype != GT_BF16 || transA || !vecA || !vecB || M < 1024 || N <= 64 || K < 64 || K >= ((int64_t)1 << 30)) return false;
    if (K > 256) return N > 128 || M <= 50000;
    if (M < 8192) return M >= 4096 || (N > 128 && (M >= 2000 || M * N >= 420000));
    if (N <= 256) return false;
    const int64_t tiles = (M + BM - 1) / BM * ((N + BN - 1) / BN), Mi = (int64_t)1 << 20;
    if (K > 128 && M <= 65536) return tiles <= 256 || tiles >= 448;
    if (vecC) return false;
    if (K > 128) return transB && N > 384 && M * N >= 200 * Mi;
    return M * N >= (transB ? 200 : 250) * Mi;
}

gt_status gt_gemm_rows_launch(GemmArgs g, int transB, hipStream_t st) {
    g.ntm = (int)((g.M + BM - 1) / BM);
    g.ntn = (int)((g.N + BN - 1) / BN);
    g.split_xcd = 0;
    return transB ? launch_rows<true>(g, st) : launch_rows<false>(g, st);
}
