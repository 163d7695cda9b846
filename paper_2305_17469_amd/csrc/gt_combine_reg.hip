// Tall bf16 products  C[M, N] = act(A op(B) + bias)  whose weights fit the registers of a CU but not its LDS (up to 320 KB).
#include "gt_combine.h"

namespace {

typedef gemm_bf16_t bf16_t;
typedef float floatx4 __attribute__((ext_vector_type(4)));

// One persistent workgroup of eight wavefronts per CU keeps the whole weight matrix in registers: a wavefront owns 16 NB columns, as the
// MFMA fragments of all KS steps of 32 terms (4 NB KS registers, at most 160).  Blocks of 32 rows of A pass through two LDS buffers; every
// wavefront reads the whole block and multiplies it by its columns; the finished rows go through LDS too and leave as whole rows.
// Why: a CU has some 80 requests towards the L2 in flight, and 128 x 256 tiles spend two thirds of them on reading the
// weights again for every 128 rows (2^19 x 602 -> 256: 211 us with A out of the L2 and nothing stored, however deep the loads).  Here only A
// is read, and what bounds the kernel is memory: 2^19 rows, 602 -> 256 320 us in such tiles, 211 here (4.3 TB/s; 490 and 206 on contiguous rows),
// 256 -> 602 with transposed weights 370 and 229 (3.9 TB/s).
// Per 32 rows and 32 terms the CU reads 16 KB of LDS (128 clocks) and multiplies for 64 NB clocks, and a block of A (20 to 64 KB) is in flight all the time.
// The last block begins at row M - 32 (rows that two blocks form are written twice with the same bits); a row's last 16 bytes
// begin at column K - 8 of A and N - 8 of C.  No operand needs an alignment past its elements'.  Terms past K are zeros in both.
constexpr int BM = 32, NT = 512;

template <int NB, int KS>
struct RegShape {
    static constexpr int CH = (KS + 3) / 4;                     // 16-byte pieces of a block of A per thread
    static constexpr int SA = CH * 128 + 8, SC = NB * 128 + 8;  // LDS row strides (elements): consecutive rows begin four banks apart
    static constexpr size_t A_ELEMS = (size_t)BM * SA, C_ELEMS = (size_t)BM * SC;
    // steps of [k][n] weights that pass through LDS at a time, and the row stride there
    static constexpr int KSB_MAX = (int)((160 * 1024 / (NB * 128) - 4 - 16) / 64), PASSES = (KS + KSB_MAX - 1) / KSB_MAX, KSB = (KS + PASSES - 1) / PASSES;
    static constexpr int SW = KSB * 32 + 8;
    static constexpr size_t RUN = 2 * (A_ELEMS + C_ELEMS) * 2, SETUP = (size_t)NB * 128 * SW * 2;
    static constexpr size_t BYTES = (RUN > SETUP ? RUN : SETUP) + (size_t)NB * 128 * 4;   // bias at the end
    static_assert(4 * NB * KS <= 160 && BYTES <= 160 * 1024 && KSB >= 1, "registers and LDS of a CU");
};

__device__ inline uint32_t lo16(uint32_t a, uint32_t b) { return __builtin_amdgcn_perm(b, a, 0x05040100u); }   // lo16(a) | lo16(b) << 16
__device__ inline uint32_t hi16(uint32_t a, uint32_t b) { return __builtin_amdgcn_perm(b, a, 0x07060302u); }   // hi16(a) | hi16(b) << 16
__device__ inline uint4 head8(uint4 v, int n) {   // the first n elements (n may be negative or past 8), zeros after them
    v.x &= n >= 2 ? ~0u : n == 1 ? 0xffffu : 0u;
    v.y &= n >= 4 ? ~0u : n == 3 ? 0xffffu : 0u;
    v.z &= n >= 6 ? ~0u : n == 5 ? 0xffffu : 0u;
    v.w &= n >= 8 ? ~0u : n == 7 ? 0xffffu : 0u;
    return v;
}

template <int NB, int KS, bool MASK>
__global__ void __launch_bounds__(NT, 2) k_gemm_reg_bf16(const GemmArgs g, const int transB, const int blocks, const int slices, const int cols) {
    using S = RegShape<NB, KS>;
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    bf16_t *As = reinterpret_cast<bf16_t *>(smem), *Cs = As + 2 * S::A_ELEMS;
    float *bias = reinterpret_cast<float *>(smem + S::BYTES) - NB * 128;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int l16 = lane & 15, kg = lane >> 4;
    // The columns may be cut into slices, a workgroup for each; those of the same rows run on one XCD and find A in its L2.
    const int xcd = blockIdx.x & 7, seq = blockIdx.x >> 3, slice = seq % slices;
    const int first = seq / slices * 8 + xcd, step = 256 / 8 / slices * 8;   // this workgroup's first block of rows, and from one to its next
    const int n0 = slice * cols, K = (int)g.K, N = (int)(g.N - n0 < cols ? g.N - n0 : cols);   // the slice's columns
    if (first >= step || first >= blocks) return;   // whole workgroups
    const bf16_t *B = static_cast<const bf16_t *>(g.B) + (transB ? (int64_t)n0 * g.ldb : n0);

    // ---- the wavefront's columns: fragment (nb, ks), lane: column ncol + 16 nb + l16, terms 32 ks + 8 kg .. + 7
    bf16x8 w[NB][KS];
    const int ncol = wave * NB * 16;
    // Eight elements of B from position i on, at any alignment.  What lies past a row's end is the next row's and takes part in nothing; the
    // vector that would leave the matrix is moved back first and then read by element.
    const int64_t left = ((transB ? g.N - n0 : g.K) - 1) * g.ldb + (transB ? g.K : g.N - n0);   // elements from B to the end of the matrix
    auto load8 = [&](int64_t i) { uint4 v; __builtin_memcpy(&v, B + (i + 8 <= left ? i : left - 8), 16); return v; };
    auto mend8 = [&](uint4 &v, int64_t i) {
        for (int64_t e = i + 8 - left; e > 0; --e)   // one element down
            v = make_uint4(v.x >> 16 | v.y << 16, v.y >> 16 | v.z << 16, v.z >> 16 | v.w << 16, v.w >> 16);
    };
    if (transB) {
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) {
            const int n = ncol + nb * 16 + l16;
            const int64_t p = (int64_t)(n < N ? n : N - 1) * g.ldb;
            uint4 v[KS];
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) v[ks] = load8(p + (ks * 32 + kg * 8 < K ? ks * 32 + kg * 8 : 0));
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) {
                const int k = ks * 32 + kg * 8;
                if (k < K) mend8(v[ks], p + k);
                v[ks] = head8(v[ks], K - k);
                __builtin_memcpy(&w[nb][ks], &v[ks], 16);
            }
        }
    } else {
        // [k][n] weights pass through LDS, KSB steps at a time, transposed on the way (patches of 4 k and 8 n): a fragment is one read
        bf16_t *Ws = As;   // [NB * 128][SW]
        constexpr int KQ = S::KSB * 8;   // patches along k
#pragma unroll
        for (int k0 = 0; k0 < KS; k0 += S::KSB) {
            __syncthreads();
            // all of a thread's loads first: a pass takes one latency of the L2
            constexpr int PT = (KQ * NB * 16 + NT - 1) / NT;
            uint4 v[PT][4];
#pragma unroll
            for (int t = 0; t < PT; ++t) {
                const int c = threadIdx.x + t * NT, kq = c % KQ, nq = c / KQ, k = k0 * 32 + kq * 4;
                const int p = (nq * 8 < N ? nq : (N - 1) / 8) * 8;
#pragma unroll
                for (int i = 0; i < 4; ++i) v[t][i] = load8((int64_t)(k + i < K ? k + i : K - 1) * g.ldb + p);
            }
#pragma unroll
            for (int t = 0; t < PT; ++t) {
                const int c = threadIdx.x + t * NT, kq = c % KQ, nq = c / KQ, k = k0 * 32 + kq * 4;
                if (nq >= NB * 16) break;
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    if (nq * 8 < N && k + i < K) mend8(v[t][i], (int64_t)(k + i) * g.ldb + nq * 8);
                    v[t][i] = head8(v[t][i], k + i < K ? 8 : 0);
                }
                const uint32_t x[4][4] = {{v[t][0].x, v[t][0].y, v[t][0].z, v[t][0].w}, {v[t][1].x, v[t][1].y, v[t][1].z, v[t][1].w},
                                          {v[t][2].x, v[t][2].y, v[t][2].z, v[t][2].w}, {v[t][3].x, v[t][3].y, v[t][3].z, v[t][3].w}};
                bf16_t *dst = Ws + nq * 8 * S::SW + kq * 4;
#pragma unroll
                for (int j = 0; j < 4; ++j) {   // columns 2 j and 2 j + 1 of the patch
                    *reinterpret_cast<uint2 *>(dst + 2 * j * S::SW) = make_uint2(lo16(x[0][j], x[1][j]), lo16(x[2][j], x[3][j]));
                    *reinterpret_cast<uint2 *>(dst + (2 * j + 1) * S::SW) = make_uint2(hi16(x[0][j], x[1][j]), hi16(x[2][j], x[3][j]));
                }
            }
            __syncthreads();
#pragma unroll
            for (int ks = k0; ks < k0 + S::KSB && ks < KS; ++ks)
#pragma unroll
                for (int nb = 0; nb < NB; ++nb)
                    w[nb][ks] = *reinterpret_cast<const bf16x8 *>(Ws + (ncol + nb * 16 + l16) * S::SW + (ks - k0) * 32 + kg * 8);
        }
        __syncthreads();
    }
    for (int n = threadIdx.x; n < NB * 128; n += NT) bias[n] = g.bias && n < N ? g.bias[n0 + n] : 0.0f;

    // terms past K are zeros in both buffers for good
    for (int i = threadIdx.x; i < 2 * BM * S::SA; i += NT)
        if (i % S::SA >= K) As[i] = 0;
    // ---- this thread's row of every block, and of it every sixteenth piece of eight elements (the last one begins at K - 8; past it that one again)
    const int r = threadIdx.x >> 4, q = threadIdx.x & 15;
    const int lastc = (N - 1) / 8;
    const bool pad = g.pad_c && n0 + (int64_t)(lastc + 1) * 8 <= g.ldc;   // a row's last piece may run past N (zeros there)
    const uint32_t arow = (uint32_t)(r * g.lda) * 2;
    auto row0 = [&](int b) -> int64_t { const int64_t m = (int64_t)b * BM; return m + BM <= g.M ? m : g.M - BM; };
    uint4 ra[S::CH];
    auto fetch = [&](int b) {
        const char *p = static_cast<const char *>(g.A) + row0(b < blocks ? b : blocks - 1) * g.lda * 2;
        int q = threadIdx.x & 15;
        asm volatile("" : "+v"(q));
#pragma unroll
        for (int i = 0; i < S::CH; ++i) {
            const int c = q + 16 * i;
            __builtin_memcpy(&ra[i], p + (arow + (uint32_t)(c * 8 < K - 8 ? c * 8 : K - 8) * 2), 16);
        }
    };
    auto put = [&](int buf) {
        bf16_t *dst = As + buf * S::A_ELEMS + r * S::SA;
#pragma unroll
        for (int i = 0; i < S::CH; ++i) {
            const int c = (q + 16 * i) * 8, k = c < K - 8 ? c : K - 8;
            if (i * 128 + 128 <= K || !(K & 7)) *reinterpret_cast<uint4 *>(dst + k) = ra[i];   // uniform
            else if (!(K & 1)) {
                uint32_t *d = reinterpret_cast<uint32_t *>(dst + k);
                d[0] = ra[i].x; d[1] = ra[i].y; d[2] = ra[i].z; d[3] = ra[i].w;
            } else {
                const uint32_t u[4] = {ra[i].x, ra[i].y, ra[i].z, ra[i].w};
#pragma unroll
                for (int j = 0; j < 4; ++j) { dst[k + 2 * j] = (bf16_t)u[j]; dst[k + 2 * j + 1] = (bf16_t)(u[j] >> 16); }
            }
        }
    };
    const bool live = ncol < N;

    int b = first;
    fetch(b);
    put(0);
    fetch(b + step);
    __syncthreads();
    for (int buf = 0; b < blocks; b += step, buf ^= 1) {
        if (live) {
            floatx4 acc[2][NB];
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) acc[0][nb] = acc[1][nb] = *reinterpret_cast<const floatx4 *>(bias + ncol + nb * 16 + 4 * kg);
            const bf16_t *a0 = As + buf * S::A_ELEMS + l16 * S::SA + kg * 8;
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) {
                bf16x8 af[2];
#pragma unroll
                for (int m = 0; m < 2; ++m) af[m] = *reinterpret_cast<const bf16x8 *>(a0 + m * 16 * S::SA + ks * 32);
#pragma unroll
                for (int m = 0; m < 2; ++m)
#pragma unroll
                    for (int nb = 0; nb < NB; ++nb) acc[m][nb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[nb][ks], af[m], acc[m][nb], 0, 0, 0);
            }
            // weights first: a lane holds four consecutive columns of row l16
            bf16_t *c0 = Cs + buf * S::C_ELEMS + l16 * S::SC + ncol + 4 * kg;
#pragma unroll
            for (int m = 0; m < 2; ++m)
#pragma unroll
                for (int nb = 0; nb < NB; ++nb) {
                    float v[4];
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        v[i] = acc[m][nb][i];
                        if (g.relu) v[i] = v[i] > 0.0f ? v[i] : 0.0f;
                    }
                    *reinterpret_cast<uint2 *>(c0 + m * 16 * S::SC + nb * 16) = make_uint2(gt_pack_bf16(v[0], v[1]), gt_pack_bf16(v[2], v[3]));
                }
        }
        put(buf ^ 1);
        fetch(b + 2 * step);   // before the stores: loads and stores complete in the order of their issue
        __syncthreads();            // this block is multiplied and its rows are in LDS; the next is there
        const int64_t m0 = row0(b);
        const bf16_t *cs = Cs + buf * S::C_ELEMS + r * S::SC;
        char *crow = static_cast<char *>(g.C) + ((m0 + r) * g.ldc + n0) * 2;
        int qc = q;
        asm volatile("" : "+v"(qc));   // columns are worked out again for every block: kept, they cost registers that the weights need
        int col[NB];
#pragma unroll
        for (int i = 0; i < NB; ++i) {
            const int c = (qc + 16 * i < lastc ? qc + 16 * i : lastc) * 8;
            col[i] = pad || c + 8 <= N ? c : N - 8;
        }
        uint4 v[NB];
        if (pad || !(N & 7)) {
#pragma unroll
            for (int i = 0; i < NB; ++i) v[i] = head8(*reinterpret_cast<const uint4 *>(cs + col[i]), N - col[i]);
        } else if (!(N & 1)) {
#pragma unroll
            for (int i = 0; i < NB; ++i) {
                const uint32_t *p = reinterpret_cast<const uint32_t *>(cs + col[i]);
                v[i] = make_uint4(p[0], p[1], p[2], p[3]);
            }
        } else {
#pragma unroll
            for (int i = 0; i < NB; ++i) {
                const bf16_t *p = cs + col[i];
                v[i] = make_uint4(p[0] | (uint32_t)p[1] << 16, p[2] | (uint32_t)p[3] << 16, p[4] | (uint32_t)p[5] << 16, p[6] | (uint32_t)p[7] << 16);
            }
        }
        if constexpr (MASK) {   // zero where the mask is not positive (NaN included)
            const bf16_t *mrow = static_cast<const bf16_t *>(g.mask) + (m0 + r) * g.ldmask + n0;
#pragma unroll
            for (int i = 0; i < NB; ++i) {
                bf16_t m[8], *o = reinterpret_cast<bf16_t *>(&v[i]);
                __builtin_memcpy(m, mrow + col[i], 16);
#pragma unroll
                for (int e = 0; e < 8; ++e)
                    if (!(gemm_bf16_to_f32(m[e]) > 0.0f)) o[e] = 0;
            }
        }
#pragma unroll
        for (int i = 0; i < NB; ++i) __builtin_memcpy(crow + col[i] * 2, &v[i], 16);
    }
}

struct Slices { int nb, ks, slices, cols; };   // instance, and how the columns are cut

// Instances in the order in which they are looked for: the first that takes the columns in the fewest slices.
constexpr int INSTANCES[][2] = {{1, 16}, {1, 20}, {1, 26}, {1, 32}, {2, 12}, {2, 16}, {2, 20}, {3, 8}, {3, 10}, {3, 13}, {4, 8}, {4, 10}, {5, 4}, {5, 8}, {8, 4}};

Slices pick(int64_t N, int64_t K) {
    Slices best{0, 0, 0, 0};
    const int64_t ks = (K + 31) / 32;
    for (const auto &c : INSTANCES) {
        if (c[1] < ks) continue;
        const int64_t s = (N + c[0] * 128 - 1) / (c[0] * 128);
        if (best.nb && (s > best.slices || (s == best.slices && c[0] * c[1] >= best.nb * best.ks))) continue;
        best = Slices{c[0], c[1], (int)s, (int)(((N + s - 1) / s + 7) / 8 * 8)};
    }
    return best;
}

template <int NB, int KS>
gt_status launch_reg(const GemmArgs &g, int transB, const Slices &s, hipStream_t st) {
    constexpr size_t lds = RegShape<NB, KS>::BYTES;
    const int blocks = (int)((g.M + BM - 1) / BM);
    const void *f = g.mask ? reinterpret_cast<const void *>(&k_gemm_reg_bf16<NB, KS, true>) : reinterpret_cast<const void *>(&k_gemm_reg_bf16<NB, KS, false>);
    GT_HIP(hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
    if (g.mask) k_gemm_reg_bf16<NB, KS, true><<<256, NT, lds, st>>>(g, transB, blocks, s.slices, s.cols);
    else k_gemm_reg_bf16<NB, KS, false><<<256, NT, lds, st>>>(g, transB, blocks, s.slices, s.cols);
    GT_LAUNCH_CHECK("k_gemm_reg_bf16");
    return GT_OK;
}

}  // namespace

// Which products come here.  us, the kernel that would take it otherwise / this one, weights as they are stored [k][n] unless said; setting the weights up
// costs 8 to 12 us (transposed ones 3 to 5, unaligned transposed ones up to 25), so the middle of the range of M stays with the row tiles
// (operands' rows aligned and padded to 16 bytes: vec) wherever a round or two of them is enough.  With few terms a block of A is 4 to 8 KB, too little in flight
// to hide its latency behind, so that a tile's round is ahead until the tiles fill many rounds; at up to 512 columns only five to seven of the eight wavefronts
// have columns besides.  The lines below are those of 16,000 random products (K 64 to 1,024, N 65 to 1,280, M 1,024 to 600,000, both orders of the weights, padded and
// contiguous) and of 1,800 at round sizes: this kernel takes 0.68 and 0.79 of the time of the others in the geometric mean of what it is given; 2 % of them are slower by more than 3 %.
//  * Rows without that alignment, which the general tiles read by element at the matrix's ends and hold a tile of weights four times as long: from 2,000
//    rows on, 1,024 with more than 256 terms (2 K rows, 602 -> 255 33.1 / 23.0, 131 K rows 166 / 69, 257 -> 602 230 / 84; 4 K rows, 65 -> 300 14.5 / 9.4); more than
//    384 columns in one slice past 18,432 with more than 256 terms (3 K rows, 320 -> 443 1.24 of the time), more than 512 from 8,192 (2.5 K rows, 150 -> 560 1.2);
//    transposed weights of more than 256 columns and others of more than 640 from 32,768 (16 K rows, 257 -> 602 transposed 29.4 / 34.7, 33 K rows 52.6 / 45.2; 16 K
//    rows, 101 -> 1000 14.8 / 22.1, 33 K rows 33.8 / 31.9).  Up to 128 terms (transposed weights past 32,768 rows only): 257 to 320 columns up to 18,432 rows and past 32,768 (32,768 rows, 75 -> 257 1.12 of
//    the time, 50 K 0.84), 321 to 512 up to 8,192, past 32,768 up to 98,304 (163,840 past 448 columns) and from 393,216 (16 K rows, 100 -> 401 1.09, 32,768 1.28, 50 K 0.96, 169 K 1.09, 2^19 0.81), 513 to 640 up to
//    8,192 and from 24,576 (12 K rows 1.1, 32,768 0.65), 641 to 768 past 32,768 but for 163,840 to 262,144 (1.0 to 1.06), more past 32,768.
//  * K past 640 and more than 128 columns (two slices of 128, A read twice): up to 8,192 rows, 16,384 of transposed weights, which are too few row tiles (4 K rows, 800 -> 130 23.0 /
//    13.5, 12 K rows 1.1 of the time; 33 K rows 25.1 / 27.0, 400 K rows, 700 -> 200 245 / 263).
//  * K up to 128 and more than 256 columns (weight-stationary from LDS, 256 columns at a time, or tiles): widths whose rows of C end inside a line, which those write in pieces: up to
//    512 columns from 2^19 rows on (128 -> 300 166 / 122, 128 -> 320 even, 154 K rows, 64 -> 325 transposed 1.8 of the time), 513 to 768 from 393,216 (2^19 rows, 100 -> 602 0.71, 64 -> 768 1.13; 131 K rows, 64 ->
//    602 1.19), more from 196,608 (2^18 rows, 128 -> 1000 0.64, 128 -> 1024 1.05; 131 K rows, 64 -> 1000 1.17).
//  * K of 129 to 256 and more than 256 columns: past 49,152 rows (400 K rows, 256 -> 602 295 / 178; 33 K rows 27.8 / 28.6), past 384 columns past 65,536 (65,536 rows, which are two full
//    rounds of tiles, 160 -> 512 1.15 of the time), past 640 from 131,072.
//  * K past 256, several slices: from 49,152 rows on (65 K rows, 512 -> 400 41.6 / 43, 320 -> 640 55 / 46, 2^18 rows 0.7 to 0.8 of the time; 16 K rows 20.7 / 21.8).
//  * K past 256, more than 256 columns in one slice: past 32,768 rows (65 K rows, 400 -> 300 54 / 38; 32,768 rows, 400 -> 384 1.20 of the time), past 384 columns past 65,536 (8 K to
//    16 K rows of transposed weights 1.2 to 1.3).
//  * K past 256, 129 to 256 columns: up to 8,192 rows of transposed weights (4 K rows, 602 -> 256 17.0 / 10.4; 10 K rows 1.03 to 1.14 of the time), 4,096 of others with up to 512 terms
//    (4,096 rows, 400 -> 256 1.11), and past 65,536 (65,536 rows, 512 -> 256 1.23, 2^18 rows 0.7), with more than 512 terms past 98,304 (131 K rows, 602 -> 256 64.9 / 58.3, 2^19 rows 306 / 211).
//  * K past 256, up to 128 columns: from 2,000 rows on (4 K rows, 300 -> 128 12.0 / 7.7, 1000 -> 70 27.0 / 13.9; 400 K rows 124 / 92, 287 / 170), but not where the row tiles come to one full
//    round, past 18,432 rows and up to 32,768 (32,768 rows, 300 -> 128 1.23 of the time, 400 -> 128 1.06; 513 to 640 terms 0.9, more of transposed weights 0.95), and with fewer than 320 terms up to 98,304
//    (50 K rows, 300 -> 128 1.13, 100 K rows 0.83), fewer than 288 up to 262,144 (1.0 to 1.2).
bool gt_gemm_reg_applicable(gt_dtype dtype, gt_dtype c_dtype, int transA, int transB, int64_t M, int64_t N, int64_t K, int64_t lda, bool vec) {
    if (dtype != GT_BF16 || c_dtype != GT_BF16 || transA || N <= 64 || K < 64 || K > 1024 || N > 2048) return false;
    if (M < 1024 || M >= ((int64_t)1 << 35) || lda >= ((int64_t)1 << 25)) return false;   // (block numbers and offsets inside a block in 32 bits)
    if (K <= 256 && N <= 256) return false;
    const int slices = pick(N, K).slices;
    if (!slices || slices > 2) return false;
    if (!vec) {
        if (K <= 128 && N > 256) {
            if (M <= 32768 && (transB || N > 640)) return false;
            if (N <= 320) return M > 32768 || (M >= 2000 && M <= 18432);
            if (N <= 512) return M >= 393216 || (M > 32768 && M < (N <= 448 ? 98304 : 163840)) || (M >= 2000 && M < 8192);
            if (N <= 640) return M >= 24576 || (M >= 2000 && M < 8192);
            return N > 768 || M < 163840 || M >= 262144;
        }
        if (N > (transB ? 256 : 640)) return M >= 32768;
        if (slices == 1 && N > 384) return M >= (K > 256 ? 18433 : N > 512 ? 8192 : 2000);
        return M >= (K > 256 ? 1024 : 2000);
    }
    if (K > 640 && N > 128) return M <= (transB ? 16384 : 8192);
    if (K <= 128) return N % 64 != 0 && M >= (N <= 512 ? 524288 : N <= 768 ? 393216 : 196608);
    if (K <= 256) return N > 640 ? M >= 131072 : M > (N > 384 ? 65536 : 49152);
    if (slices > 1) return M >= 49152;
    if (N > 256) return M > (N > 384 ? 65536 : 32768);
    if (N > 128) return M > (K > 512 ? 98304 : 65536) || (transB ? M < 8192 : M < 4096 && K <= 512);
    if (M <= 18432) return M >= 2000;
    if (K < 320) return M >= (K < 288 ? 262144 : 98304);
    return M > 32768 || (K > 512 && (transB || K <= 640));
}

gt_status gt_gemm_reg_launch(const GemmArgs &g, int transB, hipStream_t st) {
    const Slices s = pick(g.N, g.K);
#define GT_REG(NB_, KS_) if (s.nb == NB_ && s.ks == KS_) return launch_reg<NB_, KS_>(g, transB, s, st)
    GT_REG(1, 16); GT_REG(1, 20); GT_REG(1, 26); GT_REG(1, 32); GT_REG(2, 12); GT_REG(2, 16); GT_REG(2, 20); GT_REG(3, 8);
    GT_REG(3, 10); GT_REG(3, 13); GT_REG(4, 8); GT_REG(4, 10); GT_REG(5, 4); GT_REG(5, 8); GT_REG(8, 4);
#undef GT_REG
    return gt_fail(GT_ERR_INTERNAL, "gt_gemm_reg_launch: no instance");
}
