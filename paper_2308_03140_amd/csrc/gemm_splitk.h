// Tile product on the FP64 matrix cores with K split over the wavefronts of a
// workgroup, for operands read along their columns: C(m, c) = sum_k A(m, k)
// B(c, k), A and B column-major (a symmetric matrix serves as either).
#pragma once
#include "gemm_mfma.h"
#include "mbd_internal.h"
#include "splitk_extent.h"

// Each of the WK wavefronts computes the whole 16 MI x 16 NJ tile over its own
// K groups, straight from L2 into registers (no LDS staging and no barrier in
// the loop; no load is made twice, since the wavefronts read different K).  A
// lane's 16-byte load holds rows 2r, 2r + 1 (r = lane mod 16), one for each of
// two MFMA tiles: tile i covers the rows of parity i mod 2 of its 32.  The
// descriptor's size ends the K loop (columns past K read zero) and lies within
// the matrix (splitk_extent.h); rows past ld continue in the next column and
// only reach rows of C that the caller does not use.  Two register sets
// of U k-steps alternate, so U MFMA steps hide each load.
typedef double splitk_d2 __attribute__((ext_vector_type(2)));

template <int MI, int NJ, int WK, int U>
struct SplitK {
    static_assert(MI % 2 == 0 && NJ % 2 == 0 && WK >= 2, "tile and wave split");
    static constexpr int TM = 16 * MI, TN = 16 * NJ, NT = 64 * WK, LDC = TM + 2;
    static constexpr int LDS = 2 * TN * LDC;  // doubles
    typename mfma4<double>::v acc[MI][NJ];
    splitk_d2 ra[2][U][MI / 2], rb[2][U][NJ / 2];

    __device__ __forceinline__ void clear() {
#pragma unroll
        for (int i = 0; i < MI; i++)
#pragma unroll
            for (int j = 0; j < NJ; j++) acc[i][j] = typename mfma4<double>::v{0, 0, 0, 0};
    }
    // acc += (NEG: -=) sum over K columns of A(row_a .., k) B(row_b .., k); A, B at row 0
    template <bool NEG = false>
    __device__ __forceinline__ void run(const double* A, int row_a, int lda, const double* B, int row_b, int ldb, int K) {
        A += row_a;
        B += row_b;
        constexpr int G = 4 * U;  // k of one group; groups go round robin over the wavefronts
        const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
        const unsigned offa = (unsigned)((lane >> 4) * lda + 2 * (lane & 15)) * 8u;
        const unsigned offb = (unsigned)((lane >> 4) * ldb + 2 * (lane & 15)) * 8u;
        auto gload = [&](int k0, auto& xa, auto& xb) {
            const int kn = max(0, min(G, K - k0));
            const auto dA = make_rsrc(A + (long long)k0 * lda, splitk_bytes(kn, lda, row_a));
            const auto dB = make_rsrc(B + (long long)k0 * ldb, splitk_bytes(kn, ldb, row_b));
#pragma unroll
            for (int u = 0; u < U; u++) {
#pragma unroll
                for (int i = 0; i < MI / 2; i++)
                    xa[u][i] = __builtin_bit_cast(splitk_d2,
                                                  __builtin_amdgcn_raw_buffer_load_b128(dA, offa + 256u * i, 32 * u * lda, 0));
#pragma unroll
                for (int j = 0; j < NJ / 2; j++)
                    xb[u][j] = __builtin_bit_cast(splitk_d2,
                                                  __builtin_amdgcn_raw_buffer_load_b128(dB, offb + 256u * j, 32 * u * ldb, 0));
            }
        };
        auto mult = [&](auto& xa, auto& xb) {
#pragma unroll
            for (int u = 0; u < U; u++)
#pragma unroll
                for (int i = 0; i < MI; i++)
#pragma unroll
                    for (int j = 0; j < NJ; j++) {
                        const double a = xa[u][i / 2][i & 1];
                        acc[i][j] = mfma16x16x4(NEG ? -a : a, xb[u][j / 2][j & 1], acc[i][j]);
                    }
        };
        const int ng = (K + G - 1) / G;
        int g = wave;
        gload(g * G, ra[0], rb[0]);
        while (g < ng) {
            gload((g + WK) * G, ra[1], rb[1]);
            mult(ra[0], rb[0]);
            g += WK;
            if (g >= ng) break;
            gload((g + WK) * G, ra[0], rb[0]);
            mult(ra[1], rb[1]);
            g += WK;
        }
    }
    // acc += sum over K of A(row_a .., k) B(k, n0 ..), A at row 0, B column-major, columns
    // nb of them from B: a lane's 16-byte load of B holds rows k, k + 1 of one
    // column, so the k of an MFMA step are 2 apart (K even)
    __device__ __forceinline__ void run_cols(const double* A, int row_a, int lda, const double* B, int ldb, int nb, int K) {
        A += row_a;
        constexpr int D = U / 2, G = 8 * D;
        static_assert(U % 2 == 0, "pairs of k-steps");
        const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), kl = 2 * (lane >> 4);
        const unsigned offa = (unsigned)(kl * lda + 2 * (lane & 15)) * 8u;
        const unsigned offb = (unsigned)((lane & 15) * ldb + kl) * 8u;
        const auto dB = make_rsrc(B, splitk_bytes(nb, ldb, 0));
        splitk_d2 sa[2][U][MI / 2], sb[2][D][NJ];
        auto gload = [&](int k0, auto& xa, auto& xb) {
            const int kn = max(0, min(G, K - k0));
            const auto dA = make_rsrc(A + (long long)k0 * lda, splitk_bytes(kn, lda, row_a));
#pragma unroll
            for (int u = 0; u < U; u++)
#pragma unroll
                for (int i = 0; i < MI / 2; i++)
                    xa[u][i] = __builtin_bit_cast(
                        splitk_d2, __builtin_amdgcn_raw_buffer_load_b128(dA, offa + 256u * i, (u / 2 * 8 + u % 2) * lda * 8, 0));
#pragma unroll
            for (int d = 0; d < D; d++) {
                const unsigned o = 8 * d + kl < kn ? offb + (unsigned)(k0 + 8 * d) * 8u : OOB_OFFSET;
#pragma unroll
                for (int j = 0; j < NJ; j++)
                    xb[d][j] = __builtin_bit_cast(splitk_d2, __builtin_amdgcn_raw_buffer_load_b128(dB, o + (unsigned)(16 * j * ldb) * 8u, 0, 0));
            }
        };
        auto mult = [&](auto& xa, auto& xb) {
#pragma unroll
            for (int u = 0; u < U; u++)
#pragma unroll
                for (int i = 0; i < MI; i++)
#pragma unroll
                    for (int j = 0; j < NJ; j++) acc[i][j] = mfma16x16x4(xa[u][i / 2][i & 1], xb[u / 2][j][u & 1], acc[i][j]);
        };
        const int ng = (K + G - 1) / G;
        int g = wave;
        gload(g * G, sa[0], sb[0]);
        while (g < ng) {
            gload((g + WK) * G, sa[1], sb[1]);
            mult(sa[0], sb[0]);
            g += WK;
            if (g >= ng) break;
            gload((g + WK) * G, sa[0], sb[0]);
            mult(sa[1], sb[1]);
            g += WK;
        }
    }
    // The wavefronts' shares into cs (two halves of TN x LDC, column-major): two
    // write, the others add in turn; the tile is the sum of the halves.
    // COLS: after run_cols, whose tile columns are not interleaved in pairs.
    template <bool COLS = false>
    __device__ __forceinline__ void reduce(double* cs) const {
        const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
#pragma unroll
        for (int w = 0; w < WK; w += 2) {
            if (wave >= w && wave < w + 2) {
                double* c = cs + (wave & 1) * TN * LDC;
#pragma unroll
                for (int i = 0; i < MI; i++)
#pragma unroll
                    for (int j = 0; j < NJ; j++)
#pragma unroll
                        for (int r = 0; r < 4; r++) {
                            const int row = 32 * (i / 2) + 2 * mfma_rows<double>::row(lane, r) + (i & 1);
                            const int col = COLS ? 16 * j + (lane & 15) : 32 * (j / 2) + 2 * (lane & 15) + (j & 1);
                            if (w == 0) c[col * LDC + row] = acc[i][j][r];
                            else c[col * LDC + row] += acc[i][j][r];
                        }
            }
            __syncthreads();
        }
    }
};

// Tile (ti, tj) of index v: row ti of tiles holds the R (ti + 1) tiles (R = TM /
// TN) on and left of the diagonal.
__device__ __forceinline__ void splitk_lower_tile(int v, int R, int& ti, int& tj) {
    ti = (int)((sqrtf(8.0f * (float)(v / R) + 1.0f) - 1.0f) * 0.5f);
    while (R * (ti + 1) * (ti + 2) / 2 <= v) ti++;
    while (R * ti * (ti + 1) / 2 > v) ti--;
    tj = v - R * ti * (ti + 1) / 2;
}
static inline int splitk_lower_tiles(int n, int tm, int tn) {
    const int rows = (n + tm - 1) / tm;
    return tm / tn * rows * (rows + 1) / 2;
}

// Workgroup bx's index in matrix b's tiles.  The shares of the XCDs rotate with
// the matrix, or the last rows of a batch, which only its largest matrices
// have, would all fall to one XCD (512 uneven molecules, 64 x 32 tiles: 4.9 ms
// a product against 2.4).
__device__ __forceinline__ int splitk_tile_index(int bx, int b, int G) {
    const int r = bx + b % G;
    return xcd_virtual(r >= G ? r - G : r, G);
}
