// Batched Cholesky factorisation A = L L^T of symmetric positive definite
// FP64 matrices and solves with a few right-hand sides.  The screening of
// MBD@rsSCS (Sec. 2.3, eq:scs) needs alpha_bar(u) = A(u)^-1 only through
// alpha_bar B, with B = 1 (x) I_3 for the contraction (eq:contraction) and
// B = w (x) I_3 for the gradient, so one factorisation per frequency and
// two three-column solves replace the inverse.  A non-positive pivot (A not
// positive definite: the screening collapses) sets MBD_ST_COLLAPSE.
//
// Left-looking, panels of CHOL_NB = 64 columns:
//   update           A(k0.., k0..k0+63) -= L(k0.., 0..k0-1) L(k0..k0+63, 0..k0-1)^T,
//                    one long product per panel (matrix cores, K split over
//                    the wavefronts): each element is read and written once
//                    per factorisation instead of once per panel;
//   diagonal block   one workgroup per matrix factors the 64 x 64 block and
//                    inverts its factor, L11^-1, kept for the panel solve and
//                    the triangular solves;
//   panel            L21 = A21 L11^-T as a matrix-core product, in place.
// The triangular solves go by wide blocks of 256 rows: the inverses of the 64 x
// 64 blocks are first extended to those of the wide diagonal blocks, then a
// sweep alternates between a wide block's solution (its inverse times the
// residual) and the update of the rows still to come, two launches per wide
// block (16 matrices of order 3000: 0.24 ms a sweep and 0.11 for the inverses;
// steps of 64 rows took 9.3 us each, 0.44 ms a sweep).  The wide inverses take
// four times the storage; where that is refused, blocks of 64 rows serve.
#include <algorithm>

#include "gemm_splitk.h"
#include "mbd_internal.h"
#include "mbd_kernels.h"
#include "mbd_sys.h"

#define CHOL_NR 3  // right-hand sides per solve

// inverse of the 64 x 64 diagonal block at k0 (column-major, leading dimension
// wb) within that of its wide block of wb rows; matrix b's wide block w at w wb^2
__device__ __forceinline__ double* chol_inv_block(double* Linv, long long sLi, int b, int k0, int wb) {
    const int o = k0 % wb;
    return Linv + (long long)b * sLi + (long long)(k0 / wb) * wb * wb + o + (long long)o * wb;
}

// ---------------------------------------------------------------------------
// diagonal block: factor, invert the factor; identity padding past n
// ---------------------------------------------------------------------------
// One workgroup per matrix, the block in LDS, in steps of 16 columns: one
// wavefront factors the 16 columns with a row per lane (pivot and row factors
// by lane reads, no barrier), then four update the rest on the matrix cores.
// The inverse: the 16 x 16 diagonal blocks by substitution, one per wavefront,
// then the blocks below by distance from the diagonal on the matrix cores.
// Bound by the chain of 64 pivots: 21.5 us at 16 matrices, against 101 column
// by column with three barriers a column.
#define CHOL_SB 16
__global__ __launch_bounds__(256) void chol_diag_kernel(MatBatch<double> A, double* Linv, long long sLi, int wb,
                                                         int n, int k0, unsigned* status) {
    __shared__ double L[CHOL_NB][CHOL_NB + 1];
    __shared__ double X[CHOL_NB][CHOL_NB + 1];
    __shared__ double dinv[CHOL_NB];
    const int b = blockIdx.x, tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int w = min(CHOL_NB, n - k0);
    double* Ab = A.at(b) + k0 + (long long)k0 * A.ld;
    const long long ld = A.ld;
    constexpr int PER = CHOL_NB * CHOL_NB / 256;
    const int ri = tid & (CHOL_NB - 1), j0 = tid >> 6;
    {
        // all 16 loads in flight together (rows and columns clamped, values masked)
        double v[PER];
#pragma unroll
        for (int u = 0; u < PER; u++) {
            const int j = j0 + 4 * u;
            v[u] = Ab[min(ri, w - 1) + (long long)min(j, w - 1) * ld];
        }
#pragma unroll
        for (int u = 0; u < PER; u++) {
            const int j = j0 + 4 * u;
            L[ri][j] = (ri < w && j < w) ? (ri >= j ? v[u] : 0.0) : (ri == j ? 1.0 : 0.0);
            X[ri][j] = 0.0;
        }
    }
    __syncthreads();
    // C(ib, jb) += (NEG: -=) sum_k A(ib, k) B(k, jb) over 16 nk columns, one wavefront
    typedef mfma4<double>::v Acc;
    auto product = [&](Acc acc, auto a, auto bm, int nk, double sign) {
        #pragma unroll 4
        for (int k = 0; k < CHOL_SB * nk; k += 4) {
            const int kk = k + (lane >> 4);
            acc = mfma16x16x4(sign * a(lane & 15, kk), bm(kk, lane & 15), acc);
        }
        return acc;
    };
#pragma unroll 1
    for (int c0 = 0; c0 < CHOL_NB; c0 += CHOL_SB) {
        if (wave == 0) {
            double a[CHOL_SB];
#pragma unroll
            for (int j = 0; j < CHOL_SB; j++) a[j] = L[lane][c0 + j];
            bool bad = false;
#pragma unroll
            for (int j = 0; j < CHOL_SB; j++) {
                const double d = lane_value(a[j], c0 + j);
                const bool nb = !(d > 0.0);
                bad = bad || nb;
                double s, inv;
                sqrt_recip(nb ? 1.0 : d, s, inv);
                if (lane == 0) dinv[c0 + j] = inv;
                a[j] = lane == c0 + j ? s : a[j] * inv;
#pragma unroll
                for (int l = j + 1; l < CHOL_SB; l++) a[l] = fma(-a[j], lane_value(a[j], c0 + l), a[l]);
                __builtin_amdgcn_sched_barrier(0);  // the lane reads of one column at a time
            }
            // rows above the diagonal hold no factor
#pragma unroll
            for (int j = 0; j < CHOL_SB; j++) L[lane][c0 + j] = lane >= c0 + j ? a[j] : 0.0;
            if (bad && lane == 0) atomicOr(status, MBD_ST_COLLAPSE);
        }
        __syncthreads();
        const int done = c0 / CHOL_SB + 1, left = CHOL_NB / CHOL_SB - done;
        for (int t = wave; t < left * (left + 1) / 2; t += 4) {
            int ib = 0;
            while ((ib + 1) * (ib + 2) / 2 <= t) ib++;
            const int r0 = (done + ib) * CHOL_SB, q0 = (done + t - ib * (ib + 1) / 2) * CHOL_SB;
            Acc acc;
#pragma unroll
            for (int r = 0; r < 4; r++) acc[r] = L[r0 + mfma_rows<double>::row(lane, r)][q0 + (lane & 15)];
            acc = product(acc, [&](int m, int k) { return L[r0 + m][c0 + k]; },
                          [&](int k, int c) { return L[q0 + c][c0 + k]; }, 1, -1.0);
#pragma unroll
            for (int r = 0; r < 4; r++) L[r0 + mfma_rows<double>::row(lane, r)][q0 + (lane & 15)] = acc[r];
        }
        __syncthreads();
    }
    {
        // X(wave, wave): lane c holds column c, row after row
        const int o = wave * CHOL_SB, c = lane & 15;
        double x[CHOL_SB];
#pragma unroll
        for (int r = 0; r < CHOL_SB; r++) x[r] = r == c ? 1.0 : 0.0;
#pragma unroll
        for (int l = 0; l < CHOL_SB; l++) {
            x[l] *= dinv[o + l];
#pragma unroll
            for (int r = l + 1; r < CHOL_SB; r++) x[r] = fma(-L[o + r][o + l], x[l], x[r]);
        }
        if (lane < CHOL_SB) {
#pragma unroll
            for (int r = 0; r < CHOL_SB; r++) X[o + r][o + c] = x[r];
        }
    }
    __syncthreads();
    // X(i, j) = -X(i, i) sum_{j <= k < i} L(i, k) X(k, j), i - j = dist
    for (int dist = 1; dist < CHOL_NB / CHOL_SB; dist++) {
        if (dist + wave < CHOL_NB / CHOL_SB) {
            const int r0 = (dist + wave) * CHOL_SB, q0 = wave * CHOL_SB;
            Acc acc = {0, 0, 0, 0};
            acc = product(acc, [&](int m, int k) { return L[r0 + m][q0 + k]; },
                          [&](int k, int c) { return X[q0 + k][q0 + c]; }, dist, 1.0);
            // through the block's own place to the operand layout (one wavefront: in order)
#pragma unroll
            for (int r = 0; r < 4; r++) X[r0 + mfma_rows<double>::row(lane, r)][q0 + (lane & 15)] = acc[r];
            __builtin_amdgcn_wave_barrier();
            Acc acc2 = {0, 0, 0, 0};
            acc2 = product(acc2, [&](int m, int k) { return X[r0 + m][r0 + k]; },
                           [&](int k, int c) { return X[r0 + k][q0 + c]; }, 1, -1.0);
            __builtin_amdgcn_wave_barrier();
#pragma unroll
            for (int r = 0; r < 4; r++) X[r0 + mfma_rows<double>::row(lane, r)][q0 + (lane & 15)] = acc2[r];
        }
        __syncthreads();
    }
#pragma unroll
    for (int u = 0; u < PER; u++) {
        const int j = j0 + 4 * u;
        if (ri < w && j < w && ri >= j) Ab[ri + j * ld] = L[ri][j];
    }
    double* Xo = chol_inv_block(Linv, sLi, b, k0, wb);
#pragma unroll
    for (int u = 0; u < PER; u++) {
        const int j = j0 + 4 * u;
        Xo[ri + j * wb] = X[ri][j];
    }
}

// ---------------------------------------------------------------------------
// panel: L21 = A21 X^T (X = L11^-1), rows k0 + 64 .. n-1, in place: a tile
// spans the panel's 64 columns, so a workgroup reads only the rows it writes.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void chol_panel_kernel(MatBatch<double> A, double* Linv, long long sLi, int wb,
                                                          int n, int k0) {
    typedef SplitK<2, 4, 4, 4> SK;
    __shared__ __align__(16) double cs[SK::LDS];
    const int b = blockIdx.y, m0 = k0 + CHOL_NB + blockIdx.x * SK::TM, tid = threadIdx.x;
    double* Ab = A.at(b) + m0 + (long long)k0 * A.ld;
    {
        SK sk;
        sk.clear();
        // X^T(k, c) = X(c, k)
        const int o = k0 % wb;
        sk.run(Ab - m0, m0, A.ld, chol_inv_block(Linv, sLi, b, k0, wb) - o, o, wb, CHOL_NB);
        sk.reduce(cs);
    }
#pragma unroll
    for (int x = tid; x < SK::TM * SK::TN; x += SK::NT) {
        const int r = x % SK::TM, c = x / SK::TM;
        if (m0 + r < n) Ab[r + (long long)c * A.ld] = cs[c * SK::LDC + r] + cs[(SK::TN + c) * SK::LDC + r];
    }
}

// ---------------------------------------------------------------------------
// update of the panel at k0 by the k0 columns before it
// ---------------------------------------------------------------------------
// 32 x 32 tiles with K split four ways: the last panels have few rows and the
// longest K.  Bound by the matrix cores (16 matrices of order 3000: 3.2 ms, 45
// TFLOP/s; tiles of 64 x 32 3.7 ms, of 32 x 64 3.9, half or twice the
// wavefronts 4.2 and 3.9; right-looking with K = 128 from LDS 4.8 ms).
__global__ __launch_bounds__(256, 3) void chol_update_kernel(MatBatch<double> A, int n, int k0, int tiles) {
    typedef SplitK<2, 2, 4, 6> SK;
    constexpr int TC = CHOL_NB / SK::TN;  // tile columns of the panel
    __shared__ __align__(16) double cs[SK::LDS];
    // every XCD gets a run of (matrix, tile) indices: a matrix's panel rows stay in one or two L2s
    const int v = xcd_virtual(blockIdx.x, gridDim.x), b = v / tiles, t = v % tiles, tid = threadIdx.x;
    const int m0 = k0 + t / TC * SK::TM, n0 = k0 + t % TC * SK::TN;
    if (m0 + SK::TM <= n0 || n0 >= n) return;  // above the diagonal, or past the matrix
    {
        SK sk;
        sk.clear();
        sk.run(A.at(b), m0, A.ld, A.at(b), n0, A.ld, k0);
        sk.reduce(cs);
    }
    double* C = A.at(b) + m0 + (long long)n0 * A.ld;
#pragma unroll 4
    for (int x = tid; x < SK::TM * SK::TN; x += SK::NT) {
        const int r = x % SK::TM, c = x / SK::TM;
        if (m0 + r < n && n0 + c <= m0 + r) C[r + (long long)c * A.ld] -= cs[c * SK::LDC + r] + cs[(SK::TN + c) * SK::LDC + r];
    }
}

// ---------------------------------------------------------------------------
// inverses of the wide diagonal blocks: X(i, j) = -X(i, i) sum_{j <= k < i} L(i,
// k) X(k, j) over their 64 x 64 blocks, a block column per workgroup, 16 rows
// per wavefront.  Grid (WB / 64 - 1, wide blocks, matrices).
// ---------------------------------------------------------------------------
template <int WB>
__global__ __launch_bounds__(256) void chol_wide_kernel(MatBatch<double> A, double* Linv, long long sLi, int n) {
    __shared__ double T[CHOL_NB][CHOL_NB + 1];
    typedef mfma4<double>::v Acc;
    const int j = blockIdx.x, w0 = blockIdx.y * WB, b = blockIdx.z, lane = threadIdx.x & 63;
    const int nb = (min(WB, n - w0) + CHOL_NB - 1) / CHOL_NB, m0 = 16 * (threadIdx.x >> 6);
    const int m = lane & 15, kl = lane >> 4;
    double* X = chol_inv_block(Linv, sLi, b, w0, WB);
    const double* L = A.at(b) + w0 + (long long)w0 * A.ld;
    for (int i = j + 1; i < nb; i++) {
        Acc acc[4] = {{0, 0, 0, 0}, {0, 0, 0, 0}, {0, 0, 0, 0}, {0, 0, 0, 0}};
        const int row = CHOL_NB * i + m0 + m;
        const bool in = w0 + row < n;  // rows past n hold no factor
#pragma unroll 4
        for (int k = CHOL_NB * j; k < CHOL_NB * i; k += 4) {
            const double a = in ? L[row + (long long)(k + kl) * A.ld] : 0.0;
#pragma unroll
            for (int c = 0; c < 4; c++) acc[c] = mfma16x16x4(a, X[k + kl + (CHOL_NB * j + 16 * c + m) * WB], acc[c]);
        }
        __syncthreads();  // the previous block's readers of T
#pragma unroll
        for (int c = 0; c < 4; c++)
#pragma unroll
            for (int r = 0; r < 4; r++) T[m0 + mfma_rows<double>::row(lane, r)][16 * c + m] = acc[c][r];
        __syncthreads();
        Acc x[4] = {{0, 0, 0, 0}, {0, 0, 0, 0}, {0, 0, 0, 0}, {0, 0, 0, 0}};
#pragma unroll 4
        for (int k = 0; k < CHOL_NB; k += 4) {
            const double a = -X[row + (CHOL_NB * i + k + kl) * WB];
#pragma unroll
            for (int c = 0; c < 4; c++) x[c] = mfma16x16x4(a, T[k + kl][16 * c + m], x[c]);
        }
#pragma unroll
        for (int c = 0; c < 4; c++)
#pragma unroll
            for (int r = 0; r < 4; r++)
                X[CHOL_NB * i + m0 + mfma_rows<double>::row(lane, r) + (CHOL_NB * j + 16 * c + m) * WB] = x[c][r];
        __syncthreads();  // X(i, j), global memory, before the next block row reads it
    }
}

// ---------------------------------------------------------------------------
// triangular solves; right-hand sides row-major [n][CHOL_NR] per matrix
// ---------------------------------------------------------------------------
// Forward step of the wide block at w0.  SUB: 64 rows below it per workgroup,
// R -= L Y; else its own, Y = X R.  A row per lane (columns of M are
// contiguous), a quarter of the columns per wavefront.  Bandwidth bound.
template <int WB, bool SUB>
__global__ __launch_bounds__(256) void chol_fwd_kernel(MatBatch<double> A, double* Linv, long long sLi, int n, int w0,
                                                        double* R, double* Y, long long sR) {
    __shared__ double vs[WB][CHOL_NR], part[4][CHOL_NB][CHOL_NR];
    const int b = blockIdx.y, tid = threadIdx.x, lane = tid & 63, pt = tid >> 6, rb = CHOL_NB * blockIdx.x;
    const double* V = (SUB ? Y : R) + (long long)b * sR + (long long)w0 * CHOL_NR;
    const int cols = SUB ? WB : rb + CHOL_NB;  // X is lower triangular
    for (int x = tid; x < cols * CHOL_NR; x += 256)
        vs[x / CHOL_NR][x % CHOL_NR] = w0 + x / CHOL_NR < n ? V[x] : 0.0;
    const int row = (SUB ? w0 + WB : 0) + rb + lane;
    const long long ld = SUB ? A.ld : WB;
    const double* M = SUB ? A.at(b) + min(row, n - 1) + (long long)w0 * ld : chol_inv_block(Linv, sLi, b, w0, WB) + row;
    __syncthreads();
    double s[CHOL_NR] = {0.0, 0.0, 0.0};
    const int cq = cols / 4;
#pragma unroll 16
    for (int c = pt * cq; c < (pt + 1) * cq; c++) {
        const double m = M[c * ld];
        for (int k = 0; k < CHOL_NR; k++) s[k] += m * vs[c][k];
    }
    for (int k = 0; k < CHOL_NR; k++) part[pt][lane][k] = s[k];
    __syncthreads();
    if (tid < CHOL_NB * CHOL_NR) {
        const int i = tid / CHOL_NR, k = tid % CHOL_NR, g = (SUB ? w0 + WB : w0) + rb + i;
        const double v = (part[0][i][k] + part[1][i][k]) + (part[2][i][k] + part[3][i][k]);
        if (g < n) {
            const long long o = (long long)b * sR + (long long)g * CHOL_NR + k;
            if (SUB) R[o] -= v;
            else Y[o] = v;
        }
    }
}

// Backward step of the wide block at w0.  SUB: 64 columns left of it per
// workgroup, Y -= L^T Xo; else its own, Xo = X^T Y.  16 columns per wavefront,
// the rows over its lanes.
template <int WB, bool SUB>
__global__ __launch_bounds__(256) void chol_bwd_kernel(MatBatch<double> A, double* Linv, long long sLi, int n, int w0,
                                                        double* Y, double* Xo, long long sR) {
    const int b = blockIdx.y, lane = threadIdx.x & 63, c0 = CHOL_NB * blockIdx.x + 16 * (threadIdx.x >> 6);
    const double* V = (SUB ? Xo : Y) + (long long)b * sR + (long long)w0 * CHOL_NR;
    const long long ld = SUB ? A.ld : WB;
    const double* M = SUB ? A.at(b) + w0 + (long long)c0 * ld : chol_inv_block(Linv, sLi, b, w0, WB) + (long long)c0 * ld;
    const int rows = min(WB, n - w0);
    double s[CHOL_NR][16] = {};
    for (int r0 = SUB ? 0 : CHOL_NB * blockIdx.x; r0 < rows; r0 += CHOL_NB) {
        const int r = r0 + lane;
        const bool in = r < rows;
        double v[CHOL_NR], m[16];
#pragma unroll
        for (int k = 0; k < CHOL_NR; k++) v[k] = in ? V[(long long)r * CHOL_NR + k] : 0.0;
#pragma unroll
        for (int c = 0; c < 16; c++) m[c] = in ? M[r + c * ld] : 0.0;
#pragma unroll
        for (int c = 0; c < 16; c++)
#pragma unroll
            for (int k = 0; k < CHOL_NR; k++) s[k][c] += m[c] * v[k];
    }
    const int g = (SUB ? 0 : w0) + c0 + (lane >> 2);  // lane l gets the sum of column l / 4
#pragma unroll
    for (int k = 0; k < CHOL_NR; k++) {
        const double t = wave_sum16(s[k]);
        if ((lane & 3) == 0 && g < n) {
            const long long o = (long long)b * sR + (long long)g * CHOL_NR + k;
            if (SUB) Y[o] -= t;
            else Xo[o] = t;
        }
    }
}

// ---------------------------------------------------------------------------
// host
// ---------------------------------------------------------------------------
long long chol_linv_stride(int n, int wb) { return (long long)((n + wb - 1) / wb) * wb * wb; }

void chol_factor_launch(hipStream_t st, MatBatch<double> A, int n, int nbatch, double* Linv, int wb, unsigned* status) {
    const long long sLi = chol_linv_stride(n, wb);
    for (int k0 = 0; k0 < n; k0 += CHOL_NB) {
        const int rows = n - k0 - CHOL_NB;
        if (k0) {
            const int tiles = (n - k0 + 31) / 32 * (CHOL_NB / 32);
            hipLaunchKernelGGL(chol_update_kernel, dim3(tiles * nbatch), dim3(256), 0, st, A, n, k0, tiles);
        }
        hipLaunchKernelGGL(chol_diag_kernel, dim3(nbatch), dim3(256), 0, st, A, Linv, sLi, wb, n, k0, status);
        if (rows > 0)
            hipLaunchKernelGGL(chol_panel_kernel, dim3((rows + 31) / 32, nbatch), dim3(256), 0, st, A, Linv, sLi, wb, n, k0);
    }
    if (wb == CHOL_WIDE && n > CHOL_NB)
        hipLaunchKernelGGL(chol_wide_kernel<CHOL_WIDE>, dim3(CHOL_WIDE / CHOL_NB - 1, (n + CHOL_WIDE - 1) / CHOL_WIDE, nbatch),
                           dim3(256), 0, st, A, Linv, sLi, n);
}

template <int WB>
static void chol_sweeps(hipStream_t st, MatBatch<double> A, int n, int nbatch, double* Linv, double* R, double* Y, double* X,
                        long long sR) {
    const long long sLi = chol_linv_stride(n, WB);
    auto blocks = [](int k) { return (k + CHOL_NB - 1) / CHOL_NB; };
    for (int w0 = 0; w0 < n; w0 += WB) {
        hipLaunchKernelGGL((chol_fwd_kernel<WB, false>), dim3(blocks(std::min(WB, n - w0)), nbatch), dim3(256), 0, st, A, Linv,
                           sLi, n, w0, R, Y, sR);
        if (w0 + WB < n)
            hipLaunchKernelGGL((chol_fwd_kernel<WB, true>), dim3(blocks(n - w0 - WB), nbatch), dim3(256), 0, st, A, Linv, sLi, n,
                               w0, R, Y, sR);
    }
    for (int w0 = (n - 1) / WB * WB; w0 >= 0; w0 -= WB) {
        hipLaunchKernelGGL((chol_bwd_kernel<WB, false>), dim3(blocks(std::min(WB, n - w0)), nbatch), dim3(256), 0, st, A, Linv,
                           sLi, n, w0, Y, X, sR);
        if (w0 > 0)
            hipLaunchKernelGGL((chol_bwd_kernel<WB, true>), dim3(w0 / CHOL_NB, nbatch), dim3(256), 0, st, A, Linv, sLi, n, w0, Y,
                               X, sR);
    }
}

// X = A^-1 B from the factor: B in R (overwritten), Y scratch, X out; all
// [nbatch][n][CHOL_NR] with per-matrix stride sR
void chol_solve_launch(hipStream_t st, MatBatch<double> A, int n, int nbatch, double* Linv, int wb, double* R, double* Y,
                       double* X, long long sR) {
    if (wb == CHOL_WIDE) chol_sweeps<CHOL_WIDE>(st, A, n, nbatch, Linv, R, Y, X, sR);
    else chol_sweeps<CHOL_NB>(st, A, n, nbatch, Linv, R, Y, X, sR);
}
