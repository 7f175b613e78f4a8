// Eigenvalues of a symmetric tridiagonal matrix without eigenvectors, for
// calls that need no vectors (energies and eigenvalues without gradients, the
// frequency route's eigenvalues, mbd_eigh without Z): Sturm-sequence counts
// with multisection.  T = tridiag(e, d, e), d[0..n-1] the diagonal and e[i]
// the element between rows i and i+1.
//
// A group of L lanes (L a power of two, 1..64) works on one eigenvalue index
// k (k-th smallest).  The group keeps an interval [lo, hi] with count(lo) <=
// k < count(hi), count(x) = number of eigenvalues below x; each step
// evaluates the count at L interior points, lane j of the group at lo +
// (hi - lo)(j + 1)/(L + 1), and keeps the sub-interval where the count passes
// k (a ballot finds it), so the interval shrinks (L + 1)-fold per step.  L = 1
// is plain bisection (least work per eigenvalue); larger L trades work for
// fewer sequential steps and is chosen when there are too few eigenvalues to
// fill the device.
//
// The count is the number of sign changes in the leading principal minors of
// T - x I,
//   p_i = (d_i - x) p_{i-1} - e_{i-1}^2 p_{i-2},
// three FP64 operations a row of which one waits for the row before, and one
// integer operation that shifts the sign into a mask (a population count every
// 32 rows); the pivots q_i = p_i / p_{i-1} of the LDL^T factorisation take a
// division a row.  stebz_prep_kernel scales the matrix by a power of two to a
// Gershgorin norm in [1, 2), so that a block of 8 rows grows the minors less
// than 5^8-fold and each block rescales them to order one.  e^2 is kept at
// 2^-200 or more (an absolute change of 2^-100 ||T||): no two successive minors
// vanish, and one zero among them counts the same with either sign.  The error
// is that of the pivots: both are exact for a tridiagonal matrix within a few
// eps of T's elements.  All arithmetic is FP64.
#include "mbd_internal.h"
#include "mbd_kernels.h"

#define STEBZ_BLOCK 8
#define STEBZ_E2MIN 6.223015277861142e-61  // 2^-200

// Per matrix: (d_i, e_{i-1}^2) scaled by 2^-sx into pe[i], filled up to a
// multiple of STEBZ_BLOCK rows with ones that change no sign; {lo, hi} (scaled
// Gershgorin bounds) and sx into info.
template <typename T>
__global__ __launch_bounds__(256) void stebz_prep_kernel(const int* ns, const T* d, const T* e, long long sD, double2* pe,
                                                           long long sP, double* info) {
    __shared__ double red[4];
    const int b = blockIdx.x, n = ns[b];
    const T* db = d + (long long)b * sD;
    const T* eb = e + (long long)b * sD;
    double gl = 1e300, gu = -1e300;
    for (int i = threadIdx.x; i < n; i += 256) {
        const double r = (i > 0 ? fabs((double)eb[i - 1]) : 0.0) + (i < n - 1 ? fabs((double)eb[i]) : 0.0);
        gl = fmin(gl, (double)db[i] - r);
        gu = fmax(gu, (double)db[i] + r);
    }
    gl = -block_max256(-gl, red);
    gu = block_max256(gu, red);
    const double tnorm = fmax(fabs(gl), fabs(gu));
    const int sx = tnorm > 0.0 ? ilogb(tnorm) : 0;
    double2* p = pe + (long long)b * sP;
    const int np = (n + STEBZ_BLOCK - 1) / STEBZ_BLOCK * STEBZ_BLOCK;
    for (int i = threadIdx.x; i < np; i += 256) {
        if (i < n) {
            const double es = i > 0 ? scalbn((double)eb[i - 1], -sx) : 0.0;
            p[i] = make_double2(scalbn((double)db[i], -sx), i > 0 ? fmax(es * es, STEBZ_E2MIN) : 0.0);
        } else {
            p[i] = make_double2(8.0, 0.0);  // (8 - x) > 0 times the last minor
        }
    }
    if (threadIdx.x == 0) {
        const double pad = 2.0 * num_limits<double>::eps * scalbn(tnorm, -sx) * n;
        info[3 * b] = scalbn(gl, -sx) - pad;
        info[3 * b + 1] = scalbn(gu, -sx) + pad;
        info[3 * b + 2] = (double)sx;
    }
}

// Eigenvalues below x of the scaled matrix; n and p are uniform (scalar loads).
__device__ __forceinline__ int sturm_count(const double2* __restrict__ p, int n, double x) {
    double p0 = 0.0, p1 = 1.0;
    unsigned mask = 0;  // sign bits, the newest lowest
    int c = 0;
    double2 t[STEBZ_BLOCK];
#pragma unroll
    for (int u = 0; u < STEBZ_BLOCK; u++) t[u] = p[u];
    for (int i = 0, r = 0; i < n; i += STEBZ_BLOCK) {
        // the next block's rows load while this one's are used
        const double2* nx = p + (i + STEBZ_BLOCK < n ? i + STEBZ_BLOCK : 0);
        double2 tn[STEBZ_BLOCK];
#pragma unroll
        for (int u = 0; u < STEBZ_BLOCK; u++) tn[u] = nx[u];
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int u = 0; u < STEBZ_BLOCK; u++) {
            const double p2 = fma(t[u].x - x, p1, -t[u].y * p0);
            p0 = p1;
            p1 = p2;
            mask = mask << 1 | (unsigned)__double2hiint(p2) >> 31;
        }
        const int s = -__builtin_amdgcn_frexp_exp(fmax(fabs(p0), fabs(p1)));
        p0 = scalbn(p0, s);
        p1 = scalbn(p1, s);
        r += STEBZ_BLOCK;
        if (r == 24) {
            c += __popc((mask ^ mask >> 1) & 0xffffff);
            r = 0;
        } else if (i + STEBZ_BLOCK >= n) {
            c += __popc((mask ^ mask >> 1) & ((1u << r) - 1));
        }
#pragma unroll
        for (int u = 0; u < STEBZ_BLOCK; u++) t[u] = tn[u];
    }
    return c;
}

// pairs != 0: T is the tridiagonal of the real embedding [[A, -B], [B, A]]
// of a Hermitian A + iB, whose eigenvalues all come in equal pairs
// (lambda_{2m} = lambda_{2m+1}): only the odd indices are found and each is
// written to both of its pair's slots (an odd order takes every index).
template <typename T>
__global__ __launch_bounds__(256) void stebz_kernel(const int* ns, const double2* __restrict__ pe, long long sP,
                                                      const double* __restrict__ info, T* __restrict__ w, long long sW,
                                                      int L, int pairs) {
    const int b = blockIdx.z;
    const int n = ns[b];
    const bool pr = pairs && !(n & 1);
    const int nk = pr ? n / 2 : n;   // eigenvalue indices to find
    const int lane = threadIdx.x & 63;
    const int per_wave = 64 / L;
    const int wave = blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (wave * per_wave >= nk) return;  // the whole wavefront
    const int g = lane / L, j = lane % L;
    const int kq = wave * per_wave + g;
    const bool active = kq < nk;
    const int k = pr ? 2 * kq + 1 : kq;
    const double2* p = pe + (long long)b * sP;
    T* wb = w + (long long)b * sW;
    const int sx = (int)info[3 * b + 2];
    if (n == 1) {
        if (lane == 0) wb[0] = (T)scalbn(p[0].x, sx);
        return;
    }
    double lo = info[3 * b], hi = info[3 * b + 1];
    const double eps = num_limits<double>::eps;
    const double sect = (double)(L + 1);
    const unsigned long long gmask = L == 64 ? ~0ull : ((1ull << L) - 1ull);
    // stop at a relative width of 2 eps, or an absolute one of eps ||T|| (the
    // accuracy the count itself supports) for eigenvalues near zero
    const double atol = eps * fmax(fabs(lo), fabs(hi));
    for (int it = 0; it < 200; it++) {
        const double width = hi - lo;
        const bool done = !active || width <= 2.0 * eps * fmax(fabs(lo), fabs(hi)) + atol;
        if (__ballot(!done) == 0ull) break;
        const double x = lo + width * (double)(j + 1) / sect;
        const int c = sturm_count(p, n, x);
        const unsigned long long m = (__ballot(c > k) >> (g * L)) & gmask;
        const int f = m ? __ffsll((long long)m) - 1 : L;  // first lane of the group whose count passes k
        if (!done) {
            const double nlo = f == 0 ? lo : lo + width * (double)f / sect;
            const double nhi = f == L ? hi : lo + width * (double)(f + 1) / sect;
            lo = nlo;
            hi = nhi;
        }
    }
    if (active && j == 0) {
        wb[k] = (T)scalbn(0.5 * (lo + hi), sx);
        if (pr) wb[k - 1] = wb[k];
    }
}

// lanes per eigenvalue: as many as keep the launch within half the lanes the
// device holds at once (256 CUs x 4 SIMDs x 4 of 8 waves x 64 lanes), 1 to 64:
// four wavefronts on a SIMD hide each other's dependent operations, and more
// lanes add counts.  960 matrices of order 192 (184 320 eigenvalues, 2.8 waves
// per SIMD at one lane): 0.43 ms with one lane, 0.62 with two; the pivots'
// divisions took 2.3 ms with two.
static int stebz_lanes(long long eigenvalues) {
    const long long cap = 256LL * 4 * 4 * 64;
    int L = 64;
    while (L > 1 && eigenvalues * L > cap) L >>= 1;
    return L;
}

long long stebz_rows(int nmax) { return (nmax + STEBZ_BLOCK - 1) / STEBZ_BLOCK * STEBZ_BLOCK; }

template <typename T>
void stebz_launch(const int* ns, int nmax, int nbatch, const T* d, const T* e, long long sD, double2* pe, double* info,
                  T* w, long long sW, hipStream_t st, bool pairs) {
    // lanes per eigenvalue from the indices actually found; the grid still
    // covers every index of the largest order (waves past a matrix's count exit)
    const int nk = pairs ? (nmax + 1) / 2 : nmax;
    const int L = stebz_lanes((long long)nk * nbatch);
    const int per_wave = 64 / L;
    const int waves = (nmax + per_wave - 1) / per_wave;
    const long long sP = stebz_rows(nmax);
    hipLaunchKernelGGL(stebz_prep_kernel<T>, dim3(nbatch), dim3(256), 0, st, ns, d, e, sD, pe, sP, info);
    hipLaunchKernelGGL(stebz_kernel<T>, dim3((waves + 3) / 4, 1, nbatch), dim3(256), 0, st, ns, pe, sP, info, w, sW, L,
                       pairs ? 1 : 0);
}
template void stebz_launch<double>(const int*, int, int, const double*, const double*, long long, double2*, double*,
                                   double*, long long, hipStream_t, bool);
template void stebz_launch<float>(const int*, int, int, const float*, const float*, long long, double2*, double*,
                                  float*, long long, hipStream_t, bool);
