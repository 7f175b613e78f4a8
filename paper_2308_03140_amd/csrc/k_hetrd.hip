// Householder tridiagonalisation of many small Hermitian matrices K = C T C
// (order n = 3N <= 64 G, G <= 3), one workgroup each, the whole lower triangle
// in registers and LDS: the frequency route's periodic matrices at every
// frequency and q point, T the lattice sums of one q point (left block column
// [Re; Im] of the embedding) and C the frequency's diagonal, applied as the
// matrix is loaded.
//
// Eight wavefronts: wavefront w holds columns j = w + 8 t, its lanes rows i =
// lane + 64 g from the diagonal block (held whole) on: 48 complex elements a
// lane at G = 3, 40 of them in registers.  Per column k (LAPACK's zhetd2,
// lower): y = A v from the elements' rows (summed in the lane, then over the
// wavefronts through LDS) and, below the diagonal block, their columns (a
// butterfly over the lanes, four columns at once); w = tau y - |tau|^2 (v^H A
// v) v / 2; A -= v w^H + w v^H.  v_j and w_j of a column are wave-uniform,
// read from the lane that holds that row.  The wavefront of column k + 1
// updates it first and forms its reflector while the others update the rest.
// Three barriers a column; the code for each group of 64 columns leaves out
// the finished blocks.
//
// Bound by the FP64 vector units and the latency between the barriers: 8 300
// cycles a column on average at n = 192, where the products and updates alone
// are 2 100.  The real embedding of twice the order, reduced from memory by
// the general kernels, takes twice the operations, four times the elements
// and twice the columns: 960 matrices of n = 192 take 24.3 ms there and 2.75
// here (6.3 with rows on the wavefronts and the diagonal block's upper part
// kept at zero, which needs a butterfly for every row, 192 LDS stores to read
// a column, and branches per element).
#include "mbd_internal.h"
#include "mbd_kernels.h"
#include "mbd_sys.h"

namespace {

struct Cx {
    double re, im;
};
__device__ __forceinline__ Cx lane_cx(Cx v, int l) { return Cx{lane_value(v.re, l), lane_value(v.im, l)}; }
// a += x y, a += conj(x) y, a -= x conj(y): four fused operations each
__device__ __forceinline__ void cfma(Cx& a, Cx x, Cx y) {
    a.re = fma(x.re, y.re, a.re);
    a.im = fma(x.re, y.im, a.im);
    a.re = fma(-x.im, y.im, a.re);
    a.im = fma(x.im, y.re, a.im);
}
__device__ __forceinline__ void cfma_conj(Cx& a, Cx x, Cx y) {
    a.re = fma(x.re, y.re, a.re);
    a.im = fma(x.re, y.im, a.im);
    a.re = fma(x.im, y.im, a.re);
    a.im = fma(-x.im, y.re, a.im);
}
__device__ __forceinline__ void cfms_conj(Cx& a, Cx x, Cx y) {
    a.re = fma(-x.re, y.re, a.re);
    a.im = fma(x.re, y.im, a.im);
    a.re = fma(-x.im, y.im, a.re);
    a.im = fma(-x.im, y.re, a.im);
}

// Element (t, g) held in LDS instead of registers: the first columns' last rows, finished before the others.
template <int G>
__device__ constexpr bool hetrd_in_lds(int t, int g) {
    return G == 3 && t < 8 && g == 2;
}

// The shared buffers of one workgroup, order up to 64 G.
template <int G>
struct HetrdLds {
    Cx vb[2][64 * G], tau[2];
    Cx yrow[64 * G], ycol[8][64 * G], yv[64 * G];
    Cx far[G == 3 ? 8 : 1][512];  // (t < 8, g = 2) at G = 3: one slot per lane
};

// Reflector of column k, whose rows 64 g + lane a wavefront has in c: v =
// (x / (alpha - beta) with v(k+1) = 1) and tau to LDS, beta to e(k).
template <int G, int KG>
__device__ __forceinline__ void hetrd_reflector(const Cx (&c)[G], HetrdLds<G>& S, int k, int lane, double* d, double* e) {
    double xn2 = 0.0;
    Cx v[G];
#pragma unroll
    for (int g = KG; g < G; g++) {
        const int i = lane + 64 * g;
        v[g] = i > k + 1 ? c[g] : Cx{0.0, 0.0};  // rows of n and beyond are zero
        xn2 += v[g].re * v[g].re + v[g].im * v[g].im;
    }
    xn2 = wave_sum(xn2);
    Cx alpha = lane_cx(c[KG], (k + 1) & 63);
    if (KG + 1 < G && ((k + 1) & 63) == 0) alpha = lane_cx(c[KG + 1 < G ? KG + 1 : KG], 0);
    const double nrm2 = xn2 + alpha.re * alpha.re + alpha.im * alpha.im;
    // a column below the normal range, or already reduced (and real), needs no reflector: tau = 0 and no branch
    const bool none = nrm2 < num_limits<double>::tiny || (xn2 == 0.0 && alpha.im == 0.0);
    const double nrm = sqrt(nrm2), beta = none ? alpha.re : alpha.re >= 0.0 ? -nrm : nrm;
    const double bi = none ? 0.0 : 1.0 / beta;
    const double dr = alpha.re - beta, den = none ? 0.0 : 1.0 / (dr * dr + alpha.im * alpha.im);
    const Cx sc = {dr * den, -alpha.im * den};
#pragma unroll
    for (int g = KG; g < G; g++) {
        const int i = lane + 64 * g;
        const Cx p = v[g];
        S.vb[k & 1][i] = i == k + 1 ? Cx{1.0, 0.0} : Cx{p.re * sc.re - p.im * sc.im, p.re * sc.im + p.im * sc.re};
        if (i == k) d[k] = c[g].re;
    }
    if (lane == 0) {
        S.tau[k & 1] = Cx{(beta - alpha.re) * bi, -alpha.im * bi};
        e[k] = beta;
    }
}

// Columns 64 KG .. 64 KG + 63.
template <int G, int KG>
__device__ __forceinline__ void hetrd_columns(Cx (&A)[8 * G][G], HetrdLds<G>& S, int n, int tid, int lane, int wv,
                                              double* d, double* e) {
    constexpr int R = 8 * G, NP = 64 * G;
    auto get = [&](int t, int g) { return hetrd_in_lds<G>(t, g) ? S.far[t < 8 ? t : 0][tid] : A[t][g]; };
    auto set = [&](int t, int g, Cx v) {
        if (hetrd_in_lds<G>(t, g)) S.far[t < 8 ? t : 0][tid] = v;
        else A[t][g] = v;
    };
    Cx v[G], w[G];
    // A -= v w^H + w v^H on column t
    auto update = [&](int t) {
        const int j = (wv + 8 * t) & 63;
        const Cx vj = lane_cx(v[t / 8], j), wj = lane_cx(w[t / 8], j);
#pragma unroll
        for (int g = t / 8; g < G; g++) {
            Cx a = get(t, g);
            cfms_conj(a, v[g], wj);
            cfms_conj(a, w[g], vj);
            set(t, g, a);
        }
        if (t & 1) __builtin_amdgcn_sched_barrier(0);  // two columns' operands at a time: the triangle fills the registers
    };
    if (wv == 0 && 64 * KG < n - 1) {
        Cx c[G];
#pragma unroll
        for (int g = KG; g < G; g++) c[g] = get(8 * KG, g);
        hetrd_reflector<G, KG>(c, S, 64 * KG, lane, d, e);
    }
    const int kend = n - 1 < 64 * (KG + 1) ? n - 1 : 64 * (KG + 1);
    for (int k = 64 * KG; k < kend; k++) {
        __syncthreads();
#pragma unroll
        for (int g = KG; g < G; g++) v[g] = S.vb[k & 1][lane + 64 * g];
        // y = A v: every element's row sum y_i += a_ij v_j, and below the diagonal block the column sum
        // y_j += conj(a_ij) v_i
        Cx yl[G];
#pragma unroll
        for (int g = KG; g < G; g++) yl[g] = Cx{0.0, 0.0};
#pragma unroll
        for (int t4 = 8 * KG; t4 < R; t4 += 4) {
            // columns already reduced (KG's own); the branch around every block also keeps the blocks' registers apart
            if (wv + 8 * (t4 + 3) <= k) continue;
            double rs[8];
#pragma unroll
            for (int u = 0; u < 4; u++) {
                const int t = t4 + u;
                const Cx vj = lane_cx(v[t / 8], (wv + 8 * t) & 63);
                Cx yr = {0.0, 0.0};
#pragma unroll
                for (int g = t / 8; g < G; g++) {
                    const Cx a = get(t, g);
                    cfma(yl[g], a, vj);
                    if (g > t / 8) cfma_conj(yr, a, v[g]);
                }
                rs[2 * u] = yr.re;
                rs[2 * u + 1] = yr.im;
                if (u & 1) __builtin_amdgcn_sched_barrier(0);
            }
            if (t4 / 8 < G - 1) {
                const double s = wave_sum8(rs);
                // lane 8 q holds rs[q]: column t4 + q / 2
                if ((lane & 7) == 0)
                    reinterpret_cast<double*>(&S.yrow[wv + 8 * (t4 + (lane >> 4))])[(lane >> 3) & 1] = s;
            }
        }
#pragma unroll
        for (int g = KG; g < G; g++) S.ycol[wv][lane + 64 * g] = yl[g];
        __syncthreads();
        for (int q = 128 * KG + tid; q < 2 * NP; q += 512) {
            double s = q < 128 * (G - 1) ? reinterpret_cast<const double*>(S.yrow)[q] : 0.0;
#pragma unroll
            for (int u = 0; u < 8; u++) s += reinterpret_cast<const double*>(S.ycol[u])[q];
            reinterpret_cast<double*>(S.yv)[q] = q > 2 * k + 1 ? s : 0.0;
        }
        __syncthreads();
        // w = tau y - |tau|^2 (v^H y) v / 2, v^H y = v^H A v real
        const Cx tau = S.tau[k & 1];
        double vy = 0.0;
#pragma unroll
        for (int g = KG; g < G; g++) {
            w[g] = S.yv[lane + 64 * g];
            vy += v[g].re * w[g].re + v[g].im * w[g].im;
        }
        vy = wave_sum(vy);
        const double h = 0.5 * (tau.re * tau.re + tau.im * tau.im) * vy;
#pragma unroll
        for (int g = KG; g < G; g++) {
            const Cx y = w[g];
            w[g].re = tau.re * y.re - tau.im * y.im - h * v[g].re;
            w[g].im = tau.re * y.im + tau.im * y.re - h * v[g].im;
        }
        // column k + 1 first, and its reflector, while the other wavefronts update the rest
        if (k + 1 < 64 * (KG + 1) && wv == ((k + 1) & 7)) {
            __builtin_amdgcn_s_setprio(3);
            Cx c[G];
#pragma unroll
            for (int t = 8 * KG; t < 8 * KG + 8; t++)
                if (wv + 8 * t == k + 1) {
                    update(t);
#pragma unroll
                    for (int g = KG; g < G; g++) c[g] = get(t, g);
                }
            if (k + 1 < n - 1) hetrd_reflector<G, KG>(c, S, k + 1, lane, d, e);
            __builtin_amdgcn_s_setprio(0);
        }
#pragma unroll
        for (int t = 8 * KG; t < R; t++)
            if (t / 8 > KG || wv + 8 * t > k + 1) update(t);
    }
}

}  // namespace

template <int G>
__global__ __launch_bounds__(512, 2) void hetrd_kernel(MatBatch<double> T, const double* cc_f, int N, int nq, double* dout,
                                                         double* eout, long long sD) {
    __shared__ __align__(16) HetrdLds<G> S;
    const int b = blockIdx.x, n = 3 * N, tid = threadIdx.x, lane = tid & 63;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const double* cf = cc_f + (long long)(b / nq) * N;
    const double* Tb = T.at(b % nq);
    const long long ld = T.ld;
    double* d = dout + (long long)b * sD;
    double* e = eout + (long long)b * sD;
    Cx A[8 * G][G];
#pragma unroll
    for (int t = 0; t < 8 * G; t++) {
        const int j = wv + 8 * t;
#pragma unroll
        for (int g = t / 8; g < G; g++) {
            const int i = lane + 64 * g;
            Cx a = {0.0, 0.0};
            if (i < n && j < n) {
                const double s = cf[i / 3] * cf[j / 3];
                a.re = s * Tb[i + j * ld];
                a.im = j == i ? 0.0 : s * Tb[i + n + j * ld];
            }
            if (hetrd_in_lds<G>(t, g)) S.far[t < 8 ? t : 0][tid] = a;
            else A[t][g] = a;
            __builtin_amdgcn_sched_barrier(0);
        }
    }
    hetrd_columns<G, 0>(A, S, n, tid, lane, wv, d, e);
    if constexpr (G > 1) hetrd_columns<G, 1>(A, S, n, tid, lane, wv, d, e);
    if constexpr (G > 2) hetrd_columns<G, 2>(A, S, n, tid, lane, wv, d, e);
#pragma unroll
    for (int t = 0; t < 8 * G; t++)
        if (wv + 8 * t == n - 1 && lane + 64 * (t / 8) == n - 1) d[n - 1] = hetrd_in_lds<G>(t, t / 8) ? 0.0 : A[t][t / 8].re;
}

bool hetrd_fits(int n) { return n <= 192; }

// d, e of the tridiagonals of C_f T(q) C_f, matrix f nq + q, stride sD
void hetrd_launch(hipStream_t st, MatBatch<double> T, const double* cc_f, int N, int nfreq, int nq, double* d, double* e,
                  long long sD) {
    const int n = 3 * N;
    auto go = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3(nfreq * nq), dim3(512), 0, st, T, cc_f, N, nq, d, e, sD);
    };
    if (n <= 64) go(hetrd_kernel<1>);
    else if (n <= 128) go(hetrd_kernel<2>);
    else go(hetrd_kernel<3>);
}
