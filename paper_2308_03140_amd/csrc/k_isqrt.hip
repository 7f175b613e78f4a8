// Q^{-1/2} and Tr Q^{1/2} without eigenvectors: a coupled polynomial iteration
// of symmetric products on the FP64 matrix cores.
//
// With the spectrum of Q inside [lo, hi] and kappa = hi/lo, stage one takes
// Z = W(Q/hi)/sqrt(hi), W the polynomial of least max |1 - sqrt(x) W(x)| on
// [1/kappa, 1], and Y = Q Z.  Every later stage forms P = Z Y (spectrum in
// [(1-E)^2, (1+E)^2], E the error of the stage before), its own minimax W on
// that interval, and Z <- Z W, Y <- Y W: Z tends to Q^{-1/2}, Y to Q^{1/2}
// (the coupled Newton-Schulz iteration of Higham, "Functions of Matrices",
// ch. 6, with the composed minimax polynomials of Nakatsukasa & Freund, 2016,
// in place of the Taylor ones).  The later W are kept as W - I, and Z <- Z + Z (W -
// I): coefficients and sums round with the size of a correction.  Two stages of
// degree 4 to 9 reach half a unit of the last place for kappa up to 45, three up
// to 3700, in 8 to 17 products of which only the
// lower triangle is formed (n^3 flop each): the eigen-decomposition it
// replaces reads the matrix once per column (n^3/6 elements in all) and its
// 6000 columns are a serial chain.
//
// Polynomials are taken in the centred variable X = (P/scale - mid)/hw in
// [-1, 1] and evaluated by Paterson-Stockmeyer (degree 4: 2 products, 6: 3,
// 9: 4).  A product launch is one step of a per-matrix program, so matrices
// of different kappa share the launches of a batch:
//   out  = c0 A B + c1 E1 + c2 E2 + c3 I,   out2 = d0 A B + d1 E1 + d2 E2 + d3 I
// with A, B, E1, E2, out, out2 from eight buffers (buffer 0 is Q).
//
// The interval comes from a few Lanczos steps (hi: largest Ritz value plus
// twice its residual norm and 6%, lo: half of the smallest).  Afterwards the result
// is checked: up to order 64 the Frobenius norm of I - Z Q Z is formed, beyond
// it is estimated by the size of r = x - Z Q Z x for a random vector x.  A matrix
// that fails (an eigenvalue outside the interval, or not positive definite: then
// no real Z gives Z Q Z = I) is left to the eigensolver.  Both random vectors
// have generic real entries: a vector of signs is orthogonal to whole symmetry
// sectors (equal signs on two like atoms: to the modes antisymmetric under their
// exchange), which neither the interval nor the check would then see.
#include <algorithm>
#include <cmath>
#include <vector>

#include "gemm_splitk.h"
#include "mbd_internal.h"
#include "mbd_isqrt.h"
#include "mbd_kernels.h"

// products of a class's program
static int isq_products(const IsqClass& c) {
    int p = 0;
    for (int s = 0; s < 3 && c.deg[s]; s++) {
        const bool last = s == 2 || !c.deg[s + 1];
        p += (s ? 1 : 0) + (c.deg[s] == 4 ? 2 : c.deg[s] == 6 ? 3 : 4) + (last ? 1 : s ? 2 : 1);
    }
    return p;
}

const IsqTable& isq_table(bool wide) {
    static const IsqTable tab[2] = {isq_build_table(false), isq_build_table(true)};
    return tab[wide ? 1 : 0];
}

// ---------------------------------------------------------------------------
// Lanczos (batched, one launch per step)
// ---------------------------------------------------------------------------
// Entry k of a random vector, the same for every matrix: either sign,
// magnitudes uniform in [0.5, 1.5] scaled to a mean square of one.
__device__ __forceinline__ double isq_rand(int k, unsigned seed) {
    unsigned x = (unsigned)k * 2654435761u + seed;
    x ^= x >> 16; x *= 0x7feb352du; x ^= x >> 15; x *= 0x846ca68bu; x ^= x >> 16;
    const double m = 0.96076892283052 * (0.5 + (double)(x >> 1) * 0x1p-31);  // sqrt(12 / 13)
    return (x & 1u) ? m : -m;
}

// sums of acc[r] over the workgroup, valid in every thread (LDS: 4 x ISQ_MVR)
__device__ __forceinline__ void isq_row_sums(double (&acc)[ISQ_MVR], double (*red)[ISQ_MVR]) {
    static_assert(ISQ_MVR == 8, "one butterfly for all rows");
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const double t = wave_sum8(acc);
    __syncthreads();
    if ((lane & 7) == 0) red[wv][lane >> 3] = t;
    __syncthreads();
#pragma unroll
    for (int r = 0; r < ISQ_MVR; r++) acc[r] = (red[0][r] + red[1][r]) + (red[2][r] + red[3][r]);
}

// Element k of column `row` of a symmetric matrix (EMB: elements k and nr + k of
// the left block column, which make rows c and nr + c) times v (and u): row sums
// s (and t).
template <bool EMB>
__device__ __forceinline__ void isq_row_term(const double* row, int nr, int k, double v, double u, double& s, double& t) {
    const double re = row[k];
    s += re * v;
    if (EMB) {
        const double im = row[nr + k];
        s += im * u;
        t += re * u - im * v;
    }
}

// beta of the last step before a plan, from its partials s1 = v.w' and s2 =
// w'.w' with w' = M v - a v - beta v_prev and a the alpha of the step before
// (M_00 at first): alpha = a + s1, beta^2 = s2 - s1^2.  A beta at rounding level,
// of the matrix or of the difference s2 - s1^2, ends the recurrence.
__device__ __forceinline__ bool isq_beta(double alpha, double s1, double s2, double& beta) {
    const double b2 = s2 - s1 * s1;
    const bool more = b2 > fmax(1e-28 * alpha * alpha, 1e-13 * s1 * s1) && s2 < 1e300;
    beta = more ? sqrt(b2) : 0.0;
    return more;
}

// Step j: every workgroup forms v_j from the step before (elementwise, where
// it is needed) and w'_j for its ISQ_MVR rows; bandwidth bound (M read once:
// 288 MB at order 6000).  ISQ_MVR rows share the two loads behind an element
// of v_j; one launch per step, with no grid barrier.  Taking a, the alpha of the
// step before (M_00 at first), off w' keeps beta accurate where M is close to a
// multiple of the identity (weakly coupled identical atoms); its square is
// summed from the elements of v_j before their normalisation, by every
// workgroup for itself, since s2 - s1^2 cancels where one eigenvalue stands far
// above the others (as it may after squarings).  EMB: embeddings of
// Hermitian matrices, whose left block column [Re; Im] holds both rows c and n/2
// + c in column c: half the matrix is read.
template <bool EMB>
__global__ __launch_bounds__(256) void isq_lanczos_kernel(MatBatch<double> M, const int* ns, IsqLanczos L, int j) {
    __shared__ double red4[4], red[4][ISQ_MVR];
    const int b = blockIdx.z, n = ns[b], nr = EMB ? n / 2 : n;
    const int r0 = blockIdx.x * ISQ_MVR;
    if (r0 >= nr || n <= L.one) return;
    if (L.done && L.done[b]) return;
    const int nwg = (nr + ISQ_MVR - 1) / ISQ_MVR;
    double* vec = L.vec + (long long)b * L.sV * 4;
    double* vj = vec + (long long)(j & 1) * L.sV;
    const double* v1 = vec + (long long)((j + 1) & 1) * L.sV;
    double* wj = vec + (long long)(2 + (j & 1)) * L.sV;
    const double* w1 = vec + (long long)(2 + ((j + 1) & 1)) * L.sV;
    double* part = L.part + ((long long)b * 2 + (j & 1)) * 2 * L.nwg;
    const double* pprev = L.part + ((long long)b * 2 + ((j + 1) & 1)) * 2 * L.nwg;
    double* al = L.alpha + (long long)b * ISQ_LMAX;
    double* be = L.beta + (long long)b * ISQ_LMAX;
    const double* Mb = M.at(b);
    const long long ld = M.ld;
    const double a00 = Mb[0];
    double s1 = 0.0, beta = 0.0, inv = 1.0, a = a00, nrm = 0.0;
    if (j > 0) {
        double x = 0.0;
        for (int w = threadIdx.x; w < nwg; w += 256) x += pprev[2 * w];
        s1 = block_sum256(x, red4);
        a = (j > 1 ? al[j - 2] : a00) + s1;
    }
    // v_j times beta (times its own norm at first)
    auto v_at = [&](int k) -> double { return j == 0 ? isq_rand(k, 77u) : w1[k] - s1 * v1[k]; };
    const double* row[ISQ_MVR];
    double acc[ISQ_MVR], acc2[ISQ_MVR];
#pragma unroll
    for (int r = 0; r < ISQ_MVR; r++) {
        row[r] = Mb + (long long)min(r0 + r, nr - 1) * ld;
        acc[r] = acc2[r] = 0.0;
    }
    for (int k = threadIdx.x; k < nr; k += 256) {
        const double v = v_at(k), u = EMB ? v_at(nr + k) : 0.0;
        nrm += v * v + u * u;
#pragma unroll
        for (int r = 0; r < ISQ_MVR; r++) isq_row_term<EMB>(row[r], nr, k, v, u, acc[r], acc2[r]);
    }
    nrm = block_sum256(nrm, red4);
    if (j > 0) {
        const bool more = nrm > 1e-28 * a * a && nrm < 1e300;
        beta = more ? sqrt(nrm) : 0.0;
        inv = more ? 1.0 / beta : 0.0;
        if (blockIdx.x == 0 && threadIdx.x == 0) {
            al[j - 1] = a;
            be[j - 1] = beta;
            if (!more && L.len[b] == 0) L.len[b] = j;
        }
    } else {
        inv = 1.0 / sqrt(nrm);
        if (blockIdx.x == 0 && threadIdx.x == 0) L.len[b] = 0;
    }
    isq_row_sums(acc, red);
    if (EMB) isq_row_sums(acc2, red);
    if (threadIdx.x < ISQ_MVR) {
        double p1 = 0.0, p2 = 0.0;
        if (r0 + (int)threadIdx.x < nr) {
#pragma unroll
            for (int h = 0; h < (EMB ? 2 : 1); h++) {
                const int rr = h * nr + r0 + threadIdx.x;
                double sum = 0.0;
#pragma unroll
                for (int r = 0; r < ISQ_MVR; r++) sum = (int)threadIdx.x == r ? (h ? acc2[r] : acc[r]) : sum;
                const double v = v_at(rr) * inv;
                const double w = sum * inv - a * v - (j > 0 ? beta * v1[rr] : 0.0);
                vj[rr] = v;
                wj[rr] = w;
                p1 += v * w;
                p2 += w * w;
            }
        }
        // eight lanes: butterfly within the half row
        p1 = quad_sum(p1);
        p1 += dpp<DPP_HALF_MIRROR>(p1);
        p2 = quad_sum(p2);
        p2 += dpp<DPP_HALF_MIRROR>(p2);
        if (threadIdx.x == 0) {
            part[2 * blockIdx.x] = p1;
            part[2 * blockIdx.x + 1] = p2;
        }
    }
}

// Smallest (which < 0) or largest eigenvalue of the symmetric tridiagonal
// (al, be) of order m <= ISQ_LMAX: multisection on Sturm counts, one shift per
// lane of a wavefront.  The counts are the sign changes of the leading
// principal minors p_k = (al_k - x) p_{k-1} - be_{k-1}^2 p_{k-2}, two dependent
// operations a step where the quotient form takes a division (six times
// longer); with the spread scaled to 2 the minors stay far inside the range.
// known > 0 (largest only): a lower bound, the value of a leading block; the
// first round then spaces its shifts geometrically above it, so a value that
// has not moved is recognised at once.
__device__ double isq_tri_extreme(const double* al, const double* be, int m, int which, int rounds, double known = 0.0) {
    const int lane = threadIdx.x & 63;
    m = __builtin_amdgcn_readfirstlane(m);
    double lo = 1e300, hi = -1e300;
    for (int i = lane; i < m; i += 64) {
        const double r = (i ? fabs(be[i - 1]) : 0.0) + (i + 1 < m ? fabs(be[i]) : 0.0);
        lo = fmin(lo, al[i] - r);
        hi = fmax(hi, al[i] + r);
    }
    hi = wave_max(hi);
    lo = -wave_max(-lo);
    const double pad = 1e-15 * fmax(fabs(lo), fabs(hi)) + 1e-300;
    lo -= pad;
    hi += pad;
    // scaled coefficients, one per lane (and the second 64), read back with the
    // uniform index: no memory access in the recurrence
    const double sc = 2.0 / (hi - lo);
    double a0 = 0.0, a1 = 0.0, q0 = 0.0, q1 = 0.0;
    if (lane < m) { a0 = al[lane] * sc; q0 = lane ? be[lane - 1] * sc : 0.0; q0 *= q0; }
    if (lane + 64 < m) { a1 = al[lane + 64] * sc; q1 = be[lane + 63] * sc; q1 *= q1; }
    bool geo = which > 0 && known > 0.0 && known > lo && known < hi;
    if (geo) lo = known;
    for (int it = 0; it < rounds; it++) {
        const double step = (hi - lo) / 65.0, tiny = 2e-15 * hi;
        // geometric: from tiny above lo (lane 0) to just below hi
        auto shift = [&](int l) { return geo ? lo + tiny * exp2(log2((hi - lo) / tiny) * l / 64.0) : lo + step * (l + 1); };
        const double x = shift(lane), xs = x * sc;
        int cnt = 0;
        double p0 = 0.0, p1 = 1.0;
        auto pass = [&](double a, double q, int k) {
#pragma unroll 4
            for (int i = 0; i < k; i++) {
                const double p2 = (lane_value(a, i) - xs) * p1 - lane_value(q, i) * p0;
                cnt += (p2 < 0.0) != (p1 < 0.0);
                p0 = p1;
                p1 = p2;
            }
        };
        pass(a0, q0, min(m, 64));
        if (m > 64) pass(a1, q1, m - 64);
        // lanes whose shift lies above the wanted eigenvalue
        const unsigned long long above = __ballot(which < 0 ? cnt >= 1 : cnt >= m);
        const int first = above ? __ffsll((long long)above) - 1 : 64;
        const double nlo = first > 0 ? lane_value(x, first - 1) : lo;
        hi = first < 64 ? lane_value(x, first) : hi;
        lo = nlo;
        if (geo && first == 0) return known;
        geo = false;
        if (hi - lo <= 2e-16 * fabs(hi)) break;
    }
    return 0.5 * (lo + hi);
}

// Spectral interval and class from m Lanczos coefficients (one wavefront, the
// result in every lane).  exact: the recurrence ended, the Ritz values are
// eigenvalues (tmax has no residual); the margins stay, so that nothing rests on
// the start vector having met every eigenspace.  -1: no class (not positive definite, kappa above the table's
// range, non-finite).
__device__ int isq_class(const double* al, const double* be, int m, bool exact, const IsqTable& tab, double& hi) {
    // two rounds place them within 1/4000 of the spread, which the margins cover
    const double tmin = isq_tri_extreme(al, be, m, -1, 2), tmax = isq_tri_extreme(al, be, m, 1, 2);
    double res = 0.0;
    if (!exact) {
        // last component of the eigenvector of tmax, by the three-term recurrence
        double x0 = 0.0, x1 = 1.0, nn = 1.0;
        for (int i = 0; i + 1 < m; i++) {
            const double x2 = ((tmax - al[i]) * x1 - (i ? be[i - 1] * x0 : 0.0)) / be[i];
            x0 = x1;
            x1 = x2;
            nn += x2 * x2;
        }
        res = be[m - 1] * fabs(x1) / sqrt(nn);
    }
    hi = (tmax + 2.0 * res) * 1.06;
    const double lo = tmin * ISQ_LOW_FRACTION;
    int c = -1;
    if (lo > 0.0 && hi < 1e100) {
        for (int i = ISQ_CLASSES - 1; i >= 0; i--)
            if (hi <= lo * tab.cls[i].kappa) c = i;
    }
    return c;
}

// Steps between convergence checks of lambda_min, after `squares` squarings.
__host__ __device__ inline int isq_lcheck(int squares) { return squares < 2 ? 8 : 4; }

// Largest eigenvalue z of Z from that of the matrix left by the squarings,
// w = (low z^2)^(2^(squares - 1)).
__device__ __forceinline__ double isq_unsquare(double w, int squares, double low) {
    if (squares == 0) return w;
    for (int i = 1; i < squares; i++) w = sqrt(w);
    return sqrt(w / low);
}

// All Lanczos steps of a matrix in one workgroup, orders up to L.one: bound by
// one compute unit's reads of the matrix from L2 (order 256: 0.5 MB, 8 us a
// step, beyond which a launch per step is faster).  Small matrices take it also
// beside large ones: their recurrence ends, or nearly ends, within the steps,
// which its explicit norms notice and s2 - s1^2 does not.  Thread (p, r) sums every
// np-th column's share of row r (columns of M are contiguous, M symmetric), so
// the products need no cross-lane sums.  zmax != nullptr: M is what `squares`
// squarings left; run until its largest eigenvalue has converged (see
// isq_zmax_kernel) and record that of Z.
__global__ __launch_bounds__(1024) void isq_small_lanczos_kernel(MatBatch<double> M, const int* ns, IsqLanczos L, int steps,
                                                                   const int* cls, const IsqOp* ops, int squares,
                                                                   double* zmax) {
    __shared__ double v[2][ISQ_SMALL], red[16], sums[1024], al[ISQ_LMAX], be[ISQ_LMAX], zs;
    const int b = blockIdx.x, n = ns[b], tid = threadIdx.x;
    if (n > L.one) return;
    if (zmax && cls[b] < 0) {
        if (tid == 0) zmax[b] = -1.0;
        return;
    }
    const int npad = n <= 32 ? 32 : (n + 63) / 64 * 64, np = 1024 / npad;
    const int r = tid % npad, p = tid / npad;
    const double* Mb = M.at(b);
    const long long ld = M.ld;
    auto block_sum = [&](double x) {
        x = wave_sum(x);
        __syncthreads();
        if ((tid & 63) == 0) red[tid >> 6] = x;
        __syncthreads();
        double s = 0.0;
#pragma unroll
        for (int i = 0; i < 16; i++) s += red[i];
        return s;
    };
    const bool mine = p == 0 && r < n;
    double vr = mine ? isq_rand(r, 77u) : 0.0, vprev = 0.0, beta = 0.0, a = Mb[0], zp = 0.0;
    vr /= sqrt(block_sum(vr * vr));
    int m = 0;
    bool ended = false;
    const int every = isq_lcheck(squares);
    for (int j = 0; j < steps && !ended; j++) {
        double* vj = v[j & 1];
        if (mine) vj[r] = vr;
        __syncthreads();
        double s = 0.0;
        if (p < np && r < n) {
            const double* col = Mb + r;
            int k = p;
            for (; k + 7 * np < n; k += 8 * np) {
                double x[8];
#pragma unroll
                for (int u = 0; u < 8; u++) x[u] = col[(long long)(k + u * np) * ld];
#pragma unroll
                for (int u = 0; u < 8; u++) s += x[u] * vj[k + u * np];
            }
            for (; k < n; k += np) s += col[(long long)k * ld] * vj[k];
        }
        sums[tid] = s;
        __syncthreads();
        double w = 0.0;
        if (mine) {
            for (int q = 0; q < np; q++) w += sums[q * npad + r];
            w -= a * vr + beta * vprev;
        }
        const double s1 = block_sum(vr * w);
        a += s1;
        w -= s1 * vr;
        const double b2 = block_sum(w * w);
        const bool more = b2 > 1e-28 * a * a && b2 < 1e300;
        beta = more ? sqrt(b2) : 0.0;
        if (tid == 0) { al[j] = a; be[j] = beta; }
        vprev = vr;
        vr = more ? w / beta : 0.0;
        m = j + 1;
        ended = !more;
        if (zmax && (ended || m % every == 0 || m == steps)) {
            __syncthreads();
            if (tid < 64) {
                const double z = isq_tri_extreme(al, be, m, 1, 10, zp);
                if (tid == 0) zs = z;
            }
            __syncthreads();
            const double z = zs;
            const bool conv = ended || (m > 2 * every && fabs(z - zp) <= 4e-15 * z) ||
                              (m == steps && fabs(z - zp) <= 1e-11 * z);
            if (tid == 0) zmax[b] = conv ? isq_unsquare(z, squares, ops[(long long)b * ISQ_OPS + ISQ_OPMAX].c[0]) : -1.0;
            zp = z;
            if (conv) return;
        }
    }
    if (zmax) return;
    __syncthreads();
    for (int i = tid; i < m; i += 1024) {
        L.alpha[(long long)b * ISQ_LMAX + i] = al[i];
        L.beta[(long long)b * ISQ_LMAX + i] = be[i];
    }
    if (tid == 0) L.len[b] = ended ? m : 0;
}

// ---------------------------------------------------------------------------
// program of a matrix
// ---------------------------------------------------------------------------
struct IsqEmit {
    IsqOp* op;
    int k;
    __device__ void put(int a, int b, int e1, int e2, int out, int out2, double c0, double c1, double c2, double c3,
                        double d0 = 0, double d1 = 0, double d2 = 0, double d3 = 0) {
        IsqOp o;
        o.a = (signed char)a; o.b = (signed char)b; o.e1 = (signed char)e1; o.e2 = (signed char)e2;
        o.out = (signed char)out; o.out2 = (signed char)out2; o.full = 0;
        o.sa = o.sb = o.conv = 0;
        o.c[0] = c0; o.c[1] = c1; o.c[2] = c2; o.c[3] = c3;
        o.d[0] = d0; o.d[1] = d1; o.d[2] = d2; o.d[3] = d3;
        op[k++] = o;
    }
    // The polynomial of degree d in X into buffer w, scaled by f, for the symmetric matrix in
    // buffer p with X = s p + g I (s = 1, g = 0: the buffer holds X itself).
    // Buffers x2, x3, t, u hold the powers and inner sums.
    __device__ void poly(int p, double s, double g, int d, const double* b, double f, int x2, int x3, int t, int u,
                         int w) {
        // X^2 = s^2 p p + 2 s g p + g^2 I
        const double q0 = s * s, q1 = 2.0 * s * g, q3 = g * g;
        if (d == 4) {
            // T = b4 X^2 + b3 X + b2;  W = X^2 T + b1 X + b0
            put(p, p, p, -1, x2, t, q0, q1, 0, q3, b[4] * q0, b[4] * q1 + b[3] * s, 0, b[4] * q3 + b[3] * g + b[2]);
            put(x2, t, p, -1, w, -1, f, f * b[1] * s, 0, f * (b[1] * g + b[0]));
            return;
        }
        put(p, p, p, -1, x2, -1, q0, q1, 0, q3);
        // X^3 = s p X^2 + g X^2;  T = inner sum of the top coefficients
        const int o = d == 6 ? 3 : 6;
        put(p, x2, x2, p, x3, t, s, g, 0, 0, b[o + 3] * s, b[o + 3] * g + b[o + 2], b[o + 1] * s, b[o + 1] * g + b[o]);
        if (d == 9) {
            put(x3, t, x2, p, u, -1, 1.0, b[5], b[4] * s, b[4] * g + b[3]);
            put(x3, u, x2, p, w, -1, f, f * b[2], f * b[1] * s, f * (b[1] * g + b[0]));
        } else {
            put(x3, t, x2, p, w, -1, f, f * b[2], f * b[1] * s, f * (b[1] * g + b[0]));
        }
    }
};

// One wavefront per matrix: class and program (its last product always lands
// in buffer ISQ_RESULT).  No class: an empty program, and the check afterwards
// fails.
__global__ __launch_bounds__(64) void isq_plan_kernel(const int* ns, IsqLanczos L, int steps, IsqTable tab, IsqOp* ops,
                                                        int* cls, int* order, bool mod, int squares) {
    __shared__ double al[ISQ_LMAX], be[ISQ_LMAX];
    const int b = blockIdx.x, n = ns[b], lane = threadIdx.x;
    int ahead = 0;  // matrices before this one: larger, or as large and earlier
    for (int i = lane; i < (int)gridDim.x; i += 64) ahead += ns[i] > n || (ns[i] == n && i < b);
    ahead = (int)wave_sum((double)ahead);
    if (lane == 0) order[ahead] = b;
    IsqOp* op = ops + (long long)b * ISQ_OPS;
    for (int i = lane; i < steps; i += 64) {
        al[i] = L.alpha[(long long)b * ISQ_LMAX + i];
        be[i] = L.beta[(long long)b * ISQ_LMAX + i];
    }
    double blast;
    bool more = true;
    if (n > L.one) {
        // one launch per step: the last step's sums are still to be taken
        const int nwg = ((L.emb ? n / 2 : n) + ISQ_MVR - 1) / ISQ_MVR;
        const double* part = L.part + ((long long)b * 2 + ((steps + 1) & 1)) * 2 * L.nwg;
        double s1 = 0.0, s2 = 0.0;
        for (int w = lane; w < nwg; w += 64) { s1 += part[2 * w]; s2 += part[2 * w + 1]; }
        s1 = wave_sum(s1);
        s2 = wave_sum(s2);
        const double a = L.alpha[(long long)b * ISQ_LMAX + steps - 2] + s1;
        more = isq_beta(a, s1, s2, blast);
        __syncthreads();
        if (lane == 0) { al[steps - 1] = a; be[steps - 1] = blast; }
    }
    __syncthreads();
    int m = L.len[b];
    const bool exact = m > 0 || !more;
    if (m == 0) m = steps;
    double hi;
    const int c = isq_class(al, be, m, exact, tab, hi);
    if (lane == 0) {
        cls[b] = c;
        IsqEmit e = {op, 0};
        if (c >= 0) {
            const IsqClass& k = tab.cls[c];
            // stage one: X = (Q/hi - mid)/hw; buffers: 1 X^2, 2 X^3, 3 T, 4 U
            const int last = k.deg[2] ? 2 : 1;
            e.poly(0, 1.0 / (hi * k.hw[0]), -k.mid[0] / k.hw[0], k.deg[0], k.b[0], 1.0 / sqrt(hi), 1, 2, 3, 4, 5);
            e.put(0, 5, -1, -1, 6, -1, 1.0, 0, 0, 0);  // Y = Q Z
            int z = 5, y = 6;
            for (int s = 1; s <= last; s++) {
                // X = (Z Y - mid)/hw
                e.put(z, y, -1, -1, 7, -1, 1.0 / k.hw[s], 0, 0, -k.mid[s] / k.hw[s]);
                if (s < last) {
                    // buffers free here: 1 2 3 4 and, after X, none of z, y
                    e.poly(7, 1.0, 0.0, k.deg[s], k.b[s], 1.0, 1, 2, 3, 4, k.deg[s] == 9 ? 3 : 4);
                    const int w = k.deg[s] == 9 ? 3 : 4;
                    e.put(y, w, y, -1, 2, -1, 1.0, 1.0, 0, 0);
                    e.put(z, w, z, -1, 1, -1, 1.0, 1.0, 0, 0);
                    z = 1;
                    y = 2;
                } else if (z == 5) {
                    // y is free once X is formed
                    e.poly(7, 1.0, 0.0, k.deg[s], k.b[s], 1.0, 1, 2, 3, 4, 6);
                    e.put(z, 6, z, -1, ISQ_RESULT, -1, 1.0, 1.0, 0, 0);
                } else {
                    e.poly(7, 1.0, 0.0, k.deg[s], k.b[s], 1.0, 2, 3, 4, 5, 6);
                    e.put(z, 6, z, -1, ISQ_RESULT, -1, 1.0, 1.0, 0, 0);
                }
            }
        }
        if (e.k) op[e.k - 1].full = 1;
        // which operands the two residue slots hold
        int held[2] = {-1, -1};
        for (int i = 0; mod && i < e.k; i++) {
            IsqOp& o = op[i];
            int sa = held[0] == o.a ? 0 : held[1] == o.a ? 1 : -1;
            if (sa < 0) {
                sa = held[0] == o.b ? 1 : 0;
                held[sa] = o.a;
                o.conv |= 1;
            }
            int sb = o.b == o.a ? sa : 1 - sa;
            if (held[sb] != o.b) {
                held[sb] = o.b;
                o.conv |= 2;
            }
            o.sa = (signed char)sa;
            o.sb = (signed char)sb;
            for (int h = 0; h < 2; h++)
                if (held[h] == o.out || (o.out2 >= 0 && held[h] == o.out2)) held[h] = -1;
        }
        while (e.k < ISQ_OPMAX) e.put(-1, -1, -1, -1, -1, -1, 0, 0, 0, 0);
        // low Z^2, with eigenvalues up to about 1, and its squares
        for (int i = 0; i < squares; i++) {
            if (c < 0) e.put(-1, -1, -1, -1, -1, -1, 0, 0, 0, 0);
            else if (i == 0) e.put(ISQ_RESULT, ISQ_RESULT, -1, -1, 1, -1, hi / tab.cls[c].kappa, 0, 0, 0);
            else e.put(2 - (i & 1), 2 - (i & 1), -1, -1, 1 + (i & 1), -1, 1.0, 0, 0, 0);
            if (i == squares - 1) op[e.k - 1].full = 1;
        }
    }
    if (!mod || c < 0) return;
    __syncthreads();
    // bounds of the operands' norms for the residue products: the programs are
    // polynomials of Q, so 64 points of its interval are followed through one;
    // a quarter on top covers what lies between them
    double f[ISQ_NBUF];
    f[0] = hi * exp2(-log2(tab.cls[c].kappa) * lane / 63.0);
    for (int i = 0; i < ISQ_OPMAX; i++) {
        const IsqOp o = op[i];
        if (o.a < 0) break;
        auto at = [&](int k) {
            double v = 0.0;
#pragma unroll
            for (int j = 0; j < ISQ_NBUF; j++) v = j == k ? f[j] : v;
            return v;
        };
        const double x = at(o.a), y = at(o.b), e1 = at(o.e1), e2 = at(o.e2);
        const int ea = __builtin_amdgcn_frexp_exp(1.25 * wave_max(fabs(x))), eb = __builtin_amdgcn_frexp_exp(1.25 * wave_max(fabs(y)));
        if (lane == 0) {
            op[i].ea = ea;
            op[i].eb = eb;
        }
        const double o1 = o.c[0] * x * y + o.c[1] * e1 + o.c[2] * e2 + o.c[3];
        const double o2 = o.d[0] * x * y + o.d[1] * e1 + o.d[2] * e2 + o.d[3];
#pragma unroll
        for (int j = 0; j < ISQ_NBUF; j++) {
            if (j == o.out) f[j] = o1;
            if (j == o.out2) f[j] = o2;
        }
    }
}

// ---------------------------------------------------------------------------
// symmetric product step
// ---------------------------------------------------------------------------
// One TM x TN tile of the lower triangle per workgroup, K split over its WK
// wavefronts (gemm_splitk.h).  Bound by the FP64 matrix cores: at order 6000
// 62-64 TFLOP/s against 58 for 128 x 128 tiles staged through LDS (the
// library's DGEMM reaches 65), at order 2103 57 against 32 (the smaller tiles
// fill the last round of workgroups), 512 uneven molecules 2.2-2.6 ms a
// product against 4.0-4.5, one matrix of order 450 9 us against 13.
//
// EMB: the matrices are real embeddings [[Re, -Im], [Im, Re]] of Hermitian ones
// (order 2n), of which only the left block column is read and, before the last
// product, written.  Its lower triangles Re C = Re A Re B + Im A (Im B)^T (part
// 0) and Im C = Im A Re B - Re A (Im B)^T (part 1) take half the products of a
// real symmetric matrix of that order; bound by the traffic of the operands and
// the epilogue (64 matrices of order 384: 63 us a product against 118).
template <int MI, int NJ, int WK, int U, int MINW, bool EMB>
__global__ __launch_bounds__(64 * WK, MINW) void isq_prod_kernel(IsqBufs bufs, const int* ns, const IsqOp* ops,
                                                                   int step, const int* order, int nmat, int own) {
    typedef SplitK<MI, NJ, WK, U> SK;
    static_assert(MI % NJ == 0, "tile rows hold whole tile columns");
    constexpr int TM = SK::TM, TN = SK::TN, NT = SK::NT, LDC = SK::LDC;
    __shared__ __align__(16) double cs[SK::LDS];
    int b, part, v;
    if (own) {
        // whole matrices per XCD, own workgroups each, dealt out back and forth by size
        const int x = blockIdx.x % GEMM_NXCD, j = blockIdx.x / GEMM_NXCD, m = j / own;
        const int r = m * GEMM_NXCD + (m & 1 ? GEMM_NXCD - 1 - x : x);
        if (r >= nmat) return;
        b = order[r];
        v = j % own;
        part = EMB ? v & 1 : 0;
        v = EMB ? v >> 1 : v;
    } else {
        b = blockIdx.z;
        part = EMB ? blockIdx.y : 0;
        v = splitk_tile_index(blockIdx.x, b, gridDim.x);
    }
    const IsqOp& op = ops[(long long)b * ISQ_OPS + step];
    if (op.a < 0) return;
    const int n = EMB ? ns[b] / 2 : ns[b];
    int ti, tj;
    splitk_lower_tile(v, TM / TN, ti, tj);
    const int m0 = ti * TM, n0 = tj * TN;
    if (m0 >= n || n0 >= n) return;
    const int ld = bufs.ld, tid = threadIdx.x;
    {
        SK sk;
        sk.clear();
        const double* A = bufs.p[op.a] + (long long)b * bufs.stride;
        const double* B = bufs.p[op.b] + (long long)b * bufs.stride;
        if constexpr (!EMB) {
            sk.run(A, m0, ld, B, n0, ld, n);
        } else {
            sk.run(A, m0 + part * n, ld, B, n0, ld, n);
            if (part) sk.template run<true>(A, m0, ld, B, n0 + n, ld, n);
            else sk.run(A, m0 + n, ld, B, n0 + n, ld, n);
        }
        sk.reduce(cs);
    }
    const double* E1 = op.e1 >= 0 ? bufs.p[op.e1] + (long long)b * bufs.stride : nullptr;
    const double* E2 = op.e2 >= 0 ? bufs.p[op.e2] + (long long)b * bufs.stride : nullptr;
    double* C1 = bufs.p[op.out] + (long long)b * bufs.stride;
    double* C2 = op.out2 >= 0 ? bufs.p[op.out2] + (long long)b * bufs.stride : nullptr;
    double c[4], d[4];
#pragma unroll
    for (int q = 0; q < 4; q++) { c[q] = op.c[q]; d[q] = op.d[q]; }
    const bool diag = m0 < n0 + TN;
    const double sg = part ? -1.0 : 1.0;
    const bool right = EMB && op.full;  // the right block column too
    // lower triangle, in runs along m: (row, col) of the part and, in the right
    // block column, (n + row, n + col) for Re, (row, n + col) negated for Im
#pragma unroll 4
    for (int x = tid; x < TM * TN; x += NT) {
        const int r = x % TM, cl = x / TM, row = m0 + r, col = n0 + cl;
        if (row >= n || col >= n || (diag && col > row)) continue;
        const long long at = row + part * n + (long long)col * ld;
        const double s = cs[cl * LDC + r] + cs[(TN + cl) * LDC + r];
        const double e1 = E1 ? E1[at] : 0.0, e2 = E2 ? E2[at] : 0.0, id = row == col ? 1.0 : 0.0;
        double o1 = c[0] * s + c[1] * e1 + c[2] * e2 + c[3] * id;
        if (EMB && part && row == col) o1 = 0.0;  // the diagonal of Im
        const long long at2 = row + (1 - part) * n + (long long)(n + col) * ld;
        C1[at] = o1;
        if (right) C1[at2] = sg * o1;
        cs[cl * LDC + r] = o1;
        if (C2) {
            double o2 = d[0] * s + d[1] * e1 + d[2] * e2 + d[3] * id;
            if (EMB && part && row == col) o2 = 0.0;
            C2[at] = o2;
            cs[(TN + cl) * LDC + r] = o2;
        }
    }
    __syncthreads();
    // its mirror image, in runs along n
#pragma unroll 4
    for (int x = tid; x < TM * TN; x += NT) {
        const int cl = x % TN, r = x / TN, row = m0 + r, col = n0 + cl;
        if (row >= n || col >= n || (diag && col >= row)) continue;
        // (col, row) of Re, or of Im negated; then (n + col, n + row) or (col, n + row)
        const long long at = col + part * n + (long long)row * ld;
        const long long at2 = col + (1 - part) * n + (long long)(n + row) * ld;
        const double v1 = cs[cl * LDC + r];
        C1[at] = sg * v1;
        if (right) C1[at2] = v1;
        if (C2) C2[at] = sg * cs[(TN + cl) * LDC + r];
    }
}

// Tile shape of a launch.  Few tiles (at most four of 32 x 32 per compute
// unit): 32 x 32 with K over four wavefronts, the shortest chain per tile.
// Orders below 1024: 32 x 32 over two (512 uneven molecules: 2.3-2.6 ms a
// product against 2.7-3.1 for 64 x 32, whose ragged edges waste more).
// Otherwise the cheapest of three by flops, measured rate and the last round
// of workgroups left partly empty over 256 compute units (order 2103: 96 x 32
// makes 759 tiles, 2.96 rounds, 57 TFLOP/s; 64 x 32 1122, 4.4 rounds, 52).
struct IsqShape { int tm, tn; double rate; };
static const IsqShape ISQ_SHAPES[3] = {{64, 32, 1.0}, {96, 32, 0.97}, {32, 32, 0.84}};

static int isq_shape(const int* ns, int nmat, bool embed) {
    double best = 1e300;
    int pick = 2, nmax = 0;
    for (int b = 0; b < nmat; b++) nmax = std::max(nmax, embed ? ns[b] / 2 : ns[b]);
    for (int s = nmax < 1024 ? 2 : 0; s < 3; s++) {
        const IsqShape& q = ISQ_SHAPES[s];
        double tiles = 0.0, work = 0.0;
        for (int b = 0; b < nmat; b++) {
            const double t = (embed ? 2.0 : 1.0) * splitk_lower_tiles(embed ? ns[b] / 2 : ns[b], q.tm, q.tn);
            tiles += t;
            work += t * ns[b];
        }
        if (s == 2 && tiles <= 1024) return 3;
        const double rounds = tiles / 256.0, cost = work * q.tm * q.tn / q.rate * std::ceil(rounds) / rounds;
        if (cost < best) { best = cost; pick = s; }
    }
    return pick;
}

// Whether every matrix's tiles go to one XCD, whose L2 then holds its operands
// for all of them (spread over the XCDs each matrix is read into all eight):
// where the matrices fill the XCDs evenly, nmat rounded up to eights at most 9/8
// of it.  64 embeddings of order 384: 63 us a product against 80, 512 uneven
// molecules (dealt out by size, largest first) 1.42 ms a launch against 1.54,
// 60 small ones 10.3 us against 11.9.
static bool isq_own(int nmat) { return 8 * ((nmat + GEMM_NXCD - 1) / GEMM_NXCD * GEMM_NXCD) <= 9 * nmat; }

// ---------------------------------------------------------------------------
// trace and check
// ---------------------------------------------------------------------------
// pass 0: y1 = Z x (x random) and the row block's share of sum Q o Z, less its
// omega: the energy is half that difference, three digits smaller than either,
// and rounds with its own size;
// pass 1: y2 = Q y1; pass 2: x - Z y2 and the row block's sum of its squares.
// A matrix without a program is skipped (its result is never read).
template <bool EMB>
__global__ __launch_bounds__(256) void isq_check_kernel(MatBatch<double> Q, MatBatch<double> Z, const int* ns,
                                                          const int* cls, const SysDesc* sd, const double* om, double* yv,
                                                          long long sV, double* part, int nwg_max, int pass) {
    __shared__ double red[4][ISQ_MVR], red4[4];
    const int b = blockIdx.z, n = ns[b], nr = EMB ? n / 2 : n;
    const int r0 = blockIdx.x * ISQ_MVR;
    if (r0 >= nr || cls[b] < 0) return;
    const MatBatch<double>& M = pass == 1 ? Q : Z;
    double* y1 = yv + (long long)b * 2 * sV;
    double* y2 = y1 + sV;
    const double* x = pass == 1 ? y1 : y2;
    const double* row[ISQ_MVR];
    const double* qrow[ISQ_MVR];
    double acc[ISQ_MVR], acc2[ISQ_MVR], e = 0.0;
#pragma unroll
    for (int r = 0; r < ISQ_MVR; r++) {
        const long long off = (long long)min(r0 + r, nr - 1) * M.ld;
        row[r] = M.at(b) + off;
        qrow[r] = Q.at(b) + off;
        acc[r] = acc2[r] = 0.0;
    }
    for (int k = threadIdx.x; k < nr; k += 256) {
        const double v = pass == 0 ? isq_rand(k, 991u) : x[k];
        const double u = !EMB ? 0.0 : pass == 0 ? isq_rand(nr + k, 991u) : x[nr + k];
#pragma unroll
        for (int r = 0; r < ISQ_MVR; r++) {
            isq_row_term<EMB>(row[r], nr, k, v, u, acc[r], acc2[r]);
            if (pass == 0 && r0 + r < nr) {
                e += row[r][k] * qrow[r][k];
                if (EMB) e += row[r][nr + k] * qrow[r][nr + k];
            }
        }
    }
    isq_row_sums(acc, red);
    if (EMB) isq_row_sums(acc2, red);
    if (pass == 0) e = block_sum256(e, red4);
    if (threadIdx.x == 0) {
        double s = 0.0;
#pragma unroll
        for (int h = 0; h < (EMB ? 2 : 1); h++)
#pragma unroll
            for (int r = 0; r < ISQ_MVR; r++)
                if (r0 + r < nr) {
                    const int rr = h * nr + r0 + r;
                    const double y = h ? acc2[r] : acc[r];
                    if (pass == 0) y1[rr] = y;
                    else if (pass == 1) y2[rr] = y;
                    else {
                        const double dr = isq_rand(rr, 991u) - y;
                        s += dr * dr;
                    }
                }
        double* pb = part + ((long long)b * nwg_max + blockIdx.x) * 2;
        if (pass == 0) {
            const double* omp = om + sd[EMB ? 0 : b].atom_off;
            for (int r = r0; r < min(r0 + ISQ_MVR, nr); r++) e -= omp[r / 3];
            pb[0] = EMB ? 2.0 * e : e;
        }
        if (pass == 2) pb[1] = s;
    }
}

// Energy from the traces (E = w sum_q (Tr(Q Z) - Tr omega), omega per row) and the
// verdict of the check; lambda_min from the Lanczos run on Z when wanted.
// Systems whose evaluation failed keep their gradient outputs untouched: no
// gradient kernel sees an atom of them.
__global__ __launch_bounds__(256) void isq_energy_kernel(SysDesc* sd, const int* ns, const int* cls,
                                                           const double* part, int nwg_max, const double* mmult,
                                                           const double* zmax, double check, unsigned* status) {
    __shared__ double red[4];
    const int s = blockIdx.x;
    SysDesc& S = sd[s];
    double esum = 0.0, lmin = 1e300;
    bool ok = true;
    const int lane = threadIdx.x & 63;
    for (int q = threadIdx.x >> 6; q < S.nmat; q += 4) {  // a wavefront per matrix
        const int b = S.mat0 + q;
        if (cls[b] < 0) { ok = false; continue; }
        const int n = ns[b], nwg = ((S.embed ? n / 2 : n) + ISQ_MVR - 1) / ISQ_MVR;
        double e = 0.0, r = 0.0;
        for (int w = lane; w < nwg; w += 64) {
            e += part[((long long)b * nwg_max + w) * 2];
            r += part[((long long)b * nwg_max + w) * 2 + 1];
        }
        e = wave_sum(e);
        r = wave_sum(r);
        // |I - Z Q Z|_F^2, or its estimate; rounding leaves about 1e-14 sqrt(n) (measured, orders 30 to 6000)
        if (!(r <= check * check * n)) ok = false;
        if (zmax) {
            const double z = zmax[b];
            if (!(z > 0.0)) ok = false;
            lmin = fmin(lmin, 1.0 / (z * z));
        }
        if (lane == 0) esum += S.weight * (mmult ? mmult[b] : 1.0) * e;
    }
    ok = __syncthreads_and(ok);
    esum = block_sum256(esum, red);
    lmin = -block_max256(-lmin, red);
    if (threadIdx.x == 0) {
        if (!ok) status[s] |= MBD_ST_NO_ROOT;
        if (S.energy) *S.energy = esum;
        if (S.errors) {
            S.errors[0] = lmin;
            S.errors[1] = S.errors[2] = S.errors[3] = 0.0;
        }
        if (status[s] != 0) {
            S.grad_coords = S.grad_alpha0 = S.grad_omega = S.grad_rvdw = S.grad_lattice = nullptr;
            S.N = 0;
        }
    }
}

// Largest eigenvalue from the Lanczos coefficients so far; done[b] is set when
// the last isq_lcheck steps changed it by rounding only, or the recurrence
// ended, and zmax[b] is then that of Z.  Unconverged after the last step: < 0.
__global__ __launch_bounds__(64) void isq_zmax_kernel(const int* ns, const int* cls, IsqLanczos L, const IsqOp* ops,
                                                        int squares, int steps, int last, double* zmax) {
    __shared__ double al[ISQ_LMAX], be[ISQ_LMAX];
    const int b = blockIdx.x, lane = threadIdx.x;
    if (steps == 0) {
        const bool one = ns[b] <= L.one;
        if (lane == 0) L.done[b] = one || cls[b] < 0 ? 1 : 0;
        if (lane == 0 && !one) zmax[b] = -1.0;
        return;
    }
    if (L.done[b]) return;
    int m = L.len[b];
    const bool ended = m > 0;
    if (!ended) m = steps - 1;  // alpha[steps - 1] is recorded by the next step
    for (int i = lane; i < m; i += 64) {
        al[i] = L.alpha[(long long)b * ISQ_LMAX + i];
        be[i] = L.beta[(long long)b * ISQ_LMAX + i];
    }
    __syncthreads();
    const int every = isq_lcheck(squares);
    const double zp = fabs(zmax[b]);
    const double z = isq_tri_extreme(al, be, m, 1, 10, steps > every ? zp : 0.0);
    if (lane == 0) {
        const bool conv = ended || (steps > 2 * every && fabs(z - zp) <= 4e-15 * z);
        if (conv) L.done[b] = 1;
        zmax[b] = conv || (last && fabs(z - zp) <= 1e-11 * z)
                      ? isq_unsquare(z, squares, ops[(long long)b * ISQ_OPS + ISQ_OPMAX].c[0])
                      : -z;
    }
}

// ---------------------------------------------------------------------------
// orders up to 64: everything in one workgroup
// ---------------------------------------------------------------------------
// Lanczos on a matrix in LDS (row stride NP + 1, zero past n) by one wavefront,
// a row per lane, held in registers: no barrier, the vector read back from LDS
// as broadcasts.  vb: NP doubles.  zmax: stop when the largest eigenvalue has
// converged and return it (-1: it has not).
template <int NP>
__device__ double isq_tiny_lanczos(const double* M, double* vb, int n, int steps, double* al, double* be, int& m, bool& ended,
                                   bool zmax) {
    const int r = threadIdx.x & 63;
    const bool mine = r < n;
    double row[NP];
#pragma unroll
    for (int k = 0; k < NP; k++) row[k] = M[k * (NP + 1) + (r & (NP - 1))];
    double v = mine ? isq_rand(r, 77u) : 0.0, vp = 0.0, beta = 0.0, a = M[0], zp = 0.0;
    v *= rsqrt(wave_sum(v * v));
    const int c0 = min(n, 8);
    ended = false;
    m = 0;
    for (int j = 0; j < steps; j++) {
        if (r < NP) vb[r] = v;
        isq_wave_sync();
        double w[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int k = 0; k < NP; k++) w[k & 3] += row[k] * vb[k];
        isq_wave_sync();
        double u = mine ? (w[0] + w[1]) + (w[2] + w[3]) - a * v - beta * vp : 0.0;
        const double s1 = wave_sum(v * u);
        a += s1;
        u -= s1 * v;
        const double b2 = wave_sum(u * u);
        const bool more = __builtin_amdgcn_readfirstlane(b2 > 1e-28 * a * a && b2 < 1e300);
        const double inv = more ? rsqrt(b2) : 0.0;
        beta = b2 * inv;
        if (r == 0) { al[j] = a; be[j] = beta; }
        vp = v;
        v = u * inv;
        m = j + 1;
        ended = !more;
        if (zmax && (ended || m == steps || (m >= c0 && (m - c0) % 4 == 0))) {
            isq_wave_sync();
            const double z = isq_tri_extreme(al, be, m, 1, 10, zp);
            const bool conv = ended || fabs(z - zp) <= 4e-15 * z || (m == steps && fabs(z - zp) <= 1e-11 * z);
            if (__builtin_amdgcn_readfirstlane(conv)) return z;
            zp = z;
        }
        if (ended) break;
    }
    return -1.0;
}

// The whole direct root of a matrix of order <= NP in one launch (a program of
// 10 products, its Lanczos steps, check and trace are some 35 launches of 3 to
// 5 us each otherwise).  Four matrices in LDS (row stride NP + 1: the mirrored
// stores down a column spread over the banks); what enters a product only
// through the linear epilogue stays in registers.  2 x 2 wavefronts, each a quadrant; the
// upper one is mirrored from the lower.  Latency bound: 10 atoms 30 us
// against 240, and 47 us more of the call for lambda_min (67 without the
// squarings).
template <int NP>
__global__ __launch_bounds__(256) void isq_tiny_kernel(MatBatch<double> Q, MatBatch<double> Zo, const int* ns, IsqTable tab,
                                                         const SysDesc* sd, const double* om, int embed, int* cls,
                                                         double* part, int nwg_max, double* zmax) {
    constexpr int T = NP / 32;  // 16 x 16 tiles per wavefront and direction
    __shared__ __align__(16) double lds[4][NP * (NP + 1)];
    __shared__ double al[ISQ_LMAX], be[ISQ_LMAX], red[4], sh[2], vb[NP];
    __shared__ int scls;
    double *bX = lds[0], *bT = lds[1], *bZ = lds[2], *bY = lds[3];
    const int b = blockIdx.x, n = ns[b], tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = wave >> 1, wn = wave & 1;
    const double* Qb = Q.at(b);
    auto ix = [](int k, int m) { return k * (NP + 1) + m; };
    for (int x = tid; x < NP * NP; x += 256) {
        const int r = x % NP, c = x / NP;
        bY[ix(c, r)] = r < n && c < n ? Qb[r + (long long)c * Q.ld] : 0.0;
    }
    __syncthreads();
    if (wave == 0) {
        int m;
        bool ended;
        (void)isq_tiny_lanczos<NP>(bY, vb, n, ISQ_STEPS_SMALL, al, be, m, ended, false);
        isq_wave_sync();
        double hi;
        const int c = isq_class(al, be, m, ended, tab, hi);
        if (lane == 0) {
            scls = c;
            sh[0] = hi;
            cls[b] = c;
        }
    }
    __syncthreads();
    const int cl = scls;
    if (cl < 0) return;
    const IsqClass& k = tab.cls[cl];
    const double hi = sh[0];
    typedef typename mfma4<double>::v V4;
    struct Reg { V4 v[T][T]; };
    auto row_of = [&](int i, int r) { return wm * (NP / 2) + 16 * i + mfma_rows<double>::row(lane, r); };
    auto col_of = [&](int j) { return wn * (NP / 2) + 16 * j + (lane & 15); };
    const bool live = !(wm == 0 && wn == 1);
    const int nk = (n + 3) & ~3;  // the padding past it never meets the matrix
    auto mul = [&](const double* A, const double* B) {
        Reg o;
#pragma unroll
        for (int i = 0; i < T; i++)
#pragma unroll
            for (int j = 0; j < T; j++) o.v[i][j] = V4{0, 0, 0, 0};
        if (live) {
#pragma unroll 4
            for (int kk = 0; kk < nk; kk += 4) {
                const int kr = kk + (lane >> 4);
                double a[T], bb[T];
#pragma unroll
                for (int i = 0; i < T; i++) {
                    a[i] = A[ix(kr, wm * (NP / 2) + 16 * i + (lane & 15))];
                    bb[i] = B[ix(kr, wn * (NP / 2) + 16 * i + (lane & 15))];
                }
#pragma unroll
                for (int i = 0; i < T; i++)
#pragma unroll
                    for (int j = 0; j < T; j++) o.v[i][j] = mfma16x16x4(a[i], bb[j], o.v[i][j]);
            }
        }
        return o;
    };
    // f(row, col, element index) over the wavefront's own elements
    auto each = [&](auto f) {
#pragma unroll
        for (int i = 0; i < T; i++)
#pragma unroll
            for (int j = 0; j < T; j++)
#pragma unroll
                for (int r = 0; r < 4; r++) f(row_of(i, r), col_of(j), i, j, r);
    };
    auto put = [&](double* B, const Reg& x) {
        if (live)
            each([&](int r, int c, int i, int j, int q) {
                if (r >= c) B[ix(r, c)] = B[ix(c, r)] = x.v[i][j][q];
            });
    };
    auto lin = [&](double c0, const Reg& x0, double c1, const Reg& x1, double c2, const Reg& x2, double c3) {
        Reg o;
        each([&](int r, int c, int i, int j, int q) {
            o.v[i][j][q] = c0 * x0.v[i][j][q] + c1 * x1.v[i][j][q] + c2 * x2.v[i][j][q] + (r == c ? c3 : 0.0);
        });
        return o;
    };
    // the polynomial for X in bX and in registers; uses bX and bT, leaves it in registers
    auto poly = [&](const Reg& X, int d, const double* p) {
        const Reg X2 = mul(bX, bX);
        if (d == 4) {
            __syncthreads();
            put(bX, X2);
            put(bT, lin(p[4], X2, p[3], X, 0.0, X, p[2]));
            __syncthreads();
            return lin(1.0, mul(bX, bT), p[1], X, 0.0, X, p[0]);
        }
        put(bT, X2);
        __syncthreads();
        const Reg X3 = mul(bX, bT);
        const int o = d == 6 ? 3 : 6;
        __syncthreads();
        put(bX, X3);
        put(bT, lin(p[o + 3], X3, p[o + 2], X2, p[o + 1], X, p[o]));
        __syncthreads();
        if (d == 9) {
            const Reg U = lin(1.0, mul(bX, bT), p[5], X2, p[4], X, p[3]);
            __syncthreads();
            put(bT, U);
            __syncthreads();
        }
        return lin(1.0, mul(bX, bT), p[2], X2, p[1], X, p[0]);
    };
    // stage one on X = (Q/hi - mid)/hw; the padding takes X = 0
    {
        Reg X;
        const double s = 1.0 / (hi * k.hw[0]), g = k.mid[0] / k.hw[0];
        each([&](int r, int c, int i, int j, int q) {
            X.v[i][j][q] = r < n && c < n ? s * bY[ix(c, r)] - (r == c ? g : 0.0) : 0.0;
        });
        put(bX, X);
        __syncthreads();
        Reg W = poly(X, k.deg[0], k.b[0]);
        const double f = 1.0 / sqrt(hi);
        each([&](int r, int c, int i, int j, int q) { W.v[i][j][q] = r < n && c < n ? f * W.v[i][j][q] : (r == c ? 1.0 : 0.0); });
        for (int r = n + tid; r < NP; r += 256) bY[ix(r, r)] = 1.0;  // identity in the padding
        put(bZ, W);
        __syncthreads();
        const Reg Y = mul(bY, bZ);
        __syncthreads();
        put(bY, Y);
        __syncthreads();
    }
    for (int s = 1; s < 3 && k.deg[s]; s++) {
        const bool last = s == 2 || !k.deg[s + 1];
        Reg X = mul(bZ, bY);
        const double h = 1.0 / k.hw[s];
        each([&](int r, int c, int i, int j, int q) { X.v[i][j][q] = h * (X.v[i][j][q] - (r == c ? k.mid[s] : 0.0)); });
        put(bX, X);
        __syncthreads();
        const Reg W = poly(X, k.deg[s], k.b[s]);
        __syncthreads();
        put(bT, W);
        __syncthreads();
        Reg Z = mul(bZ, bT), Y;  // Z + Z (W - I)
        each([&](int r, int c, int i, int j, int q) { Z.v[i][j][q] += bZ[ix(r, c)]; });
        if (!last) {
            Y = mul(bY, bT);
            each([&](int r, int c, int i, int j, int q) { Y.v[i][j][q] += bY[ix(r, c)]; });
        }
        __syncthreads();
        put(bZ, Z);
        if (!last) put(bY, Y);
        __syncthreads();
    }
    // result, trace (less omega, row by row) and |I - Z Q Z|_F^2 from the product itself
    double e = 0.0, rr = 0.0;
    double* Zb = Zo.at(b);
    {
        const int r = tid % NP;
        for (int c = tid / NP; c < NP; c += 256 / NP) {
            const bool in = r < n && c < n;
            const double q = in ? Qb[r + (long long)c * Q.ld] : 0.0, z = bZ[ix(c, r)];
            if (in) Zb[r + (long long)c * Zo.ld] = z;
            e += in ? z * q : 0.0;
            bT[ix(c, r)] = q;
        }
    }
    bX[tid] = e;
    __syncthreads();
    e = 0.0;
    if (tid < n) {
        for (int k = 0; k < 256 / NP; k++) e += bX[tid + k * NP];
        e -= om[sd[embed ? 0 : b].atom_off + (embed ? tid % (n / 2) : tid) / 3];
    }
    e = block_sum256(e, red);
    put(bX, mul(bT, bZ));
    __syncthreads();
    {
        const Reg G = mul(bZ, bX);
        if (live)
            each([&](int r, int c, int i, int j, int q) {
                const double dr = (r == c ? 1.0 : 0.0) - G.v[i][j][q];
                if (r < n && c <= r) rr += (r == c ? 1.0 : 2.0) * dr * dr;
            });
    }
    rr = block_sum256(rr, red);
    // (low Z^2)^(2^(ISQ_SQUARES - 1)) for lambda_min
    const double low = hi / k.kappa;
    for (int i = 0; zmax && i < ISQ_SQUARES; i++) {
        Reg W = mul(i == 0 ? bZ : i & 1 ? bX : bT, i == 0 ? bZ : i & 1 ? bX : bT);
        if (i == 0) each([&](int, int, int i0, int j0, int q) { W.v[i0][j0][q] *= low; });
        put(i & 1 ? bT : bX, W);
        __syncthreads();
    }
    static_assert(ISQ_SQUARES % 2 == 0, "the last square lands in bT");
    if (wave != 0) return;
    double* pb = part + (long long)b * nwg_max * 2;
    if (lane < 2 * ((n + ISQ_MVR - 1) / ISQ_MVR)) pb[lane] = lane == 0 ? e : lane == 1 ? rr : 0.0;
    if (zmax) {
        int m;
        bool ended;
        const double w = isq_tiny_lanczos<NP>(bT, vb, n, ISQ_LMAX, al, be, m, ended, true);
        if (lane == 0) zmax[b] = w > 0.0 ? isq_unsquare(w, ISQ_SQUARES, low) : -1.0;
    }
}

// ---------------------------------------------------------------------------
// launches
// ---------------------------------------------------------------------------
int isq_lanczos_wgs(int nmax) { return (nmax + ISQ_MVR - 1) / ISQ_MVR; }

// Launches of the Lanczos run for lambda_min, and the squarings of Z before it.
// Each squaring doubles the relative gap at the upper end, so 2^(-1/2) of the
// steps do (45 on Z itself, give or take 10).  A squaring is a product at
// 45 TFLOP/s or 8 us, a step reads the matrices at 4.7 TB/s or takes 3.5 us, and
// one after convergence 3 us.  lambda_min of one matrix of order 150, 255, 447
// and 900 takes 135, 170, 175 and 267 us against 400, 635, 440 and 512 with all
// steps on Z, of 64 embeddings of order 384 0.54 ms against 0.85; from order 2300
// on the squarings cost more than they save.
static int isq_lsteps(int squares) {
    static const int most[ISQ_SQUARES + 1] = {ISQ_LMAX, 96, 64, 48, 40, 32, 24};
    return most[squares];
}
static int isq_squares(const int* ns, int nmat, bool embed) {
    double n2 = 0.0, n3 = 0.0, best = 1e300;
    for (int b = 0; b < nmat; b++) {
        const double n = ns[b];
        n2 += (embed ? 0.5 : 1.0) * n * n;
        n3 += (embed ? 0.5 : 1.0) * n * n * n;
    }
    int pick = 0;
    for (int s = 0; s <= ISQ_SQUARES; s++) {
        const double cost = s * (n3 / 45e12 + 8e-6) + (45.0 * std::pow(2.0, -0.5 * s) + 6.0) * (n2 * 8 / 4.7e12 + 3.5e-6) +
                            isq_lsteps(s) * 3e-6;
        if (cost < best) { best = cost; pick = s; }
    }
    return pick;
}

void isq_launch(hipStream_t st, const IsqWork& w, int nmax, int nmat, const int* ns_host, LaunchProfiler* prof) {
    const MatBatch<double> Q = {w.bufs.p[0], w.bufs.ld, w.bufs.stride};
    const bool wide = w.mod.mods == ISQ_MODS_SHORT;
    if (nmax <= 64) {
        const MatBatch<double> Z = {w.bufs.p[ISQ_RESULT], w.bufs.ld, w.bufs.stride};
        auto go = [&](auto kernel) {
            hipLaunchKernelGGL(kernel, dim3(nmat), dim3(256), 0, st, Q, Z, w.ns, isq_table(wide), w.sd, w.om,
                               w.embed ? 1 : 0, w.cls, w.check, isq_lanczos_wgs(nmax), w.zmax);
        };
        if (nmax <= 32) go(isq_tiny_kernel<32>);
        else go(isq_tiny_kernel<64>);
        return;
    }
    const dim3 mv(isq_lanczos_wgs(w.embed ? nmax / 2 : nmax), 1, nmat);
    IsqLanczos L = w.lan;
    L.emb = w.embed;
    const auto lanczos = w.embed ? isq_lanczos_kernel<true> : isq_lanczos_kernel<false>;
    L.done = nullptr;
    const int steps = nmax < 1024 ? ISQ_STEPS_SMALL : ISQ_STEPS_LARGE;
    const int nmin = *std::min_element(ns_host, ns_host + nmat);
    // one workgroup per matrix against one launch per step (5-6 us): an energy at order 135, 180, 225, 300, 447 takes
    // 221, 233, 264, 324, 468 us against 218, 219, 231, 249, 264; 60 molecules of up to 225 793 against 818
    L.one = nmat > 4 ? ISQ_SMALL : ISQ_SMALL / 2;
    if (nmin <= L.one)
        hipLaunchKernelGGL(isq_small_lanczos_kernel, dim3(nmat), dim3(1024), 0, st, Q, w.ns, L, steps, w.cls, w.ops, 0,
                           nullptr);
    if (nmax > L.one)
        for (int j = 0; j < steps; j++) hipLaunchKernelGGL(lanczos, mv, dim3(256), 0, st, Q, w.ns, L, j);
    const int squares = w.zmax ? isq_squares(ns_host, nmat, w.embed) : 0;
    hipLaunchKernelGGL(isq_plan_kernel, dim3(nmat), dim3(64), 0, st, w.ns, L, steps, isq_table(wide), w.ops, w.cls, w.order,
                       w.mod.mods > 0, squares);
    const int shape = isq_shape(ns_host, nmat, w.embed);
    const bool timed = prof && prof->enabled && prof->launches;
    const size_t rec0 = timed ? prof->kind.size() : 0;
    auto product = [&](int k, hipEvent_t e0, hipEvent_t e1) {
        auto go = [&](auto kernel, auto emb_kernel, int tm, int tn, int wk) {
            const int parts = w.embed ? 2 : 1, tiles = splitk_lower_tiles(nmax / parts, tm, tn);
            const int own = isq_own(nmat) ? tiles * parts : 0;
            const dim3 grid = own ? dim3((nmat + GEMM_NXCD - 1) / GEMM_NXCD * GEMM_NXCD * own) : dim3(tiles, parts, nmat);
            if (w.embed)
                hipExtLaunchKernelGGL(emb_kernel, grid, dim3(64 * wk), 0, st, e0, e1, 0, w.bufs, w.ns, w.ops, k, w.order,
                                      nmat, own);
            else
                hipExtLaunchKernelGGL(kernel, grid, dim3(64 * wk), 0, st, e0, e1, 0, w.bufs, w.ns, w.ops, k, w.order, nmat,
                                      own);
        };
        switch (shape) {
        case 0: go(isq_prod_kernel<4, 2, 4, 5, 2, false>, isq_prod_kernel<4, 2, 4, 5, 2, true>, 64, 32, 4); break;
        case 1: go(isq_prod_kernel<6, 2, 4, 2, 2, false>, isq_prod_kernel<6, 2, 4, 2, 2, true>, 96, 32, 4); break;
        case 2: go(isq_prod_kernel<2, 2, 2, 6, 3, false>, isq_prod_kernel<2, 2, 2, 6, 3, true>, 32, 32, 2); break;
        default: go(isq_prod_kernel<2, 2, 4, 6, 3, false>, isq_prod_kernel<2, 2, 4, 6, 3, true>, 32, 32, 4); break;
        }
    };
    for (int k = 0; k < ISQ_OPMAX; k++) {
        hipEvent_t e0 = nullptr, e1 = nullptr;
        if (timed) prof->pair(&e0, &e1, 1, 0.0);
        if (w.mod.mods) isq_mod_launch(st, w, nmat, k, e0, e1);
        else product(k, e0, e1);
    }
    if (timed) {
        // the flops of each launch follow from the classes found on the device;
        // launches past every program's end are no products: not counted
        std::vector<int> cls(nmat);
        (void)hipMemcpyAsync(cls.data(), w.cls, sizeof(int) * nmat, hipMemcpyDeviceToHost, st);
        (void)hipStreamSynchronize(st);
        for (int k = 0; k < ISQ_OPMAX; k++) {
            double flops = 0.0;
            for (int b = 0; b < nmat; b++)
                if (cls[b] >= 0 && k < isq_products(isq_table(wide).cls[cls[b]])) flops += (w.embed ? 0.5 : w.mod.mods ? w.mod.mods : 1.0) * ns_host[b] * ns_host[b] * ns_host[b];
            if (flops > 0.0) prof->work[rec0 + k] = flops;
            else prof->kind[rec0 + k] = -1;
        }
    }
    const MatBatch<double> Z = {w.bufs.p[ISQ_RESULT], w.bufs.ld, w.bufs.stride};
    const int nwg = isq_lanczos_wgs(nmax);
    const auto check = w.embed ? isq_check_kernel<true> : isq_check_kernel<false>;
    for (int p = 0; p < 3; p++)
        hipLaunchKernelGGL(check, mv, dim3(256), 0, st, Q, Z, w.ns, w.cls, w.sd, w.om, w.yv, w.lan.sV, w.check, nwg, p);
    if (!w.zmax) return;
    for (int i = 0; i < squares; i++) product(ISQ_OPMAX + i, nullptr, nullptr);
    const int last = isq_lsteps(squares), every = isq_lcheck(squares);
    // 24 steps at order 150, 255: 135, 192 us in one workgroup against 160, 170 by launches
    L.one = nmat > 4 ? ISQ_SMALL : 3 * ISQ_SMALL / 4;
    const MatBatch<double> W = {w.bufs.p[squares == 0 ? ISQ_RESULT : squares & 1 ? 1 : 2], w.bufs.ld, w.bufs.stride};
    if (nmin <= L.one)
        hipLaunchKernelGGL(isq_small_lanczos_kernel, dim3(nmat), dim3(1024), 0, st, W, w.ns, L, ISQ_LMAX, w.cls, w.ops,
                           squares, w.zmax);
    if (nmax <= L.one) return;
    L.done = w.lan.done;
    hipLaunchKernelGGL(isq_zmax_kernel, dim3(nmat), dim3(64), 0, st, w.ns, w.cls, L, w.ops, squares, 0, 0, w.zmax);
    for (int j = 0; j < last; j++) {
        hipLaunchKernelGGL(lanczos, mv, dim3(256), 0, st, W, w.ns, L, j);
        if ((j + 1) % every == 0)
            hipLaunchKernelGGL(isq_zmax_kernel, dim3(nmat), dim3(64), 0, st, w.ns, w.cls, L, w.ops, squares, j + 1,
                               j + 1 == last ? 1 : 0, w.zmax);
    }
}

void isq_energy_launch(hipStream_t st, const IsqWork& w, SysDesc* sd, int nsys, int nmax, const double* mmult,
                       unsigned* status) {
    hipLaunchKernelGGL(isq_energy_kernel, dim3(nsys), dim3(256), 0, st, sd, w.ns, w.cls, w.check, isq_lanczos_wgs(nmax),
                       mmult, w.zmax,
                       w.mod.mods == ISQ_MODS_SHORT ? ISQ_CHECK_SHORT : ISQ_CHECK, status);
}
