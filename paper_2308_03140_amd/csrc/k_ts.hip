// Pairwise (TS) dispersion energy and gradients (paper Sec. 2.6):
//   E = -1/2 sum_{i != j} C6_ij f(R_ij) / R_ij^6,
//   C6_ij = (3/2) alpha_i alpha_j / (1/omega_i + 1/omega_j)        (eq:pairwise)
//   f = 1/(1 + exp(-a (R/(s_R (Rv_i + Rv_j)) - 1))), TS: a = 20     (eq:fermi-damping)
// Periodic systems (energy per cell) sum over every image, the term n = 0,
// i = j excluded: the undamped R^-6 lattice sum by the Ewald split of
// eq:ts-ewald,
//   sum'_n R^-6 = sum_{0<|x_n|<Rc} gamma^6 phi_r(gamma |x_n|)
//               + (1/Omega) sum_{|G|<kc, G = 0 included} gamma^3 phi_k(|G|/gamma) cos(G.r)
//               - delta_ij gamma^6/6,
//   phi_r(z) = (z^-6 + z^-4 + z^-2/2) e^{-z^2},
//   phi_k(k) = (pi^{3/2}/12)((4 - 2k^2) e^{-k^2/4} + k^3 sqrt(pi) erfc(k/2)),
// minus the real-space sum of (1 - f)/R^6 over every image with (1-f) > 1e-18
// (the damped lattice sum exactly).  The G = 0 term, the sign of the self term
// and the cosine argument are read from the derivation of the split; the
// printed formula omits G = 0 and has them garbled.
//
// Atom i's energy share, its gradient and its parameter derivatives are sums
// over the ordered pairs (i, j) (each ordered pair's energy is counted at i;
// dE/dR_i = sum_j C6_ij grad S_ij(R_j - R_i) gathers both orders).  Per pair the
// divisions are shared: C6 and its omega derivative through 1/(omega_i +
// omega_j), the Fermi factor through 1/R0 and 1/(1 + e^{-|x|}), and 1/R.
#include <algorithm>

#include "mbd_internal.h"
#include "mbd_kernels.h"
#include "mbd_sys.h"

#define TS_DAMP_TAIL 1e-18
#define TS_FIN 128  // lanes of a finite system's row
#define TS_SQRT_PI 1.7724538509055160273

// f = 1/(1 + e^{-x}), x = a (d/R0 - 1), with 1 - f and the derivatives in d
// and R0, from e = e^{-|x|} (no overflow on either side)
__device__ __forceinline__ void ts_fermi(double d, double R0, double a, double& f, double& omf, double& df_dd,
                                         double& df_dR0) {
    if (R0 <= 0.0) { f = 1.0; omf = 0.0; df_dd = 0.0; df_dR0 = 0.0; return; }
    const double iR0 = 1.0 / R0;
    const double x = a * (d * iR0 - 1.0);
    const double e = exp(-fabs(x));
    const double p = 1.0 / (1.0 + e);
    if (x >= 0.0) { f = p; omf = e * p; }
    else { f = e * p; omf = p; }
    const double ff = a * iR0 * (f * omf);
    df_dd = ff;
    df_dR0 = -d * iR0 * ff;
}

// atom i's sums to the outputs asked for
__device__ __forceinline__ void ts_store(const SysDesc& S, int i, double ai, double wi, double Ei, double gx, double gy,
                                         double gz, double dw, double dv, double* eatom) {
    eatom[i] = Ei;
    if (S.grad_coords) {
        S.grad_coords[3 * i] = gx;
        S.grad_coords[3 * i + 1] = gy;
        S.grad_coords[3 * i + 2] = gz;
    }
    const double dEda = 2.0 * Ei / ai;
    if (S.param_kind == 1) {
        // omega = 4 C6/(3 alpha0^2)
        if (S.grad_alpha0) S.grad_alpha0[i] = dEda - 2.0 * wi / ai * dw;
        if (S.grad_omega) S.grad_omega[i] = dw * wi / S.omega_or_c6[i];
    } else {
        if (S.grad_alpha0) S.grad_alpha0[i] = dEda;
        if (S.grad_omega) S.grad_omega[i] = dw;
    }
    if (S.grad_rvdw) S.grad_rvdw[i] = dv;
}

// the six sums of a cell's atom: E, g[3], dw, dv without their factors of i
__device__ __forceinline__ void ts_store_cell(const SysDesc& S, int i, double ai, double wi, const double* r, double* eatom) {
    const double c = 1.5 * ai * wi;
    ts_store(S, i, ai, wi, -0.5 * c * r[0], c * r[1], c * r[2], c * r[3], -1.5 * ai * r[4], -S.beta * c * r[5], eatom);
}

// Finite systems: one workgroup per atom i, its two wavefronts over the j, one
// term each.  Bound by the FP64 vector units: about 120 operations a pair, the
// divisions and the square root as Newton steps on the hardware estimates, no
// branch among them, factors of i alone taken out of the loop, two pairs at
// once for their latency, the six sums in one butterfly.  N = 2000: 24.3 us
// (25.0 with four wavefronts a row), where 13.5 us are the operations; 39.7 us
// with IEEE divisions, a branch per case and a reduction per sum.
__global__ __launch_bounds__(TS_FIN) void mbd_ts_finite_kernel(const SysDesc* sd, const double* om, double* eatom,
                                                              unsigned* status) {
    __shared__ double red[TS_FIN / 64][8];
    const SysDesc& S = sd[0];
    const int N = S.N, i = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const double* __restrict__ R = S.coords;
    const double* __restrict__ al = S.alpha0;
    const double* __restrict__ rv = S.rvdw;
    const double* __restrict__ omp = om + S.atom_off;
    const double xi = R[3 * i], yi = R[3 * i + 1], zi = R[3 * i + 2];
    const double ai = al[i], wi = omp[i], rvi = rv[i], beta = S.beta, a = S.a;
    double sum[8] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0};  // E, g[3], dw, dv without their i factors
#pragma unroll 2
    for (int j = tid; j < N; j += TS_FIN) {
        const double x = R[3 * j] - xi, y = R[3 * j + 1] - yi, z = R[3 * j + 2] - zi;
        const double aj = al[j], wj = omp[j], R0 = beta * (rvi + rv[j]);
        double d2 = x * x + y * y + z * z, d, id;
        const bool close = !(d2 >= 1e-16), skip = close || j == i;
        if (close && j != i) atomicOr(&status[0], MBD_ST_COINCIDENT);
        d2 = skip ? 1.0 : fmin(d2, 1e300);
        sqrt_recip(d2, d, id);
        const double h = recip(wi + wj), wh = wj * h;
        const double c = skip ? 0.0 : aj * wh;  // C6 / ((3/2) alpha_i omega_i)
        // the Fermi factor as in ts_fermi
        const bool damp = !(R0 <= 0.0);
        const double iR0 = recip(damp ? R0 : 1.0);
        const double t = a * (d * iR0 - 1.0), e = exp(-fabs(t)), p = recip(1.0 + e), q = e * p;
        const double f = !damp ? 1.0 : t >= 0.0 ? p : q;
        const double ff = damp ? a * iR0 * (p * q) : 0.0;
        const double id2 = id * id, c6 = c * (id2 * id2 * id2);
        const double s = c6 * f, dd = c6 * (ff - 6.0 * f * id) * id;
        sum[0] += s;
        sum[1] += dd * x;
        sum[2] += dd * y;
        sum[3] += dd * z;
        sum[4] += s * wh;
        sum[5] += c6 * ff * (d * iR0);
    }
    const double w = wave_sum8(sum);
    if ((lane & 7) == 0) red[wv][lane >> 3] = w;
    __syncthreads();
    if (tid == 0) {
        double r[6];
        for (int k = 0; k < 6; k++) r[k] = red[0][k] + red[1][k];
        const double c = 1.5 * ai * wi;
        // dC6/domega_i = C6 omega_j / (omega_i (omega_i + omega_j)); dE/dR_i = sum_j C6 grad S(R_j - R_i)
        ts_store(S, i, ai, wi, -0.5 * c * r[0], c * r[1], c * r[2], c * r[3], -1.5 * ai * r[4], beta * c * r[5], eatom);
    }
}

// Reciprocal vector m and its weight, {G, gamma^3 phi_k(|G|/gamma)/Omega} (0 from
// kc on).
__device__ __forceinline__ double4 ts_recip(const SysDesc& S, const int* rec, int m) {
    double G[3];
    for (int c = 0; c < 3; c++)
        G[c] = rec[3 * m] * S.recip[c] + rec[3 * m + 1] * S.recip[3 + c] + rec[3 * m + 2] * S.recip[6 + c];
    const double k = sqrt(G[0] * G[0] + G[1] * G[1] + G[2] * G[2]), kk = k / S.gamma;
    const double phik = (TS_SQRT_PI * TS_SQRT_PI * TS_SQRT_PI / 12.0) *
                        ((4.0 - 2.0 * kk * kk) * exp(-0.25 * kk * kk) + kk * kk * kk * TS_SQRT_PI * erfc(0.5 * kk));
    return make_double4(G[0], G[1], G[2], k < S.kc ? S.gamma * S.gamma * S.gamma * phik / S.vol : 0.0);
}

// the same for every pair
__global__ __launch_bounds__(256) void mbd_ts_recip_kernel(const SysDesc* sd, const int* rec, int nrec, double4* gw) {
    const int m = blockIdx.x * 256 + threadIdx.x;
    if (m < nrec) gw[m] = ts_recip(sd[0], rec, m);
}

// Periodic systems: a wavefront per pair (i, j), TS_JPW of atom i's in a
// workgroup (and further ones in turn where the grid's y, at most TS_CHUNKS,
// does not cover them), its lanes over the images, then the reciprocal vectors:
// what depends on the pair alone is formed once, and no wavefront mixes the two
// kinds of term.  Writes the six sums of every (i, j chunk).  Bound by the exp
// and sincos of the terms (64 atoms, 602 terms a pair: 19 us, 198 with a row
// (j, term) in flat order per workgroup and the weights formed per pair).
// Without scratch (gw and part null) one workgroup takes all of atom i's pairs,
// forms the weights itself and stores the atom's results.
#define TS_JPW 4
#define TS_CHUNKS 64
__global__ __launch_bounds__(256) void mbd_ts_kernel(const SysDesc* sd, const double* om, const int* img, int nimg,
                                                       const int* rec, const double4* gw, int nrec, double* part,
                                                       double* eatom, unsigned* status) {
    __shared__ double red[4][8];
    const SysDesc& S = sd[0];
    const int N = S.N, i = blockIdx.x, tid = threadIdx.x, lane = tid & 63;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const double* R = S.coords;
    const double ai = S.alpha0[i], wi = om[S.atom_off + i], rvi = S.rvdw[i];
    const double g = S.gamma, g3 = g * g * g, g6 = g3 * g3;
    double sum[8] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0};  // E, g[3], dw, dv without their i factors
    for (int j = blockIdx.y * TS_JPW + wv; j < N; j += TS_JPW * gridDim.y) {
        const double r[3] = {R[3 * j] - R[3 * i], R[3 * j + 1] - R[3 * i + 1], R[3 * j + 2] - R[3 * i + 2]};
        const double wj = om[S.atom_off + j], wh = wj / (wi + wj), c = S.alpha0[j] * wh;  // C6 / ((3/2) alpha_i omega_i)
        const double R0 = S.beta * (rvi + S.rvdw[j]);
        double s = 0.0, ds[3] = {0.0, 0.0, 0.0}, ds0 = 0.0;
        // self term -gamma^6/6 of the reciprocal sum, once per atom
        if (j == i && lane == 0) s = -g6 / 6.0;
        for (int u = lane; u < nimg; u += 64) {
            double x[3];
            for (int k = 0; k < 3; k++)
                x[k] = r[k] + img[3 * u] * S.lat[k] + img[3 * u + 1] * S.lat[3 + k] + img[3 * u + 2] * S.lat[6 + k];
            const double d2 = x[0] * x[0] + x[1] * x[1] + x[2] * x[2];
            if (!(d2 >= 1e-16)) {  // n = 0, i = j; any other zero distance is a coincident pair
                if (j != i || d2 != 0.0) atomicOr(&status[0], MBD_ST_COINCIDENT);
                continue;
            }
            double d, id;
            sqrt_recip(d2, d, id);
            const double id2 = id * id, id6 = id2 * id2 * id2;
            double f, omf, fd, fR0;
            ts_fermi(d, R0, S.a, f, omf, fd, fR0);
            double dd = 0.0;
            if (d < S.rc) {
                const double z = g * d, iz = recip(z), iz2 = iz * iz, ez = exp(-z * z);
                s += g6 * (iz2 * iz2 * iz2 + iz2 * iz2 + 0.5 * iz2) * ez;
                dd += -g6 * g * (6.0 * iz2 * iz2 * iz2 * iz + 6.0 * iz2 * iz2 * iz + 3.0 * iz2 * iz + iz) * ez;
            }
            if (omf > TS_DAMP_TAIL) {
                s -= omf * id6;
                dd += fd * id6 + 6.0 * omf * id6 * id;
                ds0 += fR0 * id6;
            }
            for (int k = 0; k < 3; k++) ds[k] += dd * x[k] * id;
        }
        for (int m = lane; m < nrec; m += 64) {
            const double4 G = gw ? gw[m] : ts_recip(S, rec, m);
            if (G.w == 0.0) continue;
            double sn, cs;
            sincos(G.x * r[0] + G.y * r[1] + G.z * r[2], &sn, &cs);
            s += G.w * cs;
            ds[0] -= G.w * sn * G.x;
            ds[1] -= G.w * sn * G.y;
            ds[2] -= G.w * sn * G.z;
        }
        sum[0] += c * s;
        for (int k = 0; k < 3; k++) sum[1 + k] += c * ds[k];
        sum[4] += c * s * wh;
        sum[5] += c * ds0;
    }
    const double w = wave_sum8(sum);
    if ((lane & 7) == 0) red[wv][lane >> 3] = w;
    __syncthreads();
    auto total = [&](int k) { return (red[0][k] + red[1][k]) + (red[2][k] + red[3][k]); };
    if (part) {
        if (tid < 6) part[((long long)i * gridDim.y + blockIdx.y) * 6 + tid] = total(tid);
    } else if (tid == 0) {
        double r[6];
        for (int k = 0; k < 6; k++) r[k] = total(k);
        ts_store_cell(S, i, ai, wi, r, eatom);
    }
}

// energy = sum of the per-atom shares, in a fixed order; errors[0..3] = 0.  part:
// a periodic system's sums, whose rows are added here first, a lane per atom.
__global__ __launch_bounds__(1024) void mbd_ts_sum_kernel(const SysDesc* sd, const double* om, const double* part, int nchunk,
                                                            double* eatom, const unsigned* status) {
    __shared__ double red[16];
    const SysDesc& S = sd[0];
    double e = 0.0;
    for (int i = threadIdx.x; i < S.N; i += 1024) {
        if (part) {
            double r[6] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
            for (int c = 0; c < nchunk; c++)
                for (int k = 0; k < 6; k++) r[k] += part[((long long)i * nchunk + c) * 6 + k];
            ts_store_cell(S, i, S.alpha0[i], om[S.atom_off + i], r, eatom);
        }
        e += eatom[i];
    }
    e = wave_sum(e);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = e;
    __syncthreads();
    if (threadIdx.x == 0) {
        e = 0.0;
        for (int w = 0; w < 16; w++) e += red[w];
        if (S.energy) *S.energy = status[0] ? __longlong_as_double(0x7ff8000000000000LL) : e;
        if (S.errors)
            for (int k = 0; k < 4; k++) S.errors[k] = 0.0;
    }
}

static int ts_chunks(int N) { return std::min(TS_CHUNKS, (N + TS_JPW - 1) / TS_JPW); }

size_t mbd_ts_scratch(int N, int nrec) {
    return sizeof(double4) * std::max(1, nrec) + sizeof(double) * 6 * N * ts_chunks(N);
}

void mbd_ts_launch(hipStream_t st, const SysDesc* sd, int N, const double* om, const int* img, int nimg,
                   const int* rec, int nrec, int periodic, double* eatom, void* scratch, unsigned* status,
                   LaunchProfiler* prof) {
    hipEvent_t e0 = nullptr, e1 = nullptr;
    if (prof && prof->enabled && prof->launches)  // work: the pair terms of the launch
        prof->pair(&e0, &e1, 11, periodic ? (double)N * N * (nimg + nrec) : (double)N * (N - 1));
    const int nchunk = scratch ? ts_chunks(N) : 1;
    double* part = nullptr;
    if (periodic) {
        double4* gw = (double4*)scratch;
        if (scratch) part = (double*)(gw + std::max(1, nrec));
        if (scratch && nrec)
            hipLaunchKernelGGL(mbd_ts_recip_kernel, dim3((nrec + 255) / 256), dim3(256), 0, st, sd, rec, nrec, gw);
        hipExtLaunchKernelGGL(mbd_ts_kernel, dim3(N, nchunk), dim3(256), 0, st, e0, e1, 0, sd, om, img, nimg, rec, gw, nrec, part,
                              eatom, status);
    } else {
        hipExtLaunchKernelGGL(mbd_ts_finite_kernel, dim3(N), dim3(TS_FIN), 0, st, e0, e1, 0, sd, om, eatom, status);
    }
    hipLaunchKernelGGL(mbd_ts_sum_kernel, dim3(1), dim3(1024), 0, st, sd, om, part, nchunk, eatom, status);
}
