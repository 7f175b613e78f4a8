// Periodic systems: Q(q) of eq:q-matrix with T^lr(q) the Bloch sum of g T
// (paper Sec. 2.2), evaluated with the Ewald split of eq:ewald/eq:terfc plus
// a real-space damping correction, for every q of the mesh, and the matching
// adjoint contraction for dE/dR, dE/dalpha0 and dE/dA (lattice).
//
// For the pair (i, j), r = R_j - R_i and x_n = r + R_n:
//   T_ij(q) = sum_n [T^erfc(x_n) (|x_n| < Rc) - (1 - g(x_n)) T(x_n)] e^{-i q.x_n}
//           + (4 pi/Omega) sum_{0<|k|<kc} k^ k^ e^{-k^2/(4 gamma^2)} e^{+i G.r},  k = G + q
//           - delta_ij 4 gamma^3/(3 sqrt(pi)) I
// The terms with n = 0, i = j are skipped; the surface term and k = 0 are
// omitted; the damping correction runs over every image with (1 - g) > 1e-18.
// T^erfc_ab = (delta_ab r^2 B - r_a r_b C)/r^5 with B, C of eq:terfc (the
// factor 3 of the printed r_a r_b term is part of C).
//
// The reciprocal-space term is a sum of rank-one 3x3 blocks k k^T times a
// pair phase, so over all pairs it is the low-rank product U U^H with
// U_{ia,g} = sqrt(w_g) k_a e^{-i G_g.R_i}, w = (4 pi/Omega) e^{-k^2/(4 gamma^2)}/k^2,
// one column per reciprocal vector of the q point's sphere.  It is formed on
// the matrix cores (a product over the ~265 columns instead of that many
// exponentials and phases per pair and q), and the adjoint contracts M with U
// the same way: W = M C U, then per atom and column a few products of U and W.
//
// The Hermitian Q(q) is stored as its real embedding [[Re, -Im], [Im, Re]]
// (order 2n) so the batched real eigensolver serves it; every eigenvalue of
// Q(q) appears twice.  The reciprocal sums are evaluated in FP64.
#include "gemm_splitk.h"
#include "mbd_internal.h"
#include "mbd_kernels.h"
#include "mbd_sys.h"

#define DAMP_TAIL 1e-18
#define SQRT_PI 1.7724538509055160273

__device__ __forceinline__ void fermi_pair(double d, double R0, double a, double& g, double& omg, double& dg_dr) {
    if (R0 <= 0.0) { g = 1.0; omg = 0.0; dg_dr = 0.0; return; }
    const double x = a * (d / R0 - 1.0);
    if (x >= 0.0) { const double e = exp(-x); g = 1.0 / (1.0 + e); omg = e / (1.0 + e); }
    else { const double e = exp(x); g = e / (1.0 + e); omg = 1.0 / (1.0 + e); }
    dg_dr = a / R0 * g * omg;
}

// Real-space image term F(x) = T^erfc(x) [|x| < rc] - (1-g) T(x) and its
// derivatives, as the coefficients of their tensors:
//   F          = f1 delta - f2 x x^T
//   dF/dx_c    = x_c (h1 delta - h2 x x^T) - f2 (e_c x^T + x e_c^T)
//   dF/dR0     = a0 delta - b0 x x^T = (dg/dR0) T(x),
// R0 = beta (Rv_i + Rv_j) the damping radius (dg/dR0 = -(d/R0) dg/dd); f1 and f2
// only without GRAD.  Returns false when the term is empty.
struct ImageTerm {
    double f1, f2, h1, h2, a0, b0;
};
template <bool GRAD>
__device__ __forceinline__ bool image_term(const double* x, double gamma, double rc, double R0, double a, ImageTerm& T) {
    const double r2 = x[0] * x[0] + x[1] * x[1] + x[2] * x[2];
    const double d = sqrt(r2);
    const bool erfc_on = d < rc;
    double g, omg, gd;
    fermi_pair(d, R0, a, g, omg, gd);
    const bool damp_on = omg > DAMP_TAIL;
    if (!erfc_on && !damp_on) return false;
    const double inv_d = 1.0 / d;
    const double inv3 = inv_d * inv_d * inv_d, inv5 = inv3 * inv_d * inv_d;
    double B = 0.0, C = 0.0;
    T.h1 = T.h2 = T.a0 = T.b0 = 0.0;
    if (erfc_on) {
        const double z = gamma * d;
        const double ex = exp(-z * z);
        const double ec = erfc(z);
        B = ec + 2.0 * z / SQRT_PI * ex;
        C = 3.0 * ec + 2.0 * z / SQRT_PI * (3.0 + 2.0 * z * z) * ex;
        if (GRAD) {
            const double dB = -4.0 * gamma * gamma * gamma * r2 / SQRT_PI * ex;
            const double dC = -8.0 * gamma * z * z * z * z / SQRT_PI * ex;
            T.h1 = (dB * inv3 - 3.0 * B * inv3 * inv_d) * inv_d;
            T.h2 = (dC * inv5 - 5.0 * C * inv5 * inv_d) * inv_d;
        }
    }
    // the bare tensor T = delta/r^3 - 3 x x^T/r^5 scaled by (1 - g): subtracted
    const double w = damp_on ? omg : 0.0;
    T.f1 = (B - w) * inv3;
    T.f2 = (C - 3.0 * w) * inv5;
    if (GRAD && damp_on) {
        T.h1 += 3.0 * omg * inv5 + gd * inv_d * inv3;
        T.h2 += 15.0 * omg * inv5 * inv_d * inv_d + 3.0 * gd * inv_d * inv5;
        const double g0 = -gd * d / R0;
        T.a0 = g0 * inv3;
        T.b0 = 3.0 * g0 * inv5;
    }
    return true;
}

// Assembly of the embedded Q(q).  A workgroup of W wavefronts holds 64 W / lpp
// slots of lpp lanes, one lane per q-point (lpp: the q count rounded up to a
// power of two, at most 64; grid y covers further groups of q-points); spp
// slots share an atom pair i <= j and split its images.  The
// real-space image terms depend on the pair and the image only: each is
// formed once, by one lane of its slot, into LDS (lpp images per round and
// slot, the empty ones left out), and every lane of the slot adds it with its
// own phase e^{-i q.x}; the slots' sums are added at the end in a fixed order.
// Bound by those LDS reads, every lane the same address: the six components of
// the symmetric term (64 atoms, 64 q points: 71 us, 137 with all nine and a
// flag for every image).  With one slot a pair, 8 atoms on 8 q points were 8
// wavefronts that walked all images in turn (547 us, the adjoint 1374 us).
// Lanes of a pair index past the last follow the barriers and store nothing.  Writes the real-space and self terms and omega^2 into the left
// block column [Re; Im] of the embedding; the reciprocal-space product then
// adds its term and fills the right block column.
#define PER_LANES 64

// Pair index -> atoms i <= j.  The pair (j, i) is the conjugate of (i, j): the
// image terms are even in x and the image list holds -n with every n.
__device__ __forceinline__ void per_pair(long long pid, int& i, int& j) {
    j = (int)((sqrt(8.0 * (double)pid + 1.0) - 1.0) * 0.5);
    while ((long long)(j + 1) * (j + 2) / 2 <= pid) j++;
    while ((long long)j * (j + 1) / 2 > pid) j--;
    i = (int)(pid - (long long)j * (j + 1) / 2);
}
static long long per_pairs(int N) { return (long long)N * (N + 1) / 2; }

// Sum of v over the spp slots of a pair (lanes lpp, 2 lpp, .. apart within a
// wavefront, then its wavefronts through LDS), in the lanes of the pair's first
// slot.  xw: one value per thread.  Every thread of the workgroup takes part.
template <int W>
__device__ __forceinline__ double per_slot_sum(double v, int lpp, int spp, double* xw) {
    const int inw = min(spp, PER_LANES / lpp);  // slots of the pair in one wavefront
    for (int o = lpp; o < lpp * inw; o *= 2) v += __shfl_xor(v, o, 64);
    if (W > 1 && spp > inw) {
        const int nw = spp / inw;  // wavefronts of the pair (inw = 64 / lpp here)
        const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
        __syncthreads();
        xw[threadIdx.x] = v;
        __syncthreads();
        v = 0.0;
        for (int w = 0; w < nw; w++) v += xw[(wave / nw * nw + w) * 64 + lane];
    }
    return v;
}

// A slot's nonempty image terms in a row from its first entry: this lane's entry
// and the slot's count.  A slot lies in one wavefront, so its entries need no
// barrier, only the order of its own LDS accesses.
__device__ __forceinline__ int per_slot_place(bool ok, int slot, int lpp, int ql, int& cnt) {
    const unsigned long long all = __ballot(ok) >> ((threadIdx.x & 63) - ql);
    const unsigned long long m = lpp == 64 ? all : all & ((1ull << lpp) - 1ull);
    cnt = __popcll(m);
    return slot * lpp + __popcll(m & ((1ull << ql) - 1ull));
}
__device__ __forceinline__ void per_slot_fence() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

template <int W>
__global__ __launch_bounds__(PER_LANES * W) void mbd_assemble_periodic_kernel(const SysDesc* sd, const double* om,
                                                                          const double* cc, const double* qcart,
                                                                          int nq, int lpp, int spp, const int* img, int nimg,
                                                                          const double* phase, MatBatch<double> Q,
                                                                          unsigned* status) {
    __shared__ double2 Fs[PER_LANES * W][3];  // xx xy, xz yy, yz zz
    __shared__ int ts[PER_LANES * W];         // its image
    const SysDesc& S = sd[0];
    const int N = S.N, n = 3 * N;
    const int slot = threadIdx.x / lpp, ql = threadIdx.x % lpp, sub = slot % spp;
    const long long pid0 = (long long)blockIdx.x * (PER_LANES * W / lpp / spp) + slot / spp;
    const bool pv = pid0 < (long long)N * (N + 1) / 2;
    const long long pid = pv ? pid0 : 0;
    const int q = blockIdx.y * lpp + ql;
    const bool qv_ok = pv && q < nq;
    int i, j;
    per_pair(pid, i, j);
    const double* R = S.coords;
    const double r[3] = {R[3 * j] - R[3 * i], R[3 * j + 1] - R[3 * i + 1], R[3 * j + 2] - R[3 * i + 2]};
    const int qc = qv_ok ? q : 0;
    const double qv[3] = {qcart[3 * qc], qcart[3 * qc + 1], qcart[3 * qc + 2]};
    const double R0 = S.beta * (S.rvdw[i] + S.rvdw[j]);
    // e^{-i q.x} = e^{-i q.r} e^{-i q.R_n}, the second factor from the table
    double sb, cb;
    sincos(-(qv[0] * r[0] + qv[1] * r[1] + qv[2] * r[2]), &sb, &cb);
    double Tre[6], Tim[6];
    for (int k = 0; k < 6; k++) { Tre[k] = 0.0; Tim[k] = 0.0; }
    for (int r0 = 0; r0 < nimg; r0 += lpp * spp) {
        const int t = r0 + sub * lpp + ql;
        bool ok = false;
        double x[3];
        ImageTerm F;
        if (t < nimg) {
            const double n0 = img[3 * t], n1 = img[3 * t + 1], n2 = img[3 * t + 2];
            for (int c = 0; c < 3; c++) x[c] = r[c] + n0 * S.lat[c] + n1 * S.lat[3 + c] + n2 * S.lat[6 + c];
            const double d2 = x[0] * x[0] + x[1] * x[1] + x[2] * x[2];
            if (d2 != 0.0) {
                if (pv && i != j && d2 < 1e-16 && blockIdx.y == 0) atomicOr(&status[0], MBD_ST_COINCIDENT);
                ok = image_term<false>(x, S.gamma, S.rc, R0, S.a, F);
            }
        }
        int cnt;
        const int at = per_slot_place(ok, slot, lpp, ql, cnt);
        if (ok) {
            Fs[at][0] = make_double2(F.f1 - F.f2 * x[0] * x[0], -F.f2 * x[0] * x[1]);
            Fs[at][1] = make_double2(-F.f2 * x[0] * x[2], F.f1 - F.f2 * x[1] * x[1]);
            Fs[at][2] = make_double2(-F.f2 * x[1] * x[2], F.f1 - F.f2 * x[2] * x[2]);
            ts[at] = t;
        }
        per_slot_fence();
        for (int u = slot * lpp; u < slot * lpp + cnt; u++) {
            const double* pt = phase + 2 * ((long long)ts[u] * nq + qc);
            const double cph = cb * pt[0] - sb * pt[1], sph = cb * pt[1] + sb * pt[0];
            const double2 f0 = Fs[u][0], f1 = Fs[u][1], f2 = Fs[u][2];
            const double f[6] = {f0.x, f0.y, f1.x, f1.y, f2.x, f2.y};
            for (int k = 0; k < 6; k++) { Tre[k] += f[k] * cph; Tim[k] += f[k] * sph; }
        }
        per_slot_fence();
    }
    if (spp > 1) {
        double* xw = reinterpret_cast<double*>(Fs);
        __syncthreads();
        for (int k = 0; k < 6; k++) {
            Tre[k] = per_slot_sum<W>(Tre[k], lpp, spp, xw);
            Tim[k] = per_slot_sum<W>(Tim[k], lpp, spp, xw);
        }
    }
    if (!qv_ok || sub != 0) return;
    if (i == j) {
        const double self = 4.0 * S.gamma * S.gamma * S.gamma / (3.0 * SQRT_PI);
        Tre[0] -= self; Tre[3] -= self; Tre[5] -= self;
    }
    // without cc and om: the lattice sum T(q) itself (c = 1, no omega^2)
    const double pc = cc ? cc[S.atom_off + i] * cc[S.atom_off + j] : 1.0;
    double* Qb = Q.at(q);
    const long long ld = Q.ld;
    for (int a = 0; a < 3; a++)
        for (int b = 0; b < 3; b++) {
            const int k = a < b ? a * (5 - a) / 2 + b : b * (5 - b) / 2 + a;
            const double re = pc * Tre[k] +
                              ((om && i == j && a == b) ? om[S.atom_off + i] * om[S.atom_off + i] : 0.0);
            const long long r0 = 3 * i + a, c0 = 3 * j + b;
            const double im = i == j ? 0.0 : pc * Tim[k];  // the images of i = j come in +-n
            Qb[r0 + c0 * ld] = re;
            Qb[(r0 + n) + c0 * ld] = im;
            if (i != j) {
                Qb[c0 + r0 * ld] = re;
                Qb[(c0 + n) + r0 * ld] = -im;
            }
        }
}

// Reciprocal vector and weights of column g of q point q's list (t >= 0):
// G, k = G + q, sw = sqrt(w), w = (4 pi/Omega) e^{-k^2/(4 gamma^2)}/k^2, and
// f = (dw/dk_d)/(w k_d) = -1/(2 gamma^2) - 2/k^2.
__device__ __forceinline__ void recip_column(const SysDesc& S, const int* rec, int t, const double* qv, double* G,
                                             double* k, double& sw, double& f) {
    const double m0 = rec[3 * t], m1 = rec[3 * t + 1], m2 = rec[3 * t + 2];
    for (int c = 0; c < 3; c++) {
        G[c] = m0 * S.recip[c] + m1 * S.recip[3 + c] + m2 * S.recip[6 + c];
        k[c] = G[c] + qv[c];
    }
    const double k2 = k[0] * k[0] + k[1] * k[1] + k[2] * k[2];
    const double g4 = 1.0 / (4.0 * S.gamma * S.gamma);
    sw = sqrt(4.0 * M_PI / S.vol * exp(-k2 * g4) / k2);
    f = -2.0 * g4 - 2.0 / k2;
}

// Columns of C U(q), embedded: rows 0 .. n-1 Re, rows n .. 2n-1 Im, C = 1 without
// cc; the columns past the q point's count are zero.  Grid (ncol, nq), 64 threads
// over the atoms.
__global__ __launch_bounds__(64) void per_recip_basis_kernel(const SysDesc* sd, const double* cc, const double* qcart,
                                                             PerEwald pr) {
    const SysDesc& S = sd[0];
    const int N = S.N, n = 3 * N;
    const int g = blockIdx.x, q = blockIdx.y;
    double* Zc = pr.Z + (long long)q * pr.sZ + (long long)g * pr.ldz;
    const int t = pr.col[(long long)q * pr.ncol + g];
    double G[3] = {0.0, 0.0, 0.0}, k[3] = {0.0, 0.0, 0.0}, sw = 0.0, f;
    if (t >= 0) recip_column(S, pr.rec, t, qcart + 3 * q, G, k, sw, f);
    const double* R = S.coords;
    for (int i = threadIdx.x; i < N; i += 64) {
        double sn = 0.0, cs = 1.0;
        if (t >= 0) sincos(G[0] * R[3 * i] + G[1] * R[3 * i + 1] + G[2] * R[3 * i + 2], &sn, &cs);
        const double w = cc ? sw * cc[S.atom_off + i] : sw;
        for (int a = 0; a < 3; a++) {
            Zc[3 * i + a] = w * k[a] * cs;      // e^{-i G.R} = cos - i sin
            Zc[n + 3 * i + a] = -w * k[a] * sn;
        }
    }
}

// Real-space phases: phase[t][q] = (cos, sin) of -q.R_n for image t, so that
// the lanes of a pair (one q each) read consecutive entries.
__global__ __launch_bounds__(256) void per_phase_kernel(const SysDesc* sd, const double* qcart, int nq,
                                                        const int* img, int nimg, double* phase) {
    const SysDesc& S = sd[0];
    const long long e = (long long)blockIdx.x * 256 + threadIdx.x;
    if (e >= (long long)nimg * nq) return;
    const int t = (int)(e / nq), q = (int)(e % nq);
    double Rn[3];
    for (int c = 0; c < 3; c++) Rn[c] = img[3 * t] * S.lat[c] + img[3 * t + 1] * S.lat[3 + c] + img[3 * t + 2] * S.lat[6 + c];
    double sn, cs;
    sincos(-(qcart[3 * q] * Rn[0] + qcart[3 * q + 1] * Rn[1] + qcart[3 * q + 2] * Rn[2]), &sn, &cs);
    phase[2 * e] = cs;
    phase[2 * e + 1] = sn;
}

// Reciprocal term of the embedding, (C U)(C U)^H: the lower triangles of Re = U_r
// U_r^T + U_i U_i^T (part 0) and Im = U_i U_r^T - U_r U_i^T (part 1), added to
// the real-space part and copied to their other seven places (and to the FP32
// copy).  K split over the wavefronts (gemm_splitk.h); matrix-core bound: 64 q
// points of 64 atoms 90 us against 230 for the whole left block column
// through staged tiles.
template <int MI, int NJ, int WK, int U>
__global__ __launch_bounds__(64 * WK) void per_recip_asm_kernel(PerEwald pr, int n, MatBatch<double> Q,
                                                                  MatBatch<float> Q32) {
    typedef SplitK<MI, NJ, WK, U> SK;
    constexpr int TM = SK::TM, TN = SK::TN, LDC = SK::LDC;
    __shared__ __align__(16) double cs[SK::LDS];
    const int b = blockIdx.z, part = blockIdx.y;
    int ti, tj;
    splitk_lower_tile(splitk_tile_index(blockIdx.x, b, gridDim.x), TM / TN, ti, tj);
    const int m0 = ti * TM, n0 = tj * TN;
    if (m0 >= n || n0 >= n) return;
    {
        SK sk;
        sk.clear();
        const double* Z = pr.Z + (long long)b * pr.sZ;
        sk.run(Z, m0 + part * n, pr.ldz, Z, n0, pr.ldz, pr.ncol);
        if (part) sk.template run<true>(Z, m0, pr.ldz, Z, n0 + n, pr.ldz, pr.ncol);
        else sk.run(Z, m0 + n, pr.ldz, Z, n0 + n, pr.ldz, pr.ncol);
        sk.reduce(cs);
    }
    double* Qb = Q.at(b);
    float* Qf = Q32.p ? Q32.at(b) : nullptr;
    const long long ld = Q.ld;
    auto put = [&](long long at, double v) {
        Qb[at] = v;
        if (Qf) Qf[at] = (float)v;
    };
    const double sg = part ? -1.0 : 1.0;
    for (int x = threadIdx.x; x < TM * TN; x += SK::NT) {
        const int r = x % TM, cl = x / TM, row = m0 + r, col = n0 + cl;
        if (row >= n || col >= n || col > row) continue;
        const double s = cs[cl * LDC + r] + cs[(TN + cl) * LDC + r];
        double v = Qb[row + part * n + col * ld] + s;
        if (part && row == col) v = 0.0;  // the diagonal of Im
        put(row + part * n + col * ld, v);
        put(row + (1 - part) * n + (n + col) * ld, sg * v);
        cs[cl * LDC + r] = v;
    }
    __syncthreads();
    for (int x = threadIdx.x; x < TM * TN; x += SK::NT) {
        const int cl = x % TN, r = x / TN, row = m0 + r, col = n0 + cl;
        if (row >= n || col >= row) continue;
        const double v = cs[cl * LDC + r];
        put(col + part * n + row * ld, sg * v);
        put(col + (1 - part) * n + (n + row) * ld, v);
    }
}

// Adjoint contraction.  With M(q) = Q(q)^{-1/2} read from the embedded
// inverse square root (Re in the top-left block, Im in the bottom-left), the
// ordered pair (i, j) at q contributes, with X = d T_ij(q) and
// c_i c_j (1/4) (1/n_q) Re sum_ab M_{jb,ia} X_ab:
//   to dE/dR_j (+) and dE/dR_i (-)    X = dT/dr_c
//   to dE/dA_vc                        X = dT/dA_vc (Cartesian positions and
//                                      fractional q fixed: dR_n/dA_vc = n_v e_c,
//                                      dG/dA_vc = -G_c Ainv[:, v], dOmega/dA_vc =
//                                      Omega Ainv_cv)
//   to dE/dalpha_i, dE/dalpha_j        X = T_ij(q) / (2 alpha)
//   to dE/domega_i, dE/domega_j        X = T_ij(q) / omega (through c = omega
//                                      sqrt(alpha0); the omega^2 diagonal adds
//                                      (1/2) omega_i Re Tr M_ii(q) per q)
//   to dE/dRv_i, dE/dRv_j              X = beta dT_ij(q)/dR0 (damping radius
//                                      R0 = beta (Rv_i + Rv_j))
// Partial results per (q, pair i <= j) of the real-space and self terms: {P,
// dR[3], dA[9], P0} of (i, j), which (j, i) repeats (dR negated); the reciprocal-space term is contracted through U below.
// Same layout as the assembly: slots of one lane per q-point, the coefficients
// of each real-space image term formed once into LDS and added by every lane of
// its slot with its own phase and M(q).  Contracted with M, whose symmetric part
// is all that the symmetric tensors see, they need only tr M, M x and x.M x: 66
// operations and six LDS reads an image and lane (64 atoms, 64 q points: 89
// us, 288 with the 45 tensor components in LDS, which bound it).
template <int W>
__global__ __launch_bounds__(PER_LANES * W) void mbd_grad_periodic_kernel(const SysDesc* sd, const double* om,
                                                                      const double* cc, const double* qcart, int nq,
                                                                      int lpp, int spp, const int* img, int nimg,
                                                                      const double* phase, MatBatch<double> M,
                                                                      double* part) {
    __shared__ double2 Fs[PER_LANES * W][5];  // x, f1, f2, h1, h2, a0, b0
    __shared__ int4 ts[PER_LANES * W];        // the image's cell and index
    const SysDesc& S = sd[0];
    const int N = S.N, n = 3 * N;
    const int slot = threadIdx.x / lpp, ql = threadIdx.x % lpp, sub = slot % spp;
    const long long pid0 = (long long)blockIdx.x * (PER_LANES * W / lpp / spp) + slot / spp;
    const bool pv = pid0 < (long long)N * (N + 1) / 2;
    const long long pid = pv ? pid0 : 0;
    const int q0 = blockIdx.y * lpp + ql;
    const bool qv_ok = pv && q0 < nq;
    const int q = q0 < nq ? q0 : 0;
    int i, j;
    per_pair(pid, i, j);
    double* out = part + ((long long)q * N * (N + 1) / 2 + pid) * PER_PART;
    if (S.N == 0) return;
    const double* R = S.coords;
    const double r[3] = {R[3 * j] - R[3 * i], R[3 * j + 1] - R[3 * i + 1], R[3 * j + 2] - R[3 * i + 2]};
    const double qv[3] = {qcart[3 * q], qcart[3 * q + 1], qcart[3 * q + 2]};
    const double R0 = S.beta * (S.rvdw[i] + S.rvdw[j]);
    // e^{-i q.x} = e^{-i q.r} e^{-i q.R_n}, the second factor from the table
    double sb, cb;
    sincos(-(qv[0] * r[0] + qv[1] * r[1] + qv[2] * r[2]), &sb, &cb);
    // M_{jb,ia}: its trace and M + M^T (xx xy xz yy yz zz)
    double Mr[6], Mi[6];
    const double* Mb = M.at(q);
    for (int a = 0; a < 3; a++)
        for (int b = a; b < 3; b++) {
            const long long o = 3 * j + b + (long long)(3 * i + a) * M.ld, p = 3 * j + a + (long long)(3 * i + b) * M.ld;
            const int k = a * (5 - a) / 2 + b;
            Mr[k] = Mb[o] + Mb[p];
            Mi[k] = Mb[n + o] + Mb[n + p];
        }
    const double trr = 0.5 * (Mr[0] + Mr[3] + Mr[5]), tri = 0.5 * (Mi[0] + Mi[3] + Mi[5]);
    // rho = A^{-T} r  (rho_v = sum_d Ainv[d][v] r_d)
    double rho[3];
    for (int v = 0; v < 3; v++) rho[v] = S.linv[v] * r[0] + S.linv[3 + v] * r[1] + S.linv[6 + v] * r[2];
    double P = 0.0, P0 = 0.0, Ti = 0.0, dR[3] = {0, 0, 0}, dA[9];
    for (int k = 0; k < 9; k++) dA[k] = 0.0;
    for (int r0 = 0; r0 < nimg; r0 += lpp * spp) {
        const int t = r0 + sub * lpp + ql;
        bool ok = false;
        double x[3];
        int nn[3];
        ImageTerm F;
        if (t < nimg) {
            for (int c = 0; c < 3; c++) nn[c] = img[3 * t + c];
            for (int c = 0; c < 3; c++) x[c] = r[c] + nn[0] * S.lat[c] + nn[1] * S.lat[3 + c] + nn[2] * S.lat[6 + c];
            const double d2 = x[0] * x[0] + x[1] * x[1] + x[2] * x[2];
            ok = d2 != 0.0 && image_term<true>(x, S.gamma, S.rc, R0, S.a, F);
        }
        int cnt;
        const int at = per_slot_place(ok, slot, lpp, ql, cnt);
        if (ok) {
            Fs[at][0] = make_double2(x[0], x[1]);
            Fs[at][1] = make_double2(x[2], F.f1);
            Fs[at][2] = make_double2(F.f2, F.h1);
            Fs[at][3] = make_double2(F.h2, F.a0);
            Fs[at][4] = make_double2(F.b0, 0.0);
            ts[at] = make_int4(nn[0], nn[1], nn[2], t);
        }
        per_slot_fence();
        for (int u = slot * lpp; u < slot * lpp + cnt; u++) {
            const int4 m = ts[u];
            const double2 u0 = Fs[u][0], u1 = Fs[u][1], u2 = Fs[u][2], u3 = Fs[u][3];
            const double y[3] = {u0.x, u0.y, u1.x}, f1 = u1.y, f2 = u2.x, h1 = u2.y, h2 = u3.x, a0 = u3.y, b0 = Fs[u][4].x;
            const double* pt = phase + 2 * ((long long)m.w * nq + q);
            const double cph = cb * pt[0] - sb * pt[1], sph = cb * pt[1] + sb * pt[0];
            // (M + M^T) x and x.M x, then times the phase
            const double sr[3] = {Mr[0] * y[0] + Mr[1] * y[1] + Mr[2] * y[2], Mr[1] * y[0] + Mr[3] * y[1] + Mr[4] * y[2],
                                  Mr[2] * y[0] + Mr[4] * y[1] + Mr[5] * y[2]};
            const double si[3] = {Mi[0] * y[0] + Mi[1] * y[1] + Mi[2] * y[2], Mi[1] * y[0] + Mi[3] * y[1] + Mi[4] * y[2],
                                  Mi[2] * y[0] + Mi[4] * y[1] + Mi[5] * y[2]};
            const double qr = 0.5 * (y[0] * sr[0] + y[1] * sr[1] + y[2] * sr[2]);
            const double qi = 0.5 * (y[0] * si[0] + y[1] * si[1] + y[2] * si[2]);
            const double tr = trr * cph - tri * sph, ti = trr * sph + tri * cph;
            const double qc = qr * cph - qi * sph, qs = qr * sph + qi * cph;
            P += f1 * tr - f2 * qc;
            Ti += f1 * ti - f2 * qs;  // of -i F e^{i ph}: the phase's own derivatives
            P0 += a0 * tr - b0 * qc;
            const double h = h1 * tr - h2 * qc, nv[3] = {(double)m.x, (double)m.y, (double)m.z};
            for (int c = 0; c < 3; c++) {
                const double D = y[c] * h - f2 * (sr[c] * cph - si[c] * sph);
                dR[c] += D;
                for (int v = 0; v < 3; v++) dA[v * 3 + c] += nv[v] * D;
            }
        }
        per_slot_fence();
    }
    // (dF_c - i q_c F) e^{i ph} and (dF_c n_v + i q_c rho_v F) e^{i ph}
    for (int c = 0; c < 3; c++) {
        dR[c] += qv[c] * Ti;
        for (int v = 0; v < 3; v++) dA[v * 3 + c] -= qv[c] * rho[v] * Ti;
    }
    if (spp > 1) {
        double* xw = reinterpret_cast<double*>(Fs);
        __syncthreads();
        P = per_slot_sum<W>(P, lpp, spp, xw);
        P0 = per_slot_sum<W>(P0, lpp, spp, xw);
        for (int c = 0; c < 3; c++) dR[c] = per_slot_sum<W>(dR[c], lpp, spp, xw);
        for (int k = 0; k < 9; k++) dA[k] = per_slot_sum<W>(dA[k], lpp, spp, xw);
    }
    if (i == j) {
        const double self = 4.0 * S.gamma * S.gamma * S.gamma / (3.0 * SQRT_PI);
        P -= self * trr;
    }
    if (!qv_ok || sub != 0) return;
    out[0] = P;
    for (int c = 0; c < 3; c++) out[1 + c] = dR[c];
    for (int k = 0; k < 9; k++) out[4 + k] = dA[k];
    out[13] = P0;
}

// Reciprocal term of the adjoint, W = M C U: M(q) the full embedded inverse
// square root (2n x 2n), C U the basis; W (2n x ncol) is [Re; Im] of the complex
// product.  32 x 32 tiles, K split over two wavefronts, runs of tiles of one q
// point on an XCD; matrix-core bound (64 q points of 64 atoms: 135 us, 202
// through staged 64 x 64 tiles).
__global__ __launch_bounds__(128) void per_recip_mz_kernel(MatBatch<double> M, PerEwald pr, int n2, int tiles_m, int tiles) {
    typedef SplitK<2, 2, 2, 6> SK;
    constexpr int TM = SK::TM, TN = SK::TN, LDC = SK::LDC;
    __shared__ __align__(16) double cs[SK::LDS];
    const int v = xcd_virtual(blockIdx.x, gridDim.x), q = v / tiles, t = v % tiles;
    const int m0 = t % tiles_m * TM, g0 = t / tiles_m * TN;
    {
        SK sk;
        sk.clear();
        const double* Z = pr.Z + (long long)q * pr.sZ + (long long)g0 * pr.ldz;
        sk.run_cols(M.at(q), m0, M.ld, Z, pr.ldz, min(TN, pr.ncol - g0), n2);
        sk.reduce<true>(cs);
    }
    double* W = pr.W + (long long)q * pr.sZ + (long long)g0 * pr.ldz + m0;
#pragma unroll
    for (int x = threadIdx.x; x < TM * TN; x += SK::NT) {
        const int r = x % TM, c = x / TM;
        if (m0 + r < n2 && g0 + c < pr.ncol) W[r + (long long)c * pr.ldz] = cs[c * LDC + r] + cs[(TN + c) * LDC + r];
    }
}

// Reciprocal term of the adjoint, per atom k and column g (k = G + q,
// u = U_{k., g}, z = c_k sum_a conj(u_a) W_{ka, g}):
//   dE/dalpha, dE/domega partial  2 Re z (the pair sum over both orders)
//   dE/dR_k                        -2 G Im z
//   dE/dA_vc  -Ainv_cv s - sum_d Ainv_dv [k_c k_d f s + 2 sw k_c b_d
//             + G_c sum_k R_kd e_k], s = sum_k Re z, e_k = -2 Im z,
//             b_d = sum_k c_k Re(conj(W_{kd,g}) e^{-i G.R_k})
// (derivatives of the weight w, of k and of the pair phase through G with
// the fractional q fixed, and of the prefactor through Omega).  Grid (nq,
// chunks of PER_RCOLS columns); writes per (q, chunk, atom) {2 Re z, dR[3]}
// and per (q, chunk) {s, L[c][d]}, L the bracket's matrix without Ainv.
#define PER_RCOLS 16
__global__ __launch_bounds__(64) void per_recip_grad_kernel(const SysDesc* sd, const double* cc, const double* qcart,
                                                            PerEwald pr, int nchunk, double* rq, double* rl) {
    const SysDesc& S = sd[0];
    const int N = S.N, n = 3 * N;
    const int q = blockIdx.x, ch = blockIdx.y;
    const double* Wq = pr.W + (long long)q * pr.sZ;
    const int* cols = pr.col + (long long)q * pr.ncol;
    const double* qv = qcart + 3 * q;
    const double* R = S.coords;
    const int g0 = ch * PER_RCOLS, g1 = min(pr.ncol, g0 + PER_RCOLS);
    double sre = 0.0, L[9];
    for (int v = 0; v < 9; v++) L[v] = 0.0;
    for (int k = threadIdx.x; k < N; k += 64) {
        const double ck = cc[S.atom_off + k];
        const double Rk[3] = {R[3 * k], R[3 * k + 1], R[3 * k + 2]};
        double ga = 0.0, gr[3] = {0.0, 0.0, 0.0};
        for (int g = g0; g < g1; g++) {
            const int t = cols[g];
            if (t < 0) break;
            double G[3], kv[3], sw, f;
            recip_column(S, pr.rec, t, qv, G, kv, sw, f);
            double sn, cs;
            sincos(G[0] * Rk[0] + G[1] * Rk[1] + G[2] * Rk[2], &sn, &cs);
            const double pr_ = cs, pi_ = -sn;  // e^{-i G.R_k}
            double zr = 0.0, zi = 0.0, bd[3];
            for (int a = 0; a < 3; a++) {
                const double wr = Wq[3 * k + a + (long long)g * pr.ldz];
                const double wi = Wq[n + 3 * k + a + (long long)g * pr.ldz];
                const double ur = sw * kv[a] * pr_, ui = sw * kv[a] * pi_;
                zr += ur * wr + ui * wi;
                zi += ur * wi - ui * wr;
                bd[a] = ck * (wr * pr_ + wi * pi_);
            }
            zr *= ck;
            zi *= ck;
            const double e = -2.0 * zi;
            ga += 2.0 * zr;
            for (int c = 0; c < 3; c++) gr[c] += G[c] * e;
            sre += zr;
            for (int c = 0; c < 3; c++)
                for (int d = 0; d < 3; d++)
                    L[c * 3 + d] += f * zr * kv[c] * kv[d] + 2.0 * sw * kv[c] * bd[d] + e * G[c] * Rk[d];
        }
        double* o = rq + (((long long)q * nchunk + ch) * N + k) * 4;
        o[0] = ga;
        for (int c = 0; c < 3; c++) o[1 + c] = gr[c];
    }
    sre = wave_sum(sre);
    for (int v = 0; v < 9; v++) L[v] = wave_sum(L[v]);
    if (threadIdx.x == 0) {
        double* o = rl + ((long long)q * nchunk + ch) * 10;
        o[0] = sre;
        for (int v = 0; v < 9; v++) o[1 + v] = L[v];
    }
}

// Per-atom reduction in a fixed order: the pair partials (k as either atom)
// over all q, the reciprocal partials of every (q, chunk), and the lattice
// partials of the pairs of k, to latpart[k].
__global__ __launch_bounds__(256) void mbd_grad_periodic_reduce_kernel(const SysDesc* sd, int nq, const double* qmult,
                                                                         double wq, const double* om,
                                                                         const double* cc, const double* part,
                                                                         MatBatch<double> M, const double* rq,
                                                                         int nchunk, double* latpart) {
    __shared__ double red[4];
    const SysDesc& S = sd[0];
    const int N = S.N;
    if (N == 0) return;
    const int k = blockIdx.x;
    double g0 = 0, g1 = 0, g2 = 0, ga = 0, gv = 0, tr = 0, la[9];
    for (int v = 0; v < 9; v++) la[v] = 0.0;
    const long long NP = (long long)N * (N + 1) / 2;
    for (long long idx = threadIdx.x; idx < (long long)nq * N; idx += 256) {
        const int q = (int)(idx / N), o = (int)(idx % N);
        // the pair of k and o, i <= j; both orders contribute the same to dR_k
        // (with the sign of k's place), P and P0, and to dA
        const int i = min(o, k), j = max(o, k);
        const double* pp = part + ((long long)q * NP + (long long)j * (j + 1) / 2 + i) * PER_PART;
        const double cj = qmult[q] * cc[S.atom_off + o] * cc[S.atom_off + k];
        if (o != k) {
            const double sg = k == j ? 2.0 * cj : -2.0 * cj;
            g0 += sg * pp[1];
            g1 += sg * pp[2];
            g2 += sg * pp[3];
        }
        ga += 2.0 * cj * pp[0];
        gv += 2.0 * cj * pp[13];
        // each pair once over its two orders: half of it at either atom
        for (int v = 0; v < 9; v++) la[v] += cj * pp[4 + v];
    }
    for (long long idx = threadIdx.x; idx < (long long)nq * nchunk; idx += 256) {
        const double w = qmult[idx / nchunk];
        const double* r = rq + (idx * N + k) * 4;
        ga += w * r[0];
        g0 += w * r[1];
        g1 += w * r[2];
        g2 += w * r[3];
    }
    // Re Tr M_kk(q), summed over q
    for (int q = threadIdx.x; q < nq; q += 256) {
        const double* Mb = M.at(q);
        for (int c = 0; c < 3; c++) tr += qmult[q] * Mb[(3 * k + c) + (long long)(3 * k + c) * M.ld];
    }
    g0 = block_sum256(g0, red);
    g1 = block_sum256(g1, red);
    g2 = block_sum256(g2, red);
    ga = block_sum256(ga, red);
    gv = block_sum256(gv, red);
    tr = block_sum256(tr, red);
    for (int v = 0; v < 9; v++) la[v] = block_sum256(la[v], red);
    if (threadIdx.x == 0) {
        for (int v = 0; v < 9; v++) latpart[9 * k + v] = la[v];
        if (S.grad_coords) {
            S.grad_coords[3 * k] = wq * g0;
            S.grad_coords[3 * k + 1] = wq * g1;
            S.grad_coords[3 * k + 2] = wq * g2;
        }
        const double a0 = S.alpha0[k];
        const double w = om[S.atom_off + k];
        const double dEda = wq * ga / (2.0 * a0);
        const double dEdw = wq * ga / w + wq * 2.0 * w * tr - 1.5;
        if (S.param_kind == 1) {
            // omega = 4 C6/(3 alpha0^2)
            if (S.grad_alpha0) S.grad_alpha0[k] = dEda - 2.0 * w / a0 * dEdw;
            if (S.grad_omega) S.grad_omega[k] = dEdw * w / S.omega_or_c6[k];
        } else {
            if (S.grad_alpha0) S.grad_alpha0[k] = dEda;
            if (S.grad_omega) S.grad_omega[k] = dEdw;
        }
        if (S.grad_rvdw) S.grad_rvdw[k] = wq * S.beta * gv;
    }
}

// dE/dA: the per-atom pair partials and the reciprocal (q, chunk) partials,
// each summed in a fixed order, the latter contracted with Ainv once.
__global__ __launch_bounds__(256) void mbd_grad_periodic_lattice_kernel(const SysDesc* sd, int nq, int nchunk,
                                                                          const double* qmult, double wq,
                                                                          const double* latpart, const double* rl) {
    __shared__ double red[4];
    const SysDesc& S = sd[0];
    const int N = S.N;
    double la[9], r[10];
    for (int v = 0; v < 9; v++) la[v] = 0.0;
    for (int v = 0; v < 10; v++) r[v] = 0.0;
    for (int k = threadIdx.x; k < N; k += 256)
        for (int v = 0; v < 9; v++) la[v] += latpart[9 * k + v];
    for (long long idx = threadIdx.x; idx < (long long)nq * nchunk; idx += 256) {
        const double w = qmult[idx / nchunk];
        for (int v = 0; v < 10; v++) r[v] += w * rl[idx * 10 + v];
    }
    for (int v = 0; v < 9; v++) la[v] = block_sum256(la[v], red);
    for (int v = 0; v < 10; v++) r[v] = block_sum256(r[v], red);
    if (threadIdx.x != 0 || !S.grad_lattice) return;
    // linv[d * 3 + v] = Ainv[d][v]
    for (int v = 0; v < 3; v++)
        for (int c = 0; c < 3; c++) {
            double t = -S.linv[c * 3 + v] * r[0];
            for (int d = 0; d < 3; d++) t -= S.linv[d * 3 + v] * r[1 + c * 3 + d];
            S.grad_lattice[v * 3 + c] = wq * (la[v * 3 + c] + t);
        }
}

// lanes per atom pair: the q count rounded up to a power of two, at most 64
static int per_lanes_per_pair(int nq) {
    int l = 1;
    while (l < nq && l < PER_LANES) l *= 2;
    return l;
}

// Wavefronts per workgroup and slots per pair: pairs are split over their
// images until the launch has two wavefronts per SIMD (2048), but a slot keeps
// at least two rounds of lpp images; first within a wavefront, then over the
// four of a workgroup.
static void per_split(long long pairs, int nq, int lpp, int nimg, int& waves, int& spp) {
    waves = spp = 1;
    const long long groups = (nq + lpp - 1) / lpp;
    auto more = [&]() { return pairs * groups * lpp * spp / PER_LANES < 2048 && 4LL * lpp * spp <= nimg; };
    while (spp < PER_LANES / lpp && more()) spp *= 2;
    while (spp >= PER_LANES / lpp && spp < 4 * PER_LANES / lpp && more()) {
        spp *= 2;
        waves = 4;
    }
}

void per_recip_basis_launch(hipStream_t st, const SysDesc* sd, const double* cc, const double* qcart, int nq,
                            const int* img, int nimg, const PerEwald& pr) {
    if (nq == 0) return;
    if (nimg > 0)
        hipLaunchKernelGGL(per_phase_kernel, dim3((unsigned)(((long long)nimg * nq + 255) / 256)), dim3(256), 0, st,
                           sd, qcart, nq, img, nimg, pr.phase);
    if (pr.ncol == 0) return;
    hipLaunchKernelGGL(per_recip_basis_kernel, dim3(pr.ncol, nq), dim3(64), 0, st, sd, cc, qcart, pr);
}

void mbd_assemble_periodic_launch(hipStream_t st, const SysDesc* sd, const double* om, const double* cc,
                                  const double* qcart, int nq, const int* img, int nimg, const PerEwald& pr,
                                  MatBatch<double> Q, MatBatch<float> Q32, unsigned* status, int N) {
    const long long pairs = per_pairs(N);
    const int lpp = per_lanes_per_pair(nq);
    int wv, spp;
    per_split(pairs, nq, lpp, nimg, wv, spp);
    const int ppw = PER_LANES * wv / lpp / spp;
    auto go = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3((unsigned)((pairs + ppw - 1) / ppw), (nq + lpp - 1) / lpp), dim3(PER_LANES * wv), 0,
                           st, sd, om, cc, qcart, nq, lpp, spp, img, nimg, pr.phase, Q, status);
    };
    if (wv == 1) go(mbd_assemble_periodic_kernel<1>);
    else go(mbd_assemble_periodic_kernel<4>);
    // always launched: besides the reciprocal term, the epilogue fills the
    // right block column and the FP32 copy
    hipLaunchKernelGGL((per_recip_asm_kernel<2, 2, 2, 4>), dim3(splitk_lower_tiles(3 * N, 32, 32), 2, nq), dim3(128), 0, st,
                       pr, 3 * N, Q, Q32);
}

int per_recip_chunks(int ncol) { return (ncol + PER_RCOLS - 1) / PER_RCOLS; }

void mbd_grad_periodic_launch(hipStream_t st, const SysDesc* sd, const double* om, const double* cc,
                              const double* qcart, const double* qmult, double wq, int nq, const int* img,
                              int nimg, const PerEwald& pr, MatBatch<double> M, double* partial, double* rq,
                              double* rl, double* latpart, int N) {
    const long long pairs = per_pairs(N);
    const int lpp = per_lanes_per_pair(nq);
    int wv, spp;
    per_split(pairs, nq, lpp, nimg, wv, spp);
    const int ppw = PER_LANES * wv / lpp / spp;
    auto go = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3((unsigned)((pairs + ppw - 1) / ppw), (nq + lpp - 1) / lpp), dim3(PER_LANES * wv), 0,
                           st, sd, om, cc, qcart, nq, lpp, spp, img, nimg, pr.phase, M, partial);
    };
    if (wv == 1) go(mbd_grad_periodic_kernel<1>);
    else go(mbd_grad_periodic_kernel<4>);
    const int nchunk = per_recip_chunks(pr.ncol);
    if (nchunk > 0) {
        const int tiles_m = (6 * N + 31) / 32, tiles = tiles_m * ((pr.ncol + 31) / 32);
        hipLaunchKernelGGL(per_recip_mz_kernel, dim3(tiles * nq), dim3(128), 0, st, M, pr, 6 * N, tiles_m, tiles);
        hipLaunchKernelGGL(per_recip_grad_kernel, dim3(nq, nchunk), dim3(64), 0, st, sd, cc, qcart, pr, nchunk, rq,
                           rl);
    }
    hipLaunchKernelGGL(mbd_grad_periodic_reduce_kernel, dim3(N), dim3(256), 0, st, sd, nq, qmult, wq, om, cc,
                       partial, M, rq, nchunk, latpart);
    hipLaunchKernelGGL(mbd_grad_periodic_lattice_kernel, dim3(1), dim3(256), 0, st, sd, nq, nchunk, qmult, wq,
                       latpart, rl);
}
