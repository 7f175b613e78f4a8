// Symmetric products of the direct root on the INT8 matrix cores, for large
// matrices: C = A B by residues (the modular scheme of Ozaki, Uchino & Imamura,
// "Ozaki scheme II", 2025).  A and B are scaled by powers of two to norms
// of at most 2^p (the plan follows a bound of each matrix's norm) and rounded
// to integers a', b'; x_ij = sum_k a'_ik b'_jk, at most the product of two rows'
// norms, |x| <= 2^2p, is an integer that its residues modulo pairwise coprime
// m_1 .. m_s (256 and the largest below 236) determine once their product M
// exceeds 2^(2p+1).  So C is formed from s exact INT8 products with 32-bit
// sums, and
//   x / M = frac(sum_i r_i theta_i),  theta_i = ((M / m_i)^-1 mod m_i) / m_i,
// with theta_i split into a multiple of 2^-42 (its sum is exact in FP64) and a
// remainder.  The only errors are the roundings of a' and b', 2^-(p+1) of the
// norm each, and those of the result.  s = 15, p = 57, serves FP64: an element 16
// times below the norm keeps 53 bits, and gradients at order 2700 and 6000 are
// 6.0e-15 and 7.1e-15 from 64-bit ones, 6.5e-15 and 8.4e-15 with FP64 products
// (each sum rounds n times), 7.3e-15 and 8.7e-15 by diagonalisation; s = 14, p =
// 53, left 1.9e-14 and 2.1e-14, since small elements lost bits that an FP64 one
// has.  s = 12, p = 46, serves the FP32-with-refinement precision.
//
// Three launches a product: residues of the operands that are not already held
// (the plan tracks which two are), the s integer products, and the combination
// with the epilogue of the FP64 product kernel.  Residues are laid out in the
// order of the matrix instructions' operands (blocks of 32 rows x 32 columns, 1
// KB, lane after lane), so every load is a whole line.
//
// At order 6000 and s = 15 (12) the integer products take 1.91 (1.57) ms, 1.7
// PetaOP/s (2.4 with neither loads nor LDS, the rate that the card holds), the
// conversion of an operand 0.18 (0.13) and the combination 0.18 (0.16); the FP64
// product takes 3.4 ms.
#include <hip/hip_ext.h>

#include "gemm_mfma.h"
#include "mbd_internal.h"
#include "mbd_isqrt.h"

#define MM_TB 8      // blocks of 32 per tile side
#define MM_USPLIT 42  // bits of theta in its leading part

typedef int mm_i4 __attribute__((ext_vector_type(4)));
typedef int mm_i16 __attribute__((ext_vector_type(16)));

// 256 and coprime numbers up to 236: a residue of a number below 2^53 that missed
// its centre by the rounding of a quotient (at most 4) still fits eight bits
__device__ __constant__ const int MM_MOD[ISQ_MODS_MAX] = {256, 235, 233, 229, 227, 223, 221, 217, 213, 211, 209, 199, 197, 193, 191};
static const int MM_MOD_HOST[ISQ_MODS_MAX] = {256, 235, 233, 229, 227, 223, 221, 217, 213, 211, 209, 199, 197, 193, 191};

struct ModCoef {
    double u[ISQ_MODS_MAX], v[ISQ_MODS_MAX], M;
};

static ModCoef mod_coef(int mods) {
    ModCoef c = {};
    long double M = 1.0L;
    for (int i = 0; i < mods; i++) {
        const int m = MM_MOD_HOST[i];
        M *= m;
        long long w = 1;
        for (int j = 0; j < mods; j++)
            if (j != i) w = w * MM_MOD_HOST[j] % m;
        long long inv = 1;
        while (w * inv % m != 1) inv++;
        if (2 * inv > m) inv -= m;
        const long long num = inv * (1LL << MM_USPLIT);
        const long long q = (num >= 0 ? num + m / 2 : num - m / 2) / m;
        c.u[i] = (double)q / (double)(1LL << MM_USPLIT);
        c.v[i] = (double)(num - q * m) / ((double)m * (double)(1LL << MM_USPLIT));
    }
    c.M = (double)M;
    return c;
}

// Residues of one 32 x 32 block per wavefront: lane l holds row l mod 32,
// columns 16 (l / 32) .. + 15.  Bound by HBM (order 6000: 288 MB read, 432 or 504
// written) where consecutive lanes read consecutive addresses: 156 us an operand
// with 12 moduli, against 267 with 16 columns of a row, 128 B, to each lane.
template <int MODS>
__global__ __launch_bounds__(256) void mod_split_kernel(IsqBufs bufs, const int* ns, const IsqOp* ops, int step, IsqMod w) {
    const int b = blockIdx.z >> 1, which = blockIdx.z & 1, lane = threadIdx.x & 63;
    const IsqOp& op = ops[(long long)b * ISQ_OPS + step];
    if (op.a < 0 || !(op.conv >> which & 1)) return;
    const int kb = blockIdx.x * 4 + (threadIdx.x >> 6), rb = blockIdx.y, n = ns[b];
    if (kb >= w.kb) return;
    const int slot = which ? op.sb : op.sa, row = rb * 32 + (lane & 31), k0 = kb * 32 + 16 * (lane >> 5);
    // the operand is symmetric: element (row, k0 + i) from column k0 + i
    const double* a = bufs.p[which ? op.b : op.a] + (long long)b * bufs.stride + row + (long long)k0 * bufs.ld;
    const int sh = w.bits - (which ? op.eb : op.ea);
    double t[16];
#pragma unroll
    for (int i = 0; i < 16; i++) t[i] = row < n && k0 + i < n ? a[(long long)i * bufs.ld] : 0.0;
#pragma unroll
    for (int i = 0; i < 16; i++) t[i] = rint(scalbn(t[i], sh));
    const long long sm = (long long)w.nb * w.kb * 64;
    mm_i4* out = w.res + (((long long)b * 2 + slot) * MODS) * sm + ((long long)rb * w.kb + kb) * 64 + lane;
#pragma unroll
    for (int m = 0; m < MODS; m++) {
        const double p = MM_MOD[m], ip = 1.0 / p;
        mm_i4 o;
#pragma unroll
        for (int q = 0; q < 4; q++) {
            unsigned pk = 0;
#pragma unroll
            for (int e = 0; e < 4; e++) {
                double x = t[4 * q + e];
                x = fma(-p, rint(x * ip), x);
                if (MODS == ISQ_MODS_MAX) x = fma(-p, rint(x * ip), x);  // 2^57: the quotient may be one off
                pk |= ((unsigned)(int)x & 255u) << (8 * e);
            }
            o[q] = (int)pk;
        }
        out[m * sm] = o;
    }
}

// One 256 x 256 tile of one residue product per workgroup, each wavefront 128 x
// 128 in 16 accumulators; K steps of 64 staged through three LDS buffers (two
// steps ahead of the products, so neither the loads nor the first operands of a
// step are waited for).  Each XCD gets a run of (residue, banded tile) indices.
__global__ __launch_bounds__(256, 1) void mod_prod_kernel(const int* ns, const IsqOp* ops, int step, IsqMod w, int mods,
                                                            int tiles) {
    constexpr int KS = 2;
    __shared__ mm_i4 S[3][16 * KS][64];
    const int b = blockIdx.z, tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const IsqOp& op = ops[(long long)b * ISQ_OPS + step];
    if (op.a < 0) return;
    const int v = xcd_virtual(blockIdx.x, gridDim.x), mod = v / tiles, t = v % tiles;
    int ti, tj;
    band_lower_tile(t, w.nb / MM_TB, ti, tj);
    const int n = ns[b];
    if (ti * 32 * MM_TB >= n) return;
    const long long sm = (long long)w.nb * w.kb * 64;
    const mm_i4* A = w.res + (((long long)b * 2 + op.sa) * mods + mod) * sm + (long long)ti * MM_TB * w.kb * 64 + lane;
    const mm_i4* B = w.res + (((long long)b * 2 + op.sb) * mods + mod) * sm + (long long)tj * MM_TB * w.kb * 64 + lane;
    const int wm = wv & 1, wn = wv >> 1;
    mm_i16 acc[4][4];
#pragma unroll
    for (int i = 0; i < 4; i++)
#pragma unroll
        for (int j = 0; j < 4; j++) acc[i][j] = mm_i16{0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
    mm_i4 st0[4 * KS], st1[4 * KS], a0[4], b0[4], a1[4], b1[4];
    // slot s of a step: block s mod 16 (eight of A, eight of B) of its column block s / 16
    auto gload = [&](int kb, mm_i4 (&st)[4 * KS]) {
#pragma unroll
        for (int u = 0; u < 4 * KS; u++) {
            const int s = wv + 4 * u, blk = s & 15;
            const mm_i4* p = blk < MM_TB ? A + (long long)blk * w.kb * 64 : B + (long long)(blk - MM_TB) * w.kb * 64;
            st[u] = p[(kb + (s >> 4)) * 64];
        }
    };
    auto sstore = [&](int buf, const mm_i4 (&st)[4 * KS]) {
#pragma unroll
        for (int u = 0; u < 4 * KS; u++) S[buf][wv + 4 * u][lane] = st[u];
    };
    auto frag = [&](int buf, int k, mm_i4 (&a)[4], mm_i4 (&bb)[4]) {
#pragma unroll
        for (int i = 0; i < 4; i++) {
            a[i] = S[buf][16 * k + 4 * wm + i][lane];
            bb[i] = S[buf][16 * k + 8 + 4 * wn + i][lane];
        }
    };
    auto mult = [&](const mm_i4 (&a)[4], const mm_i4 (&bb)[4]) {
#pragma unroll
        for (int i = 0; i < 4; i++)
#pragma unroll
            for (int j = 0; j < 4; j++) acc[i][j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(a[i], bb[j], acc[i][j], 0, 0, 0);
    };
    const int nst = (n + 127) / 128 * 2;  // an even number of steps: the blocks past n hold zeros
    gload(0, st0);
    gload(KS, st1);
    sstore(0, st0);
    sstore(1, st1);
    if (nst > 2) gload(2 * KS, st0);
    __syncthreads();
    frag(0, 0, a0, b0);
    int cur = 0, nxt = 1, aft = 2;
    // one step: loads three ahead, LDS stores (of the loads made a step ago) two ahead
    auto kstep = [&](int s, mm_i4 (&in)[4 * KS], const mm_i4 (&have)[4 * KS]) {
        if (s + 3 < nst) gload((s + 3) * KS, in);
        frag(cur, 1, a1, b1);
        __builtin_amdgcn_sched_barrier(0);
        mult(a0, b0);
        __builtin_amdgcn_sched_barrier(0);
        frag(nxt, 0, a0, b0);  // past the last step: not used
        __builtin_amdgcn_sched_barrier(0);
        mult(a1, b1);
        __builtin_amdgcn_sched_barrier(0);
        if (s + 2 < nst) sstore(aft, have);
        __syncthreads();
        const int o = cur;
        cur = nxt;
        nxt = aft;
        aft = o;
    };
    for (int s = 0; s < nst; s += 2) {
        kstep(s, st1, st0);
        kstep(s + 1, st0, st1);
    }
    // the sums to residues (x / m from the high word of x (2^38 / m), rounded), 16 bytes a lane and block
    const int m = MM_MOD[mod], magic = (int)((1LL << 38) / m + 1);
    mm_i4* C = w.prod + (((long long)b * mods + mod) * tiles + t) * 4096 + lane;
#pragma unroll
    for (int i = 0; i < 4; i++)
#pragma unroll
        for (int j = 0; j < 4; j++) {
            mm_i4 o;
#pragma unroll
            for (int q = 0; q < 4; q++) {
                unsigned pk = 0;
#pragma unroll
                for (int e = 0; e < 4; e++) {
                    const int x = acc[i][j][4 * q + e];
                    pk |= (unsigned)((x - ((__mulhi(x, magic) + 32) >> 6) * m) & 255) << (8 * e);
                }
                o[q] = (int)pk;
            }
            C[((4 * wm + i) * MM_TB + 4 * wn + j) * 64] = o;
        }
}

// The products from their residues, and the step's two outputs as
// isq_prod_kernel writes them: one 32 x 32 block of the lower triangle per
// wavefront; lane l holds its column l mod 32, rows 8 q + 4 (l / 32) + e.
// Bound by HBM (order 6000, 12 moduli: 216 MB read, 288 written, more with
// epilogue matrices and a second output); the lower triangle is stored from a
// transposed copy in LDS, 256 B to 32 lanes: 142 us against 176 with 32 B
// segments straight from the registers.
template <int MODS>
__global__ __launch_bounds__(256) void mod_combine_kernel(IsqBufs bufs, const int* ns, const IsqOp* ops, int step,
                                                            IsqMod w, ModCoef cf, int tiles) {
    __shared__ double tr[4][32 * 33];
    const int b = blockIdx.z, lane = threadIdx.x & 63;
    double* T = tr[threadIdx.x >> 6];
    const IsqOp& op = ops[(long long)b * ISQ_OPS + step];
    if (op.a < 0) return;
    const int t = blockIdx.x / 16, s = (blockIdx.x % 16) * 4 + (threadIdx.x >> 6), n = ns[b], ld = bufs.ld;
    int ti, tj;
    band_lower_tile(t, w.nb / MM_TB, ti, tj);
    const int bi = ti * MM_TB + s / MM_TB, bj = tj * MM_TB + s % MM_TB;
    if (bj > bi || 32 * bi >= n) return;
    const mm_i4* P = w.prod + ((long long)b * MODS * tiles + t) * 4096 + s * 64 + lane;
    mm_i4 r[MODS];
#pragma unroll
    for (int m = 0; m < MODS; m++) r[m] = P[(long long)m * tiles * 4096];
    const double* E1 = op.e1 >= 0 ? bufs.p[op.e1] + (long long)b * bufs.stride : nullptr;
    const double* E2 = op.e2 >= 0 ? bufs.p[op.e2] + (long long)b * bufs.stride : nullptr;
    double* C1 = bufs.p[op.out] + (long long)b * bufs.stride;
    double* C2 = op.out2 >= 0 ? bufs.p[op.out2] + (long long)b * bufs.stride : nullptr;
    const int col = 32 * bj + (lane & 31);
    const double scale = scalbn(cf.M, op.ea + op.eb - 2 * w.bits);
    double o2[16];
#pragma unroll
    for (int q = 0; q < 4; q++) {
#pragma unroll
        for (int e = 0; e < 4; e++) {
            const int rr = 8 * q + 4 * (lane >> 5) + e, row = 32 * bi + rr;
            double s1 = 0.0, s2 = 0.0;
#pragma unroll
            for (int m = 0; m < MODS; m++) {
                const double x = (double)((r[m][q] << (24 - 8 * e)) >> 24);
                s1 = fma(x, cf.u[m], s1);
                s2 = fma(x, cf.v[m], s2);
            }
            const double f = ((s1 - rint(s1)) + s2) * scale;
            // the symmetric epilogue matrices at (col, row): consecutive lanes, consecutive addresses
            const bool in = row < n && col < n && row >= col;
            const long long at = col + (long long)row * ld;
            const double e1 = E1 && in ? E1[at] : 0.0, e2 = E2 && in ? E2[at] : 0.0, id = row == col ? 1.0 : 0.0;
            const double o1 = op.c[0] * f + op.c[1] * e1 + op.c[2] * e2 + op.c[3] * id;
            o2[4 * q + e] = op.d[0] * f + op.d[1] * e1 + op.d[2] * e2 + op.d[3] * id;
            if (in) {
                C1[at] = o1;
                if (C2) C2[at] = o2[4 * q + e];
            }
            T[(lane & 31) * 33 + rr] = o1;
        }
    }
    // the other triangle from the transposed block, in runs along the rows
    const int row = 32 * bi + (lane & 31);
    auto mirror = [&](double* C) {
        isq_wave_sync();
#pragma unroll
        for (int i = 0; i < 16; i++) {
            const int cc = 2 * i + (lane >> 5);
            if (row < n && row > 32 * bj + cc) C[row + (long long)(32 * bj + cc) * ld] = T[cc * 33 + (lane & 31)];
        }
        isq_wave_sync();
    };
    mirror(C1);
    if (!C2) return;
#pragma unroll
    for (int i = 0; i < 16; i++) T[(lane & 31) * 33 + 8 * (i / 4) + 4 * (lane >> 5) + i % 4] = o2[i];
    mirror(C2);
}

// Large orders only: conversions and combination grow with n^2, and 256 x 256
// tiles waste their edges.  One matrix of order 2202, 2256, 2304, 2400, 2550, 2700,
// 3000, 3600, 5100 with 15 moduli: 2.67, 2.70, 2.72, 3.36, 3.51, 3.88, 4.77, 7.88,
// 17.0 ms an evaluation, with FP64 products 2.54, 2.89, 3.00, 3.15, 3.73, 4.40, 5.46,
// 8.98, 24.0; with 12 moduli at 2112, 2124, 2160, 2199: 2.29, 2.29, 2.29, 2.39 against
// 2.24, 2.43, 2.42, 2.50, and 2.58, 3.66, 5.81, 12.3 at 2550, 3000, 3600, 5100.  Embedded
// (periodic) matrices never are that large.
bool isq_mod_fits(const int* ns_host, int nmat, bool embed, int mods) {
    if (embed) return false;
    for (int b = 0; b < nmat; b++)
        if (ns_host[b] < (mods == ISQ_MODS_MAX ? 2470 : 2128)) return false;
    return true;
}

void isq_mod_sizes(int nmax, int mods, IsqMod& w, size_t& res, size_t& prod) {
    const int nt = (nmax + 32 * MM_TB - 1) / (32 * MM_TB), tiles = nt * (nt + 1) / 2;
    w.mods = mods;
    // 2p + 1 bits below the moduli's product: 2^116.3 (15), 2^93.5 (12)
    w.bits = mods == ISQ_MODS_MAX ? 57 : 46;
    w.nb = nt * MM_TB;
    w.kb = (nmax + 127) / 128 * 4;
    res = (size_t)2 * mods * w.nb * w.kb * 1024;
    prod = (size_t)mods * tiles * 65536;
}

template <int MODS>
static void mod_launch(hipStream_t st, const IsqWork& w, int nmat, int step, hipEvent_t e0, hipEvent_t e1) {
    static const ModCoef cf = mod_coef(MODS);
    const int nt = w.mod.nb / MM_TB, tiles = nt * (nt + 1) / 2;
    hipLaunchKernelGGL(mod_split_kernel<MODS>, dim3((w.mod.kb + 3) / 4, w.mod.nb, 2 * nmat), dim3(256), 0, st, w.bufs,
                       w.ns, w.ops, step, w.mod);
    hipExtLaunchKernelGGL(mod_prod_kernel, dim3(tiles * MODS, 1, nmat), dim3(256), 0, st, e0, e1, 0, w.ns, w.ops, step,
                          w.mod, MODS, tiles);
    hipLaunchKernelGGL(mod_combine_kernel<MODS>, dim3(tiles * 16, 1, nmat), dim3(256), 0, st, w.bufs, w.ns, w.ops, step,
                       w.mod, cf, tiles);
}

void isq_mod_launch(hipStream_t st, const IsqWork& w, int nmat, int step, hipEvent_t e0, hipEvent_t e1) {
    if (w.mod.mods == ISQ_MODS_MAX) mod_launch<ISQ_MODS_MAX>(st, w, nmat, step, e0, e1);
    else mod_launch<ISQ_MODS_SHORT>(st, w, nmat, step, e0, e1);
}
