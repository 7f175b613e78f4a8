// Workspaces and launches of the direct inverse square root (k_isqrt.hip).
#pragma once
#include "isq_table.h"
#include "mbd_internal.h"
#include "mbd_sys.h"

#define ISQ_SQUARES 6      // most squarings of Q^{-1/2} before the Lanczos run for lambda_min
#define ISQ_OPS (ISQ_OPMAX + ISQ_SQUARES)
#define ISQ_NBUF 8         // matrix buffers, buffer 0 = Q
#define ISQ_RESULT 7       // buffer that receives Q^{-1/2}
#define ISQ_MVR 8          // rows per workgroup of a matrix-vector pass
#define ISQ_LMAX 128       // most Lanczos steps
#define ISQ_SMALL 256      // largest order whose Lanczos steps run in one workgroup
#define ISQ_STEPS_SMALL 10 // Lanczos steps for the interval, orders below 1024
#define ISQ_STEPS_LARGE 14 // and from 1024 on
// The smallest Ritz value overstates lambda_min by up to 1.4 after 10 steps
// (orders up to 900) and 1.9 after 14 (order 6000), and the largest plus its
// residual norm falls up to 2.4% short of lambda_max (clusters, both densities);
// twice the residual and 6% on top left none of 12 288 molecules of 10 to 300
// atoms to the eigensolver, 4% left five.
#define ISQ_LOW_FRACTION 0.5
#define ISQ_CHECK 1e-12    // largest accepted |I - Z Q Z|_F / sqrt(n)
#define ISQ_CHECK_SHORT 1e-10  // with the shorter residue products

const IsqTable& isq_table(bool wide);

struct IsqOp {
    signed char a, b, e1, e2, out, out2;
    signed char full;  // the last product: an embedding is written whole
    signed char sa, sb, conv;  // residue products: slots of a and b, bits: a, b to convert first
    int ea, eb;        // their norms are below 2^ea, 2^eb
    double c[4], d[4];
};
struct IsqBufs {
    double* p[ISQ_NBUF];
    int ld;
    long long stride;
};
struct IsqLanczos {
    double* vec;    // [nmat][4][sV]: two vectors v and two w
    long long sV;
    double* part;   // [nmat][2][nwg][2]
    int nwg;
    bool emb;       // embeddings: half the rows' workgroups
    int one;        // matrices up to this order have all their steps in one workgroup
    double* alpha;  // [nmat][ISQ_LMAX]
    double* beta;
    int* len;       // order at which the recurrence ended, 0: it has not
    int* done;      // matrices that need no further step (nullptr: all run)
};
// Residue products (k_modmul.hip): 15 moduli for FP64, 12 for FP32 with
// refinement
#define ISQ_MODS_MAX 15
#define ISQ_MODS_SHORT 12
typedef int isq_i4 __attribute__((ext_vector_type(4)));
struct IsqMod {
    int mods = 0;   // 0: FP64 products
    int bits;       // p: operands scaled to a norm of 2^p
    int nb, kb;     // 32-row and 32-column blocks
    isq_i4* res;    // [nmat][2 slots][mods][nb][kb][64]
    isq_i4* prod;   // [nmat][mods][tiles][64 blocks][64]
};
struct IsqWork {
    const int* ns;
    const SysDesc* sd;  // of the systems (matrix b's, or the one cell's)
    const double* om;
    IsqMod mod;
    bool embed;     // real embeddings of Hermitian matrices (order even)
    IsqBufs bufs;
    IsqLanczos lan;
    IsqOp* ops;     // [nmat][ISQ_OPS]: the program, then the squarings
    int* cls;       // [nmat]
    int* order;     // [nmat] matrices by order, largest first
    double* yv;     // [nmat][2][sV]
    double* check;  // [nmat][nwg][2]
    double* zmax;   // [nmat], or nullptr when lambda_min is not wanted
};

// LDS written by a wavefront becomes visible to its other lanes
__device__ __forceinline__ void isq_wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

int isq_lanczos_wgs(int nmax);
// whether products of these orders go by residues of so many moduli; buffer sizes per matrix
// (bytes) and layout for order nmax; the launches of program step `step`
// (events around the integer products)
bool isq_mod_fits(const int* ns_host, int nmat, bool embed, int mods);
void isq_mod_sizes(int nmax, int mods, IsqMod& w, size_t& res, size_t& prod);
void isq_mod_launch(hipStream_t st, const IsqWork& w, int nmat, int step, hipEvent_t e0, hipEvent_t e1);
// Q^{-1/2} of every matrix into buffer ISQ_RESULT (both triangles), traces and
// check sums, and the largest eigenvalue of Q^{-1/2} when wanted.  ns_host: the
// orders; prof: each product launch as kind 1 when launch timing is on
struct LaunchProfiler;
void isq_launch(hipStream_t st, const IsqWork& w, int nmax, int nmat, const int* ns_host, LaunchProfiler* prof);
// energies, errors[0..3] and MBD_ST_NO_ROOT of the systems; a failed system's
// descriptor loses its atoms and gradient outputs
void isq_energy_launch(hipStream_t st, const IsqWork& w, SysDesc* sd, int nsys, int nmax, const double* mmult,
                       unsigned* status);
