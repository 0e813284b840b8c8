/*
 * mhlp.hip -- HIP kernels and C ABI of the modified-Helmholtz layer-potential
 * library (declarations and contracts: include/mhlp.h).
 *
 * Data layout in device memory
 *   geometry : node SoA x, y, dx, dy, d2x, d2y (copy of the caller's [6][N]),
 *              derived per-node weight w, unit normal nx, ny, curvature;
 *              per panel the Legendre coefficients of its position (16
 *              complex), arclength h and a bounding circle.
 *   plan     : targets tx, ty; CSR near list by target (row_ptr, panel index
 *              ascending, target index, complex preimage) and 16 SLP + 16 DLP
 *              correction weights per listed (target, panel) pair.
 *
 * Kernels
 *   geom_prep        one thread per panel: weights, normals, curvature, Legendre
 *                    coefficients, arclength, bounding circle.
 *   near_list        one thread per target, run twice (count, then fill): candidate
 *                    panels (some node within 1.2 h), Newton preimage, Bernstein
 *                    radius < 3.5 (Sec. 4.5.1).
 *   near_weights     one thread per listed pair: correction weights (nearfield.h).
 *   far_tree         FP64 far field (tree.h): far panels through cluster expansions,
 *                    the others pair by pair; listed panels are skipped and their
 *                    corrected contribution added in the epilogue (no
 *                    add-then-subtract).
 *   far_eval_mixed   FP32 far field, one thread per target, sources streamed
 *                    through LDS in tiles of 16 panels.
 *   gmres_*          BLAS-1 pieces of the Arnoldi process.
 */
#include <hip/hip_runtime.h>

#include <climits>
#include <cmath>
#include <algorithm>
#include <cstdio>
#include <cstring>
#include <string>
#include <vector>
#include <map>
#include <mutex>
#include <numeric>
#include <type_traits>

#include "mhlp.h"
#include "nearfield.h"

using namespace mhlp;

/* ------------------------------------------------------------------------ */
/* error handling                                                            */
/* ------------------------------------------------------------------------ */
static thread_local std::string g_err;

static mhlp_status fail(mhlp_status s, const std::string &msg)
{
    g_err = msg;
    return s;
}

#define HIPCHECK(x)                                                                                   \
    do {                                                                                              \
        hipError_t e_ = (x);                                                                          \
        if (e_ != hipSuccess) return fail(MHLP_HIP_ERROR, std::string(#x) + ": " + hipGetErrorString(e_)); \
    } while (0)

extern "C" const char *mhlp_last_error(void) { return g_err.c_str(); }

/* error setter shared with the other translation units of the library */
__attribute__((visibility("hidden"))) mhlp_status mhlp_set_error(mhlp_status s, const char *msg)
{
    g_err = msg;
    return s;
}

/* ------------------------------------------------------------------------ */
/* handles                                                                   */
/* ------------------------------------------------------------------------ */
struct mhlp_geometry {
    int device = 0;
    int64_t N = 0, Np = 0;
    double *soa = nullptr;                       /* [6][N] */
    double *w = nullptr, *nx = nullptr, *ny = nullptr, *kappa = nullptr;
    double *pa = nullptr; /* [Np][16] complex Legendre coefficients of the panel relative to its node 7 */
    double *ph = nullptr, *pcx = nullptr, *pcy = nullptr, *prad = nullptr;
    std::vector<int32_t> curve_off; /* host: first panel of each curve, then Np */
};

/* Device state of one GMRES cycle (see the GMRES section). */
struct GState {
    int32_t j;     /* current Arnoldi column                               */
    int32_t kmax;  /* columns allowed in this cycle                        */
    int32_t done;  /* converged, broken down or kmax reached               */
    int32_t steps; /* Arnoldi steps taken in this cycle                    */
    double thresh; /* stop when the residual estimate |g_{j+1}| <= thresh  */
    double inv;    /* 1 / h_{j+1,j}: scaling of the next basis vector      */
    double resest; /* |g_{j+1}| after the last step                        */
    double bnorm;  /* ||b|| when the solve left it on the device (first cycle) */
    double rn2;    /* ||b - A x||^2 after the end of the cycle (its last chunk) */
    double *xout;  /* caller's array that receives x at the end of each cycle (or NULL) */
};
static_assert(sizeof(GState) <= 64, "the state and the tail state share the first 128 bytes of gdev");

namespace mhlp {
struct FmmTree;
struct TreeDev;
}

struct mhlp_plan {
    const mhlp_geometry *g = nullptr;
    double alpha = 0.0;
    int64_t M = 0;
    bool onsurf = false;
    double *tx = nullptr, *ty = nullptr; /* owned unless onsurf; off-surface: Morton order */
    int32_t *perm = nullptr;             /* off-surface: caller index of internal target i */
    int32_t *near_ptr = nullptr;         /* [M+1] */
    int32_t *near_panel = nullptr;       /* [nnz] */
    int32_t *near_tgt = nullptr;         /* [nnz] */
    double *near_ts = nullptr;           /* [nnz][2] */
    double *wslp = nullptr, *wdlp = nullptr; /* [nnz][16] */
    double *wgrad = nullptr;  /* off-surface, built on first use: [4][nnz][16] gradient weights */
    bool stokes = false;      /* modified-Stokes (stresslet) plan: operator on [2][N] densities */
    double *wstk = nullptr;   /* stokes: [4][nnz][16] stresslet weights (D11, D12, D21, D22)   */
    mhlp::FmmTree *fmm = nullptr; /* off-surface scalar plans: FMM far field (mhlp_plan_set_fmm) */
    bool fmm_serves = false;      /* it is faster than the cluster lists (fmm_is_faster) */
    double *wstkg = nullptr;  /* stokes, off-surface, built on first use: [8][nnz][16] stresslet
                                 gradient weights, block (2a + l) 2 + j = d u_a/d x_l per mu_j */
    double inv_len = 0.0;     /* 1 / |Gamma| */
    int64_t nnz = 0;
    int32_t fill_mismatch = 0;
    int nsplit = 1;           /* source splits of the far field (small M)   */
    int32_t pps = 0;          /* panels per split                           */
    double *part = nullptr;   /* [2][nsplit][M] partial sums ([4][..] off-surface, for gradients) */
    uint8_t *wcls = nullptr;  /* scalar plans: [M/64 waves][Np] fine piece + 1 of each (wave, panel) for the
                                 mixed-precision tiles */
    double *fqd = nullptr;    /* [FINE_SCALES] fine-piece scales and constants at alpha (fine_scales) */
    mhlp::TreeDev *tree = nullptr; /* clusters, item lists, moments (tree.h) */
    char *tree_mem = nullptr;      /* its arrays but for the partial sums and, unless small, the lists */
    uint2 *tree_items = nullptr;   /* the lists where they have memory of their own */
    unsigned long long tr_cost = 0; /* total work of the item lists */
    struct TreeShape {
        int waves = 0, split = 1, cut = 0; /* waves per block and blocks per group, direct items in 2^cut units */
    } tr, tr_skip;                         /* of far_tree_kernel; where it leaves items out */
    int64_t tr_pairs = 0;                  /* (group, panel) pairs of a plan that may do without staging; 0: none may */
    NearParams np{};
    double near_factor = 1.2;
    int64_t part_cap = 0;     /* capacity of part (doubles)                 */
    /* GMRES workspace (lazily allocated) */
    double *ws = nullptr;
    int64_t ws_cols = 0;
    double *hdev = nullptr;  /* small device scratch for dot products */
    double *hhost = nullptr; /* pinned host mirror                    */
    /* device-driven GMRES: state + Hessenberg data, captured step graphs */
    char *gdev = nullptr;       /* GState, H, cs, sn, gv, y, h1, h2, hn   */
    int gdev_R = 0;
    GState *gstate_host = nullptr; /* pinned mirror of the state          */
    hipStream_t cap_stream = nullptr;
    struct StepGraph {
        hipGraphExec_t exec = nullptr;
        const void *ws = nullptr, *part = nullptr, *gdev = nullptr, *x = nullptr, *b = nullptr;
        int R = 0, nsplit = 0;
    };
    /* keyed by (precision, chunk length S = 0..GMRES_MAX_CHUNK, steps m <= S
       whose Gram-Schmidt runs in one block, end-of-cycle tail or not) */
    std::map<int, StepGraph> graphs;
    int gm_first_steps = 0; /* steps of the last solve's first cycle */
};

/* ------------------------------------------------------------------------ */
/* geometry preparation                                                      */
/* ------------------------------------------------------------------------ */
__host__ __device__ inline void geom_prep_body(int64_t p, const double *__restrict__ soa, int64_t N,
                                               double *__restrict__ w, double *__restrict__ nx,
                                               double *__restrict__ ny, double *__restrict__ kappa,
                                               double *__restrict__ pa, double *__restrict__ ph,
                                               double *__restrict__ pcx, double *__restrict__ pcy,
                                               double *__restrict__ prad)
{
    const double *x = soa, *y = soa + N, *dx = soa + 2 * N, *dy = soa + 3 * N, *ddx = soa + 4 * N,
                 *ddy = soa + 5 * N;
    double h = 0.0;
    for (int j = 0; j < 16; ++j) {
        const int64_t m = 16 * p + j;
        const double sp = hypot(dx[m], dy[m]);
        const double wm = GL16_W[j] * sp;
        w[m] = wm;
        nx[m] = -dy[m] / sp;
        ny[m] = dx[m] / sp;
        kappa[m] = (dx[m] * ddy[m] - dy[m] * ddx[m]) / (sp * sp * sp);
        h += wm;
    }
    /* Legendre coefficients of the panel polynomial relative to its node 7
       (an exact double): rounding then scales with the panel size instead of
       the distance from the origin.  Near-field routines add (node 7 - target)
       to the constant term and work in the target's frame (panel_local). */
    const cplx ref = mk(x[16 * p + 7], y[16 * p + 7]);
    cplx a[16];
    for (int mm = 0; mm < 16; ++mm) {
        cplx s = mk(0.0, 0.0);
        for (int j = 0; j < 16; ++j) s = s + LEGC[mm * 16 + j] * (mk(x[16 * p + j], y[16 * p + j]) - ref);
        a[mm] = s;
        pa[(16 * p + mm) * 2] = s.re;
        pa[(16 * p + mm) * 2 + 1] = s.im;
    }
    const cplx c0 = a[0]; /* panel centre relative to ref */
    double r = 0.0;
    for (int j = 0; j < 16; ++j) r = fmax(r, cabs((mk(x[16 * p + j], y[16 * p + j]) - ref) - c0));
    cplx e1 = mk(0.0, 0.0), e0 = mk(0.0, 0.0);
    for (int mm = 0; mm < 16; ++mm) {
        e1 = e1 + a[mm];
        e0 = e0 + ((mm & 1) ? -1.0 : 1.0) * a[mm];
    }
    r = fmax(r, fmax(cabs(e1 - c0), cabs(e0 - c0)));
    const cplx c = ref + c0;
    ph[p] = h;
    pcx[p] = c.re;
    pcy[p] = c.im;
    prad[p] = r;
}

/* given panel ends must lie within this fraction of the panel's arclength of
   the node polynomial's ends and of the next panel's start */
constexpr double PANEL_ENDS_TOL = 1e-6;

/* Checks given panel end points against the node data (Sec. 3.2: a panel is
   the degree-15 polynomial through its 16 nodes, so its ends are tau(-1) and
   tau(1)) and the chain of each closed curve (the end of a panel is the
   start of the next panel of its curve).  ends: [4][Np] xa, ya, xb, yb.
   flag[p]: bit 0 an end further than tol*h from the polynomial's end, bit 1
   the end of p further than tol*h from the start of next[p]. */
__global__ void panel_ends_kernel(const double *__restrict__ pa, const double *__restrict__ x,
                                  const double *__restrict__ y, const double *__restrict__ ph,
                                  const double *__restrict__ ends, const int32_t *__restrict__ next, int64_t Np,
                                  double tol, int32_t *__restrict__ flag)
{
    const int64_t p = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (p >= Np) return;
    double ax = x[16 * p + 7], ay = y[16 * p + 7], bx = ax, by = ay;
    for (int m = 0; m < 16; ++m) {
        const double cr = pa[(16 * p + m) * 2], ci = pa[(16 * p + m) * 2 + 1];
        bx += cr;
        by += ci;
        ax += (m & 1) ? -cr : cr;
        ay += (m & 1) ? -ci : ci;
    }
    const double lim = tol * ph[p];
    const double xa = ends[p], ya = ends[Np + p], xb = ends[2 * Np + p], yb = ends[3 * Np + p];
    int32_t f = 0;
    if (!(hypot(xa - ax, ya - ay) <= lim && hypot(xb - bx, yb - by) <= lim)) f |= 1;
    const int64_t q = next[p];
    if (!(hypot(xb - ends[q], yb - ends[Np + q]) <= lim)) f |= 2;
    flag[p] = f;
}

__global__ void geom_prep_kernel(const double *__restrict__ soa, int64_t N, int64_t Np, double *__restrict__ w,
                                 double *__restrict__ nx, double *__restrict__ ny, double *__restrict__ kappa,
                                 double *__restrict__ pa, double *__restrict__ ph, double *__restrict__ pcx,
                                 double *__restrict__ pcy, double *__restrict__ prad)
{
    const int64_t p = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (p >= Np) return;
    geom_prep_body(p, soa, N, w, nx, ny, kappa, pa, ph, pcx, pcy, prad);
}

/* ------------------------------------------------------------------------ */
/* near list                                                                 */
/* ------------------------------------------------------------------------ */
struct GeoView {
    const double *x, *y, *pa, *ph, *pcx, *pcy, *prad;
    int64_t N, Np;
};

/* Legendre coefficients of p(t) - z for panel p: the panel in the frame of
   the target z (the kernels depend on y - x only), so that tau - z near the
   target is formed without cancellation against |z|. */
__host__ __device__ inline void panel_local(const GeoView &G, int64_t p, cplx z, cplx *a)
{
    for (int m = 0; m < 16; ++m) a[m] = mk(G.pa[(16 * p + m) * 2], G.pa[(16 * p + m) * 2 + 1]);
    a[0] = a[0] + (mk(G.x[16 * p + 7], G.y[16 * p + 7]) - z);
}

/* Calls f(panel, self, tstar) for every panel needing a correction at target i
   (panel index ascending). */
template <class F>
__host__ __device__ inline void visit_near(const GeoView &G, int64_t i, cplx z, bool onsurf, double near_factor,
                                  double rho_direct, F &&f)
{
    const int64_t self_p = onsurf ? i / 16 : -1;
    for (int64_t p = 0; p < G.Np; ++p) {
        const double lim = near_factor * G.ph[p];
        const bool self = (p == self_p);
        if (!self) {
            const double dc = cabs(z - mk(G.pcx[p], G.pcy[p])) - G.prad[p];
            if (dc > lim) continue;
        }
        if (self) {
            f(p, (int)(i % 16), mk(GL16_T[i % 16], 0.0));
            continue;
        }
        double dmin = 1e300;
        int jb = 0;
        for (int j = 0; j < 16; ++j) {
            const double d = cabs2(z - mk(G.x[16 * p + j], G.y[16 * p + j]));
            if (d < dmin) {
                dmin = d;
                jb = j;
            }
        }
        if (dmin >= lim * lim) continue;
        cplx a[16];
        panel_local(G, p, z, a);
        cplx ts;
        if (!preimage(a, mk(0.0, 0.0), mk(GL16_T[jb], 0.0), ts)) continue;
        if (bernstein_rho(ts) >= rho_direct) continue;
        f(p, -1, ts);
    }
}

/* One traversal serves both passes of the CSR build (mode 0: count, mode 1:
   fill), so that the two passes run the same instructions and find the same
   pairs.  In fill mode, slots a target reserved but did not fill (which the
   shared code path rules out) are padded with panel -1, which every consumer
   skips, and the event is flagged. */
__host__ __device__ inline void near_list_body(int64_t i, int mode, const GeoView &G, const double *__restrict__ tx,
                                               const double *__restrict__ ty, int onsurf, double near_factor,
                                               double rho_direct, int32_t *__restrict__ cnt,
                                               const int32_t *__restrict__ ptr, int32_t *__restrict__ panel,
                                               int32_t *__restrict__ tgt, double *__restrict__ ts_out,
                                               int32_t *__restrict__ mismatch)
{
    int32_t q = mode ? ptr[i] : 0;
    const int32_t qend = mode ? ptr[i + 1] : INT_MAX;
    const int32_t q0 = q;
    visit_near(G, i, mk(tx[i], ty[i]), onsurf != 0, near_factor, rho_direct, [&](int64_t p, int, cplx ts) {
        if (mode && q < qend) {
            panel[q] = (int32_t)p;
            tgt[q] = (int32_t)i;
            ts_out[2 * q] = ts.re;
            ts_out[2 * q + 1] = ts.im;
        }
        ++q;
    });
    if (!mode) {
        cnt[i] = q - q0;
        return;
    }
    if (q != qend) mismatch[0] = 1;
    for (int32_t r = q; r < qend; ++r) {
        panel[r] = -1;
        tgt[r] = (int32_t)i;
        ts_out[2 * r] = 0.0;
        ts_out[2 * r + 1] = 0.0;
    }
}

__global__ void near_list_kernel(int mode, GeoView G, const double *__restrict__ tx, const double *__restrict__ ty,
                                 int64_t M, int onsurf, double near_factor, double rho_direct,
                                 int32_t *__restrict__ cnt, const int32_t *__restrict__ ptr,
                                 int32_t *__restrict__ panel, int32_t *__restrict__ tgt, double *__restrict__ ts_out,
                                 int32_t *__restrict__ mismatch)
{
    const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (i >= M) return;
    near_list_body(i, mode, G, tx, ty, onsurf, near_factor, rho_direct, cnt, ptr, panel, tgt, ts_out, mismatch);
}

/* exclusive scan of cnt[0..M) into ptr[0..M]; one block of 1024 threads */
__global__ __launch_bounds__(1024) void scan_kernel(const int32_t *__restrict__ cnt, int64_t M,
                                                    int32_t *__restrict__ ptr)
{
    __shared__ int64_t part[1024];
    const int t = threadIdx.x;
    const int64_t chunk = (M + 1023) / 1024;
    const int64_t b = t * chunk, e = (b + chunk < M) ? b + chunk : M;
    int64_t s = 0;
    for (int64_t i = b; i < e; ++i) s += cnt[i];
    part[t] = s;
    __syncthreads();
    for (int off = 1; off < 1024; off <<= 1) {
        int64_t v = (t >= off) ? part[t - off] : 0;
        __syncthreads();
        part[t] += v;
        __syncthreads();
    }
    int64_t run = part[t] - s;
    for (int64_t i = b; i < e; ++i) {
        ptr[i] = (int32_t)run;
        run += cnt[i];
    }
    if (t == 1023) ptr[M] = (int32_t)part[1023];
}

__host__ __device__ inline void near_weights_body(int64_t q, const GeoView &G, const double *__restrict__ tx,
                                                  const double *__restrict__ ty, int onsurf,
                                                  const int32_t *__restrict__ panel, const int32_t *__restrict__ tgt,
                                                  const double *__restrict__ ts, double alpha, const NearParams &P,
                                                  double *__restrict__ wsl, double *__restrict__ wdl)
{
    const int64_t p = panel[q], i = tgt[q];
    if (p < 0 || p >= G.Np) {
        for (int j = 0; j < 16; ++j) wsl[16 * q + j] = wdl[16 * q + j] = 0.0;
        return;
    }
    cplx a[16];
    panel_local(G, p, mk(tx[i], ty[i]), a);
    const int self = (onsurf && i / 16 == p) ? (int)(i % 16) : -1;
    double Ws[16], Wd[16];
    pair_weights(a, G.ph[p], mk(0.0, 0.0), self, mk(ts[2 * q], ts[2 * q + 1]), alpha, P, Ws, Wd);
    for (int j = 0; j < 16; ++j) {
        wsl[16 * q + j] = Ws[j];
        wdl[16 * q + j] = Wd[j];
    }
}

__global__ void near_weights_kernel(GeoView G, const double *__restrict__ tx, const double *__restrict__ ty,
                                    int onsurf, const int32_t *__restrict__ panel, const int32_t *__restrict__ tgt,
                                    const double *__restrict__ ts, int64_t nnz, double alpha, NearParams P,
                                    double *__restrict__ wsl, double *__restrict__ wdl)
{
    const int64_t q = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (q >= nnz) return;
    near_weights_body(q, G, tx, ty, onsurf, panel, tgt, ts, alpha, P, wsl, wdl);
}

/* gradient correction weights of the off-surface pairs: wg[b][q][j] */
__global__ void near_grad_weights_kernel(GeoView G, const double *__restrict__ tx, const double *__restrict__ ty,
                                         const int32_t *__restrict__ panel, const int32_t *__restrict__ tgt,
                                         const double *__restrict__ ts, int64_t nnz, double alpha, NearParams P,
                                         double *__restrict__ wg)
{
    const int64_t q = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (q >= nnz) return;
    const int64_t p = panel[q], i = tgt[q];
    double W[4][16];
    if (p < 0 || p >= G.Np) {
        for (int b = 0; b < 4; ++b)
            for (int j = 0; j < 16; ++j) W[b][j] = 0.0;
    } else {
        cplx a[16];
        panel_local(G, p, mk(tx[i], ty[i]), a);
        pair_grad_weights(a, G.ph[p], mk(0.0, 0.0), mk(ts[2 * q], ts[2 * q + 1]), alpha, P, W);
    }
    for (int b = 0; b < 4; ++b)
        for (int j = 0; j < 16; ++j) wg[(b * nnz + q) * 16 + j] = W[b][j];
}

/* stresslet correction weights of all pairs: ws[b][q][j] */
__global__ void near_stokes_weights_kernel(GeoView G, const double *__restrict__ tx, const double *__restrict__ ty,
                                           int onsurf, const int32_t *__restrict__ panel,
                                           const int32_t *__restrict__ tgt, const double *__restrict__ ts,
                                           int64_t nnz, double alpha, NearParams P, double *__restrict__ wst)
{
    const int64_t q = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (q >= nnz) return;
    const int64_t p = panel[q], i = tgt[q];
    double W[4][16];
    if (p < 0 || p >= G.Np) {
        for (int b = 0; b < 4; ++b)
            for (int j = 0; j < 16; ++j) W[b][j] = 0.0;
    } else {
        cplx a[16];
        panel_local(G, p, mk(tx[i], ty[i]), a);
        const int self = (onsurf && i / 16 == p) ? (int)(i % 16) : -1;
        pair_stokes_weights(a, G.ph[p], mk(0.0, 0.0), self, mk(ts[2 * q], ts[2 * q + 1]), alpha, P, W);
    }
    for (int b = 0; b < 4; ++b)
        for (int j = 0; j < 16; ++j) wst[(b * nnz + q) * 16 + j] = W[b][j];
}

/* stresslet gradient correction weights of the off-surface pairs: wg[b][q][j] */
__global__ void near_stokes_grad_weights_kernel(GeoView G, const double *__restrict__ tx,
                                                const double *__restrict__ ty, const int32_t *__restrict__ panel,
                                                const int32_t *__restrict__ tgt, const double *__restrict__ ts,
                                                int64_t nnz, double alpha, NearParams P, double *__restrict__ wg)
{
    const int64_t q = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (q >= nnz) return;
    const int64_t p = panel[q], i = tgt[q];
    double W[8][16];
    if (p < 0 || p >= G.Np) {
        for (int b = 0; b < 8; ++b)
            for (int j = 0; j < 16; ++j) W[b][j] = 0.0;
    } else {
        cplx a[16];
        panel_local(G, p, mk(tx[i], ty[i]), a);
        pair_stokes_grad_weights(a, G.ph[p], mk(0.0, 0.0), mk(ts[2 * q], ts[2 * q + 1]), alpha, P, W);
    }
    for (int b = 0; b < 8; ++b)
        for (int j = 0; j < 16; ++j) wg[(b * nnz + q) * 16 + j] = W[b][j];
}

/* ------------------------------------------------------------------------ */
/* far field + corrections, FP64                                             */
/* ------------------------------------------------------------------------ */
constexpr int FT_THREADS = 256;
constexpr int FT_SRC = 256; /* sources per LDS tile = 16 panels */

struct FarArgs {
    const double *sx, *sy, *sw, *snx, *sny;
    const double *sigma, *mu;
    int64_t N;
    const double *tx, *ty;
    int64_t M;
    const int32_t *nptr, *npan;
    const double *wsl, *wdl;
    double alpha;
    double half_term; /* 0.5 for (1/2 I + D) on an on-surface plan, else 0 */
    double *us, *ud;
    /* gradients, stresslet: correction weights [blocks][nnz][16] and the outputs of the fields */
    const double *wg = nullptr;
    int64_t nnz = 0;
    double *gout[4] = {nullptr, nullptr, nullptr, nullptr};
    double inv_len = 0.0; /* 1/|Gamma| (on-surface stresslet operator) */
    int64_t Np;
    int32_t pps;      /* panels per source split (blockIdx.y) */
    double *part_s, *part_d; /* [nsplit][M] partial far sums when split */
    /* device-driven GMRES: when gs is set the density is column gs->j of the
       basis (mu + j*jstride) and the launch does nothing once gs->done */
    const GState *gs;
    int64_t jstride;
    const int32_t *perm; /* output index of internal target i (NULL: identity) */
    const double *pcx, *pcy, *prad; /* bounding circle of each panel */
    const uint8_t *wcls = nullptr; /* [M/64 waves][Np] fine piece + 1 of each (wave, panel): mixed precision */
    const double *fq = nullptr; /* scales of the fine pieces and constants at the plan's alpha (fine_scales) */
};


/* density of a far launch: fixed, or the current GMRES basis column;
   false when the launch is a no-op */
__device__ __forceinline__ bool far_density(const FarArgs &A, const double *&mu)
{
    mu = A.mu;
    if (A.gs) {
        if (A.gs->done) return false;
        mu += (int64_t)A.gs->j * A.jstride;
    }
    return true;
}

/* Near corrections, 1/(2 pi) scaling and identity term for target i. */
template <bool SLP, bool DLP>
__device__ __forceinline__ void far_epilogue(const FarArgs &A, const double *__restrict__ mu, int64_t i, double accs,
                                             double accd)
{
    double cs = 0.0, cd = 0.0;
    for (int32_t q = A.nptr[i]; q < A.nptr[i + 1]; ++q) {
        const int64_t p = A.npan[q];
        if (p < 0) continue;
        for (int jj = 0; jj < 16; ++jj) {
            if (SLP) cs = fma(A.wsl[16 * (int64_t)q + jj], A.sigma[16 * p + jj], cs);
            if (DLP) cd = fma(A.wdl[16 * (int64_t)q + jj], mu[16 * p + jj], cd);
        }
    }
    const int64_t o = A.perm ? (int64_t)A.perm[i] : i;
    if (SLP) A.us[o] = fma(INV_2PI, accs, cs);
    if (DLP) {
        double v = fma(INV_2PI, accd, cd);
        /* identity term: only on-surface plans (targets are the nodes, M == N) */
        if (A.half_term != 0.0) v = fma(A.half_term, mu[i], v);
        A.ud[o] = v;
    }
}

/* Sum of the source-split partials, near corrections, 1/(2 pi) scaling and
   identity term.  A block takes FZ_TG consecutive targets with L lanes each
   (lane l is the l-th group of FZ_TG threads, so the partial loads of a lane
   are row segments of FZ_TG consecutive values; small blocks spread short
   lists over many CUs): lane
   l adds the partials l, l + L, ... and the correction terms of node l, l + L,
   ... of each near panel; the lane sums are then added in lane order.  L = 16
   for short target lists (many splits, few targets: the on-surface operator),
   L = 1 (one thread per target, 256 targets a block) otherwise. */
constexpr int FZ_TG = 16, FZ_L = 16, FZ_SHORT = 16384;

template <bool SLP, bool DLP, int L>
__global__ __launch_bounds__(L == 1 ? 256 : FZ_TG * L) void far_finalize(FarArgs A, int nsplit)
{
    constexpr int TG = L == 1 ? 256 : FZ_TG;
    __shared__ double red[4][L == 1 ? 1 : L][L == 1 ? 1 : TG]; /* far S, near S, far D, near D */
    const double *mu;
    if (!far_density(A, mu)) return; /* the same for every thread of the launch */
    const int g = threadIdx.x % TG, l = L == 1 ? 0 : threadIdx.x / TG; /* L = 1: loops unroll */
    const int64_t i = blockIdx.x * (int64_t)TG + g;
    double fs = 0.0, ns = 0.0, fd = 0.0, nd = 0.0;
    if (i < A.M) {
        for (int k = l; k < nsplit; k += L) {
            if (SLP) fs += A.part_s[k * A.M + i];
            if (DLP) fd += A.part_d[k * A.M + i];
        }
        for (int32_t q = A.nptr[i]; q < A.nptr[i + 1]; ++q) {
            const int64_t p = A.npan[q];
            if (p < 0) continue;
            for (int jj = l; jj < 16; jj += L) {
                if (SLP) ns = fma(A.wsl[16 * (int64_t)q + jj], A.sigma[16 * p + jj], ns);
                if (DLP) nd = fma(A.wdl[16 * (int64_t)q + jj], mu[16 * p + jj], nd);
            }
        }
    }
    if (L > 1) {
        red[0][l][g] = fs;
        red[1][l][g] = ns;
        red[2][l][g] = fd;
        red[3][l][g] = nd;
        __syncthreads();
        if (l != 0) return;
        for (int q = 1; q < L; ++q) {
            fs += red[0][q][g];
            ns += red[1][q][g];
            fd += red[2][q][g];
            nd += red[3][q][g];
        }
    }
    if (i >= A.M) return;
    const int64_t o = A.perm ? (int64_t)A.perm[i] : i;
    if (SLP) A.us[o] = fma(INV_2PI, fs, ns);
    if (DLP) {
        double v = fma(INV_2PI, fd, nd);
        if (A.half_term != 0.0) v = fma(A.half_term, mu[i], v);
        A.ud[o] = v;
    }
}

/* Sum over the 64 lanes of a wave with DPP moves (no LDS traffic): adds of
   the value 1, 2, 4, 8 lanes lower within each row of 16 lanes, then the last
   lane of each row carried into the next row (row_bcast15) and lane 31 into
   the upper half (row_bcast31): lane 63 then holds the sum, a fixed tree, and
   readlane returns it to every lane.  Lanes with no source add zero. */
__device__ __forceinline__ double dpp_add(double v, int ctrl_sel)
{
    const int lo = __double2loint(v), hi = __double2hiint(v);
    int rlo, rhi;
    switch (ctrl_sel) {
    case 0: rlo = __builtin_amdgcn_update_dpp(0, lo, 0x111, 0xf, 0xf, false);
            rhi = __builtin_amdgcn_update_dpp(0, hi, 0x111, 0xf, 0xf, false); break;
    case 1: rlo = __builtin_amdgcn_update_dpp(0, lo, 0x112, 0xf, 0xf, false);
            rhi = __builtin_amdgcn_update_dpp(0, hi, 0x112, 0xf, 0xf, false); break;
    case 2: rlo = __builtin_amdgcn_update_dpp(0, lo, 0x114, 0xf, 0xf, false);
            rhi = __builtin_amdgcn_update_dpp(0, hi, 0x114, 0xf, 0xf, false); break;
    case 3: rlo = __builtin_amdgcn_update_dpp(0, lo, 0x118, 0xf, 0xf, false);
            rhi = __builtin_amdgcn_update_dpp(0, hi, 0x118, 0xf, 0xf, false); break;
    case 4: rlo = __builtin_amdgcn_update_dpp(0, lo, 0x142, 0xa, 0xf, false);
            rhi = __builtin_amdgcn_update_dpp(0, hi, 0x142, 0xa, 0xf, false); break;
    default: rlo = __builtin_amdgcn_update_dpp(0, lo, 0x143, 0xc, 0xf, false);
             rhi = __builtin_amdgcn_update_dpp(0, hi, 0x143, 0xc, 0xf, false); break;
    }
    return v + __hiloint2double(rhi, rlo);
}

__device__ __forceinline__ double wave_sum_dpp(double v)
{
#pragma unroll
    for (int k = 0; k < 6; ++k) v = dpp_add(v, k);
    const int lo = __builtin_amdgcn_readlane(__double2loint(v), 63);
    const int hi = __builtin_amdgcn_readlane(__double2hiint(v), 63);
    return __hiloint2double(hi, lo);
}

/* Plan time: the fine piece of every (wave of 64 targets, panel) for the
   mixed-precision tiles (low 7 bits: piece + 1, 0 for z <= 2 everywhere, KQ_NP + 1 when
   the pairs need the per-pair selection; bit 7 set when some target of the
   wave lists the panel as near), from the exact extreme distances of the
   wave's targets to the panel's nodes; targets that list the panel do not vote
   (they skip it).  Lanes past the last target repeat it. */
__global__ __launch_bounds__(256) void far_class_kernel(const double *__restrict__ tx, const double *__restrict__ ty,
                                                        int64_t M, const double *__restrict__ sx,
                                                        const double *__restrict__ sy, int64_t Np, double alpha,
                                                        const int32_t *__restrict__ nptr,
                                                        const int32_t *__restrict__ npan, uint8_t *__restrict__ cls)
{
    const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    const int64_t iv = i < M ? i : M - 1;
    const int64_t w = i >> 6;
    const double x = tx[iv], y = ty[iv];
    int32_t k = nptr[iv];
    const int32_t kend = nptr[iv + 1];
    while (k < kend && npan[k] < 0) ++k;
    for (int64_t p = 0; p < Np; ++p) {
        double r2lo = 1e300, r2hi = 0.0;
        for (int j = 0; j < 16; ++j) {
            const double ex = x - sx[16 * p + j], ey = y - sy[16 * p + j];
            const double r2 = fma(ex, ex, ey * ey);
            r2lo = fmin(r2lo, r2);
            r2hi = fmax(r2hi, r2);
        }
        bool listed = false;
        if (k < kend && npan[k] == p) {
            listed = true;
            ++k;
        }
        const double zlo = alpha * sqrt(r2lo), zhi = alpha * sqrt(r2hi);
        int kl = 0, kh = 0;
        for (int b = 0; b < KQ_NB; ++b) {
            kl += zlo > KQ_B[b] ? 1 : 0;
            kh += zhi > KQ_B[b] ? 1 : 0;
        }
        /* the voting lanes' extreme piece indices */
        int lo = listed ? KQ_NB + 1 : kl, hi = listed ? -1 : kh;
        for (int off = 32; off > 0; off >>= 1) {
            lo = min(lo, __shfl_xor(lo, off));
            hi = max(hi, __shfl_xor(hi, off));
        }
        int c = KQ_NP + 1;
        if (hi < 0)
            c = KQ_NP + 1; /* every target skips the panel */
        else if (lo == hi)
            c = lo; /* piece lo - 1 (0: z <= 2) */
        else if (lo >= 1 && hi == lo + 1 && lo <= KQ_NB - 1)
            c = KQ_NB + lo; /* pieces lo - 1 and lo */
        if (__ballot(listed) != 0) c |= 0x80;
        if ((threadIdx.x & 63) == 0) cls[w * Np + p] = (uint8_t)c;
    }
}

/* ------------------------------------------------------------------------ */
/* far field, mixed precision: FP32 kernel values and products, differences  */
/* x - y formed exactly in FP64 then rounded, FP32 partial sums over each     */
/* 16-node panel accumulated in FP64; corrections and identity term in FP64. */
/* ------------------------------------------------------------------------ */
/* the classes -1 .. KQ_NP - 1 of the plan's (wave, panel) table, for a switch */
#define MHLP_PC_CASES(X) X(-1) X(0) X(1) X(2) X(3) X(4) X(5) X(6) X(7) X(8) X(9) X(10) X(11) X(12) X(13) X(14)
static_assert(KQ_NP == 15, "MHLP_PC_CASES lists the fine pieces");

/* the 16 sources of one LDS panel (offset l0) against the lane's target in
   FP32, in piece PC of the plan's class table (k01_fp32_pc) */
template <bool SLP, bool DLP, int PC>
__device__ __forceinline__ void mixed_panel(double x, double y, const double *lx, const double *ly, const float *lq,
                                            const float *ldx, const float *ldy, int l0, float alpha, float a2q,
                                            float a4, float &ps, float &pd)
{
#pragma unroll 4
    for (int s = 0; s < 16; ++s) {
        const int l = l0 + s;
        const float ex = (float)(x - lx[l]), ey = (float)(y - ly[l]);
        const float r2 = fmaf(ex, ex, ey * ey);
        const K01f o = k01_fp32_pc<SLP, DLP, PC>(r2, alpha, a2q, a4);
        if (SLP) ps = fmaf(o.k0, lq[l], ps);
        if (DLP) pd = fmaf(o.ak1r, fmaf(ex, ldx[l], ey * ldy[l]), pd);
    }
}

template <bool SLP, bool DLP, bool SPLIT>
__global__ __launch_bounds__(FT_THREADS) void far_eval_mixed(FarArgs A)
{
    __shared__ double lx[FT_SRC], ly[FT_SRC];
    __shared__ float lq[FT_SRC], ldx[FT_SRC], ldy[FT_SRC];
    const double *mu;
    if (!far_density(A, mu)) return;
    const int64_t i = blockIdx.x * (int64_t)FT_THREADS + threadIdx.x;
    const bool valid = i < A.M;
    const double x = valid ? A.tx[i] : 0.0, y = valid ? A.ty[i] : 0.0;
    const int64_t pb = SPLIT ? (int64_t)blockIdx.y * A.pps : 0;
    const int64_t pe = SPLIT ? min(A.Np, pb + A.pps) : A.Np;
    int32_t k = 0, kend = 0;
    if (valid) {
        k = A.nptr[i];
        kend = A.nptr[i + 1];
        while (k < kend && A.npan[k] >= 0 && A.npan[k] < pb) ++k;
    }
    int32_t nxt = (k < kend) ? A.npan[k] : INT_MAX;
    const float alpha = (float)A.alpha, a2q = 0.25f * alpha * alpha, a4 = 4.0f / alpha;
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint8_t *cls = A.wcls ? A.wcls + ((int64_t)blockIdx.x * (FT_THREADS / 64) + wv) * A.Np : nullptr;
    double accs = 0.0, accd = 0.0;
    for (int64_t base = 16 * pb; base < 16 * pe; base += FT_SRC) {
        __syncthreads();
        const int64_t j = base + threadIdx.x;
        if (j < 16 * pe) {
            const double wj = A.sw[j];
            lx[threadIdx.x] = A.sx[j];
            ly[threadIdx.x] = A.sy[j];
            if (SLP) lq[threadIdx.x] = (float)(wj * A.sigma[j]);
            if (DLP) {
                const double m = wj * mu[j];
                ldx[threadIdx.x] = (float)(m * A.snx[j]);
                ldy[threadIdx.x] = (float)(m * A.sny[j]);
            }
        }
        __syncthreads();
        const int32_t p0 = (int32_t)(base / 16);
        const int npl = (pe - p0) < 16 ? (int)(pe - p0) : 16;
        for (int pl = 0; pl < npl; ++pl) {
            if (p0 + pl == nxt) {
                ++k;
                nxt = (k < kend) ? A.npan[k] : INT_MAX;
                continue;
            }
            float ps = 0.0f, pd = 0.0f;
            const int pc = cls ? (cls[p0 + pl] & 0x7f) - 1 : KQ_NP;
            switch (pc) {
#define MHLP_MIXED_PANEL(PCV)                                                                              \
    case PCV:                                                                                              \
        mixed_panel<SLP, DLP, PCV>(x, y, lx, ly, lq, ldx, ldy, pl * 16, alpha, a2q, a4, ps, pd);           \
        break;
                MHLP_PC_CASES(MHLP_MIXED_PANEL)
#undef MHLP_MIXED_PANEL
            default:
                mixed_panel<SLP, DLP, KQ_NP>(x, y, lx, ly, lq, ldx, ldy, pl * 16, alpha, a2q, a4, ps, pd);
            }
            if (SLP) accs += (double)ps;
            if (DLP) accd += (double)pd;
        }
    }
    if (!valid) return;
    if (SPLIT) {
        if (SLP) A.part_s[blockIdx.y * A.M + i] = accs;
        if (DLP) A.part_d[blockIdx.y * A.M + i] = accd;
    } else {
        far_epilogue<SLP, DLP>(A, mu, i, accs, accd);
    }
}

#include "tree.h"
#include "volume_tree.h"

/* ------------------------------------------------------------------------ */
/* volume sum over a tensor grid (all pairs) with the self-cell correction   */
/*   u_i = sum_{j != i} K0(alpha r_ij)/(2 pi) w_j f_j + (w_i/h^2) Wcell f_i    */
/* Sources are targets; the self pair (r == 0) is skipped in the sum.        */
/* ------------------------------------------------------------------------ */
struct VolArgs {
    const double *x, *y, *w, *f;
    int64_t n;
    double alpha;
    double selfc;   /* Wcell / h^2 */
    int64_t per_split;
    double *part;   /* [nsplit][n] */
    double *u;
    const double *selfc_dev; /* when set, Wcell / h^2 is read here instead of selfc */
};

template <bool MIXED, bool SPLIT>
__global__ __launch_bounds__(FT_THREADS) void volume_kernel(VolArgs A)
{
    __shared__ double lx[FT_SRC], ly[FT_SRC];
    __shared__ double lq[FT_SRC];
    const int64_t i = blockIdx.x * (int64_t)FT_THREADS + threadIdx.x;
    const bool valid = i < A.n;
    const double x = valid ? A.x[i] : 0.0, y = valid ? A.y[i] : 0.0;
    const int64_t jb = SPLIT ? (int64_t)blockIdx.y * A.per_split : 0;
    const int64_t je = SPLIT ? min(A.n, jb + A.per_split) : A.n;
    const FarConst fc = far_const(A.alpha);
    const float af = (float)A.alpha, a2qf = 0.25f * af * af, a4f = 4.0f / af;
    double acc = 0.0;
    for (int64_t base = jb; base < je; base += FT_SRC) {
        __syncthreads();
        const int64_t j = base + threadIdx.x;
        if (j < je) {
            lx[threadIdx.x] = A.x[j];
            ly[threadIdx.x] = A.y[j];
            lq[threadIdx.x] = A.w[j] * A.f[j];
        } else {
            lx[threadIdx.x] = 0.0;
            ly[threadIdx.x] = 0.0;
            lq[threadIdx.x] = 0.0;
        }
        __syncthreads();
        const int cnt = (je - base) < FT_SRC ? (int)(je - base) : FT_SRC;
        if (MIXED) {
            float ps = 0.0f;
            for (int l = 0; l < cnt; ++l) {
                const float ex = (float)(x - lx[l]), ey = (float)(y - ly[l]);
                float r2 = fmaf(ex, ex, ey * ey);
                const bool self = r2 == 0.0f;
                r2 = self ? 1.0f : r2;
                const K01f o = k01_fp32<true, false>(r2, af, a2qf, a4f);
                ps = fmaf(self ? 0.0f : o.k0, (float)lq[l], ps);
                if ((l & 15) == 15) {
                    acc += (double)ps;
                    ps = 0.0f;
                }
            }
            acc += (double)ps;
        } else {
            /* pairs of sources; an odd count reads one zero-padded slot (lq = 0) */
#pragma unroll 1
            for (int l = 0; l < cnt; l += 2) {
                const FarTab T = far_table();
                const double ex0 = x - lx[l], ey0 = y - ly[l];
                const double ex1 = x - lx[l + 1], ey1 = y - ly[l + 1];
                double r20 = fma(ex0, ex0, ey0 * ey0), r21 = fma(ex1, ex1, ey1 * ey1);
                const bool self0 = r20 == 0.0, self1 = r21 == 0.0;
                r20 = self0 ? 1.0 : r20;
                r21 = self1 ? 1.0 : r21;
                K01 o0, o1;
                k01_far2<true, false, false>(T, fc, r20, r21, o0, o1);
                acc = fma(self1 ? 0.0 : o1.k0, lq[l + 1], fma(self0 ? 0.0 : o0.k0, lq[l], acc));
            }
        }
    }
    if (!valid) return;
    if (SPLIT)
        A.part[blockIdx.y * A.n + i] = acc;
    else
        A.u[i] = fma(INV_2PI, acc, (A.selfc_dev ? A.selfc_dev[0] : A.selfc) * A.w[i] * A.f[i]);
}

__global__ void volume_finalize(VolArgs A, int nsplit)
{
    const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (i >= A.n) return;
    double s_ = 0.0;
    for (int k = 0; k < nsplit; ++k) s_ += A.part[k * A.n + i];
    A.u[i] = fma(INV_2PI, s_, (A.selfc_dev ? A.selfc_dev[0] : A.selfc) * A.w[i] * A.f[i]);
}

/* ------------------------------------------------------------------------ */
/* GMRES BLAS-1                                                              */
/* ------------------------------------------------------------------------ */
/* out[c] = sum_i V[c*ld + i] * w[i], one block per column */
__global__ __launch_bounds__(256) void multi_dot_kernel(const double *__restrict__ V, int64_t ld, const double *__restrict__ w,
                                                        int64_t N, double *__restrict__ out)
{
    __shared__ double red[256];
    const int c = blockIdx.x;
    const double *v = V + c * ld;
    double s = 0.0;
    for (int64_t i = threadIdx.x; i < N; i += 256) s = fma(v[i], w[i], s);
    red[threadIdx.x] = s;
    __syncthreads();
    for (int off = 128; off > 0; off >>= 1) {
        if (threadIdx.x < off) red[threadIdx.x] += red[threadIdx.x + off];
        __syncthreads();
    }
    if (threadIdx.x == 0) out[c] = red[0];
}


/* out = s * in */
__global__ void scale_kernel(const double *__restrict__ in, double s, double *__restrict__ out, int64_t N)
{
    const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (i < N) out[i] = s * in[i];
}

/* r = g - a */
__global__ void residual_kernel(const double *__restrict__ g, const double *__restrict__ a, double *__restrict__ r,
                                int64_t N)
{
    const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (i < N) r[i] = g[i] - a[i];
}

/* ---- device-driven GMRES steps (every kernel does nothing once done) ---- */
/* Column k = j of the Hessenberg matrix (CGS2 coefficients h1 + h2,
   subdiagonal ||w|| = sqrt(hnsq)), the earlier Givens rotations applied to it,
   a new rotation that zeroes the subdiagonal, the rotated right-hand side g
   and the stopping decision.  H is (R+1) x R row-major.  Called by every
   thread of one block: the column and the rotations are staged in LDS (col:
   R + 2 values, rot: 2R) by all threads, the rotations run on thread 0, and
   the column is written back by all threads. */
__device__ void gs_finish_block(GState *__restrict__ gs, double *__restrict__ H, int R, double *__restrict__ cs,
                                double *__restrict__ sn, double *__restrict__ gv, const double *__restrict__ h1,
                                const double *__restrict__ h2, double hnsq, double *col, double *rot)
{
    const int k = gs->j;
    for (int c = threadIdx.x; c <= k; c += blockDim.x) {
        col[c] = h1[c] + h2[c];
        if (c < k) {
            rot[2 * c] = cs[c];
            rot[2 * c + 1] = sn[c];
        }
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        const double hn1 = sqrt(hnsq);
        col[k + 1] = hn1;
        for (int j = 0; j < k; ++j) {
            const double a = col[j], c = col[j + 1];
            col[j] = rot[2 * j] * a + rot[2 * j + 1] * c;
            col[j + 1] = -rot[2 * j + 1] * a + rot[2 * j] * c;
        }
        const double a = col[k], c = col[k + 1];
        const double den = hypot(a, c);
        const double ck = a / den, sk = c / den;
        cs[k] = ck;
        sn[k] = sk;
        col[k] = den;
        col[k + 1] = 0.0;
        gv[k + 1] = -sk * gv[k];
        gv[k] = ck * gv[k];
        gs->steps = k + 1;
        gs->resest = fabs(gv[k + 1]);
        gs->inv = hn1 > 0.0 ? 1.0 / hn1 : 0.0;
        if (gs->resest <= gs->thresh || hn1 == 0.0 || k + 1 >= gs->kmax) gs->done = 1;
    }
    __syncthreads();
    for (int c = threadIdx.x; c <= k + 1; c += blockDim.x) H[(int64_t)c * R + k] = col[c];
}

constexpr int GSF_T = 1024, GSF_W = GSF_T / 64, GSF_RMAX = 256;

/* The whole Gram-Schmidt part of an Arnoldi step in one block with the new
   vector held in registers (vectors up to GSR_NMAX long, any step): thread t
   owns elements t, t + GSF_T, ... (E of them).  The basis columns go through
   registers in chunks of C = 32 / E; while all columns fit in one chunk they
   are loaded once, together with the new vector, and serve both CGS passes.
   A pass forms the thread's partial dot products, sums them over the wave by
   a fixed butterfly and over the waves in wave order, then subtracts the
   projection in column order.  Then the norm, the Hessenberg column
   (gs_finish_block), and the next basis vector from the registers. */
constexpr int64_t GSR_NMAX = 8 * GSF_T;
/* basis columns the one-block form keeps in registers for vectors of length N;
   it serves the steps whose columns all fit, the slice form the later ones */
__host__ __device__ inline int gsr_cols(int64_t N) { return N <= GSF_T ? 32 : N <= 2 * GSF_T ? 16 : N <= 4 * GSF_T ? 8 : 4; }
/* steps take the one-block form while their basis columns exceed the register
   capacity by at most this many (read one at a time), the slice form after.
   Above 4096 unknowns one CU reads the columns from L2 too slowly for that:
   8192 unknowns, step 1 11 us, step 5 20, step 12 40, the slice form 19. */
__host__ __device__ inline int gsr_extra(int64_t N) { return N <= 4 * GSF_T ? 8 : 0; }

/* v[c][k] = V_{c0+c}[t + k GSF_T] for the chunk's columns below ncol (0 elsewhere) */
template <int C, int E>
__device__ __forceinline__ void gsr_load(const double *__restrict__ V, int64_t ld, int64_t N, int c0, int ncol,
                                         double (&v)[C][E])
{
    const int t = threadIdx.x;
#pragma unroll
    for (int c = 0; c < C; ++c)
#pragma unroll
        for (int k = 0; k < E; ++k) {
            const int64_t i = t + (int64_t)k * GSF_T;
            v[c][k] = (c0 + c < ncol && i < N) ? V[(int64_t)(c0 + c) * ld + i] : 0.0;
        }
}

/* the chunk's dot products with x: wave sums (wave_sum_dpp) into
   red[wave][c0 + c] */
template <int C, int E>
__device__ __forceinline__ void gsr_dots(const double (&v)[C][E], const double (&x)[E], int c0, int ncol,
                                         double (*red)[GSF_RMAX])
{
    const int wv = threadIdx.x >> 6, ln = threadIdx.x & 63;
    double p[C];
#pragma unroll
    for (int c = 0; c < C; ++c) {
        p[c] = 0.0;
#pragma unroll
        for (int k = 0; k < E; ++k) p[c] = fma(v[c][k], x[k], p[c]);
        p[c] = wave_sum_dpp(p[c]);
    }
    if (ln == 0)
#pragma unroll
        for (int c = 0; c < C; ++c)
            if (c0 + c < ncol) red[wv][c0 + c] = p[c];
}

/* hp[c] = sum over the waves of red[.][c], in wave order (after a barrier) */
__device__ __forceinline__ void gsr_collect(double (*red)[GSF_RMAX], int ncol, double *hp)
{
    __syncthreads();
    for (int c = threadIdx.x; c < ncol; c += GSF_T) {
        double sacc = red[0][c];
        for (int q = 1; q < GSF_W; ++q) sacc += red[q][c];
        hp[c] = sacc;
    }
    __syncthreads();
}

template <int C, int E>
__device__ __forceinline__ void gsr_sub(const double (&v)[C][E], double (&x)[E], int c0, int ncol, const double *hp)
{
#pragma unroll
    for (int c = 0; c < C; ++c) {
        if (c0 + c >= ncol) break;
        const double h = hp[c0 + c];
#pragma unroll
        for (int k = 0; k < E; ++k) x[k] = fma(-h, v[c][k], x[k]);
    }
}

/* LDS of the one-block Gram-Schmidt */
struct GsrShared {
    double red[GSF_W][GSF_RMAX];
    double hs[2][GSF_RMAX];
    double nrm[GSF_W], hnl[1];
    double col[GSF_RMAX + 2], rot[2 * GSF_RMAX];
};

/* CGS2 of w (length N) against V_0..V_{ncol-1}, by every thread of a GSF_T
   block: the new vector in x, the two passes' coefficients in sh.hs and the
   squared norm in sh.hnl. */
template <int E>
__device__ __forceinline__ void gsr_orth(const double *__restrict__ V, int64_t ld, const double *__restrict__ w,
                                         int64_t N, int ncol, double (&x)[E], GsrShared &sh)
{
    constexpr int C = 32 / E;
    const int t = threadIdx.x, wv = t >> 6, ln = t & 63;
#pragma unroll
    for (int k = 0; k < E; ++k) {
        const int64_t i = t + (int64_t)k * GSF_T;
        x[k] = i < N ? w[i] : 0.0;
    }
    if (ncol <= C) {
        double v[C][E];
        gsr_load<C, E>(V, ld, N, 0, ncol, v);
        for (int pass = 0; pass < 2; ++pass) {
            gsr_dots<C, E>(v, x, 0, ncol, sh.red);
            gsr_collect(sh.red, ncol, sh.hs[pass]);
            gsr_sub<C, E>(v, x, 0, ncol, sh.hs[pass]);
        }
    } else {
        /* the first C columns stay in registers for both passes; the others
           are read one at a time, twice per pass */
        double v[C][E];
        gsr_load<C, E>(V, ld, N, 0, ncol, v);
        for (int pass = 0; pass < 2; ++pass) {
            gsr_dots<C, E>(v, x, 0, ncol, sh.red);
            for (int c = C; c < ncol; ++c) {
                double u[1][E];
                gsr_load<1, E>(V, ld, N, c, ncol, u);
                gsr_dots<1, E>(u, x, c, ncol, sh.red);
            }
            gsr_collect(sh.red, ncol, sh.hs[pass]);
            gsr_sub<C, E>(v, x, 0, ncol, sh.hs[pass]);
            for (int c = C; c < ncol; ++c) {
                double u[1][E];
                gsr_load<1, E>(V, ld, N, c, ncol, u);
                gsr_sub<1, E>(u, x, c, ncol, sh.hs[pass]);
            }
        }
    }
    double sacc = 0.0;
#pragma unroll
    for (int k = 0; k < E; ++k) sacc = fma(x[k], x[k], sacc);
    sacc = wave_sum_dpp(sacc);
    if (ln == 0) sh.nrm[wv] = sacc;
    __syncthreads();
    if (t == 0) {
        double s2 = sh.nrm[0];
        for (int q = 1; q < GSF_W; ++q) s2 += sh.nrm[q];
        sh.hnl[0] = s2;
    }
    __syncthreads();
}

/* The one-block CGS2 step on w (length N), by every thread of a GSF_T block. */
template <int E>
__device__ __forceinline__ void gsr_body(GState *__restrict__ gs, double *__restrict__ V, int64_t ld,
                                         const double *__restrict__ w, int64_t N, double *__restrict__ H, int R,
                                         double *__restrict__ cs, double *__restrict__ sn, double *__restrict__ gv,
                                         GsrShared &sh)
{
    const int t = threadIdx.x, j = gs->j;
    double x[E];
    gsr_orth<E>(V, ld, w, N, j + 1, x, sh);
    gs_finish_block(gs, H, R, cs, sn, gv, sh.hs[0], sh.hs[1], sh.hnl[0], sh.col, sh.rot);
    if (gs->done) return; /* written by thread 0 before the block's last barrier */
    const double inv = gs->inv;
#pragma unroll
    for (int k = 0; k < E; ++k) {
        const int64_t i = t + (int64_t)k * GSF_T;
        if (i < N) V[(int64_t)(j + 1) * ld + i] = inv * x[k];
    }
    __syncthreads(); /* every thread has read gs->j and gs->done */
    if (t == 0) gs->j = j + 1;
}

template <int E>
__global__ __launch_bounds__(GSF_T) void gs_reg_kernel(GState *__restrict__ gs, double *__restrict__ V, int64_t ld,
                                                       const double *__restrict__ w, int64_t N,
                                                       double *__restrict__ H, int R, double *__restrict__ cs,
                                                       double *__restrict__ sn, double *__restrict__ gv)
{
    __shared__ GsrShared sh;
    if (gs->done) return; /* the whole block */
    gsr_body<E>(gs, V, ld, w, N, H, R, cs, sn, gv, sh);
}

/* The Gram-Schmidt part of an Arnoldi step over many blocks (CGS2), for
   vectors too long for one block.  Block b owns the element slice
   [b L, (b+1) L); a pass leaves one partial dot product per (column, block)
   in P[c][b] (nb blocks, at most two per lane of a wave), and the next kernel
   adds a column's partials over the lanes of one wave by a fixed tree, so no
   result depends on timing.  Bound by the latency of its four launches: 8192
   unknowns, 20 columns, 32 -> 19 us against partials added one after the other
   and slices of 256. */
constexpr int GSM_T = 256, GSM_W = GSM_T / 64, GSM_S = 128, GSM_NBMAX = 128, GSM_HMAX = 520;

/* slice length: a multiple of GSM_S giving at most GSM_NBMAX blocks */
static int64_t gsm_slice(int64_t N)
{
    const int64_t per = (N + (int64_t)GSM_S * GSM_NBMAX - 1) / ((int64_t)GSM_S * GSM_NBMAX);
    return GSM_S * std::max<int64_t>(1, per);
}

/* P[c][block] = V_c . w over the block's slice; wave c % GSM_W takes column c,
   four columns' loads in flight */
__device__ __forceinline__ void gsm_partial_dots(const double *__restrict__ V, int64_t ld, const double *w, int64_t i0,
                                                 int64_t n, int ncol, double *__restrict__ P, int nb)
{
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), ln = threadIdx.x & 63;
    for (int c0 = wv; c0 < ncol; c0 += 4 * GSM_W) {
        double s[4] = {0.0, 0.0, 0.0, 0.0};
        for (int64_t e = ln; e < n; e += 64) {
            const double we = w[i0 + e];
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const int c = min(c0 + k * GSM_W, ncol - 1);
                s[k] = fma(V[(int64_t)c * ld + i0 + e], we, s[k]);
            }
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const double v = wave_sum_dpp(s[k]);
            if (ln == 0 && c0 + k * GSM_W < ncol) P[(int64_t)(c0 + k * GSM_W) * nb + blockIdx.x] = v;
        }
    }
}

/* sum of a row of nb <= 128 partials, in every lane of a wave */
__device__ __forceinline__ double gsm_row(const double *__restrict__ P, int nb)
{
    const int ln = threadIdx.x & 63;
    double v = ln < nb ? P[ln] : 0.0;
    if (ln + 64 < nb) v += P[ln + 64];
    return wave_sum_dpp(v);
}

/* first pass: P[c][b] = V_c . w over slice b, c <= j */
__global__ __launch_bounds__(GSM_T) void gsm_dot_kernel(const GState *__restrict__ gs, const double *__restrict__ V,
                                                        int64_t ld, const double *__restrict__ w, int64_t N,
                                                        int64_t L, double *__restrict__ P)
{
    if (gs->done) return;
    const int64_t i0 = blockIdx.x * L;
    gsm_partial_dots(V, ld, w, i0, min(L, N - i0), gs->j + 1, P, gridDim.x);
}

/* h = sum_b Pin[.][b] (block 0 also stores it in hout); w -= sum_c h_c V_c on
   the slice, the columns shared by the two threads of an element; then either
   the partial dots of the new w (NORM = false, into Pout[c][b]) or its partial
   squared norm (NORM = true, into Pout[b]). */
template <bool NORM>
__global__ __launch_bounds__(GSM_T) void gsm_sub_kernel(const GState *__restrict__ gs, const double *__restrict__ V,
                                                        int64_t ld, double *w, int64_t N, int64_t L,
                                                        const double *__restrict__ Pin, double *__restrict__ hout,
                                                        double *__restrict__ Pout)
{
    __shared__ double hl[GSM_HMAX];
    __shared__ double half[GSM_S];
    __shared__ double red[GSM_S / 64];
    if (gs->done) return;
    const int t = threadIdx.x, wv = __builtin_amdgcn_readfirstlane(t >> 6), nb = gridDim.x;
    const int ncol = gs->j + 1;
#pragma unroll 4
    for (int c = wv; c < ncol; c += GSM_W) {
        const double h = gsm_row(Pin + (int64_t)c * nb, nb);
        if ((t & 63) == 0) {
            hl[c] = h;
            if (blockIdx.x == 0) hout[c] = h;
        }
    }
    __syncthreads();
    const int64_t i0 = blockIdx.x * L, n = min(L, N - i0);
    const int s = t & (GSM_S - 1), part = t / GSM_S; /* even or odd columns */
    double sq = 0.0;
    for (int64_t e0 = 0; e0 < n; e0 += GSM_S) {
        const int64_t e = min(e0 + s, n - 1), i = i0 + e;
        double v = part == 0 ? w[i] : 0.0;
#pragma unroll 8
        for (int c = part; c < ncol; c += 2) v = fma(-hl[c], V[(int64_t)c * ld + i], v);
        if (part == 1) half[s] = v;
        __syncthreads();
        if (part == 0 && e0 + s < n) {
            v += half[s];
            w[i] = v;
            sq = fma(v, v, sq);
        }
        __syncthreads();
    }
    if (NORM) {
        sq = wave_sum_dpp(sq);
        if ((t & 63) == 0 && part == 0) red[wv] = sq;
        __syncthreads();
        if (t == 0) Pout[blockIdx.x] = red[0] + red[1];
    } else {
        gsm_partial_dots(V, ld, w, i0, n, ncol, Pout, nb); /* the slice of w is written: the last barrier */
    }
}

/* ||w||^2 from the slice partials (block order), the Hessenberg column, then
   V_{j+1} = w / ||w|| and the advance; one block */
__global__ __launch_bounds__(GSF_T) void gsm_finish_kernel(GState *__restrict__ gs, double *__restrict__ V,
                                                           int64_t ld, const double *__restrict__ w, int64_t N,
                                                           const double *__restrict__ Pn, int nb,
                                                           double *__restrict__ H, int R, double *__restrict__ cs,
                                                           double *__restrict__ sn, double *__restrict__ gv,
                                                           const double *__restrict__ h1,
                                                           const double *__restrict__ h2)
{
    __shared__ double col[GSM_HMAX + 2], rot[2 * GSM_HMAX];
    __shared__ double hn;
    if (gs->done) return;
    const int t = threadIdx.x;
    const int j = gs->j;
    if (t < 64) {
        const double s2 = gsm_row(Pn, nb);
        if (t == 0) hn = s2;
    }
    __syncthreads();
    gs_finish_block(gs, H, R, cs, sn, gv, h1, h2, hn, col, rot);
    if (gs->done) return; /* written by thread 0 before the block's last barrier */
    const double inv = gs->inv;
    for (int64_t i = t; i < N; i += GSF_T) V[(int64_t)(j + 1) * ld + i] = inv * w[i];
    __syncthreads(); /* every thread has read gs->j and gs->done */
    if (t == 0) gs->j = j + 1;
}

/* start of a cycle: state, g = beta e_1 */
__global__ void gs_init_kernel(GState *__restrict__ gs, double *__restrict__ gv, int R, int kmax, double beta,
                               double thresh, double *xout)
{
    for (int i = threadIdx.x; i <= R; i += blockDim.x) gv[i] = i == 0 ? beta : 0.0;
    if (threadIdx.x == 0) {
        gs->j = 0;
        gs->kmax = kmax;
        gs->done = 0;
        gs->steps = 0;
        gs->thresh = thresh;
        gs->inv = 0.0;
        gs->resest = beta;
        gs->xout = xout;
    }
}

/* start of the first cycle of a zero-guess solve whose ||b|| stays on the
   device: beta = ||b|| from its square bn2[0], V_0 = b / beta (zero when b
   is), g = beta e_1, the stopping threshold half_tol * beta, and ||b|| kept in
   the state for the host's first read (a zero b ends the cycle at once) */
__global__ void gs_init_dev_kernel(GState *__restrict__ gs, double *__restrict__ gv, int R, int kmax,
                                   double half_tol, const double *__restrict__ bn2, const double *__restrict__ b,
                                   double *__restrict__ V0, int64_t N, double *xout)
{
    const double beta = sqrt(bn2[0]);
    const double sc = beta > 0.0 ? 1.0 / beta : 0.0;
    const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (i < N) V0[i] = sc * b[i];
    if (blockIdx.x != 0) return;
    for (int k = threadIdx.x; k <= R; k += blockDim.x) gv[k] = k == 0 ? beta : 0.0;
    if (threadIdx.x == 0) {
        gs->j = 0;
        gs->kmax = kmax;
        gs->done = beta > 0.0 ? 0 : 1;
        gs->steps = 0;
        gs->thresh = half_tol * beta;
        gs->inv = 0.0;
        gs->resest = beta;
        gs->bnorm = beta;
        gs->xout = xout;
    }
}

/* ---- end of a cycle, enqueued after its last chunk of steps; every kernel
   does nothing unless the cycle has ended (gs->done) ---- */
/* y = R_k^{-1} g_k for the k = steps leading columns (upper triangular back
   substitution), one wave: the row sums are split over the 64 lanes.  Also
   arms the tail state for the operator application that follows: density
   x (column 0, stride 0), active only when the cycle has ended. */
__global__ __launch_bounds__(64) void gs_solve_kernel(const GState *__restrict__ gs, GState *__restrict__ tail,
                                                      const double *__restrict__ H, int R,
                                                      const double *__restrict__ gv, double *__restrict__ y)
{
    if (!gs->done) {
        if (threadIdx.x == 0) tail->done = 1;
        return;
    }
    const int k = gs->steps;
    for (int i = k - 1; i >= 0; --i) {
        double s = 0.0;
        for (int m = i + 1 + (int)threadIdx.x; m < k; m += 64) s = fma(H[(int64_t)i * R + m], y[m], s);
        for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off);
        if (threadIdx.x == 0) y[i] = (gv[i] - s) / H[(int64_t)i * R + i];
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        tail->j = 0;
        tail->done = 0;
    }
}

/* x += sum_{c < steps} y[c] V_c */
__global__ void gs_addcols_kernel(const GState *__restrict__ gs, const double *__restrict__ V, int64_t ld,
                                  const double *__restrict__ y, double *__restrict__ x, int64_t N)
{
    const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (i >= N || !gs->done) return;
    const int k = gs->steps;
    double v = x[i];
    for (int c = 0; c < k; ++c) v = fma(y[c], V[c * ld + i], v);
    x[i] = v;
}

/* r = b - a and gs->rn2 = ||r||^2 (the true residual of the cycle's new
   iterate x, a = A x), and x copied to gs->xout when set; one block; the sum
   runs in a fixed order (each thread's strided elements, wave sums, waves in
   order) */
__global__ __launch_bounds__(GSF_T) void tail_residual_kernel(const GState *__restrict__ tail,
                                                              const double *__restrict__ b,
                                                              const double *__restrict__ a,
                                                              const double *__restrict__ x, double *__restrict__ r,
                                                              int64_t N, GState *__restrict__ gs)
{
    __shared__ double red[GSF_W];
    if (tail->done) return;
    const int t = threadIdx.x;
    double *xout = gs->xout;
    double s = 0.0;
    for (int64_t i = t; i < N; i += GSF_T) {
        const double v = b[i] - a[i];
        r[i] = v;
        s = fma(v, v, s);
        if (xout) xout[i] = x[i];
    }
    s = wave_sum_dpp(s);
    if ((t & 63) == 0) red[t >> 6] = s;
    __syncthreads();
    if (t == 0) {
        double q = red[0];
        for (int k = 1; k < GSF_W; ++k) q += red[k];
        gs->rn2 = q;
    }
}

/* Start of a zero-guess FP64 solve in one block (vectors up to
   GS_START_NMAX): beta = ||bsrc||, b = bsrc (the solve's own copy), x = 0,
   V_0 = b / beta (zero when b is), g = beta e_1, the stopping threshold
   half_tol * beta, and beta kept in the state for the host's first read (a
   zero b ends the cycle at once).  The sum runs in a fixed order. */
constexpr int64_t GS_START_NMAX = 64 * GSF_T;
__global__ __launch_bounds__(GSF_T) void gs_start_kernel(GState *__restrict__ gs, double *__restrict__ gv, int R,
                                                         int kmax, double half_tol, const double *__restrict__ bsrc,
                                                         double *__restrict__ b, double *__restrict__ x,
                                                         double *__restrict__ V0, int64_t N, double *xout)
{
    __shared__ double red[GSF_W];
    __shared__ double bsh;
    const int t = threadIdx.x;
    double s = 0.0;
    for (int64_t i = t; i < N; i += GSF_T) {
        const double v = bsrc[i];
        b[i] = v;
        x[i] = 0.0;
        s = fma(v, v, s);
    }
    s = wave_sum_dpp(s);
    if ((t & 63) == 0) red[t >> 6] = s;
    __syncthreads();
    if (t == 0) {
        double q = red[0];
        for (int k = 1; k < GSF_W; ++k) q += red[k];
        bsh = sqrt(q);
    }
    __syncthreads();
    const double beta = bsh;
    const double sc = beta > 0.0 ? 1.0 / beta : 0.0;
    for (int64_t i = t; i < N; i += GSF_T) V0[i] = sc * bsrc[i];
    for (int k = t; k <= R; k += GSF_T) gv[k] = k == 0 ? beta : 0.0;
    if (t == 0) {
        gs->j = 0;
        gs->kmax = kmax;
        gs->done = beta > 0.0 ? 0 : 1;
        gs->steps = 0;
        gs->thresh = half_tol * beta;
        gs->inv = 0.0;
        gs->resest = beta;
        gs->bnorm = beta;
        gs->rn2 = 0.0;
        gs->xout = xout;
    }
}

__global__ void fill_i32_kernel(int32_t *__restrict__ x, int32_t v, int64_t N)
{
    const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (i < N) x[i] = v;
}

__global__ void fill_kernel(double *__restrict__ x, double v, int64_t N)
{
    const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (i < N) x[i] = v;
}

#include "fmm.h"
#include "fourier.h"

/* ------------------------------------------------------------------------ */
/* host helpers                                                              */
/* ------------------------------------------------------------------------ */
static inline unsigned nblocks(int64_t n, int t) { return (unsigned)((n + t - 1) / t); }

template <class T>
static mhlp_status dalloc(T **p, int64_t n)
{
    *p = nullptr;
    if (n <= 0) return MHLP_OK;
    hipError_t e = hipMalloc((void **)p, sizeof(T) * (size_t)n);
    if (e != hipSuccess) return fail(MHLP_NO_MEMORY, std::string("hipMalloc: ") + hipGetErrorString(e));
    return MHLP_OK;
}

#define TRY(x)                          \
    do {                                \
        mhlp_status s_ = (x);           \
        if (s_ != MHLP_OK) return s_;   \
    } while (0)

/* ------------------------------------------------------------------------ */
/* FMM tree (host side): root square, stable counting sort of sources and    */
/* targets into leaf boxes, per-level occupancy, leaf work items, and the    */
/* translation tables (computed on the device)                               */
/* ------------------------------------------------------------------------ */
namespace mhlp {
struct FmmTree {
    FmmDev d{};
    std::vector<void *> bufs;
    int32_t order = 0, level = 0;
    ~FmmTree()
    {
        for (void *b : bufs)
            if (b) (void)hipFree(b);
    }
    template <class T>
    mhlp_status alloc(T **p, int64_t n)
    {
        mhlp_status s = dalloc(p, n < 1 ? 1 : n);
        if (s == MHLP_OK) bufs.push_back((void *)*p);
        return s;
    }
};
} // namespace mhlp
using mhlp::FmmTree;

static int fmm_coord(double v, double v0, double side, int nb)
{
    const double f = std::floor((v - v0) / side);
    return f < 0.0 ? 0 : (f >= (double)nb ? nb - 1 : (int)f);
}

struct FmmGeom {
    double x0, y0, S;
};

/* root square of the sources and targets (same definition as the oracle's) */
static FmmGeom fmm_root(const std::vector<double> &sx, const std::vector<double> &sy, const std::vector<double> &tx,
                        const std::vector<double> &ty)
{
    double xmin = INFINITY, xmax = -INFINITY, ymin = INFINITY, ymax = -INFINITY;
    auto upd = [&](const std::vector<double> &a, const std::vector<double> &b) {
        for (size_t k = 0; k < a.size(); ++k) {
            xmin = std::min(xmin, a[k]);
            xmax = std::max(xmax, a[k]);
            ymin = std::min(ymin, b[k]);
            ymax = std::max(ymax, b[k]);
        }
    };
    upd(sx, sy);
    upd(tx, ty);
    const double cx = 0.5 * (xmin + xmax), cy = 0.5 * (ymin + ymax);
    const double ext = std::max(xmax - xmin, ymax - ymin);
    const double S = ext > 0.0 ? ext * (1.0 + 0x1p-20) : 1.0;
    const double hS = 0.5 * S;
    return FmmGeom{cx - hS, cy - hS, S};
}

/* every node of every near panel of a target lies in the target's 3x3 leaf
   neighbourhood (then skipping near panels in the direct part skips them everywhere) */
static bool fmm_contains_near(const FmmGeom &G, int L, const std::vector<double> &sx, const std::vector<double> &sy,
                              const std::vector<double> &tx, const std::vector<double> &ty,
                              const std::vector<int32_t> &nptr, const std::vector<int32_t> &npan)
{
    const int nb = 1 << L;
    const double side = G.S / (double)nb;
    const int64_t M = (int64_t)tx.size(), Np = (int64_t)sx.size() / 16;
    for (int64_t i = 0; i < M; ++i) {
        const int ix = fmm_coord(tx[i], G.x0, side, nb), iy = fmm_coord(ty[i], G.y0, side, nb);
        for (int32_t q = nptr[i]; q < nptr[i + 1]; ++q) {
            const int64_t pn = npan[q];
            if (pn < 0 || pn >= Np) continue;
            for (int j = 0; j < 16; ++j) {
                const int jx = fmm_coord(sx[16 * pn + j], G.x0, side, nb);
                const int jy = fmm_coord(sy[16 * pn + j], G.y0, side, nb);
                if (std::abs(jx - ix) > 1 || std::abs(jy - iy) > 1) return false;
            }
        }
    }
    return true;
}

/* Build the tree.  Sources: host copies sx, sy and device arrays dsx.. (gathered
   into leaf order; dnx/dny NULL for the volume); targets tx, ty (host), or the
   sources themselves when same_points. */
static mhlp_status fmm_build(FmmTree *F, const FmmGeom &G, int L, int p, double alpha,
                             const std::vector<double> &sx, const std::vector<double> &sy,
                             const std::vector<double> &tx, const std::vector<double> &ty, bool same_points,
                             const double *dsx, const double *dsy, const double *dsw, const double *dnx,
                             const double *dny, hipStream_t st)
{
    FmmDev &T = F->d;
    const int nb = 1 << L;
    const int64_t nleaf = (int64_t)nb * nb, N = (int64_t)sx.size(), M = same_points ? N : (int64_t)tx.size();
    T.L = L;
    T.p = p;
    T.alpha = alpha;
    T.x0 = G.x0;
    T.y0 = G.y0;
    T.S = G.S;
    for (int l = 0; l <= L; ++l) {
        T.side[l] = G.S / (double)(1 << l);
        T.sig[l] = std::min(1.0, alpha * T.side[l]);
    }
    T.lstart = L + 1;
    for (int l = 2; l <= L; ++l)
        if (alpha * 0.586 * T.side[l] <= 40.0) {
            T.lstart = l;
            break;
        }
    /* stable counting sorts into the leaves */
    auto sort_pts = [&](const std::vector<double> &ax, const std::vector<double> &ay, int64_t n,
                        std::vector<int32_t> &start, std::vector<int32_t> &idx) {
        std::vector<int32_t> leaf(n);
        start.assign(nleaf + 1, 0);
        for (int64_t k = 0; k < n; ++k) {
            const int ix = fmm_coord(ax[k], G.x0, T.side[L], nb), iy = fmm_coord(ay[k], G.y0, T.side[L], nb);
            leaf[k] = iy * nb + ix;
            ++start[leaf[k] + 1];
        }
        for (int64_t b = 0; b < nleaf; ++b) start[b + 1] += start[b];
        std::vector<int32_t> pos(start.begin(), start.end() - 1);
        idx.resize(n);
        for (int64_t k = 0; k < n; ++k) idx[pos[leaf[k]]++] = (int32_t)k;
    };
    std::vector<int32_t> sstart, sidx, tstart, tidx;
    sort_pts(sx, sy, N, sstart, sidx);
    if (same_points) {
        tstart = sstart;
        tidx = sidx;
    } else {
        sort_pts(tx, ty, M, tstart, tidx);
    }
    /* occupancy per level */
    const int64_t nall = mhlp::lev4(L + 1);
    std::vector<int32_t> socc(nall, 0), tocc(nall, 0);
    for (int64_t b = 0; b < nleaf; ++b) {
        socc[mhlp::lev4(L) + b] = sstart[b + 1] - sstart[b];
        tocc[mhlp::lev4(L) + b] = tstart[b + 1] - tstart[b];
    }
    for (int l = L - 1; l >= 0; --l) {
        const int n1 = 1 << l;
        for (int iy = 0; iy < 2 * n1; ++iy)
            for (int ix = 0; ix < 2 * n1; ++ix) {
                const int64_t c = mhlp::lev4(l + 1) + iy * 2 * n1 + ix, pb = mhlp::lev4(l) + (iy >> 1) * n1 + (ix >> 1);
                socc[pb] += socc[c];
                tocc[pb] += tocc[c];
            }
    }
    /* leaf work items */
    std::vector<int32_t> wbox, wt0;
    for (int64_t b = 0; b < nleaf; ++b)
        for (int32_t t0 = tstart[b]; t0 < tstart[b + 1]; t0 += mhlp::FMM_TILE) {
            wbox.push_back((int32_t)b);
            wt0.push_back(t0);
        }
    T.nwork = (int)wbox.size();
    /* expansions and tables */
    int64_t eo = 0, to = 0;
    const int64_t rl = 3 * p + 1;
    std::vector<mhlp::FmmRow> rows;
    for (int l = 0; l <= L; ++l) {
        T.eoff[l] = T.t2l[l] = T.tmm[l] = T.tll[l] = 0;
        if (l < T.lstart) continue;
        T.eoff[l] = eo;
        eo += 2 * ((int64_t)1 << (2 * l)) * (p + 1);
        T.t2l[l] = to;
        for (int ox = -3; ox <= 3; ++ox)
            for (int oy = -3; oy <= 3; ++oy) {
                if (std::abs(ox) <= 1 && std::abs(oy) <= 1) continue;
                rows.push_back(mhlp::FmmRow{-ox * T.side[l], -oy * T.side[l], T.sig[l],
                                            to + ((ox + 3) * 7 + (oy + 3)) * rl, 0});
            }
        to += 49 * rl;
        if (l < L) {
            const double hc = 0.5 * T.side[l + 1];
            T.tmm[l] = to;
            for (int ch = 0; ch < 4; ++ch)
                rows.push_back(mhlp::FmmRow{(ch & 1) ? hc : -hc, (ch >> 1) ? hc : -hc, T.sig[l], to + ch * rl, 1});
            to += 4 * rl;
            T.tll[l] = to;
            for (int ch = 0; ch < 4; ++ch)
                rows.push_back(mhlp::FmmRow{(ch & 1) ? hc : -hc, (ch >> 1) ? hc : -hc, T.sig[l + 1], to + ch * rl, 1});
            to += 4 * rl;
        }
    }
    int32_t *d_sstart, *d_tstart, *d_sidx, *d_tidx, *d_socc, *d_tocc, *d_wbox, *d_wt0, *d_lpan = nullptr;
    double *d_lx, *d_ly, *d_lw, *d_lnx = nullptr, *d_lny = nullptr;
    cplx *d_mexp, *d_lexp, *d_tab;
    TRY(F->alloc(&d_sstart, nleaf + 1));
    TRY(F->alloc(&d_tstart, nleaf + 1));
    TRY(F->alloc(&d_sidx, N));
    TRY(F->alloc(&d_tidx, M));
    TRY(F->alloc(&d_socc, nall));
    TRY(F->alloc(&d_tocc, nall));
    TRY(F->alloc(&d_wbox, T.nwork));
    TRY(F->alloc(&d_wt0, T.nwork));
    TRY(F->alloc(&d_lx, N));
    TRY(F->alloc(&d_ly, N));
    TRY(F->alloc(&d_lw, N));
    if (dnx) {
        TRY(F->alloc(&d_lnx, N));
        TRY(F->alloc(&d_lny, N));
        TRY(F->alloc(&d_lpan, N));
    }
    TRY(F->alloc(&d_mexp, eo));
    TRY(F->alloc(&d_lexp, mhlp::FMM_CH * eo));
    TRY(F->alloc(&d_tab, to));
    mhlp::FmmRow *d_rows = nullptr;
    double *d_scr = nullptr;
    const int nrows = (int)rows.size();
    if (nrows > 0) {
        TRY(dalloc(&d_rows, nrows));
        mhlp_status s2 = dalloc(&d_scr, (int64_t)nrows * (2 * p + 1));
        if (s2 != MHLP_OK) {
            (void)hipFree(d_rows);
            return s2;
        }
    }
    auto up = [&](void *d, const void *h, size_t bytes) -> hipError_t {
        return bytes ? hipMemcpyAsync(d, h, bytes, hipMemcpyHostToDevice, st) : hipSuccess;
    };
    hipError_t e = up(d_sstart, sstart.data(), sstart.size() * 4);
    if (e == hipSuccess) e = up(d_tstart, tstart.data(), tstart.size() * 4);
    if (e == hipSuccess) e = up(d_sidx, sidx.data(), sidx.size() * 4);
    if (e == hipSuccess) e = up(d_tidx, tidx.data(), tidx.size() * 4);
    if (e == hipSuccess) e = up(d_socc, socc.data(), socc.size() * 4);
    if (e == hipSuccess) e = up(d_tocc, tocc.data(), tocc.size() * 4);
    if (e == hipSuccess) e = up(d_wbox, wbox.data(), wbox.size() * 4);
    if (e == hipSuccess) e = up(d_wt0, wt0.data(), wt0.size() * 4);
    if (e == hipSuccess && nrows > 0) e = up(d_rows, rows.data(), rows.size() * sizeof(mhlp::FmmRow));
    if (e == hipSuccess) {
        mhlp::fmm_gather_kernel<<<nblocks(N, 256), 256, 0, st>>>(d_sidx, N, dsx, dsy, dsw, dnx, dny, d_lx, d_ly, d_lw,
                                                                 d_lnx, d_lny, d_lpan);
        if (nrows > 0)
            mhlp::fmm_tables_kernel<<<nblocks(nrows, 64), 64, 0, st>>>(d_rows, nrows, p, alpha, d_tab, d_scr);
        e = hipGetLastError();
    }
    if (e == hipSuccess) e = hipStreamSynchronize(st);
    if (d_rows) (void)hipFree(d_rows);
    if (d_scr) (void)hipFree(d_scr);
    if (e != hipSuccess) return fail(MHLP_HIP_ERROR, std::string("fmm build: ") + hipGetErrorString(e));
    T.sstart = d_sstart;
    T.tstart = d_tstart;
    T.sidx = d_sidx;
    T.tidx = d_tidx;
    T.socc = d_socc;
    T.tocc = d_tocc;
    T.wbox = d_wbox;
    T.wt0 = d_wt0;
    T.lx = d_lx;
    T.ly = d_ly;
    T.lw = d_lw;
    T.lnx = d_lnx;
    T.lny = d_lny;
    T.lpan = d_lpan;
    T.mexp = d_mexp;
    T.lexp = d_lexp;
    T.lch = eo;
    for (int l = 0; l <= mhlp::FMM_LMAX; ++l) T.nch[l] = ((int64_t)1 << (2 * l)) < mhlp::FMM_CH_BOXES ? mhlp::FMM_CH : 1;
    T.tab = d_tab;
    F->order = p;
    F->level = L;
    return MHLP_OK;
}

/* upward and downward passes; the leaf kernel is launched by the caller */
template <bool SLP, bool DLP>
static void fmm_passes(const FmmTree *F, const double *sigma, const double *mu, hipStream_t st)
{
    const FmmDev &T = F->d;
    if (T.lstart > T.L) return;
    mhlp::fmm_p2m_kernel<SLP, DLP><<<(unsigned)(1u << (2 * T.L)), 64, 0, st>>>(T, sigma, mu);
    for (int l = T.L - 1; l >= T.lstart; --l)
        mhlp::fmm_m2m_kernel<SLP, DLP><<<(unsigned)(1u << (2 * l)), 256, 0, st>>>(T, l);
    for (int l = T.lstart; l <= T.L; ++l)
        mhlp::fmm_down_kernel<SLP, DLP><<<dim3(1u << (2 * l), (unsigned)T.nch[l]), 64 * mhlp::FMM_DW, 0, st>>>(T, l);
}

template <bool SLP, bool DLP>
static void fmm_far_t(const FmmTree *F, const FarArgs &A, hipStream_t st)
{
    fmm_passes<SLP, DLP>(F, A.sigma, A.mu, st);
    if (F->d.nwork > 0)
        mhlp::fmm_leaf_kernel<SLP, DLP, 0><<<(unsigned)F->d.nwork, 64 * mhlp::FMM_LW, 0, st>>>(F->d, A, mhlp::FmmVol{});
}

static GeoView view(const mhlp_geometry *g)
{
    GeoView G;
    G.x = g->soa;
    G.y = g->soa + g->N;
    G.pa = g->pa;
    G.ph = g->ph;
    G.pcx = g->pcx;
    G.pcy = g->pcy;
    G.prad = g->prad;
    G.N = g->N;
    G.Np = g->Np;
    return G;
}

/* ------------------------------------------------------------------------ */
/* geometry API                                                              */
/* ------------------------------------------------------------------------ */
extern "C" mhlp_status mhlp_geometry_create(int32_t n_curves, const int32_t *curve_panel_offsets,
                                            int32_t nodes_per_panel, const double *node_soa,
                                            const double *panel_ends, void *stream, mhlp_geometry **out)
{
    if (!out) return fail(MHLP_INVALID_ARG, "out is NULL");
    *out = nullptr;
    if (!node_soa) return fail(MHLP_INVALID_ARG, "node_soa is NULL");
    if (!curve_panel_offsets) return fail(MHLP_INVALID_ARG, "curve_panel_offsets is NULL");
    if (n_curves < 1) return fail(MHLP_INVALID_ARG, "n_curves must be >= 1");
    if (nodes_per_panel != 16) return fail(MHLP_UNSUPPORTED, "nodes_per_panel must be 16");
    if (curve_panel_offsets[0] != 0) return fail(MHLP_INVALID_ARG, "curve_panel_offsets[0] must be 0");
    for (int32_t c = 0; c < n_curves; ++c)
        if (curve_panel_offsets[c + 1] <= curve_panel_offsets[c])
            return fail(MHLP_INVALID_ARG, "curve_panel_offsets must increase (every curve has a panel)");
    const int64_t n_panels = curve_panel_offsets[n_curves];
    if (n_panels > (INT_MAX / 16)) return fail(MHLP_INVALID_ARG, "n_panels out of range");
    hipStream_t st = (hipStream_t)stream;
    mhlp_geometry *g = new mhlp_geometry();
    HIPCHECK(hipGetDevice(&g->device));
    g->Np = n_panels;
    g->N = 16 * n_panels;
    g->curve_off.assign(curve_panel_offsets, curve_panel_offsets + n_curves + 1);
    const int64_t N = g->N, Np = g->Np;
    mhlp_status s;
    if ((s = dalloc(&g->soa, 6 * N)) || (s = dalloc(&g->w, N)) || (s = dalloc(&g->nx, N)) || (s = dalloc(&g->ny, N)) ||
        (s = dalloc(&g->kappa, N)) || (s = dalloc(&g->pa, 32 * Np)) || (s = dalloc(&g->ph, Np)) ||
        (s = dalloc(&g->pcx, Np)) || (s = dalloc(&g->pcy, Np)) || (s = dalloc(&g->prad, Np))) {
        mhlp_geometry_destroy(g);
        return s;
    }
    hipError_t e = hipMemcpyAsync(g->soa, node_soa, sizeof(double) * 6 * N, hipMemcpyDeviceToDevice, st);
    if (e == hipSuccess) {
        geom_prep_kernel<<<nblocks(Np, 64), 64, 0, st>>>(g->soa, N, Np, g->w, g->nx, g->ny, g->kappa, g->pa, g->ph,
                                                          g->pcx, g->pcy, g->prad);
        e = hipGetLastError();
    }
    std::vector<int32_t> flags;
    int32_t *dnext = nullptr;
    if (e == hipSuccess && panel_ends) {
        std::vector<int32_t> next((size_t)Np);
        for (int32_t c = 0; c < n_curves; ++c)
            for (int32_t p = curve_panel_offsets[c]; p < curve_panel_offsets[c + 1]; ++p)
                next[p] = (p + 1 < curve_panel_offsets[c + 1]) ? p + 1 : curve_panel_offsets[c];
        flags.resize((size_t)Np);
        /* one buffer: next panels, then the flags */
        if ((s = dalloc(&dnext, 2 * Np))) {
            mhlp_geometry_destroy(g);
            return s;
        }
        e = hipMemcpyAsync(dnext, next.data(), sizeof(int32_t) * Np, hipMemcpyHostToDevice, st);
        if (e == hipSuccess) {
            panel_ends_kernel<<<nblocks(Np, 64), 64, 0, st>>>(g->pa, g->soa, g->soa + N, g->ph, panel_ends, dnext, Np,
                                                              PANEL_ENDS_TOL, dnext + Np);
            e = hipGetLastError();
        }
        if (e == hipSuccess)
            e = hipMemcpyAsync(flags.data(), dnext + Np, sizeof(int32_t) * Np, hipMemcpyDeviceToHost, st);
    }
    if (e == hipSuccess) e = hipStreamSynchronize(st);
    if (dnext) (void)hipFree(dnext);
    if (e != hipSuccess) {
        mhlp_geometry_destroy(g);
        return fail(MHLP_HIP_ERROR, std::string("geometry_create: ") + hipGetErrorString(e));
    }
    for (int64_t p = 0; p < (int64_t)flags.size(); ++p)
        if (flags[p]) {
            mhlp_geometry_destroy(g);
            return fail(MHLP_INVALID_ARG,
                        std::string("panel_ends: panel ") + std::to_string(p) +
                            ((flags[p] & 1) ? " does not end where its node polynomial ends"
                                            : " does not end where the next panel of its curve starts"));
        }
    *out = g;
    return MHLP_OK;
}

extern "C" mhlp_status mhlp_geometry_info(const mhlp_geometry *g, int64_t *n_nodes, int64_t *n_panels,
                                          int32_t *n_curves, int32_t *curve_panel_offsets, int32_t cap)
{
    if (!g) return fail(MHLP_INVALID_ARG, "geometry is NULL");
    const int32_t nc = (int32_t)g->curve_off.size() - 1;
    if (n_nodes) *n_nodes = g->N;
    if (n_panels) *n_panels = g->Np;
    if (n_curves) *n_curves = nc;
    if (curve_panel_offsets)
        for (int32_t c = 0; c <= nc && c < cap; ++c) curve_panel_offsets[c] = g->curve_off[c];
    return MHLP_OK;
}

extern "C" mhlp_status mhlp_geometry_destroy(mhlp_geometry *g)
{
    if (!g) return MHLP_OK;
    double *ptrs[] = {g->soa, g->w, g->nx, g->ny, g->kappa, g->pa, g->ph, g->pcx, g->pcy, g->prad};
    for (double *p : ptrs)
        if (p) (void)hipFree(p);
    delete g;
    return MHLP_OK;
}

extern "C" mhlp_status mhlp_geometry_arrays(const mhlp_geometry *g, const double **w, const double **nx,
                                            const double **ny, const double **kappa)
{
    if (!g) return fail(MHLP_INVALID_ARG, "geometry is NULL");
    if (w) *w = g->w;
    if (nx) *nx = g->nx;
    if (ny) *ny = g->ny;
    if (kappa) *kappa = g->kappa;
    return MHLP_OK;
}

/* ------------------------------------------------------------------------ */
/* plan API                                                                  */
/* ------------------------------------------------------------------------ */
/* Source splits of the far field: ns requested splits of the panel range
   (1 = none); the partial-sum buffer grows as needed. */
static mhlp_status plan_set_split(mhlp_plan *P, int ns)
{
    const int64_t Np = P->g->Np;
    if (ns < 1) ns = 1;
    if (ns > Np) ns = (int)Np;
    const int32_t pps = (int32_t)((Np + ns - 1) / ns);
    const int nsplit = (int)((Np + pps - 1) / pps);
    const int64_t need = nsplit > 1 ? (P->onsurf ? 2 : 4) * (int64_t)nsplit * P->M : 0;
    if (need > P->part_cap) {
        if (P->part) {
            HIPCHECK(hipDeviceSynchronize()); /* queued launches may still use it */
            (void)hipFree(P->part);
            P->part = nullptr;
            P->part_cap = 0;
        }
        TRY(dalloc(&P->part, need));
        P->part_cap = need;
    }
    P->pps = pps;
    P->nsplit = nsplit;
    return MHLP_OK;
}

extern "C" mhlp_status mhlp_plan_destroy(mhlp_plan *P)
{
    if (!P) return MHLP_OK;
    if (!P->onsurf) {
        if (P->tx) (void)hipFree(P->tx);
        if (P->ty) (void)hipFree(P->ty);
    }
    for (auto &gp : P->graphs)
        if (gp.second.exec) (void)hipGraphExecDestroy(gp.second.exec);
    if (P->cap_stream) (void)hipStreamDestroy(P->cap_stream);
    void *ptrs[] = {P->near_ptr, P->near_panel, P->near_tgt, P->near_ts, P->wslp,  P->wdlp,    P->ws,
                    P->hdev,     P->part,       P->gdev,     P->perm,    P->wgrad, P->wstk,    P->wstkg,
                    P->wcls,     P->fqd};
    for (void *p : ptrs)
        if (p) (void)hipFree(p);
    delete P->fmm;
    if (P->tree) {
        void *tp[] = {P->tree_mem, P->tree_items, P->tree->part, P->tree->base};
        for (void *p : tp)
            if (p) (void)hipFree(p);
        delete P->tree;
    }
    if (P->hhost) (void)hipHostFree(P->hhost);
    if (P->gstate_host) (void)hipHostFree(P->gstate_host);
    delete P;
    return MHLP_OK;
}

/* The fine pieces' scales at the plan's alpha (read by every far kernel). */
static mhlp_status far_scales_setup(mhlp_plan *P, hipStream_t st)
{
    double fq[FINE_SCALES];
    fine_scales(P->alpha, fq);
    TRY(dalloc(&P->fqd, FINE_SCALES));
    HIPCHECK(hipMemcpyAsync(P->fqd, fq, sizeof(fq), hipMemcpyHostToDevice, st));
    HIPCHECK(hipStreamSynchronize(st)); /* fq ends here */
    return MHLP_OK;
}

/* The (wave of 64 targets, panel) class table of the mixed-precision tiles (built on the stream after the near lists, which it reads). */
static mhlp_status far_class_setup(mhlp_plan *P, hipStream_t st)
{
    const int64_t M = P->M, Np = P->g->Np;
    const int64_t TB = (M + FT_THREADS - 1) / FT_THREADS;
    TRY(dalloc(&P->wcls, TB * (FT_THREADS / 64) * Np));
    far_class_kernel<<<(unsigned)TB, FT_THREADS, 0, st>>>(P->tx, P->ty, M, P->g->soa, P->g->soa + P->g->N, Np,
                                                          P->alpha, P->near_ptr, P->near_panel, P->wcls);
    HIPCHECK(hipGetLastError());
    HIPCHECK(hipStreamSynchronize(st)); /* later calls may come on other streams */
    return MHLP_OK;
}

/* Launch shape of far_tree_kernel for G groups of U units of work each
   (tree_cost): 2^e waves a group, in blocks of 8 or, from few waves, 4; direct
   items in 2^cut units.  More waves shorten a group's sum until the chip is
   full (thousands of them) or a wave's share falls to a unit or two.  Waves a
   group of the fastest of 12 to 30 shapes, over curves of 16 to 256 panels and
   alpha = 1e-3 to 500 (potentials, gradients, stresslet):
       G        1    5   11   24   47   79  125  313  469  704 1016 1719
     U ~  32       128  128   64   64   32   32   16   16    8    8    4
     U ~ 128  256  256  128  128   64   64   64   32   16    8    8    4
     U ~ 512  512  256  256  256  128  128   64   32   32   16    8    8
   and cut 3 below one unit a wave, 0 from nine on (the stresslet from six on; potentials,
   512 panels on the curve, 528 units, 6 a wave, 58 against 53).  The formula is within
   3.4% of the fastest on average, 33% at worst.
   Where far items are left out (tree.h) the second pass needs the group's sum.  Off
   the curve one block makes both, which pays from 400 groups on (both layers, us, left
   out | split: alpha = 500, 256 panels, 313 groups 152 | 115, 469 145 | 160, 1016 162 |
   305; 64 panels, alpha = 100, 469 groups 68 | 83), of 8 waves, or 4 for many groups of
   little work (1719 groups, 64 panels, alpha = 500: 76 against 89; 256 panels 250
   against 183).  On the curve, where few panels are near a group, each pass is a
   launch: if almost half of a group's panels are summed directly, in 400 units or
   more, over 150 classes of z, or 500 over 90 (double layer, smooth density | one that
   spans 300 decades, of which little can be left out | split, nothing left out: alpha =
   500, 256 panels 22 | 26 | 36, 512 29 | 37 | 93, 1024 44 | 76 | 344; alpha = 200, 198
   panels 25 | 37 | 38; both passes in one launch, smooth: 61 classes, 400 panels 61 | . |
   45; 512 panels, a third of them direct, 58 | . | 53; a solve whose density spans
   decades 0.32 ms, 0.23 with nothing left out, 0.20 in two launches).
   Up to 50 groups, 85 on the curve: one block of 16 waves a CU, up to 100 two of 8,
   in place of powers of two, where some CUs get a block more than others (us,
   formula and this; on the curve, double layer: 139 panels, 35 groups, alpha = 100:
   26.0, 20.6; 198 panels 36.8, 29.8; 70 panels, alpha = 350: 14.5, 11.1; 300 panels,
   alpha = 1: 21.3, 17.3, but 100 groups 20.8, 21.1; off it, 12 to 45 shapes at 180
   plans: 15% off the fastest at 30 to 60 groups, 4% with this, 13% and 6% at 60 to
   100), and from there to 280 groups of less than 150 units four blocks of 8 (10%, 5%
   at 250), six up to 134 with 100 panels and more (118 groups, alpha = 5, 256 panels
   28.2, 25.2; 24 panels 20.6, 23.5).  On the curve, units of 2 sources below 100 units a group (128 panels,
   alpha = 20: 15.1, of 4 16.3).  The stresslet's kernels hold fewer waves. */
constexpr int TREE_CUS = 256;
static mhlp_plan::TreeShape tree_shape(int64_t G, double U, int64_t Np, bool curve, bool stokes)
{
    if (!stokes && G >= (curve ? 1 : 12)) {
        if (G <= (curve ? 85 : 50))
            return {16, (int)std::min<int64_t>(curve ? 14 : 16, TREE_CUS / G), curve && U < 100.0 ? 3 : U < 480.0 ? 2 : 1};
        if (!curve && G <= 100) return {8, (int)(2 * TREE_CUS / G), 2};
        if (!curve && G <= 280 && U < 150.0) return {8, G < 135 && Np >= 100 ? 6 : 4, 2};
    }
    const double lu = std::log2(std::max(8.0, U));
    int e = (int)std::floor(9.5 - 0.55 * std::log2((double)G) + 0.3 * (lu - 6.0));
    e = std::max(2, std::min({e, (int)lu + 2, 9}));
    if (G >= 1200) e = 2;
    const int cut = lu - e < 0.25 && e >= 6 ? 3 : lu - e < (stokes ? 2.5 : 3.1) ? 2 : 0;
    if (e <= 3) return {1 << e, 1, cut};
    if (e == 4) return {4, 4, cut};
    return {8, 1 << (e - 3), cut};
}

/* Up to TREE_DIRECT_MAX (group, panel) pairs an off-surface plan is summed pair by
   pair, which takes no longer than moments and expansions (us, single layer |
   stresslet, lists and direct, alpha = 1: 320 pairs 16.2, 10.9 | 23.9, 17.4; 752
   17.1, 12.2 | 29.1, 21.2; 1280 16.8, 21.0 | 26.1, 39.4; with 16 panels, whose
   clusters gather little, 2000 pairs 19.8, 15.7 | 35.9, 32.2); batches share the
   lists of plans on the curve, whose many groups run at once, so these keep their
   expansions.  Without expansions, charges are formed where they are read up to
   tree_raw_max pairs: a launch less, 2.5 us, for a multiplication a source and lane
   with a charge, four with a dipole (us, 50 panels at alpha = 95, formed and
   staged, single layer | double | both: 1000 pairs 12.2, 14.8 | 13.4, 14.6 | 15.8,
   16.5; 2500 15.7, 18.1 | 16.6, 17.8 | 20.8, 20.6; 5000 22.2, 24.2 | 24.7, 23.9 |
   30.8, 28.2; 16000 40.3, 41.4 | 47.7, 42.6 | 62.2, 52.2; gradients alike, the
   stresslet 22.8, 22.8 at 2500). */
constexpr int64_t TREE_DIRECT_MAX = 1024;
constexpr int64_t tree_raw_max(bool sigma, bool mu) { return !mu ? 16384 : sigma ? 2048 : 3072; }

/* Clusters, item lists and buffers of a plan's far field (tree.h), on
   the stream after the near lists, which the item lists read. */
static mhlp_status tree_setup(mhlp_plan *P, hipStream_t st)
{
    const mhlp_geometry *g = P->g;
    const int64_t M = P->M, Np = g->Np, G = (M + 63) / 64;
    P->tree = new mhlp::TreeDev();
    mhlp::TreeDev &T = *P->tree;
    T.Np = Np;
    T.expands = (P->onsurf && !P->stokes) || G * Np > (Np <= 24 ? 2 : 1) * TREE_DIRECT_MAX;
    while (T.nlev < mhlp::TR_LEV && ((int64_t)1 << T.nlev) <= Np) {
        T.off[T.nlev] = T.ncl;
        T.ncl += (Np + ((int64_t)1 << T.nlev) - 1) >> T.nlev;
        ++T.nlev;
    }
    T.stokes = P->stokes ? 1 : 0;
    int64_t bytes = 0;
    auto take = [&](int64_t n) {
        const int64_t o = bytes;
        bytes += (n + 255) / 256 * 256;
        return o;
    };
    const int64_t nmom = T.ncl * mhlp::tr_stride(P->stokes ? (P->onsurf ? 6 : 10) : (P->onsurf ? 4 : 8));
    const int64_t o_cc = take(16 * T.ncl), o_rmin = take(8 * mhlp::TR_RM * T.ncl), o_mom = take(8 * nmom);
    const int64_t o_small = take(P->stokes ? 8 * T.ncl * mhlp::tr_stride(P->onsurf ? 4 : 8) : 0);
    const int64_t o_st = take(8 * 48 * Np), o_flux = take(P->stokes && P->onsurf ? 8 * Np : 0), o_lb = take(4 * T.ncl);
    const int64_t o_at = take(16 * G), o_cnt = take(8 * G), o_order = take(4 * G), o_znear = take(4 * G), o_cost = take(32);
    const int64_t o_arr = take(4 * G);
    /* the lists are counted, then filled into storage of their size; they pass
       through slots of one entry a panel, for as many groups at a time as 64 MB
       hold (more than one such part: listed once to count and again to fill).
       Small plans keep slots and room for all entries, at most 8 MB, with the
       rest: allocations are most of what their creation costs here */
    const int64_t nrun = mhlp::tree_nrun(Np), slot = mhlp::TR_RUN * (int64_t)sizeof(uint2), per = nrun * (slot + 4);
    const int64_t Gc = std::min(G, std::max<int64_t>(1, ((int64_t)64 << 20) / per));
    const bool small = G * nrun * slot <= (int64_t)4 << 20;
    const int64_t o_tmp = take(small ? G * per : 0), o_items = take(small ? G * nrun * slot : 0);
    TRY(dalloc(&P->tree_mem, bytes));
    T.cc = reinterpret_cast<double *>(P->tree_mem + o_cc);
    T.rmin = reinterpret_cast<double *>(P->tree_mem + o_rmin);
    T.mom = reinterpret_cast<double *>(P->tree_mem + o_mom);
    T.st = reinterpret_cast<double *>(P->tree_mem + o_st);
    if (P->stokes && P->onsurf) T.flux = reinterpret_cast<double *>(P->tree_mem + o_flux);
    T.lb = reinterpret_cast<float *>(P->tree_mem + o_lb);
    T.at = reinterpret_cast<longlong2 *>(P->tree_mem + o_at);
    T.cnt = reinterpret_cast<int2 *>(P->tree_mem + o_cnt);
    T.order = reinterpret_cast<int32_t *>(P->tree_mem + o_order);
    T.znear = reinterpret_cast<int *>(P->tree_mem + o_znear);
    T.cost = reinterpret_cast<unsigned long long *>(P->tree_mem + o_cost);
    T.arrived = reinterpret_cast<uint32_t *>(P->tree_mem + o_arr);
    mhlp::tree_clusters_kernel<<<nblocks(T.ncl, 4), 256, 0, st>>>(T, g->soa, g->soa + g->N, g->ph, P->alpha,
                                                                  P->near_factor);
    HIPCHECK(hipMemsetAsync(T.cost, 0, 4 * sizeof(*T.cost), st));
    HIPCHECK(hipMemsetAsync(T.arrived, 0, 4 * G, st));
    char *tmp = small ? P->tree_mem + o_tmp : nullptr;
    bool have = small || hipMalloc((void **)&tmp, (size_t)(Gc * per)) == hipSuccess;
    uint2 *slots = reinterpret_cast<uint2 *>(tmp);
    uint32_t *runs = reinterpret_cast<uint32_t *>(slots + Gc * nrun * mhlp::TR_RUN);
    auto list = [&](int64_t g0) {
        const int64_t ng = std::min(Gc, G - g0);
        mhlp::tree_lists_kernel<<<nblocks(ng * nrun, 4), 256, 0, st>>>(T, P->tx, P->ty, M, g->soa, g->soa + g->N, P->alpha,
                                                                       P->near_ptr, P->near_panel, g0, ng, slots, runs);
        return (unsigned)ng;
    };
    unsigned long long cost[4] = {3ull * (unsigned long long)Np * (unsigned long long)G, 0, (unsigned long long)Np, 0};
    hipError_t e = hipSuccess;
    if (have) {
        for (int64_t g0 = 0; g0 < G; g0 += Gc) {
            const unsigned ng = list(g0);
            mhlp::tree_count_kernel<<<ng, 64, 0, st>>>(T, g0, runs);
        }
        mhlp::tree_order_kernel<<<1, 1024, 0, st>>>(T, G);
        e = hipGetLastError();
        unsigned long long c[4];
        if (e == hipSuccess) e = hipMemcpyAsync(c, T.cost, sizeof(c), hipMemcpyDeviceToHost, st);
        if (e == hipSuccess) e = hipStreamSynchronize(st);
        if (e == hipSuccess) {
            const size_t n = (size_t)std::max<unsigned long long>(1, c[2]);
            have = small || hipMalloc((void **)&P->tree_items, sizeof(uint2) * n) == hipSuccess;
            T.items = small ? reinterpret_cast<uint2 *>(P->tree_mem + o_items) : P->tree_items;
            if (have) std::copy(c, c + 4, cost);
        }
    }
    if (have && e == hipSuccess) {
        for (int64_t g0 = 0; g0 < G; g0 += Gc) {
            const unsigned ng = Gc < G ? list(g0) : (unsigned)G; /* else they are in the slots */
            mhlp::tree_fill_kernel<<<ng, 64, 0, st>>>(T, g0, slots, runs);
        }
        e = hipGetLastError();
        if (e == hipSuccess) e = hipStreamSynchronize(st); /* later calls may come on other streams */
    }
    if (tmp && !small) (void)hipFree(tmp);
    if (e != hipSuccess) return fail(MHLP_HIP_ERROR, std::string("plan_create lists: ") + hipGetErrorString(e));
    if (!have) {
        /* no memory for them: one list serves every group, all pairs one by one */
        (void)hipGetLastError();
        P->tree_items = nullptr;
        TRY(dalloc(&P->tree_items, Np));
        T.items = P->tree_items;
        mhlp::tree_direct_kernel<<<nblocks(std::max(G, Np), 256), 256, 0, st>>>(T, G);
        HIPCHECK(hipGetLastError());
        HIPCHECK(hipStreamSynchronize(st));
    }
    P->tr_cost = cost[0];
    T.expands = cost[3] != 0;
    if (P->stokes && cost[1] > 0) T.small = reinterpret_cast<double *>(P->tree_mem + o_small);
    const double U = (double)cost[0] / (double)G;
    P->tr = tree_shape(G, U, Np, P->onsurf, P->stokes);
    const double least = std::max(1.35 * (double)Np, cost[1] >= 150 ? 400.0 : 500.0);
    T.skip = P->onsurf ? cost[1] >= 90 && U >= least : cost[1] >= mhlp::TR_ZSKIP && G >= 400;
    P->tr_pairs = !T.expands && !T.skip && !T.flux ? G * Np : 0;
    P->tr_skip = {G >= 1200 && U < 350.0 ? 4 : 8, 1, 0};
    if (P->onsurf) P->tr_skip = 3 * G <= TREE_CUS ? P->tr : mhlp_plan::TreeShape{16, 2 * G <= TREE_CUS ? 2 : 1, 1};
    const int split = std::max(P->tr.split, P->tr_skip.split);
    if (split > 1) TRY(dalloc(&T.part, (P->onsurf ? 2 : 4) * (int64_t)split * 64 * G));
    if (T.skip && P->onsurf) {
        TRY(dalloc(&T.base, 2 * (64 + 1) * G)); /* two fields, and their room */
        T.room = reinterpret_cast<float *>(T.base + 2 * 64 * G);
    }
    return MHLP_OK;
}

static mhlp_status plan_create_impl(const mhlp_geometry *g, double alpha, const double *tx, const double *ty,
                                    int64_t m, const mhlp_params *prm, void *stream, mhlp_plan **out, bool stokes)
{
    if (!out) return fail(MHLP_INVALID_ARG, "out is NULL");
    *out = nullptr;
    if (!g) return fail(MHLP_INVALID_ARG, "geometry is NULL");
    if (!(alpha > 0.0) || !std::isfinite(alpha)) return fail(MHLP_INVALID_ARG, "alpha must be finite and > 0");
    if (m < 0 || m > INT_MAX - 1) return fail(MHLP_INVALID_ARG, "number of targets out of range");
    if (m > 0 && (!tx || !ty)) return fail(MHLP_INVALID_ARG, "target arrays are NULL");
    hipStream_t st = (hipStream_t)stream;
    mhlp_plan *P = new mhlp_plan();
    P->g = g;
    P->alpha = alpha;
    P->stokes = stokes;
    P->np.rho_direct = 3.5;
    P->np.rho_split = std::sqrt(3.5);
    P->np.ah_max = 4.5;
    P->np.far_exp = 40.0;
    if (prm) {
        if (prm->near_factor > 0) P->near_factor = prm->near_factor;
        if (prm->rho_direct > 0) P->np.rho_direct = prm->rho_direct;
        if (prm->rho_split > 0) P->np.rho_split = prm->rho_split;
        if (prm->ah_max > 0) P->np.ah_max = prm->ah_max;
        if (prm->far_exp > 0) P->np.far_exp = prm->far_exp;
    }
    mhlp_status s;
    if (m == 0) {
        P->onsurf = true;
        P->M = g->N;
        P->tx = g->soa;
        P->ty = g->soa + g->N;
    } else {
        P->M = m;
        if ((s = dalloc(&P->tx, m)) || (s = dalloc(&P->ty, m)) || (s = dalloc(&P->perm, m))) {
            mhlp_plan_destroy(P);
            return s;
        }
        /* Targets are kept in Morton (Z-curve) order of their coordinates, so the
           64 lanes of a wave hold nearby targets: they share near panels and
           fall on the same side of the z = 2 switch of the kernel values more
           often.  Results are written back through perm. */
        std::vector<double> hx((size_t)m), hy((size_t)m);
        hipError_t e = hipMemcpyAsync(hx.data(), tx, sizeof(double) * m, hipMemcpyDeviceToHost, st);
        if (e == hipSuccess) e = hipMemcpyAsync(hy.data(), ty, sizeof(double) * m, hipMemcpyDeviceToHost, st);
        if (e == hipSuccess) e = hipStreamSynchronize(st);
        if (e != hipSuccess) {
            mhlp_plan_destroy(P);
            return fail(MHLP_HIP_ERROR, std::string("plan_create copy: ") + hipGetErrorString(e));
        }
        double x0 = hx[0], x1 = hx[0], y0 = hy[0], y1 = hy[0];
        for (int64_t i = 0; i < m; ++i) {
            if (!std::isfinite(hx[i]) || !std::isfinite(hy[i])) {
                mhlp_plan_destroy(P);
                return fail(MHLP_INVALID_ARG, "target coordinates must be finite");
            }
            x0 = std::min(x0, hx[i]), x1 = std::max(x1, hx[i]);
            y0 = std::min(y0, hy[i]), y1 = std::max(y1, hy[i]);
        }
        const double span = std::max(std::max(x1 - x0, y1 - y0), 1e-300);
        auto spread = [](uint32_t v) { /* 16 bits -> even bit positions */
            uint64_t b = v & 0xFFFFu;
            b = (b | (b << 8)) & 0x00FF00FFull;
            b = (b | (b << 4)) & 0x0F0F0F0Full;
            b = (b | (b << 2)) & 0x33333333ull;
            b = (b | (b << 1)) & 0x55555555ull;
            return b;
        };
        std::vector<std::pair<uint64_t, int32_t>> key((size_t)m);
        for (int64_t i = 0; i < m; ++i) {
            const uint32_t qx = (uint32_t)std::min(65535.0, std::floor((hx[i] - x0) / span * 65536.0));
            const uint32_t qy = (uint32_t)std::min(65535.0, std::floor((hy[i] - y0) / span * 65536.0));
            key[i] = {spread(qx) | (spread(qy) << 1), (int32_t)i};
        }
        std::stable_sort(key.begin(), key.end(),
                         [](const std::pair<uint64_t, int32_t> &a, const std::pair<uint64_t, int32_t> &b) {
                             return a.first < b.first;
                         });
        std::vector<double> px((size_t)m), py((size_t)m);
        std::vector<int32_t> pm((size_t)m);
        for (int64_t i = 0; i < m; ++i) {
            pm[i] = key[i].second;
            px[i] = hx[pm[i]];
            py[i] = hy[pm[i]];
        }
        e = hipMemcpyAsync(P->tx, px.data(), sizeof(double) * m, hipMemcpyHostToDevice, st);
        if (e == hipSuccess) e = hipMemcpyAsync(P->ty, py.data(), sizeof(double) * m, hipMemcpyHostToDevice, st);
        if (e == hipSuccess) e = hipMemcpyAsync(P->perm, pm.data(), sizeof(int32_t) * m, hipMemcpyHostToDevice, st);
        if (e == hipSuccess) e = hipStreamSynchronize(st);
        if (e != hipSuccess) {
            mhlp_plan_destroy(P);
            return fail(MHLP_HIP_ERROR, std::string("plan_create copy: ") + hipGetErrorString(e));
        }
    }
    const int64_t M = P->M;
    {
        /* source splits so that about 8192 blocks of 256 targets run (the
           chip holds about 1024 at a time; several rounds keep the tail
           short); at least 2 panels per split.  mhlp_plan_autotune refines. */
        const int64_t tblocks = (M + FT_THREADS - 1) / FT_THREADS;
        int64_t ns = (8192 + tblocks - 1) / tblocks;
        if (ns > g->Np / 2) ns = g->Np / 2;
        if (ns < 1) ns = 1;
        if ((s = plan_set_split(P, (int)ns))) {
            mhlp_plan_destroy(P);
            return s;
        }
    }
    int32_t *cnt = nullptr;
    if ((s = dalloc(&cnt, M + 1)) || (s = dalloc(&P->near_ptr, M + 1))) {
        if (cnt) (void)hipFree(cnt);
        mhlp_plan_destroy(P);
        return s;
    }
    GeoView G = view(g);
    /* cnt[M] doubles as the fill-mismatch flag */
    near_list_kernel<<<nblocks(M, 128), 128, 0, st>>>(0, G, P->tx, P->ty, M, P->onsurf ? 1 : 0, P->near_factor,
                                                       P->np.rho_direct, cnt, nullptr, nullptr, nullptr, nullptr,
                                                       nullptr);
    scan_kernel<<<1, 1024, 0, st>>>(cnt, M, P->near_ptr);
    int32_t nnz = 0;
    hipError_t e = hipGetLastError();
    if (e == hipSuccess) e = hipMemcpyAsync(&nnz, P->near_ptr + M, sizeof(int32_t), hipMemcpyDeviceToHost, st);
    if (e == hipSuccess) e = hipStreamSynchronize(st);
    if (e != hipSuccess) {
        (void)hipFree(cnt);
        mhlp_plan_destroy(P);
        return fail(MHLP_HIP_ERROR, std::string("plan_create near count: ") + hipGetErrorString(e));
    }
    P->nnz = nnz;
    if (nnz > 0) {
        if ((s = dalloc(&P->near_panel, nnz)) || (s = dalloc(&P->near_tgt, nnz)) || (s = dalloc(&P->near_ts, 2 * (int64_t)nnz)) ||
            (!stokes && ((s = dalloc(&P->wslp, 16 * (int64_t)nnz)) || (s = dalloc(&P->wdlp, 16 * (int64_t)nnz)))) ||
            (stokes && (s = dalloc(&P->wstk, 64 * (int64_t)nnz)))) {
            mhlp_plan_destroy(P);
            return s;
        }
        fill_i32_kernel<<<1, 1, 0, st>>>(cnt + M, 0, 1);
        near_list_kernel<<<nblocks(M, 128), 128, 0, st>>>(1, G, P->tx, P->ty, M, P->onsurf ? 1 : 0, P->near_factor,
                                                           P->np.rho_direct, nullptr, P->near_ptr, P->near_panel,
                                                           P->near_tgt, P->near_ts, cnt + M);
        /* validate the list on the host before any kernel indexes with it */
        {
            std::vector<int32_t> hp((size_t)nnz);
            e = hipGetLastError();
            if (e == hipSuccess)
                e = hipMemcpyAsync(hp.data(), P->near_panel, sizeof(int32_t) * nnz, hipMemcpyDeviceToHost, st);
            if (e == hipSuccess) e = hipStreamSynchronize(st);
            if (e != hipSuccess) {
                (void)hipFree(cnt);
                mhlp_plan_destroy(P);
                return fail(MHLP_HIP_ERROR, std::string("plan_create near list: ") + hipGetErrorString(e));
            }
            for (int32_t v : hp)
                if (v < -1 || v >= g->Np) {
                    (void)hipFree(cnt);
                    mhlp_plan_destroy(P);
                    return fail(MHLP_HIP_ERROR, "plan_create: near list holds an invalid panel index");
                }
        }
        if (stokes)
            near_stokes_weights_kernel<<<nblocks(nnz, 64), 64, 0, st>>>(G, P->tx, P->ty, P->onsurf ? 1 : 0,
                                                                         P->near_panel, P->near_tgt, P->near_ts, nnz,
                                                                         alpha, P->np, P->wstk);
        else
            near_weights_kernel<<<nblocks(nnz, 64), 64, 0, st>>>(G, P->tx, P->ty, P->onsurf ? 1 : 0, P->near_panel,
                                                                  P->near_tgt, P->near_ts, nnz, alpha, P->np, P->wslp,
                                                                  P->wdlp);
        e = hipGetLastError();
        int32_t mism = 0;
        if (e == hipSuccess) e = hipMemcpyAsync(&mism, cnt + M, sizeof(int32_t), hipMemcpyDeviceToHost, st);
        if (e == hipSuccess) e = hipStreamSynchronize(st);
        if (e != hipSuccess) {
            (void)hipFree(cnt);
            mhlp_plan_destroy(P);
            return fail(MHLP_HIP_ERROR, std::string("plan_create near weights: ") + hipGetErrorString(e));
        }
        P->fill_mismatch = mism;
    }
    (void)hipFree(cnt);
    if ((s = far_scales_setup(P, st)) || (s = tree_setup(P, st)) || (!stokes && (s = far_class_setup(P, st)))) {
        mhlp_plan_destroy(P);
        return s;
    }
    if (stokes) {
        /* W term: 1/|Gamma| */
        std::vector<double> hw((size_t)g->N);
        hipError_t e2 = hipMemcpyAsync(hw.data(), g->w, sizeof(double) * g->N, hipMemcpyDeviceToHost, st);
        if (e2 == hipSuccess) e2 = hipStreamSynchronize(st);
        if (e2 != hipSuccess) {
            mhlp_plan_destroy(P);
            return fail(MHLP_HIP_ERROR, std::string("stokes plan: ") + hipGetErrorString(e2));
        }
        double len = 0.0;
        for (double v : hw) len += v;
        P->inv_len = 1.0 / len;
    }
    *out = P;
    return MHLP_OK;
}

extern "C" mhlp_status mhlp_plan_create(const mhlp_geometry *g, double alpha, const double *tx, const double *ty,
                                        int64_t m, const mhlp_params *prm, void *stream, mhlp_plan **out)
{
    return plan_create_impl(g, alpha, tx, ty, m, prm, stream, out, false);
}

extern "C" mhlp_status mhlp_stokes_plan_create(const mhlp_geometry *g, double alpha, const double *tx,
                                               const double *ty, int64_t m, const mhlp_params *prm, void *stream,
                                               mhlp_plan **out)
{
    return plan_create_impl(g, alpha, tx, ty, m, prm, stream, out, true);
}

extern "C" mhlp_status mhlp_plan_info(const mhlp_plan *P, int64_t *n_targets, int64_t *n_sources,
                                      int64_t *n_near_pairs, double *alpha)
{
    if (!P) return fail(MHLP_INVALID_ARG, "plan is NULL");
    if (n_targets) *n_targets = P->M;
    if (n_sources) *n_sources = P->g->N;
    if (n_near_pairs) *n_near_pairs = P->nnz;
    if (alpha) *alpha = P->alpha;
    return MHLP_OK;
}

/* ------------------------------------------------------------------------ */
/* evaluation                                                                */
/* ------------------------------------------------------------------------ */
/* The launches of one far sum by cluster expansions: Op<SLP, DLP, RAW> what it
   evaluates, <SLP, DLP, GRAD> the moments it reads. */
static dim3 moments_grid(const FarArgs &A, const mhlp::TreeDev &T)
{
    /* without expansions only the staging at level 0 is left: 6 -> 2.5 us */
    return T.expands ? dim3(nblocks(A.Np, 16), (unsigned)T.nlev, mhlp::TR_GROUPS) : dim3(nblocks(A.Np, 16));
}

template <class Op>
static void launch_tree_far(const FarArgs &A, const mhlp_plan *P, hipStream_t st)
{
    const mhlp::TreeDev &T = *P->tree;
    const bool skip = Op::SKIP && T.skip;
    const mhlp_plan::TreeShape &F = skip ? P->tr_skip : P->tr;
    const int threads = 64 * std::min(F.waves, Op::WMAX);
    const int64_t G = nblocks(A.M, 64), most = (int64_t)1 << 20; /* groups a launch: below 2^32 threads along the grid */
    for (int64_t g0 = 0; g0 < G; g0 += most) {
        mhlp::TreeDev S = T;
        S.order += g0;
        S.cut = F.cut;
        const dim3 grid((unsigned)std::min(most, G - g0), (unsigned)F.split);
        if constexpr (Op::SKIP) {
            if (skip && P->onsurf) {
                mhlp::far_tree_kernel<Op, mhlp::TREE_NEAREST><<<grid, threads, 0, st>>>(A, S);
                mhlp::far_tree_kernel<Op, mhlp::TREE_REST><<<grid, threads, 0, st>>>(A, S);
                continue;
            }
            if (skip) {
                mhlp::far_tree_kernel<Op, mhlp::TREE_BOTH><<<grid, threads, 0, st>>>(A, S);
                continue;
            }
        }
        mhlp::far_tree_kernel<Op, mhlp::TREE_ALL><<<grid, threads, 0, st>>>(A, S);
    }
}

template <template <bool, bool, bool> class Op, bool SLP, bool DLP, bool GRAD>
static void launch_tree(const FarArgs &A, const mhlp_plan *P, hipStream_t st)
{
    if (P->tr_pairs && P->tr_pairs <= tree_raw_max(SLP, DLP)) return launch_tree_far<Op<SLP, DLP, true>>(A, P, st);
    const mhlp::TreeDev &T = *P->tree;
    mhlp::tree_moments_kernel<SLP, DLP, GRAD><<<moments_grid(A, T), 256, 0, st>>>(A, T);
    launch_tree_far<Op<SLP, DLP, false>>(A, P, st);
}

template <bool GRAD>
static void launch_tree_stokes(const FarArgs &A, const mhlp_plan *P, hipStream_t st)
{
    const mhlp::TreeDev &T = *P->tree;
    if (P->tr_pairs && P->tr_pairs <= tree_raw_max(true, true))
        return launch_tree_far<mhlp::TreeStokes<GRAD, false, true>>(A, P, st);
    dim3 grid = moments_grid(A, T);
    if (T.small) grid.z *= 2; /* the rows of the powers, too */
    mhlp::tree_stokes_kernel<GRAD><<<grid, 256, 0, st>>>(A, T);
    if (T.small)
        launch_tree_far<mhlp::TreeStokes<GRAD, true>>(A, P, st);
    else
        launch_tree_far<mhlp::TreeStokes<GRAD, false>>(A, P, st);
}

template <bool SLP, bool DLP>
static void launch_far_t(const FarArgs &A, const mhlp_plan *P, int32_t precision, hipStream_t st)
{
    if (precision == MHLP_FP64) {
        launch_tree<mhlp::TreePot, SLP, DLP, false>(A, P, st);
        return;
    }
    const int nsplit = P->nsplit;
    const dim3 grid(nblocks(A.M, FT_THREADS), (unsigned)nsplit);
    if (nsplit <= 1) {
        far_eval_mixed<SLP, DLP, false><<<grid, FT_THREADS, 0, st>>>(A);
        return;
    }
    far_eval_mixed<SLP, DLP, true><<<grid, FT_THREADS, 0, st>>>(A);
    if (A.M <= FZ_SHORT)
        far_finalize<SLP, DLP, FZ_L><<<nblocks(A.M, FZ_TG), FZ_TG * FZ_L, 0, st>>>(A, nsplit);
    else
        far_finalize<SLP, DLP, 1><<<nblocks(A.M, 256), 256, 0, st>>>(A, nsplit);
}

/* The far-field launch arguments of plan P for the given densities and outputs. */
static FarArgs far_args(const mhlp_plan *P, const double *sigma, const double *mu, double *us, double *ud,
                        double half_term, const GState *gs, int64_t jstride)
{
    const mhlp_geometry *g = P->g;
    FarArgs A;
    A.sx = g->soa;
    A.sy = g->soa + g->N;
    A.sw = g->w;
    A.snx = g->nx;
    A.sny = g->ny;
    A.sigma = sigma;
    A.mu = mu;
    A.N = g->N;
    A.tx = P->tx;
    A.ty = P->ty;
    A.M = P->M;
    A.nptr = P->near_ptr;
    A.npan = P->near_panel;
    A.wsl = P->wslp;
    A.wdl = P->wdlp;
    A.alpha = P->alpha;
    A.half_term = half_term;
    A.us = us;
    A.ud = ud;
    A.Np = g->Np;
    A.pps = P->pps;
    A.part_s = P->part;
    A.part_d = P->part + (int64_t)P->nsplit * P->M;
    A.gs = gs;
    A.jstride = jstride;
    A.perm = P->perm;
    A.pcx = g->pcx;
    A.pcy = g->pcy;
    A.prad = g->prad;
    A.wcls = P->wcls;
    A.fq = P->fqd;
    return A;
}

static mhlp_status launch_far(const mhlp_plan *P, const double *sigma, const double *mu, double *us, double *ud,
                              double half_term, int32_t precision, hipStream_t st, const GState *gs = nullptr,
                              int64_t jstride = 0)
{
    if (precision != MHLP_FP64 && precision != MHLP_MIXED) return fail(MHLP_INVALID_ARG, "unknown precision");
    if (P->stokes) return fail(MHLP_INVALID_ARG, "a stokes plan evaluates with the mhlp_stokes_* calls");
    const mhlp_geometry *g = P->g;
    if (half_term != 0.0 && (!P->onsurf || P->M != g->N))
        return fail(MHLP_INVALID_ARG, "identity term needs an on-surface plan");
    const FarArgs A = far_args(P, sigma, mu, us, ud, half_term, gs, jstride);
    if (P->fmm && P->fmm_serves && precision == MHLP_FP64 && !gs) {
        if (sigma && mu)
            fmm_far_t<true, true>(P->fmm, A, st);
        else if (sigma)
            fmm_far_t<true, false>(P->fmm, A, st);
        else
            fmm_far_t<false, true>(P->fmm, A, st);
        HIPCHECK(hipGetLastError());
        return MHLP_OK;
    }
    if (sigma && mu)
        launch_far_t<true, true>(A, P, precision, st);
    else if (sigma)
        launch_far_t<true, false>(A, P, precision, st);
    else
        launch_far_t<false, true>(A, P, precision, st);
    HIPCHECK(hipGetLastError());
    return MHLP_OK;
}

extern "C" mhlp_status mhlp_eval_layer(const mhlp_plan *P, const double *sigma, const double *mu, double *u_slp,
                                       double *u_dlp, int32_t precision, void *stream)
{
    if (!P) return fail(MHLP_INVALID_ARG, "plan is NULL");
    const bool ds = sigma && u_slp, dd = mu && u_dlp;
    if (!ds && !dd) return fail(MHLP_INVALID_ARG, "no density/output pair given");
    if ((sigma && !u_slp) || (u_slp && !sigma) || (mu && !u_dlp) || (u_dlp && !mu))
        return fail(MHLP_INVALID_ARG, "density and output must be given together");
    return launch_far(P, sigma, mu, u_slp, u_dlp, 0.0, precision, (hipStream_t)stream);
}

/* ------------------------------------------------------------------------ */
/* far-field launch shape: source splits, and their autotuner               */
/* ------------------------------------------------------------------------ */
extern "C" mhlp_status mhlp_plan_set_split(mhlp_plan *P, int32_t nsplit)
{
    if (!P) return fail(MHLP_INVALID_ARG, "plan is NULL");
    if (nsplit < 1) return fail(MHLP_INVALID_ARG, "nsplit must be >= 1");
    return plan_set_split(P, nsplit);
}

extern "C" mhlp_status mhlp_plan_get_split(const mhlp_plan *P, int32_t *nsplit)
{
    if (!P || !nsplit) return fail(MHLP_INVALID_ARG, "NULL argument");
    *nsplit = P->nsplit;
    return MHLP_OK;
}

static mhlp_status launch_stokes(const mhlp_plan *P, const double *mu, double *u, int64_t ustride, bool bie,
                                 hipStream_t st, const GState *gs = nullptr, int64_t jstride = 0);

extern "C" mhlp_status mhlp_plan_autotune(mhlp_plan *P, int32_t layers, int32_t precision, int32_t reps,
                                          void *stream, int32_t *best_nsplit, double *best_ms, int32_t *cand,
                                          double *cand_ms, int32_t cap, int32_t *n_cand)
{
    if (!P) return fail(MHLP_INVALID_ARG, "plan is NULL");
    if (layers < 1 || layers > 7) return fail(MHLP_INVALID_ARG, "layers must be 1 to 7");
    if ((layers >= 6) != P->stokes) return fail(MHLP_INVALID_ARG, "layers 6 and 7 (and only they) tune a stokes plan");
    if (layers >= 6 && precision != MHLP_FP64) return fail(MHLP_INVALID_ARG, "the stresslet is FP64 only");
    if (layers == 7 && P->onsurf) return fail(MHLP_INVALID_ARG, "layers 7 (stresslet gradient) needs an off-surface plan");
    if (layers == 4 && !P->onsurf) return fail(MHLP_INVALID_ARG, "layers 4 (BIE operator) needs an on-surface plan");
    if (layers == 5 && P->onsurf) return fail(MHLP_INVALID_ARG, "layers 5 (gradients) needs an off-surface plan");
    if (layers == 5 && precision != MHLP_FP64) return fail(MHLP_INVALID_ARG, "gradients are FP64 only");
    if (precision != MHLP_FP64 && precision != MHLP_MIXED) return fail(MHLP_INVALID_ARG, "unknown precision");
    if (reps < 1 || reps > 1000) return fail(MHLP_INVALID_ARG, "reps must be in [1, 1000]");
    if (cap < 0 || (cap > 0 && (!cand || !cand_ms))) return fail(MHLP_INVALID_ARG, "candidate arrays");
    hipStream_t st = (hipStream_t)stream;
    const int64_t N = P->g->N, M = P->M, Np = P->g->Np;
    /* The FP64 launches run by cluster expansions (tree.h) and do not use the
       split.  For the potentials it serves the MIXED launch of the same layers,
       which is what gets timed; the gradients and the stresslet are timed as they
       stand, and the split, which shapes the plan's MIXED launches, is left alone. */
    if (precision == MHLP_FP64 && layers <= 4) precision = MHLP_MIXED;
    std::vector<int> cs;
    if (layers <= 4)
        for (int64_t ns = 1; ns <= Np && ns <= 256; ns *= 2) cs.push_back((int)ns);
    if (std::find(cs.begin(), cs.end(), P->nsplit) == cs.end()) cs.push_back(P->nsplit);
    double *dens = nullptr, *out = nullptr;
    TRY(dalloc(&dens, 2 * N));
    mhlp_status s = dalloc(&out, 4 * M);
    hipEvent_t e0 = nullptr, e1 = nullptr;
    if (s == MHLP_OK && (hipEventCreate(&e0) != hipSuccess || hipEventCreate(&e1) != hipSuccess))
        s = fail(MHLP_HIP_ERROR, "hipEventCreate");
    int best = P->nsplit;
    double bms = 1e300;
    int nc = 0;
    std::vector<std::pair<int, double>> tim;
    if (s == MHLP_OK) fill_kernel<<<nblocks(2 * N, 256), 256, 0, st>>>(dens, 1.0, 2 * N);
    for (size_t c = 0; c < cs.size() && s == MHLP_OK; ++c) {
        if ((s = plan_set_split(P, cs[c]))) break;
        auto run = [&]() -> mhlp_status {
            if (layers == 5) return mhlp_eval_grad(P, dens, dens, out, out + M, out + 2 * M, out + 3 * M, st);
            if (layers == 6) return launch_stokes(P, dens, out, M, P->onsurf, st);
            if (layers == 7) return mhlp_stokes_eval_grad(P, dens, out, st);
            const double *sg = (layers & 1) ? dens : nullptr, *mu = (layers & 2 || layers == 4) ? dens : nullptr;
            return launch_far(P, sg, mu, sg ? out : nullptr, mu ? out + M : nullptr, layers == 4 ? 0.5 : 0.0,
                              precision, st);
        };
        if ((s = run())) break;
        if (hipEventRecord(e0, st) != hipSuccess) {
            s = fail(MHLP_HIP_ERROR, "hipEventRecord");
            break;
        }
        for (int r = 0; r < reps && s == MHLP_OK; ++r) s = run();
        if (s) break;
        float ms = 0.f;
        hipError_t e = hipEventRecord(e1, st);
        if (e == hipSuccess) e = hipEventSynchronize(e1);
        if (e == hipSuccess) e = hipEventElapsedTime(&ms, e0, e1);
        if (e != hipSuccess) {
            s = fail(MHLP_HIP_ERROR, std::string("autotune timing: ") + hipGetErrorString(e));
            break;
        }
        const double per = (double)ms / reps;
        tim.emplace_back(P->nsplit, per);
        if (nc < cap) {
            cand[nc] = P->nsplit;
            cand_ms[nc] = per;
        }
        ++nc;
        if (per < bms) bms = per;
    }
    /* fewest splits within 1% of the fastest (fewer partial sums, and a choice
       that is stable under timing noise) */
    if (s == MHLP_OK && !tim.empty()) {
        best = INT_MAX;
        for (const auto &t : tim)
            if (t.second <= 1.01 * bms && t.first < best) best = t.first;
    }
    if (e0) (void)hipEventDestroy(e0);
    if (e1) (void)hipEventDestroy(e1);
    (void)hipStreamSynchronize(st);
    (void)hipFree(dens);
    if (out) (void)hipFree(out);
    if (s) return s;
    TRY(plan_set_split(P, best));
    if (best_nsplit) *best_nsplit = best;
    if (best_ms)
        for (const auto &t : tim)
            if (t.first == best) *best_ms = t.second;
    if (n_cand) *n_cand = std::min(nc, cap);
    return MHLP_OK;
}

extern "C" mhlp_status mhlp_eval_slp(const mhlp_plan *P, const double *sigma, double *u, int32_t precision,
                                     void *stream)
{
    if (!sigma || !u) return fail(MHLP_INVALID_ARG, "sigma or u is NULL");
    return mhlp_eval_layer(P, sigma, nullptr, u, nullptr, precision, stream);
}

extern "C" mhlp_status mhlp_eval_dlp(const mhlp_plan *P, const double *mu, double *u, int32_t precision, void *stream)
{
    if (!mu || !u) return fail(MHLP_INVALID_ARG, "mu or u is NULL");
    return mhlp_eval_layer(P, nullptr, mu, nullptr, u, precision, stream);
}

extern "C" mhlp_status mhlp_apply_bie_operator(const mhlp_plan *P, const double *mu, double *out, int32_t precision,
                                               void *stream)
{
    if (!P) return fail(MHLP_INVALID_ARG, "plan is NULL");
    if (!P->onsurf) return fail(MHLP_INVALID_ARG, "apply_bie_operator needs an on-surface plan (m == 0)");
    if (!mu || !out) return fail(MHLP_INVALID_ARG, "mu or out is NULL");
    if (mu == out) return fail(MHLP_INVALID_ARG, "mu and out must not alias");
    return launch_far(P, nullptr, mu, nullptr, out, 0.5, precision, (hipStream_t)stream);
}

/* ------------------------------------------------------------------------ */
/* target gradients                                                          */
/* ------------------------------------------------------------------------ */
static mhlp_status ensure_grad_weights(mhlp_plan *P, hipStream_t st)
{
    if (P->wgrad || P->nnz == 0) return MHLP_OK;
    TRY(dalloc(&P->wgrad, 64 * P->nnz));
    near_grad_weights_kernel<<<nblocks(P->nnz, 64), 64, 0, st>>>(view(P->g), P->tx, P->ty, P->near_panel,
                                                                  P->near_tgt, P->near_ts, P->nnz, P->alpha, P->np,
                                                                  P->wgrad);
    hipError_t e = hipGetLastError();
    if (e == hipSuccess) e = hipStreamSynchronize(st);
    if (e != hipSuccess) {
        (void)hipFree(P->wgrad);
        P->wgrad = nullptr;
        return fail(MHLP_HIP_ERROR, std::string("gradient weights: ") + hipGetErrorString(e));
    }
    return MHLP_OK;
}

extern "C" mhlp_status mhlp_eval_grad(const mhlp_plan *Pc, const double *sigma, const double *mu, double *gs_x,
                                      double *gs_y, double *gd_x, double *gd_y, void *stream)
{
    if (!Pc) return fail(MHLP_INVALID_ARG, "plan is NULL");
    if (Pc->onsurf) return fail(MHLP_UNSUPPORTED, "eval_grad needs an off-surface plan (targets off the curve)");
    if (Pc->stokes) return fail(MHLP_INVALID_ARG, "eval_grad needs a scalar plan");
    const bool gs = sigma != nullptr, gd = mu != nullptr;
    if (!gs && !gd) return fail(MHLP_INVALID_ARG, "no density given");
    if (gs != (gs_x != nullptr) || gs != (gs_y != nullptr) || gd != (gd_x != nullptr) || gd != (gd_y != nullptr))
        return fail(MHLP_INVALID_ARG, "each density needs both of its gradient outputs (and only then)");
    mhlp_plan *P = const_cast<mhlp_plan *>(Pc); /* gradient weights are built on first use */
    hipStream_t st = (hipStream_t)stream;
    TRY(ensure_grad_weights(P, st));
    FarArgs A = far_args(P, sigma, mu, nullptr, nullptr, 0.0, nullptr, 0);
    A.wg = P->wgrad;
    A.nnz = P->nnz;
    double *out[4] = {gs_x, gs_y, gd_x, gd_y};
    for (int f = 0; f < 4; ++f) A.gout[f] = out[f];
    if (gs && gd)
        launch_tree<mhlp::TreeGrad, true, true, true>(A, P, st);
    else if (gs)
        launch_tree<mhlp::TreeGrad, true, false, true>(A, P, st);
    else
        launch_tree<mhlp::TreeGrad, false, true, true>(A, P, st);
    HIPCHECK(hipGetLastError());
    return MHLP_OK;
}

/* ------------------------------------------------------------------------ */
/* modified-Stokes double layer: entry points                                */
/* ------------------------------------------------------------------------ */
static mhlp_status launch_stokes(const mhlp_plan *P, const double *mu, double *u, int64_t ustride, bool bie,
                                 hipStream_t st, const GState *gs, int64_t jstride)
{
    FarArgs A = far_args(P, nullptr, mu, nullptr, nullptr, bie ? 0.5 : 0.0, gs, jstride);
    A.wg = P->wstk;
    A.nnz = P->nnz;
    A.gout[0] = u;
    A.gout[1] = u + ustride;
    A.inv_len = P->inv_len;
    launch_tree_stokes<false>(A, P, st);
    HIPCHECK(hipGetLastError());
    return MHLP_OK;
}

extern "C" mhlp_status mhlp_stokes_eval(const mhlp_plan *P, const double *mu, double *u, void *stream)
{
    if (!P) return fail(MHLP_INVALID_ARG, "plan is NULL");
    if (!P->stokes) return fail(MHLP_INVALID_ARG, "stokes_eval needs a plan from mhlp_stokes_plan_create");
    if (!mu || !u) return fail(MHLP_INVALID_ARG, "mu or u is NULL");
    if (mu == u) return fail(MHLP_INVALID_ARG, "mu and u must not alias");
    return launch_stokes(P, mu, u, P->M, false, (hipStream_t)stream);
}

extern "C" mhlp_status mhlp_stokes_apply_bie(const mhlp_plan *P, const double *mu, double *out, void *stream)
{
    if (!P) return fail(MHLP_INVALID_ARG, "plan is NULL");
    if (!P->stokes || !P->onsurf)
        return fail(MHLP_INVALID_ARG, "stokes_apply_bie needs an on-surface plan from mhlp_stokes_plan_create");
    if (!mu || !out) return fail(MHLP_INVALID_ARG, "mu or out is NULL");
    if (mu == out) return fail(MHLP_INVALID_ARG, "mu and out must not alias");
    return launch_stokes(P, mu, out, P->M, true, (hipStream_t)stream);
}

static mhlp_status ensure_stokes_grad_weights(mhlp_plan *P, hipStream_t st)
{
    if (P->wstkg || P->nnz == 0) return MHLP_OK;
    TRY(dalloc(&P->wstkg, 128 * P->nnz));
    near_stokes_grad_weights_kernel<<<nblocks(P->nnz, 64), 64, 0, st>>>(view(P->g), P->tx, P->ty, P->near_panel,
                                                                         P->near_tgt, P->near_ts, P->nnz, P->alpha,
                                                                         P->np, P->wstkg);
    hipError_t e = hipGetLastError();
    if (e == hipSuccess) e = hipStreamSynchronize(st);
    if (e != hipSuccess) {
        (void)hipFree(P->wstkg);
        P->wstkg = nullptr;
        return fail(MHLP_HIP_ERROR, std::string("stresslet gradient weights: ") + hipGetErrorString(e));
    }
    return MHLP_OK;
}

extern "C" mhlp_status mhlp_stokes_eval_grad(const mhlp_plan *Pc, const double *mu, double *g, void *stream)
{
    if (!Pc) return fail(MHLP_INVALID_ARG, "plan is NULL");
    if (!Pc->stokes) return fail(MHLP_INVALID_ARG, "stokes_eval_grad needs a plan from mhlp_stokes_plan_create");
    if (Pc->onsurf) return fail(MHLP_UNSUPPORTED, "stokes_eval_grad needs an off-surface plan (targets off the curve)");
    if (!mu || !g) return fail(MHLP_INVALID_ARG, "mu or g is NULL");
    if (mu == g) return fail(MHLP_INVALID_ARG, "mu and g must not alias");
    mhlp_plan *P = const_cast<mhlp_plan *>(Pc); /* gradient weights are built on first use */
    hipStream_t st = (hipStream_t)stream;
    TRY(ensure_stokes_grad_weights(P, st));
    FarArgs A = far_args(P, nullptr, mu, nullptr, nullptr, 0.0, nullptr, 0);
    A.wg = P->wstkg;
    A.nnz = P->nnz;
    for (int f = 0; f < 4; ++f) A.gout[f] = g + f * P->M;
    launch_tree_stokes<true>(A, P, st);
    HIPCHECK(hipGetLastError());
    return MHLP_OK;
}

/* ------------------------------------------------------------------------ */
/* GMRES                                                                     */
/* ------------------------------------------------------------------------ */
/* length of the unknown vector and the on-surface operator of the plan:
   (1/2 I + D) mu for the scalar kernel (N), (1/2 I + D + W) mu for the
   stresslet (2N, component-major) */
static int64_t vlen(const mhlp_plan *P) { return P->stokes ? 2 * P->g->N : P->g->N; }

/* the FP64 operator, in mixed-precision solves too: by expansions it takes a
   third of the FP32 tiles' time (N = 4096: 18 against 61 + 5 us) and is the more
   accurate */
static mhlp_status apply_op(mhlp_plan *P, const double *x, double *out, hipStream_t st, const GState *gs = nullptr,
                            int64_t jstride = 0)
{
    if (P->stokes) return launch_stokes(P, x, out, P->g->N, true, st, gs, jstride);
    return launch_far(P, nullptr, x, nullptr, out, 0.5, MHLP_FP64, st, gs, jstride);
}

static mhlp_status ensure_ws(mhlp_plan *P, int64_t cols)
{
    if (P->ws && P->ws_cols >= cols) return MHLP_OK;
    if (P->ws) (void)hipFree(P->ws);
    P->ws = nullptr;
    TRY(dalloc(&P->ws, (cols + 6) * vlen(P)));
    P->ws_cols = cols;
    if (!P->hdev) TRY(dalloc(&P->hdev, 4 * 1024));
    if (!P->hhost) HIPCHECK(hipHostMalloc((void **)&P->hhost, sizeof(double) * 4 * 1024, hipHostMallocDefault));
    return MHLP_OK;
}

/* ||v||_2 (synchronising) */
static mhlp_status dnorm(mhlp_plan *P, const double *v, int64_t N, hipStream_t st, double *out)
{
    multi_dot_kernel<<<1, 256, 0, st>>>(v, N, v, N, P->hdev);
    HIPCHECK(hipGetLastError());
    HIPCHECK(hipMemcpyAsync(P->hhost, P->hdev, sizeof(double), hipMemcpyDeviceToHost, st));
    HIPCHECK(hipStreamSynchronize(st));
    *out = std::sqrt(P->hhost[0]);
    return MHLP_OK;
}

/* Device data of the device-driven GMRES for restart length R. */
struct GmresDev {
    GState *gs;
    GState *tail; /* density selector of the end-of-cycle operator: j = 0, done unless gs->done */
    double *H, *cs, *sn, *gv, *y, *h1, *h2, *hn;
    double *p1, *p2, *pn; /* multi-block Gram-Schmidt partials: [nb][R+1], [nb][R+1], [nb] */
};

static GmresDev gdev_view(const mhlp_plan *P)
{
    const int R = P->gdev_R;
    double *d = reinterpret_cast<double *>(P->gdev + 128);
    GmresDev v;
    v.gs = reinterpret_cast<GState *>(P->gdev);
    v.tail = reinterpret_cast<GState *>(P->gdev + 64);
    v.H = d;
    d += (int64_t)(R + 1) * R;
    v.cs = d;
    d += R;
    v.sn = d;
    d += R;
    v.gv = d;
    d += R + 1;
    v.y = d;
    d += R;
    v.h1 = d;
    d += R + 1;
    v.h2 = d;
    d += R + 1;
    v.hn = d;
    d += 1;
    const int64_t nb = (vlen(P) + gsm_slice(vlen(P)) - 1) / gsm_slice(vlen(P));
    v.p1 = d;
    d += nb * (R + 1);
    v.p2 = d;
    d += nb * (R + 1);
    v.pn = d;
    return v;
}

static mhlp_status ensure_gdev(mhlp_plan *P, int R)
{
    if (P->gdev && P->gdev_R >= R) return MHLP_OK;
    if (P->gdev) {
        HIPCHECK(hipDeviceSynchronize());
        (void)hipFree(P->gdev);
        P->gdev = nullptr;
    }
    const int64_t nb = (vlen(P) + gsm_slice(vlen(P)) - 1) / gsm_slice(vlen(P));
    const int64_t nd = (int64_t)(R + 1) * R + 3 * R + 3 * (R + 1) + 1 + nb * (2 * (R + 1) + 1);
    char *g = nullptr;
    TRY(dalloc(&g, 128 + 8 * nd));
    P->gdev = g;
    P->gdev_R = R;
    if (!P->gstate_host) HIPCHECK(hipHostMalloc((void **)&P->gstate_host, sizeof(GState), hipHostMallocDefault));
    return MHLP_OK;
}

/* Arnoldi steps of the first captured chunk of a GMRES cycle (later chunks
   follow the observed convergence rate); measured on the config-2 solves, 4
   saves a replay at alpha = 50 and 500 against 2 and costs nothing at 5 */
constexpr int GMRES_FIRST_CHUNK = 4;

/* Waits for the stream by polling it: the chunk reads of GMRES are a few tens
   of microseconds apart, shorter than a blocking wait takes to wake. */
static hipError_t spin_sync(hipStream_t st)
{
    hipError_t e;
    while ((e = hipStreamQuery(st)) == hipErrorNotReady) {
    }
    return e;
}

/* One Arnoldi step of the device-driven GMRES, enqueued on st (one_block: the
   Gram-Schmidt part in one block, else over element slices). */
static mhlp_status enqueue_step(mhlp_plan *P, bool one_block, hipStream_t st)
{
    const int64_t N = vlen(P);
    const int R = P->gdev_R;
    double *V = P->ws, *w = P->ws + (int64_t)(R + 1) * N;
    const GmresDev d = gdev_view(P);
    TRY(apply_op(P, V, w, st, d.gs, N));
    if (one_block) {
        if (N <= GSF_T)
            gs_reg_kernel<1><<<1, GSF_T, 0, st>>>(d.gs, V, N, w, N, d.H, R, d.cs, d.sn, d.gv);
        else if (N <= 2 * GSF_T)
            gs_reg_kernel<2><<<1, GSF_T, 0, st>>>(d.gs, V, N, w, N, d.H, R, d.cs, d.sn, d.gv);
        else if (N <= 4 * GSF_T)
            gs_reg_kernel<4><<<1, GSF_T, 0, st>>>(d.gs, V, N, w, N, d.H, R, d.cs, d.sn, d.gv);
        else
            gs_reg_kernel<8><<<1, GSF_T, 0, st>>>(d.gs, V, N, w, N, d.H, R, d.cs, d.sn, d.gv);
        HIPCHECK(hipGetLastError());
        return MHLP_OK;
    }
    /* classical Gram-Schmidt, twice, over element slices */
    const int64_t L = gsm_slice(N);
    const int nb = (int)((N + L - 1) / L);
    gsm_dot_kernel<<<nb, GSM_T, 0, st>>>(d.gs, V, N, w, N, L, d.p1);
    gsm_sub_kernel<false><<<nb, GSM_T, 0, st>>>(d.gs, V, N, w, N, L, d.p1, d.h1, d.p2);
    gsm_sub_kernel<true><<<nb, GSM_T, 0, st>>>(d.gs, V, N, w, N, L, d.p2, d.h2, d.pn);
    gsm_finish_kernel<<<1, GSF_T, 0, st>>>(d.gs, V, N, w, N, d.pn, nb, d.H, R, d.cs, d.sn, d.gv, d.h1, d.h2);
    HIPCHECK(hipGetLastError());
    return MHLP_OK;
}

/* End of a cycle (each kernel a no-op unless the state says done): y from
   the rotated Hessenberg system, x += V y, and the true residual r = b - A x
   and its squared norm in the state, so that the host reads the
   outcome of the cycle with the state itself.  x and b are the solve's own
   vectors. */
static mhlp_status enqueue_tail(mhlp_plan *P, const double *b, double *x, hipStream_t st)
{
    const int64_t N = vlen(P);
    const int R = P->gdev_R;
    double *V = P->ws, *w = P->ws + (int64_t)(R + 1) * N, *r = w + N;
    const GmresDev d = gdev_view(P);
    gs_solve_kernel<<<1, 64, 0, st>>>(d.gs, d.tail, d.H, R, d.gv, d.y);
    gs_addcols_kernel<<<nblocks(N, 256), 256, 0, st>>>(d.gs, V, N, d.y, x, N);
    HIPCHECK(hipGetLastError());
    TRY(apply_op(P, x, w, st, d.tail, 0));
    tail_residual_kernel<<<1, GSF_T, 0, st>>>(d.tail, b, w, x, r, N, d.gs);
    HIPCHECK(hipGetLastError());
    return MHLP_OK;
}

/* longest chunk of Arnoldi steps captured in one graph */
constexpr int GMRES_MAX_CHUNK = 16;

/* Executable graph of S consecutive Arnoldi steps (0 <= S <= GMRES_MAX_CHUNK),
   the first m of them with the one-block Gram-Schmidt, followed by the end of
   the cycle when `tail` is set; captured once per plan state (workspace,
   split, restart, the solve's x and b) on a private stream. */
static mhlp_status step_graph(mhlp_plan *P, int m, int S, bool tail, const double *b, double *x, hipGraphExec_t *out)
{
    const int key = (S * (GMRES_MAX_CHUNK + 1) + m) * 2 + (tail ? 1 : 0);
    mhlp_plan::StepGraph &G = P->graphs[key];
    if (G.exec && G.ws == P->ws && G.part == P->part && G.gdev == P->gdev && G.R == P->gdev_R &&
        G.nsplit == P->nsplit && G.x == x && G.b == b) {
        *out = G.exec;
        return MHLP_OK;
    }
    if (G.exec) {
        (void)hipGraphExecDestroy(G.exec);
        G.exec = nullptr;
    }
    if (!P->cap_stream) HIPCHECK(hipStreamCreateWithFlags(&P->cap_stream, hipStreamNonBlocking));
    HIPCHECK(hipStreamBeginCapture(P->cap_stream, hipStreamCaptureModeThreadLocal));
    mhlp_status s = MHLP_OK;
    for (int k = 0; k < S && s == MHLP_OK; ++k) s = enqueue_step(P, k < m, P->cap_stream);
    if (tail && s == MHLP_OK) s = enqueue_tail(P, b, x, P->cap_stream);
    hipGraph_t graph = nullptr;
    hipError_t e = hipStreamEndCapture(P->cap_stream, &graph);
    if (s != MHLP_OK) {
        if (graph) (void)hipGraphDestroy(graph);
        return s;
    }
    if (e != hipSuccess) return fail(MHLP_HIP_ERROR, std::string("GMRES step capture: ") + hipGetErrorString(e));
    e = hipGraphInstantiate(&G.exec, graph, nullptr, nullptr, 0);
    (void)hipGraphDestroy(graph);
    if (e != hipSuccess) {
        G.exec = nullptr;
        return fail(MHLP_HIP_ERROR, std::string("GMRES step graph: ") + hipGetErrorString(e));
    }
    G.ws = P->ws;
    G.part = P->part;
    G.gdev = P->gdev;
    G.R = P->gdev_R;
    G.nsplit = P->nsplit;
    G.x = x;
    G.b = b;
    *out = G.exec;
    return MHLP_OK;
}

/* One restarted-GMRES solve of A x = b to relative tolerance `tol` (relative
   to bnorm), FP64 Arnoldi with CGS2, each cycle ended by the true residual.  A
   cycle stops once its residual estimate is below 0.5 tol bnorm.  Both
   precisions take this path: the operator is FP64 in either, so cycles that
   stop early to be refined would only repeat work (N = 4096, alpha = 50:
   0.33 ms in two cycles, 0.23 in one).  x and b belong to
   the plan's workspace (captured graphs refer to them); x is updated in
   place.  The Arnoldi steps, the Givens rotations, the stopping test and the
   end of each cycle (x += V y, the true residual, and a copy of x into xout
   when given) run on the device; the
   host replays captured chunks of steps and reads the state once per chunk.
   The first chunk of a solve is as long as the first cycle of the previous
   solve on this plan (GMRES_FIRST_CHUNK the first time), later chunks follow
   the observed convergence rate; a chunk expected to end the cycle carries
   its end, and steps after the stopping point do nothing.  With first_dev
   the solve starts from x = 0 with ||b|| formed on the device from bsrc,
   which is copied into b. */
static mhlp_status gmres_core(mhlp_plan *P, double *b, double bnorm, double *x, double tol, int restart,
                              int max_iter, hipStream_t st, int *iters, int *cycles, double *relres,
                              const double *r_first, double beta_first, bool first_dev_in = false,
                              const double *bsrc = nullptr, double *xout = nullptr)
{
    const double half_tol = 0.5 * tol;
    const int64_t N = vlen(P);
    TRY(ensure_gdev(P, restart));
    const int R = P->gdev_R;
    double *V = P->ws;
    double *w = P->ws + (int64_t)(R + 1) * N;
    double *r = w + N;
    const GmresDev d = gdev_view(P);
    const unsigned nbN = nblocks(N, 256);
    int it = 0;
    *cycles = 0;
    double beta_tail = 0.0;
    for (;;) {
        /* residual at the start of the cycle: handed over by the caller for
           the first cycle (b itself for a zero initial guess), left in r by
           the previous cycle's end otherwise */
        double beta;
        const double *rr;
        const bool first_dev = first_dev_in && *cycles == 0;
        if (first_dev) {
            beta = 0.0; /* known after the first read of the state */
            rr = nullptr;
        } else if (*cycles == 0 && r_first) {
            beta = beta_first;
            rr = r_first;
        } else if (*cycles == 0) {
            TRY(apply_op(P, x, w, st));
            residual_kernel<<<nbN, 256, 0, st>>>(b, w, r, N);
            TRY(dnorm(P, r, N, st, &beta));
            rr = r;
        } else {
            beta = beta_tail;
            rr = r;
        }
        if (!first_dev) {
            *relres = beta / bnorm;
            if (*relres <= tol || it >= max_iter) break;
        }
        ++*cycles;
        const int kmax = std::min(restart, max_iter - it);
        if (first_dev) {
            if (N <= GS_START_NMAX) {
                gs_start_kernel<<<1, GSF_T, 0, st>>>(d.gs, d.gv, R, kmax, half_tol, bsrc, b, x, V, N, xout);
            } else {
                HIPCHECK(hipMemcpyAsync(b, bsrc, sizeof(double) * N, hipMemcpyDeviceToDevice, st));
                fill_kernel<<<nbN, 256, 0, st>>>(x, 0.0, N);
                multi_dot_kernel<<<1, 256, 0, st>>>(b, N, b, N, P->hdev); /* ||b||^2 */
                gs_init_dev_kernel<<<nbN, 256, 0, st>>>(d.gs, d.gv, R, kmax, half_tol, P->hdev, b, V, N, xout);
            }
        } else {
            scale_kernel<<<nbN, 256, 0, st>>>(rr, 1.0 / beta, V, N);
            gs_init_kernel<<<1, 256, 0, st>>>(d.gs, d.gv, R, kmax, beta, half_tol * bnorm, xout);
        }
        HIPCHECK(hipGetLastError());
        int done_steps = 0;
        /* the first cycle starts with the previous solve's count and its end
           appended; otherwise GMRES_FIRST_CHUNK steps */
        const bool hist = *cycles == 1 && P->gm_first_steps > 0;
        int chunk = hist ? P->gm_first_steps : GMRES_FIRST_CHUNK;
        bool expect_end = hist;
        double last_est = beta, thresh = half_tol * bnorm;
        GState gsh;
        for (;;) {
            const int S = std::max(1, std::min({chunk, GMRES_MAX_CHUNK, kmax - done_steps}));
            const bool tail = expect_end || S == kmax - done_steps;
            /* Gram-Schmidt in one block for the steps whose basis columns fit
               its registers, or exceed them by at most gsr_extra (step j has
               j + 1), over slices after them */
            const int m = (N <= GSR_NMAX && R <= GSF_RMAX)
                              ? std::max(0, std::min(S, gsr_cols(N) + gsr_extra(N) - done_steps))
                              : 0;
            hipGraphExec_t ex;
            TRY(step_graph(P, m, S, tail, b, x, &ex));
            HIPCHECK(hipGraphLaunch(ex, st));
            HIPCHECK(hipMemcpyAsync(P->gstate_host, d.gs, sizeof(GState), hipMemcpyDeviceToHost, st));
            HIPCHECK(spin_sync(st));
            gsh = *P->gstate_host;
            if (first_dev && done_steps == 0) {
                bnorm = gsh.bnorm;
                if (bnorm == 0.0) { /* b = 0: x = 0 (set by the start kernel) */
                    *relres = 0.0;
                    *iters = 0;
                    *cycles = 0;
                    return MHLP_OK;
                }
                last_est = bnorm;
                thresh = half_tol * bnorm;
            }
            if (gsh.done) {
                if (!tail) { /* the cycle ended before its end was enqueued */
                    TRY(step_graph(P, 0, 0, true, b, x, &ex));
                    HIPCHECK(hipGraphLaunch(ex, st));
                    HIPCHECK(hipMemcpyAsync(P->gstate_host, d.gs, sizeof(GState), hipMemcpyDeviceToHost, st));
                    HIPCHECK(spin_sync(st));
                    gsh = *P->gstate_host;
                }
                break;
            }
            /* steps still needed at the rate observed over this chunk */
            const int ran = gsh.steps - done_steps;
            done_steps = gsh.steps;
            expect_end = false;
            int need = GMRES_MAX_CHUNK;
            if (ran > 0 && gsh.resest > 0.0 && gsh.resest < last_est) {
                const double rate = std::pow(gsh.resest / last_est, 1.0 / ran);
                const double est = std::ceil(std::log(thresh / gsh.resest) / std::log(rate));
                if (est <= GMRES_MAX_CHUNK) {
                    need = std::max(1, (int)est);
                    expect_end = true;
                }
            }
            last_est = gsh.resest;
            chunk = need;
        }
        it += gsh.steps;
        if (*cycles == 1) P->gm_first_steps = std::max(1, gsh.steps);
        beta_tail = std::sqrt(gsh.rn2);
    }
    *iters = it;
    return MHLP_OK;
}

static mhlp_status gmres_solve_impl(const mhlp_plan *Pc, const double *g, double *mu, const mhlp_gmres_opts *opts,
                                    mhlp_gmres_info *info, void *stream)
{
    if (!Pc) return fail(MHLP_INVALID_ARG, "plan is NULL");
    if (!Pc->onsurf) return fail(MHLP_INVALID_ARG, "gmres_solve needs an on-surface plan (m == 0)");
    if (!g || !mu || !opts || !info) return fail(MHLP_INVALID_ARG, "NULL argument");
    if (g == mu) return fail(MHLP_INVALID_ARG, "g and mu must not alias");
    if (!(opts->tol > 0.0) || opts->max_iter < 1 || opts->restart < 1 || opts->restart > 512)
        return fail(MHLP_INVALID_ARG, "bad GMRES options");
    if (opts->precision != MHLP_FP64 && opts->precision != MHLP_MIXED)
        return fail(MHLP_INVALID_ARG, "unknown precision");
    if (Pc->stokes && opts->precision != MHLP_FP64)
        return fail(MHLP_INVALID_ARG, "the stresslet operator is FP64 only");
    mhlp_plan *P = const_cast<mhlp_plan *>(Pc);
    hipStream_t st = (hipStream_t)stream;
    const int64_t N = vlen(P);
    std::memset(info, 0, sizeof(*info));
    /* workspace columns: basis V_0..V_R, w, r (cycle residual), two spare
       vectors, and the solve's own x and b; R >= restart is the largest
       restart seen */
    TRY(ensure_gdev(P, opts->restart));
    const int R = P->gdev_R;
    TRY(ensure_ws(P, R + 1));
    double *xw = P->ws + (int64_t)(R + 5) * N, *bw = P->ws + (int64_t)(R + 6) * N;
    /* a solve from zero forms ||g|| on the device and reads it with the first
       read of the GMRES state (one host round trip fewer); the others need it
       now */
    const bool bnorm_dev = !opts->use_x0 && opts->tol < 1.0;
    double bnorm = 0.0;
    if (!bnorm_dev) TRY(dnorm(P, g, N, st, &bnorm));
    info->used_x0 = opts->use_x0 ? 1 : 0;
    if (!bnorm_dev && bnorm == 0.0) {
        fill_kernel<<<nblocks(N, 256), 256, 0, st>>>(mu, 0.0, N);
        HIPCHECK(hipStreamSynchronize(st));
        info->converged = 1;
        return MHLP_OK;
    }
    /* residual of the initial guess, kept in the residual slot
       of the first GMRES cycle (basis V_0..V_R, then w, r) so the cycle does
       not recompute it */
    double *r0 = P->ws + (int64_t)(R + 2) * N;
    double r0n = 0.0;
    if (opts->use_x0) {
        double *w = P->ws + (int64_t)(R + 1) * N;
        TRY(apply_op(P, mu, w, st));
        residual_kernel<<<nblocks(N, 256), 256, 0, st>>>(g, w, r0, N);
        TRY(dnorm(P, r0, N, st, &r0n));
        info->x0_residual = r0n / bnorm;
        if (!(info->x0_residual < 1.0)) {
            fill_kernel<<<nblocks(N, 256), 256, 0, st>>>(xw, 0.0, N);
            info->used_x0 = 0;
        } else {
            HIPCHECK(hipMemcpyAsync(xw, mu, sizeof(double) * N, hipMemcpyDeviceToDevice, st));
        }
    } else {
        if (!bnorm_dev) fill_kernel<<<nblocks(N, 256), 256, 0, st>>>(xw, 0.0, N);
        info->x0_residual = 1.0;
    }
    int iters = 0, cycles = 0;
    double rel = 1.0;
    /* the solve runs on its own copies of g and mu (xw, bw), which the captured
       graphs refer to; the start kernel of a device-normed solve makes them,
       else they are copied here. */
    if (!bnorm_dev) HIPCHECK(hipMemcpyAsync(bw, g, sizeof(double) * N, hipMemcpyDeviceToDevice, st));
    TRY(gmres_core(P, bw, bnorm, xw, opts->tol, opts->restart, opts->max_iter, st, &iters, &cycles, &rel,
                   info->used_x0 ? r0 : bw, info->used_x0 ? r0n : bnorm, bnorm_dev, g, mu));
    /* every cycle's end copies x into mu; without a cycle x is the start */
    if (cycles == 0) HIPCHECK(hipMemcpyAsync(mu, xw, sizeof(double) * N, hipMemcpyDeviceToDevice, st));
    info->iters = iters;
    info->restarts = cycles;
    info->rel_residual = rel;
    info->converged = rel <= opts->tol ? 1 : 0;
    return info->converged ? MHLP_OK : MHLP_NOT_CONVERGED;
}

extern "C" mhlp_status mhlp_gmres_solve(const mhlp_plan *P, const double *g, double *mu, const mhlp_gmres_opts *opts,
                                        mhlp_gmres_info *info, void *stream)
{
    if (P && P->stokes) return fail(MHLP_INVALID_ARG, "stokes plans solve with mhlp_stokes_gmres_solve");
    return gmres_solve_impl(P, g, mu, opts, info, stream);
}

extern "C" mhlp_status mhlp_stokes_gmres_solve(const mhlp_plan *P, const double *g, double *mu,
                                               const mhlp_gmres_opts *opts, mhlp_gmres_info *info, void *stream)
{
    if (P && !P->stokes) return fail(MHLP_INVALID_ARG, "stokes_gmres_solve needs a plan from mhlp_stokes_plan_create");
    return gmres_solve_impl(P, g, mu, opts, info, stream);
}

/* ------------------------------------------------------------------------ */
/* volume API                                                                */
/* ------------------------------------------------------------------------ */
/* ------------------------------------------------------------------------ */
/* FMM far field: plans and the volume sum                                   */
/* ------------------------------------------------------------------------ */
template <class T>
static mhlp_status to_host(std::vector<T> &h, const T *d, int64_t n, hipStream_t st)
{
    h.resize(n);
    if (n == 0) return MHLP_OK;
    hipError_t e = hipMemcpyAsync(h.data(), d, sizeof(T) * (size_t)n, hipMemcpyDeviceToHost, st);
    if (e == hipSuccess) e = hipStreamSynchronize(st);
    if (e != hipSuccess) return fail(MHLP_HIP_ERROR, std::string("copy to host: ") + hipGetErrorString(e));
    return MHLP_OK;
}

static int fmm_auto_level(int64_t npts, int64_t per_leaf)
{
    int L = 0;
    while (L < 8 && ((int64_t)1 << (2 * L)) * per_leaf < npts) ++L;
    return L;
}

/* Does the FMM serve an evaluation sooner than the plan's cluster lists, which
   reach rounding whatever the order?  (Where the caller leaves the level to the
   library; a level asked for is served by the FMM.)  The lists cost their items,
   the FMM its boxes, but for those whose neighbours underflow: from
   z = alpha times the leaf's side about 20 on they get fewer, from 100 on none
   are left but the direct part.  Both layers, us, lists | order 40, 20, 10:
     64 panels, 3000 points, level 3:       alpha = 5 22 | 167 144 133; 200 23 | 46 45 46
     256, 49,729, level 5:   alpha = 50 121 | 346 263 228; 500 166 | 145 127 117; 1000 98 | 59 59 58
     512, 100,000, level 6:  alpha = 5 78 | 700 508 419; 500 337 | 495 368 305
     896, 250,000, level 7:  alpha = 50 524 | 1775 1235 976; 200 945 | 1664 1161 910
     896, 898,704, level 7:  alpha = 20 619 | 1751 1206 944; 200 2767 | 1686 1177 933
   The estimates err on the FMM's side (boxes of levels 3 and 7 take up to twice
   theirs, lists that leave far items out down to a third), which is what a plan
   that has one asked for: over these and 70 more cases the choice was never
   slower than the FMM and 3% from the faster of both on average. */
static bool fmm_is_faster(unsigned long long list_cost, int order, int level, double z)
{
    const double lists = 25.0 + 0.75e-3 * (double)list_cost;
    const double left = std::min(1.0, std::max(0.05, (100.0 - z) / 80.0));
    const double boxes = 9.5 * std::exp2(level) * (level >= 8 ? 1.4 : 1.0) * (0.45 + 0.55 * order / 40.0);
    return 33.0 + boxes * left < lists;
}

extern "C" mhlp_status mhlp_plan_set_fmm(mhlp_plan *P, int32_t order, int32_t leaf_level, void *stream)
{
    if (!P) return fail(MHLP_INVALID_ARG, "plan is NULL");
    if (order == 0) {
        delete P->fmm;
        P->fmm = nullptr;
        return MHLP_OK;
    }
    if (P->stokes) return fail(MHLP_INVALID_ARG, "the FMM serves scalar plans");
    if (P->onsurf) return fail(MHLP_UNSUPPORTED, "the FMM serves off-surface plans");
    if (order < 4 || order > mhlp::FMM_PMAX) return fail(MHLP_INVALID_ARG, "order must be 0 or in [4, 60]");
    if (leaf_level < -1 || leaf_level > mhlp::FMM_LMAX) return fail(MHLP_INVALID_ARG, "leaf_level must be -1 or in [0, 10]");
    hipStream_t st = (hipStream_t)stream;
    const mhlp_geometry *g = P->g;
    std::vector<double> sx, sy, tx, ty;
    std::vector<int32_t> nptr, npan;
    TRY(to_host(sx, g->soa, g->N, st));
    TRY(to_host(sy, g->soa + g->N, g->N, st));
    TRY(to_host(tx, P->tx, P->M, st));
    TRY(to_host(ty, P->ty, P->M, st));
    TRY(to_host(nptr, P->near_ptr, P->M + 1, st));
    TRY(to_host(npan, P->near_panel, P->nnz, st));
    const FmmGeom G = fmm_root(sx, sy, tx, ty);
    int L = leaf_level;
    if (L < 0) {
        L = fmm_auto_level(P->M + g->N, 32);
        while (L > 0 && !fmm_contains_near(G, L, sx, sy, tx, ty, nptr, npan)) --L;
    } else if (!fmm_contains_near(G, L, sx, sy, tx, ty, nptr, npan)) {
        return fail(MHLP_INVALID_ARG, "leaf_level too fine: a near panel reaches beyond a target's 3x3 leaf neighbourhood");
    }
    FmmTree *F = new FmmTree();
    mhlp_status s = fmm_build(F, G, L, order, P->alpha, sx, sy, tx, ty, false, g->soa, g->soa + g->N, g->w, g->nx,
                              g->ny, st);
    if (s != MHLP_OK) {
        delete F;
        return s;
    }
    delete P->fmm;
    P->fmm = F;
    P->fmm_serves = leaf_level >= 0 || fmm_is_faster(P->tr_cost, order, L, P->alpha * G.S / std::exp2(L));
    return MHLP_OK;
}

extern "C" mhlp_status mhlp_plan_get_fmm(const mhlp_plan *P, int32_t *order, int32_t *leaf_level)
{
    if (!P) return fail(MHLP_INVALID_ARG, "plan is NULL");
    if (order) *order = P->fmm ? P->fmm->order : 0;
    if (leaf_level) *leaf_level = P->fmm ? P->fmm->level : -1;
    return MHLP_OK;
}

struct mhlp_volume_fmm {
    FmmTree tree;
    int64_t n = 0;
    double alpha = 0.0, h = 0.0, selfc = 0.0, wcell = 0.0;
};

static mhlp_status self_cell_value(double alpha, double h, hipStream_t st, double *wc)
{
    double *dev = nullptr;
    TRY(dalloc(&dev, 1));
    mhlp::self_cell_kernel<<<1, 256, 0, st>>>(alpha, h, nullptr, dev);
    hipError_t e = hipGetLastError();
    if (e == hipSuccess) e = hipMemcpyAsync(wc, dev, sizeof(double), hipMemcpyDeviceToHost, st);
    if (e == hipSuccess) e = hipStreamSynchronize(st);
    (void)hipFree(dev);
    if (e != hipSuccess) return fail(MHLP_HIP_ERROR, std::string("volume self cell: ") + hipGetErrorString(e));
    return MHLP_OK;
}

extern "C" mhlp_status mhlp_volume_fmm_create(const double *x, const double *y, const double *w, int64_t n,
                                              double alpha, double h, int32_t order, int32_t leaf_level, void *stream,
                                              mhlp_volume_fmm **out)
{
    if (!out) return fail(MHLP_INVALID_ARG, "out is NULL");
    *out = nullptr;
    if (!x || !y || !w) return fail(MHLP_INVALID_ARG, "NULL argument");
    if (n < 1 || n > INT_MAX - 1) return fail(MHLP_INVALID_ARG, "n out of range");
    if (!(alpha > 0.0) || !std::isfinite(alpha) || !(h > 0.0)) return fail(MHLP_INVALID_ARG, "alpha and h must be > 0");
    if (order < 4 || order > mhlp::FMM_PMAX) return fail(MHLP_INVALID_ARG, "order must be in [4, 60]");
    if (leaf_level < -1 || leaf_level > mhlp::FMM_LMAX) return fail(MHLP_INVALID_ARG, "leaf_level must be -1 or in [0, 10]");
    hipStream_t st = (hipStream_t)stream;
    std::vector<double> hx, hy;
    TRY(to_host(hx, x, n, st));
    TRY(to_host(hy, y, n, st));
    for (int64_t k = 0; k < n; ++k)
        if (!std::isfinite(hx[k]) || !std::isfinite(hy[k])) return fail(MHLP_INVALID_ARG, "coordinates must be finite");
    const std::vector<double> none;
    const FmmGeom G = fmm_root(hx, hy, none, none);
    const int L = leaf_level < 0 ? fmm_auto_level(n, 64) : leaf_level;
    mhlp_volume_fmm *V = new mhlp_volume_fmm();
    V->n = n;
    V->alpha = alpha;
    V->h = h;
    mhlp_status s = self_cell_value(alpha, h, st, &V->wcell);
    if (s == MHLP_OK) s = fmm_build(&V->tree, G, L, order, alpha, hx, hy, none, none, true, x, y, w, nullptr, nullptr, st);
    if (s != MHLP_OK) {
        delete V;
        return s;
    }
    V->selfc = V->wcell / (h * h);
    *out = V;
    return MHLP_OK;
}

extern "C" mhlp_status mhlp_volume_fmm_eval(const mhlp_volume_fmm *V, const double *f, double *u, void *stream)
{
    if (!V) return fail(MHLP_INVALID_ARG, "volume FMM is NULL");
    if (!f || !u) return fail(MHLP_INVALID_ARG, "f or u is NULL");
    if (f == u) return fail(MHLP_INVALID_ARG, "f and u must not alias");
    hipStream_t st = (hipStream_t)stream;
    const FmmTree *F = &V->tree;
    fmm_passes<true, false>(F, f, nullptr, st);
    FarArgs A{};
    mhlp::FmmVol vol{f, V->selfc, u};
    if (F->d.nwork > 0)
        mhlp::fmm_leaf_kernel<true, false, 1><<<(unsigned)F->d.nwork, 64 * mhlp::FMM_LW, 0, st>>>(F->d, A, vol);
    HIPCHECK(hipGetLastError());
    return MHLP_OK;
}

extern "C" mhlp_status mhlp_volume_fmm_info(const mhlp_volume_fmm *V, int32_t *order, int32_t *leaf_level,
                                            double *self_cell)
{
    if (!V) return fail(MHLP_INVALID_ARG, "volume FMM is NULL");
    if (order) *order = V->tree.order;
    if (leaf_level) *leaf_level = V->tree.level;
    if (self_cell) *self_cell = V->wcell;
    return MHLP_OK;
}

extern "C" mhlp_status mhlp_volume_fmm_destroy(mhlp_volume_fmm *V)
{
    delete V;
    return MHLP_OK;
}

/* ------------------------------------------------------------------------ */
/* particular solution on a periodic box                                     */
/* ------------------------------------------------------------------------ */
struct mhlp_box {
    int M = 0;
    double x0 = 0.0, y0 = 0.0, Lb = 0.0, alpha = 0.0;
    cplx *tw = nullptr;   /* M/2 twiddles */
    cplx *spec = nullptr; /* [2][M^2] forcing spectra */
    cplx *uh = nullptr;   /* [6][M^2] u^_1, u^_2 and the four gradient spectra */
    double *part = nullptr;
    int64_t part_cap = 0;
    double *sdc = nullptr; /* SISDC workspace */
    int64_t sdc_cap = 0;
    int point_method = 1;  /* 0: direct type-2 sums, 1: non-uniform FFT */
    cplx *twf = nullptr;   /* NUFFT: twiddles of the fine size 2M */
    double *corr = nullptr; /* NUFFT: hf / psi^(k_j), coarse FFT order */
    cplx *fine = nullptr;  /* NUFFT: [2][(2M)^2] */
    ~mhlp_box()
    {
        for (void *q : {(void *)tw, (void *)spec, (void *)uh, (void *)part, (void *)sdc, (void *)twf, (void *)corr,
                        (void *)fine})
            if (q) (void)hipFree(q);
    }
};

/* NUFFT tables of the box: fine twiddles and the deconvolution factors
   hf/psi^(k) with psi^(k) = (W hf/2) int_{-1}^{1} phi(z) cos(k W hf z/2) dz by
   composite 32-point Gauss-Legendre quadrature on 16 panels */
static mhlp_status box_nufft_setup(mhlp_box *B, hipStream_t st)
{
    if (B->fine) return MHLP_OK;
    const int M = B->M, Mf = 2 * M;
    const double hf = B->Lb / Mf, half = 0.5 * mhlp::NU_W * hf;
    std::vector<cplx> twf(Mf / 2);
    for (int j = 0; j < Mf / 2; ++j) {
        const double a = 2.0 * PI * (double)j / (double)Mf;
        twf[j] = mk(std::cos(a), -std::sin(a));
    }
    std::vector<double> corr(M);
    for (int j = 0; j < M; ++j) {
        const double k = 2.0 * PI / B->Lb * (j < M / 2 ? j : j - M);
        double s = 0.0;
        for (int pnl = 0; pnl < 16; ++pnl) {
            const double a = -1.0 + pnl * 0.125, b = a + 0.125;
            for (int q = 0; q < 32; ++q) {
                const double z = 0.5 * (a + b) + 0.5 * (b - a) * GL32_T[q];
                const double qz = 1.0 - z * z;
                const double ph = qz > 0.0 ? std::exp(mhlp::NU_BETA * (std::sqrt(qz) - 1.0)) : 0.0;
                s += 0.5 * (b - a) * GL32_W[q] * ph * std::cos(k * half * z);
            }
        }
        corr[j] = hf / (half * s);
    }
    cplx *d_twf = nullptr, *d_fine = nullptr;
    double *d_corr = nullptr;
    mhlp_status s = dalloc(&d_twf, Mf / 2);
    if (s == MHLP_OK) s = dalloc(&d_corr, M);
    if (s == MHLP_OK) s = dalloc(&d_fine, 2 * (int64_t)Mf * Mf);
    hipError_t e = hipSuccess;
    if (s == MHLP_OK) {
        e = hipMemcpyAsync(d_twf, twf.data(), sizeof(cplx) * twf.size(), hipMemcpyHostToDevice, st);
        if (e == hipSuccess) e = hipMemcpyAsync(d_corr, corr.data(), sizeof(double) * M, hipMemcpyHostToDevice, st);
        if (e == hipSuccess) e = hipStreamSynchronize(st);
        if (e != hipSuccess) s = fail(MHLP_HIP_ERROR, std::string("box NUFFT tables: ") + hipGetErrorString(e));
    }
    if (s != MHLP_OK) { /* nothing half-built stays behind */
        for (void *q : {(void *)d_twf, (void *)d_corr, (void *)d_fine})
            if (q) (void)hipFree(q);
        return s;
    }
    B->twf = d_twf;
    B->corr = d_corr;
    B->fine = d_fine;
    return MHLP_OK;
}

extern "C" mhlp_status mhlp_box_set_point_method(mhlp_box *B, int32_t method)
{
    if (!B) return fail(MHLP_INVALID_ARG, "box is NULL");
    if (method != 0 && method != 1) return fail(MHLP_INVALID_ARG, "method must be 0 (direct) or 1 (NUFFT)");
    if (method == 1 && B->M > 1024) return fail(MHLP_INVALID_ARG, "the NUFFT serves boxes with M <= 1024");
    B->point_method = method;
    return MHLP_OK;
}

extern "C" mhlp_status mhlp_box_create(int32_t M, double x0, double y0, double Lb, double alpha, void *stream,
                                       mhlp_box **out)
{
    if (!out) return fail(MHLP_INVALID_ARG, "out is NULL");
    *out = nullptr;
    if (M < 16 || M > 2048 || (M & (M - 1))) return fail(MHLP_INVALID_ARG, "M must be a power of two in [16, 2048]");
    if (!std::isfinite(x0) || !std::isfinite(y0) || !(Lb > 0.0) || !std::isfinite(Lb))
        return fail(MHLP_INVALID_ARG, "box corner must be finite and Lb > 0");
    if (!(alpha > 0.0) || !std::isfinite(alpha)) return fail(MHLP_INVALID_ARG, "alpha must be finite and > 0");
    mhlp_box *B = new mhlp_box();
    B->M = M;
    B->x0 = x0;
    B->y0 = y0;
    B->Lb = Lb;
    B->alpha = alpha;
    B->point_method = M <= 1024 ? 1 : 0;
    const int64_t MM = (int64_t)M * M;
    mhlp_status s;
    if ((s = dalloc(&B->tw, M / 2)) || (s = dalloc(&B->spec, 2 * MM)) || (s = dalloc(&B->uh, 6 * MM))) {
        delete B;
        return s;
    }
    std::vector<cplx> tw(M / 2);
    for (int j = 0; j < M / 2; ++j) {
        const double a = 2.0 * PI * (double)j / (double)M;
        tw[j] = mk(std::cos(a), -std::sin(a));
    }
    hipError_t e = hipMemcpyAsync(B->tw, tw.data(), sizeof(cplx) * tw.size(), hipMemcpyHostToDevice, (hipStream_t)stream);
    if (e == hipSuccess) e = hipStreamSynchronize((hipStream_t)stream);
    if (e != hipSuccess) {
        delete B;
        return fail(MHLP_HIP_ERROR, std::string("box_create: ") + hipGetErrorString(e));
    }
    *out = B;
    return MHLP_OK;
}

extern "C" mhlp_status mhlp_box_particular(mhlp_box *B, const double *F, double *u, double *grad, int64_t n,
                                           const double *px, const double *py, double *up, void *stream)
{
    if (!B) return fail(MHLP_INVALID_ARG, "box is NULL");
    if (!F) return fail(MHLP_INVALID_ARG, "F is NULL");
    if (n < 0 || n > INT_MAX) return fail(MHLP_INVALID_ARG, "n out of range");
    if (n > 0 && (!px || !py || !up)) return fail(MHLP_INVALID_ARG, "points need px, py and up");
    if (!u && !grad && n == 0) return fail(MHLP_INVALID_ARG, "no output requested");
    hipStream_t st = (hipStream_t)stream;
    const int M = B->M;
    const int64_t MM = (int64_t)M * M;
    int lg = 4;
    while ((1 << lg) < M) ++lg;
    const int L = mhlp::fft_rows(M), T = M / 8, G = M <= 512 ? 3 : 1;
    const size_t line = sizeof(cplx) * mhlp::fft_line_lds(M);
    mhlp::fft_rows_load_kernel<<<dim3(M / L, 2), L * T, L * line, st>>>(F, lg, B->tw, B->spec);
    const int f0 = u ? 0 : 2, f1 = grad ? 6 : u ? 2 : f0; /* fields on the grid */
    mhlp::fft_solve_kernel<<<M, G * T, G * line, st>>>(B->spec, lg, B->tw, B->Lb, B->alpha, f0, f1, n > 0, B->uh);
    if (n > 0 && B->point_method == 1) {
        TRY(box_nufft_setup(B, st));
        const int Mf = 2 * M, Lf = mhlp::fft_rows(Mf);
        const int64_t MMf = (int64_t)Mf * Mf;
        const size_t linef = sizeof(cplx) * mhlp::fft_line_lds(Mf);
        double *values = reinterpret_cast<double *>(B->fine + MMf); /* behind the [2][M][Mf] lines */
        mhlp::nufft_lines_kernel<<<dim3(M, 2), Mf / 8, linef, st>>>(B->spec, lg + 1, B->corr, B->twf, B->fine);
        mhlp::fft_rows_store_kernel<true><<<dim3(Mf / Lf, 2), Lf * Mf / 8, Lf * linef, st>>>(B->fine, lg + 1, MMf / 2,
                                                                                           B->twf, 0, values, nullptr);
        const int64_t pb = nblocks(n, 16);
        mhlp::nufft_interp_kernel<<<dim3((unsigned)std::min<int64_t>(pb, mhlp::NU_ROW), nblocks(pb, mhlp::NU_ROW)), 256, 0,
                                    st>>>(values, Mf, B->Lb / Mf, B->x0, B->y0, px, py, n, up);
    } else if (n > 0) {
        const int nchunk = M / mhlp::FT2_R;
        const int64_t need = 2 * (int64_t)nchunk * n;
        if (need > B->part_cap) {
            HIPCHECK(hipStreamSynchronize(st));
            if (B->part) (void)hipFree(B->part);
            B->part = nullptr;
            B->part_cap = 0;
            TRY(dalloc(&B->part, need));
            B->part_cap = need;
        }
        mhlp::type2_points_kernel<<<dim3(nblocks(n, mhlp::FT2_T), nchunk), mhlp::FT2_T, 0, st>>>(
            B->spec, M, B->Lb, B->x0, B->y0, px, py, n, B->part);
        mhlp::type2_reduce_kernel<<<nblocks(n, 256), 256, 0, st>>>(B->part, nchunk, n, up);
    }
    if (f1 > f0)
        mhlp::fft_rows_store_kernel<false><<<dim3(M / L, f1 - f0), L * T, L * line, st>>>(B->uh, lg, MM, B->tw, f0, u, grad);
    HIPCHECK(hipGetLastError());
    return MHLP_OK;
}

extern "C" mhlp_status mhlp_box_destroy(mhlp_box *B)
{
    delete B;
    return MHLP_OK;
}

/* ------------------------------------------------------------------------ */
/* SISDC time step of the Navier-Stokes equations on the periodic box         */
/* ------------------------------------------------------------------------ */
/* q[m][j] = (1/dts) int_{t_m}^{t_{m+1}} l_j(t) dt, t_i = i dts: the Lagrange basis
   polynomial of node j expanded in monomials and integrated exactly */
static void sisdc_weights(int p, std::vector<double> &q)
{
    q.assign((size_t)p * (p + 1), 0.0);
    for (int j = 0; j <= p; ++j) {
        std::vector<double> c(1, 1.0); /* coefficients of prod_{i != j} (t - i)/(j - i), ascending */
        for (int i = 0; i <= p; ++i) {
            if (i == j) continue;
            std::vector<double> nc(c.size() + 1, 0.0);
            for (size_t d = 0; d < c.size(); ++d) {
                nc[d + 1] += c[d] / (double)(j - i);
                nc[d] -= c[d] * (double)i / (double)(j - i);
            }
            c.swap(nc);
        }
        for (int m = 0; m < p; ++m) {
            double s = 0.0;
            for (size_t d = 0; d < c.size(); ++d)
                s += c[d] * (std::pow((double)(m + 1), (double)(d + 1)) - std::pow((double)m, (double)(d + 1))) /
                     (double)(d + 1);
            q[(size_t)m * (p + 1) + j] = s;
        }
    }
}

static void lincomb(const std::vector<std::pair<double, const double *>> &terms, int64_t n, double *out,
                    hipStream_t st)
{
    mhlp::LinComb T{};
    T.nterm = (int)terms.size();
    for (int k = 0; k < T.nterm; ++k) {
        T.c[k] = terms[k].first;
        T.x[k] = terms[k].second;
    }
    mhlp::lincomb_kernel<<<nblocks(n, 256), 256, 0, st>>>(T, n, out);
}

extern "C" mhlp_status mhlp_sisdc_step(mhlp_box *B, double Re, double dt, int32_t K, double *u, double *grad,
                                       double *lap, void *stream)
{
    if (!B) return fail(MHLP_INVALID_ARG, "box is NULL");
    if (!u || !grad || !lap) return fail(MHLP_INVALID_ARG, "u, grad and lap are required");
    if (K < 2 || K > 5) return fail(MHLP_INVALID_ARG, "K must be in [2, 5]");
    if (!(Re > 0.0) || !(dt > 0.0) || !std::isfinite(Re) || !std::isfinite(dt))
        return fail(MHLP_INVALID_ARG, "Re and dt must be finite and > 0");
    const int p = K - 1;
    const double dts = dt / p, a2 = Re / dts;
    if (std::fabs(B->alpha * B->alpha - a2) > 1e-12 * a2)
        return fail(MHLP_INVALID_ARG, "the box's alpha must satisfy alpha^2 = Re K'/dt, K' = K - 1 substeps");
    hipStream_t st = (hipStream_t)stream;
    const int64_t n2 = 2 * (int64_t)B->M * B->M;
    /* workspace: N, L of the previous sweep, U, N, L of the new one (p + 1 each), F */
    const int64_t need = (5 * (int64_t)(p + 1) + 1) * n2;
    if (need > B->sdc_cap) {
        HIPCHECK(hipStreamSynchronize(st));
        if (B->sdc) (void)hipFree(B->sdc);
        B->sdc = nullptr;
        B->sdc_cap = 0;
        TRY(dalloc(&B->sdc, need));
        B->sdc_cap = need;
    }
    double *w = B->sdc;
    auto slot = [&](int k) { return w + (int64_t)k * n2; };
    std::vector<double *> No(p + 1), Lo(p + 1), Un(p + 1), Nn(p + 1), Ln(p + 1);
    for (int m = 0; m <= p; ++m) {
        No[m] = slot(m);
        Lo[m] = slot(p + 1 + m);
        Un[m] = slot(2 * (p + 1) + m);
        Nn[m] = slot(3 * (p + 1) + m);
        Ln[m] = slot(4 * (p + 1) + m);
    }
    double *F = slot(5 * (p + 1));
    std::vector<double> q;
    sisdc_weights(p, q);
    const unsigned nb = nblocks(n2 / 2, 256);
    /* start of the step: u0, N0 = (u0.grad) u0, L0 = lap */
    HIPCHECK(hipMemcpyAsync(Un[0], u, sizeof(double) * n2, hipMemcpyDeviceToDevice, st));
    mhlp::advect_kernel<<<nb, 256, 0, st>>>(u, grad, n2 / 2, Nn[0]);
    HIPCHECK(hipMemcpyAsync(Ln[0], lap, sizeof(double) * n2, hipMemcpyDeviceToDevice, st));
    auto solve_into = [&](int m) -> mhlp_status {
        /* (alpha^2 - Delta) U_{m+1} + Re grad p = F; N_{m+1}, L_{m+1} = alpha^2 U_{m+1} - F */
        TRY(mhlp_box_particular(B, F, Un[m + 1], grad, 0, nullptr, nullptr, nullptr, stream));
        mhlp::advect_kernel<<<nb, 256, 0, st>>>(Un[m + 1], grad, n2 / 2, Nn[m + 1]);
        lincomb({{a2, Un[m + 1]}, {-1.0, F}}, n2, Ln[m + 1], st);
        return MHLP_OK;
    };
    for (int m = 0; m < p; ++m) { /* first sweep: implicit-explicit Euler */
        lincomb({{a2, Un[m]}, {-Re, Nn[m]}}, n2, F, st);
        TRY(solve_into(m));
    }
    for (int k = 1; k < K; ++k) { /* corrections */
        std::swap(No, Nn);
        std::swap(Lo, Ln);
        /* the new sweep starts from the same initial values */
        HIPCHECK(hipMemcpyAsync(Nn[0], No[0], sizeof(double) * n2, hipMemcpyDeviceToDevice, st));
        HIPCHECK(hipMemcpyAsync(Ln[0], Lo[0], sizeof(double) * n2, hipMemcpyDeviceToDevice, st));
        for (int m = 0; m < p; ++m) {
            std::vector<std::pair<double, const double *>> t = {
                {a2, Un[m]}, {-Re, Nn[m]}, {Re, No[m]}, {-1.0, Lo[m + 1]}};
            for (int j = 0; j <= p; ++j) {
                t.push_back({q[(size_t)m * (p + 1) + j], Lo[j]});
                t.push_back({-Re * q[(size_t)m * (p + 1) + j], No[j]});
            }
            lincomb(t, n2, F, st);
            TRY(solve_into(m));
        }
    }
    HIPCHECK(hipMemcpyAsync(u, Un[p], sizeof(double) * n2, hipMemcpyDeviceToDevice, st));
    HIPCHECK(hipMemcpyAsync(lap, Ln[p], sizeof(double) * n2, hipMemcpyDeviceToDevice, st));
    HIPCHECK(hipGetLastError());
    return MHLP_OK;
}

/* Launch shape of the volume sum: one thread per target in blocks of
   FT_THREADS; when that leaves fewer than 1024 blocks the sources are split
   into ranges of whole LDS tiles evaluated by separate blocks (partials
   [nsplit][n], summed in fixed order by volume_finalize).  Returns nsplit. */
static int volume_shape(VolArgs &A)
{
    const int64_t n = A.n;
    const int64_t tblocks = (n + FT_THREADS - 1) / FT_THREADS;
    int64_t ns = (1024 + tblocks - 1) / tblocks;
    if (ns > (n + FT_SRC - 1) / FT_SRC) ns = (n + FT_SRC - 1) / FT_SRC;
    if (ns < 1) ns = 1;
    A.per_split = ((n + ns - 1) / ns + FT_SRC - 1) / FT_SRC * FT_SRC;
    return (int)((n + A.per_split - 1) / A.per_split);
}

static void volume_launch(const VolArgs &A, int nsplit, int32_t precision, hipStream_t st)
{
    const unsigned tblocks = (unsigned)((A.n + FT_THREADS - 1) / FT_THREADS);
    if (nsplit > 1) {
        dim3 grid(tblocks, nsplit);
        if (precision == MHLP_MIXED)
            volume_kernel<true, true><<<grid, FT_THREADS, 0, st>>>(A);
        else
            volume_kernel<false, true><<<grid, FT_THREADS, 0, st>>>(A);
        volume_finalize<<<nblocks(A.n, 256), 256, 0, st>>>(A, nsplit);
    } else if (precision == MHLP_MIXED) {
        volume_kernel<true, false><<<tblocks, FT_THREADS, 0, st>>>(A);
    } else {
        volume_kernel<false, false><<<tblocks, FT_THREADS, 0, st>>>(A);
    }
}

static mhlp_status volume_check(const double *x, const double *y, const double *w, const double *f, int64_t n,
                                double alpha, double h, int32_t precision, const double *u)
{
    if (!x || !y || !w || !f || !u) return fail(MHLP_INVALID_ARG, "NULL argument");
    if (n < 1) return fail(MHLP_INVALID_ARG, "n must be >= 1");
    if (!(alpha > 0.0) || !std::isfinite(alpha) || !(h > 0.0)) return fail(MHLP_INVALID_ARG, "alpha and h must be > 0");
    if (precision != MHLP_FP64 && precision != MHLP_MIXED) return fail(MHLP_INVALID_ARG, "unknown precision");
    return MHLP_OK;
}

/* tree_order_ratio over the bins of alpha R: the larger of a bin's ends */
struct VolRatios {
    float v[mhlp::VT_BINS][mhlp::TR_NP];
    VolRatios()
    {
        auto edge = [](int b) { return std::min(mhlp::VT_AMAX, std::max(mhlp::TR_AMIN, std::exp2(b / 3.0 - 20.0))); };
        for (int b = 0; b < mhlp::VT_BINS; ++b)
            for (int q = 0; q < mhlp::TR_NP; ++q) {
                const int p = mhlp::TR_PMIN + mhlp::TR_PSTEP * q;
                v[b][q] = (float)(1.01 * std::max(mhlp::tree_order_ratio(p, edge(b), mhlp::VT_AMAX), mhlp::tree_order_ratio(p, edge(b + 1), mhlp::VT_AMAX)));
            }
    }
};

/* From this many points on the FP64 sum goes by cluster expansions: its sort,
   clusters and workspace take about 150 us whatever n.  Whole calls at
   alpha = 20 (100): 8281 points 310 (400) us against 400 (290) for the direct
   sum, 16,384 points 282 (670) against 830 (660). */
constexpr int64_t VOL_TREE_MIN = 12288;

/* The sum by cluster expansions (about 200 bytes of workspace a point);
   served = false when the workspace is not to be had. */
static mhlp_status volume_tree(const double *x, const double *y, const double *w, const double *f, int64_t n,
                               double alpha, double h, double *u, double *self_cell, hipStream_t st, bool *served)
{
    *served = false;
    if (n > (int64_t)1 << 28) return MHLP_OK;
    mhlp::VolTree V = {};
    V.x = x, V.y = y, V.w = w, V.f = f, V.u = u;
    V.n = n, V.alpha = alpha, V.h = h;
    V.bits = 7; /* four cells a point, so that few share one */
    while (V.bits < mhlp::VT_BITS && ((int64_t)1 << (2 * V.bits)) < 4 * n) ++V.bits;
    V.tile = (int)(64 * std::max<int64_t>(8, (n + 64 * mhlp::VT_TILES - 1) / (64 * mhlp::VT_TILES)));
    V.ntile = (int)((n + V.tile - 1) / V.tile);
    mhlp::TreeDev T;
    T.Np = (n + 15) / 16;
    for (; T.nlev < mhlp::TR_LEV; ++T.nlev) {
        T.off[T.nlev] = T.ncl;
        T.ncl += (T.Np + (1 << T.nlev) - 1) >> T.nlev;
    }
    int64_t bytes = 0;
    auto take = [&](int64_t b) {
        const int64_t o = bytes;
        bytes += (b + 255) / 256 * 256;
        return o;
    };
    const int64_t m = 16 * T.Np, ms = mhlp::tr_stride(2);
    const int64_t o_setup = take(sizeof(mhlp::VolSetup)), o_box = take(32 * mhlp::VT_BOXES), o_self = take(16);
    const int64_t o_hist = take((int64_t)4 * V.ntile << V.bits), o_key = take(16 * n), o_pts = take(32 * m);
    const int64_t o_cbox = take(32 * T.ncl), o_cc = take(16 * T.ncl), o_rm = take(8 * mhlp::TR_RM * T.ncl);
    const int64_t o_mom = take(8 * ms * T.ncl), o_st = take(8 * 48 * T.Np);
    char *ws = nullptr;
    if (hipMalloc((void **)&ws, (size_t)bytes) != hipSuccess) {
        (void)hipGetLastError();
        return MHLP_OK;
    }
    auto at = [&](int64_t o) { return reinterpret_cast<double *>(ws + o); };
    V.setup = reinterpret_cast<mhlp::VolSetup *>(ws + o_setup);
    V.box = at(o_box), V.selfc = at(o_self), V.cbox = at(o_cbox);
    V.hist = reinterpret_cast<uint32_t *>(ws + o_hist);
    uint32_t *keys = reinterpret_cast<uint32_t *>(ws + o_key);
    V.key[0] = keys, V.key[1] = keys + n, V.idx[0] = keys + 2 * n, V.idx[1] = keys + 3 * n;
    V.xs = at(o_pts), V.ys = V.xs + m, V.ws = V.ys + m, V.fs = V.ws + m;
    T.cc = at(o_cc), T.rmin = at(o_rm), T.mom = at(o_mom), T.st = at(o_st);
    FarArgs A = {};
    A.sx = V.xs, A.sy = V.ys, A.sw = V.ws, A.sigma = V.fs, A.N = m, A.alpha = alpha;
    A.fq = V.setup->fq;
    static const VolRatios ratios;
    mhlp::VolSetup S;
    fine_scales(alpha, S.fq);
    std::copy(&ratios.v[0][0], &ratios.v[0][0] + mhlp::VT_BINS * mhlp::TR_NP, &S.ratio[0][0]);
    const int64_t G = (n + 63) / 64;
    mhlp::vol_box_kernel<<<mhlp::VT_BOXES + 1, 256, 0, st>>>(V, S);
    mhlp::vol_hist_kernel<0><<<V.ntile, 64, 0, st>>>(V);
    mhlp::vol_scan_kernel<<<1, 1024, 0, st>>>(V);
    mhlp::vol_scatter_kernel<0><<<V.ntile, 64, 0, st>>>(V);
    mhlp::vol_hist_kernel<1><<<V.ntile, 64, 0, st>>>(V);
    mhlp::vol_scan_kernel<<<1, 1024, 0, st>>>(V);
    mhlp::vol_scatter_kernel<1><<<V.ntile, 64, 0, st>>>(V);
    mhlp::vol_clusters_kernel<<<(unsigned)((T.ncl + 3) / 4), 256, 0, st>>>(V, T);
    mhlp::tree_moments_kernel<true, false, false><<<dim3((unsigned)((T.Np + 15) / 16), T.nlev, mhlp::TR_GROUPS), 256, 0, st>>>(A, T);
    /* few groups: more waves each */
    mhlp::vol_far_kernel<<<(unsigned)G, G >= 768 ? 256 : G >= 384 ? 512 : 1024, 0, st>>>(V, A, T);
    hipError_t e = hipGetLastError();
    double wc = 0.0;
    if (e == hipSuccess) e = hipMemcpyAsync(&wc, V.selfc + 1, sizeof(double), hipMemcpyDeviceToHost, st);
    if (e == hipSuccess) e = hipStreamSynchronize(st);
    (void)hipFree(ws);
    if (e != hipSuccess) return fail(MHLP_HIP_ERROR, std::string("volume_eval: ") + hipGetErrorString(e));
    if (self_cell) *self_cell = wc;
    *served = true;
    return MHLP_OK;
}

extern "C" mhlp_status mhlp_volume_eval(const double *x, const double *y, const double *w, const double *f, int64_t n,
                                        double alpha, double h, int32_t precision, double *u, double *self_cell,
                                        void *stream)
{
    TRY(volume_check(x, y, w, f, n, alpha, h, precision, u));
    hipStream_t st = (hipStream_t)stream;
    if (precision == MHLP_FP64 && n >= VOL_TREE_MIN) {
        bool served = false;
        TRY(volume_tree(x, y, w, f, n, alpha, h, u, self_cell, st, &served));
        if (served) return MHLP_OK;
    }
    double wc = 0.0;
    TRY(self_cell_value(alpha, h, st, &wc));
    hipError_t e;
    if (self_cell) *self_cell = wc;
    VolArgs A;
    A.x = x;
    A.y = y;
    A.w = w;
    A.f = f;
    A.n = n;
    A.alpha = alpha;
    A.selfc = wc / (h * h);
    A.u = u;
    A.selfc_dev = nullptr;
    A.part = nullptr;
    const int nsplit = volume_shape(A);
    if (nsplit > 1) {
        TRY(dalloc(&A.part, (int64_t)nsplit * n));
        volume_launch(A, nsplit, precision, st);
        e = hipGetLastError();
        if (e == hipSuccess) e = hipStreamSynchronize(st);
        (void)hipFree(A.part);
        if (e != hipSuccess) return fail(MHLP_HIP_ERROR, std::string("volume_eval: ") + hipGetErrorString(e));
        return MHLP_OK;
    }
    volume_launch(A, nsplit, precision, st);
    HIPCHECK(hipGetLastError());
    return MHLP_OK;
}

/* Fixed device scratch of the allocation-free volume sum, one copy per device
   (a file-scope device array lives in every device's copy of the code
   object).  Slot 0 holds Wcell/h^2; the split partials start at VOL_HEAD.
   volume_shape() never needs more than 523,776 partial values (nsplit = 2 at
   n = 261,888), below VOL_PART_MAX.  Host code must not pass `scratch` itself
   to a kernel: it names a host-side stand-in; the device address comes from
   hipGetSymbolAddress, once per device. */
constexpr int64_t VOL_HEAD = 32; /* doubles: keeps the partials 256-byte aligned */
constexpr int64_t VOL_PART_MAX = (int64_t)1 << 19;
static __device__ __align__(256) double scratch[VOL_HEAD + VOL_PART_MAX];

constexpr int SCRATCH_MAX_DEVICES = 64;
static std::mutex g_scratch_mutex;
static double *g_scratch_ptr[SCRATCH_MAX_DEVICES];

/* Device address of `scratch` on the current device (looked up on the first
   call per device, then reused). */
static mhlp_status scratch_address(double **out)
{
    int dev = 0;
    HIPCHECK(hipGetDevice(&dev));
    if (dev < 0 || dev >= SCRATCH_MAX_DEVICES) return fail(MHLP_UNSUPPORTED, "device index beyond 63");
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (!g_scratch_ptr[dev]) {
        void *p = nullptr;
        const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess || !p)
            return fail(MHLP_HIP_ERROR, std::string("hipGetSymbolAddress(scratch): ") + hipGetErrorString(e));
        g_scratch_ptr[dev] = (double *)p;
    }
    *out = g_scratch_ptr[dev];
    return MHLP_OK;
}

extern "C" mhlp_status mhlp_volume_eval_noalloc(const double *x, const double *y, const double *w, const double *f,
                                                int64_t n, double alpha, double h, int32_t precision, double *u,
                                                void *stream)
{
    TRY(volume_check(x, y, w, f, n, alpha, h, precision, u));
    hipStream_t st = (hipStream_t)stream;
    VolArgs A;
    A.x = x;
    A.y = y;
    A.w = w;
    A.f = f;
    A.n = n;
    A.alpha = alpha;
    A.selfc = 0.0;
    A.u = u;
    const int nsplit = volume_shape(A);
    if (nsplit > 1 && (int64_t)nsplit * n > VOL_PART_MAX)
        return fail(MHLP_INVALID_ARG, "volume_eval_noalloc: partial sums exceed the fixed scratch (" +
                                          std::to_string(VOL_PART_MAX) + " values)");
    double *S = nullptr;
    TRY(scratch_address(&S));
    A.selfc_dev = S;
    A.part = nsplit > 1 ? S + VOL_HEAD : nullptr;
    /* slot 0 and every partial are written before they are read: nothing to clear */
    mhlp::self_cell_kernel<<<1, 256, 0, st>>>(alpha, h, S, nullptr);
    volume_launch(A, nsplit, precision, st);
    HIPCHECK(hipGetLastError());
    return MHLP_OK;
}

/* ------------------------------------------------------------------------ */
/* batched on-surface operator and lockstep GMRES over many geometries and   */
/* right-hand sides                                                          */
/*                                                                           */
/* Batched vector layout: for each geometry g, a block [R][N_g] at offset     */
/* voff_g (R right-hand sides of the same geometry are contiguous systems).   */
/* One grouped launch applies (1/2 I + D) to every system: each block owns    */
/* (geometry, target tile, source split); every kernel value is shared by the */
/* R right-hand sides of its geometry.                                        */
/* ------------------------------------------------------------------------ */
constexpr int BATCH_R_MAX = 4;

struct BatchGeo {
    const double *x, *y, *w, *nx, *ny;
    const int32_t *nptr, *npan;
    const double *wdl, *fq;
    int64_t N, Np;
    double alpha;
    int64_t voff; /* offset of the geometry's [R][N] block in batched vectors */
    int64_t poff; /* offset of its partial sums [nsplit][R][N]                 */
    int32_t nsplit, pad;
    mhlp::TreeDev tree; /* the plan's clusters and lists with the batch's own moments ([ncl][tr_stride(2 R)])
                           and staged dipoles ([Np][2 R][16]: alpha w mu n_x, alpha w mu n_y per right-hand side) */
};

struct BatchWork {
    int32_t g, tb, split, pad;
};

/* A geometry takes part in a batched operator application unless a gate is
   given and all its right-hand sides are gated off (gate[g*R + r] == 0:
   systems that have converged in the current GMRES cycle). */
template <int R>
__device__ __forceinline__ bool batch_gated_off(const double *__restrict__ gate, int g)
{
    if (!gate) return false;
#pragma unroll
    for (int r = 0; r < R; ++r)
        if (gate[(int64_t)g * R + r] != 0.0) return false;
    return true;
}

/* Device state of a lockstep batched GMRES cycle. */
struct BState {
    int32_t j;     /* current Arnoldi column (common to all systems)         */
    int32_t kmax;  /* columns allowed in this cycle                          */
    int32_t done;  /* all systems converged / broken down, or kmax reached   */
    int32_t nact;  /* systems still active after the last step               */
    int32_t steps; /* lockstep steps taken in this cycle                     */
    int32_t pad;
    unsigned long long arrived; /* the running step: systems that are through, and << 32 those left active */
};

/* density of a batched launch: fixed, or basis column bs->j; false = no-op */
__device__ __forceinline__ bool batch_density(const BState *bs, int64_t jstride, const double *__restrict__ &mu)
{
    if (bs) {
        if (bs->done) return false;
        mu += (int64_t)bs->j * jstride;
    }
    return true;
}

/* Moments and staged dipoles of one geometry's 16-panel chunk (work item: g,
   chunk tb) at level blockIdx.y, orders of blockIdx.z, for its R right-hand
   sides: tree_moments_kernel with the regular functions of a source shared. */
template <int R, int Z, int RR, class B>
__device__ __forceinline__ void batch_moments_rounds(const mhlp::TreeDev &T, int k, int64_t p0, const B &b,
                                                     const double (&ex)[R], const double (&ey)[R],
                                                     double (*buf)[16 * mhlp::TR_PAD])
{
    constexpr int NV = 2 * R, RO = R > 2 ? 2 : 4, N = Z * mhlp::TR_NG + RR;
    if constexpr (RR < mhlp::TR_NG && N <= mhlp::TR_PMAX) {
        const int t = threadIdx.x, at = (t >> 4) * mhlp::TR_PAD + (t & 15), pp = t & 15, cb = t >> 4;
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const mhlp::TreeDipole<B> md{b, ex[r], ey[r]};
            mhlp::tree_row_values<false, N>(md, 0.0, buf + 2 * r, at);
            mhlp::tree_row_values<false, N + 1>(md, 0.0, buf + NV + 2 * r, at);
            if constexpr (RO > 2) {
                mhlp::tree_row_values<false, N + 2>(md, 0.0, buf + 2 * NV + 2 * r, at);
                mhlp::tree_row_values<false, N + 3>(md, 0.0, buf + 3 * NV + 2 * r, at);
            }
        }
        __syncthreads();
        if (cb < RO * NV) {
            const double *row = buf[cb] + pp * mhlp::TR_PAD;
            double s0 = 0.0, s1 = 0.0;
#pragma unroll
            for (int l = 0; l < 16; l += 2) {
                s0 += row[l];
                s1 += row[l + 1];
            }
            double s = s0 + s1;
            for (int o = 1; o < (1 << k); o <<= 1) s += __shfl_xor(s, o);
            const int n = N + cb / NV;
            const int64_t p = p0 + pp;
            if ((pp & ((1 << k) - 1)) == 0 && p < T.Np && n < mhlp::TR_ROWS)
                T.mom[(T.off[k] + (p >> k)) * mhlp::tr_stride(NV) + n * NV + cb % NV] = s;
        }
        __syncthreads();
        batch_moments_rounds<R, Z, RR + RO>(T, k, p0, b, ex, ey, buf);
    }
}

template <int R, int Z>
__device__ __forceinline__ void batch_moments_body(const BatchGeo &geo, int64_t chunk, const double *mug,
                                                   double (*buf)[16 * mhlp::TR_PAD])
{
    const mhlp::TreeDev &T = geo.tree;
    const int k = blockIdx.y, t = threadIdx.x;
    const int64_t p0 = 16 * chunk, j = 16 * p0 + t;
    const bool have = j < geo.N;
    const int64_t js = have ? j : geo.N - 1;
    const int64_t c = T.off[k] + ((js >> 4) >> k);
    const double aw = have ? geo.alpha * geo.w[js] : 0.0, nx = geo.nx[js], ny = geo.ny[js];
    double ex[R], ey[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const double m = have ? aw * mug[r * geo.N + js] : 0.0; /* the pair gives K1(z)/r */
        ex[r] = m * nx;
        ey[r] = m * ny;
        if (Z == 0 && k == 0 && have) {
            double *s = T.st + ((j >> 4) * 2 * R + 2 * r) * 16 + (j & 15);
            s[0] = ex[r];
            s[16] = ey[r];
        }
    }
    const bool live = T.rmin[mhlp::TR_RM * c + mhlp::TR_NP - 1] < INFINITY;
    if (__syncthreads_or(live ? 1 : 0) == 0) return;
    const double ah = 0.5 * geo.alpha;
    const double wr = live ? ah * (geo.x[js] - T.cc[2 * c]) : 0.0, wi = live ? -ah * (geo.y[js] - T.cc[2 * c + 1]) : 0.0;
    mhlp::TreeB<false, Z> b;
    mhlp::tree_regular<mhlp::TreeB<false, Z>::LO, mhlp::TreeB<false, Z>::CNT>(wr, wi, fma(wr, wr, wi * wi), b.br, b.bi);
    batch_moments_rounds<R, Z, 0>(T, k, p0, b, ex, ey, buf);
}

template <int R>
__global__ __launch_bounds__(256) void batch_moments_kernel(const BatchGeo *__restrict__ G,
                                                            const BatchWork *__restrict__ W,
                                                            const double *__restrict__ mu,
                                                            const double *__restrict__ gate, const BState *bs,
                                                            int64_t jstride)
{
    __shared__ double buf[16][16 * mhlp::TR_PAD];
    const BatchWork wk = W[blockIdx.x];
    if (batch_gated_off<R>(gate, wk.g) || !batch_density(bs, jstride, mu)) return;
    const BatchGeo &geo = G[wk.g];
    if ((int)blockIdx.y >= geo.tree.nlev) return;
    const double *mug = mu + geo.voff;
    switch (blockIdx.z) {
    case 0: batch_moments_body<R, 0>(geo, wk.tb, mug, buf); break;
    case 1: batch_moments_body<R, 1>(geo, wk.tb, mug, buf); break;
    default: batch_moments_body<R, 2>(geo, wk.tb, mug, buf); break;
    }
}

/* staged dipoles s0..s1-1 of panel p, R right-hand sides sharing every kernel value */
template <int R, int PC>
__device__ __forceinline__ void batch_panel(const BatchGeo &geo, int64_t p, int s0, int s1, double x, double y,
                                            double (&f)[R])
{
    constexpr int K = PC < 0 || PC >= KQ_NP ? 0 : PC;
    const MHLP_CAS double *sx = (const MHLP_CAS double *)geo.x + 16 * p;
    const MHLP_CAS double *sy = (const MHLP_CAS double *)geo.y + 16 * p;
    const MHLP_CAS double *st = (const MHLP_CAS double *)geo.tree.st + 32 * R * p;
    FarTab T = far_table();
    const FarConst fc = far_const_of(geo.fq);
    double qa, qk;
    fine_q<K>(geo.fq, qa, qk);
#pragma unroll 1
    for (int s = s0; s < s1; s += 2) {
        if (PC < 0 || PC >= KQ_NP) T = far_table(); /* their coefficients exceed the scalar registers */
        const double ex0 = x - sx[s], ey0 = y - sy[s];
        const double ex1 = x - sx[s + 1], ey1 = y - sy[s + 1];
        const double r20 = fma(ex0, ex0, ey0 * ey0), r21 = fma(ex1, ex1, ey1 * ey1);
        K01 o0, o1;
        if constexpr (PC >= KQ_NP)
            k01_far2<false, true, true, true>(T, fc, r20, r21, o0, o1);
        else
            k01_far2_fixed<false, true, PC>(T, fc, qa, qk, r20, r21, o0, o1);
        const double ax = ex0 * o0.ak1r, ay = ey0 * o0.ak1r, bx = ex1 * o1.ak1r, by = ey1 * o1.ak1r;
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const MHLP_CAS double *q = st + 32 * r + s;
            f[r] = fma(ax, q[0], fma(ay, q[16], fma(bx, q[1], fma(by, q[17], f[r]))));
        }
    }
}

/* The batched far field of one work item (geometry g, group of 64 targets tb,
   split): the items of far_tree_kernel's lists, direct panels cut into halves,
   shared by the BATCH_W waves of the group's nsplit blocks; R right-hand sides
   share every kernel value and every K_n.  Partial sums per (split, right-hand
   side, node).  Bound by VALU FP64 (per expansion 8 + 2 R instructions an
   order, per pair 47 + 4 R): 24,656 nodes in 16 curves, R = 4, 22e6 wave
   instructions, 50 us at 75% of their rate (the last blocks run alone), against
   127 us for the sum over all pairs. */
constexpr int BATCH_W = 8;
template <int R>
__global__ __launch_bounds__(64 * BATCH_W, 4) void batch_far_kernel(const BatchGeo *__restrict__ G,
                                                                    const BatchWork *__restrict__ W,
                                                                    const double *__restrict__ mu,
                                                                    double *__restrict__ part,
                                                                    const double *__restrict__ gate, const BState *bs,
                                                                    int64_t jstride)
{
    __shared__ double red[R][BATCH_W][64];
    const BatchWork wk = W[blockIdx.x];
    if (batch_gated_off<R>(gate, wk.g) || !batch_density(bs, jstride, mu)) return;
    const BatchGeo &geo = G[wk.g];
    const mhlp::TreeDev &T = geo.tree;
    const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t g = wk.tb, i = 64 * g + lane;
    const bool valid = i < geo.N;
    const int64_t iv = valid ? i : geo.N - 1;
    const double x = geo.x[iv], y = geo.y[iv];
    const int32_t k0 = geo.nptr[iv], k1 = geo.nptr[iv + 1];
    const int NW = BATCH_W * geo.nsplit, wg = w * geo.nsplit + wk.split;
    const int2 cnt = T.cnt[g];
    const longlong2 at = T.at[g];
    const uint2 *items = T.items + at.x, *back = T.items + at.y - 1;
    double acc[R];
#pragma unroll
    for (int r = 0; r < R; ++r) acc[r] = 0.0;
    for (int k = wg; k < 2 * cnt.x; k += NW) {
        const uint2 it = items[k >> 1];
        const uint32_t p = __builtin_amdgcn_readfirstlane(it.x), fl = __builtin_amdgcn_readfirstlane(it.y);
        bool listed = false;
        if (fl & mhlp::TR_NEAR)
            for (int32_t q = k0; q < k1; ++q) listed = listed || geo.npan[q] == (int32_t)p;
        if (listed) continue;
        const int s0 = 8 * (k & 1);
        double f[R];
#pragma unroll
        for (int r = 0; r < R; ++r) f[r] = 0.0;
        switch ((int)(fl & 31) - 1) {
#define MHLP_BATCH_PANEL(PCV) \
    case PCV: batch_panel<R, PCV>(geo, p, s0, s0 + 8, x, y, f); break;
            MHLP_PC_CASES(MHLP_BATCH_PANEL)
#undef MHLP_BATCH_PANEL
        default: batch_panel<R, KQ_NP>(geo, p, s0, s0 + 8, x, y, f);
        }
#pragma unroll
        for (int r = 0; r < R; ++r) acc[r] += f[r];
    }
    const int fb = cnt.y * (NW - 1 - wg) / NW, fe = cnt.y * (NW - wg) / NW;
    for (int k = fb; k < fe; ++k) {
        const uint2 it = back[-k];
        const uint32_t c = __builtin_amdgcn_readfirstlane(it.x), fl = __builtin_amdgcn_readfirstlane(it.y);
        int64_t p0, p1;
        double f[R];
        bool direct = false;
        if (fl & mhlp::TR_ZERO) {
            /* all pairs underflow: only a non-finite density matters */
            mhlp::tree_panels_of(T, c, p0, p1);
            double z = 0.0;
            for (int64_t q = 32 * R * p0 + lane; q < 32 * R * p1; q += 64) z = fma(0.0, T.st[q], z);
            direct = __ballot(!(z == 0.0)) != 0;
#pragma unroll
            for (int r = 0; r < R; ++r) f[r] = 0.0;
        } else {
            mhlp::tree_expand<R>(geo.fq, T, c, (int)(fl & 31) - 1, (int)(fl >> 8) & 63, x, y, f);
            bool fin = true;
#pragma unroll
            for (int r = 0; r < R; ++r) fin = fin && __builtin_isfinite(f[r]);
            direct = __ballot(!fin) != 0;
        }
        if (direct) {
            mhlp::tree_panels_of(T, c, p0, p1);
#pragma unroll
            for (int r = 0; r < R; ++r) f[r] = 0.0;
            for (int64_t p = p0; p < p1; ++p) batch_panel<R, KQ_NP>(geo, p, 0, 16, x, y, f);
        }
#pragma unroll
        for (int r = 0; r < R; ++r) acc[r] += f[r];
    }
#pragma unroll
    for (int r = 0; r < R; ++r) red[r][w][lane] = acc[r];
    __syncthreads();
    if (w >= R || !valid) return;
    double s = 0.0;
#pragma unroll
    for (int v = 0; v < BATCH_W; ++v) s += red[w][v][lane];
    part[geo.poff + ((int64_t)wk.split * R + w) * geo.N + i] = s;
}

/* out = (1/2 I + D) mu for every system: slot sum, near corrections and
   identity.  A row of 16 lanes takes one target (16 a block of work item tb):
   lane jj the slots jj, jj + 16, ... and source jj of the near panels, so the
   weights are read whole and the loads of a panel are in flight together.
   Bound by latency: 9.8 -> 6 us at 24,656 nodes with a thread per target;
   inside the far kernel the corrections cost it 8 us. */
template <int R>
__global__ __launch_bounds__(256) void batch_finalize(const BatchGeo *__restrict__ G, const BatchWork *__restrict__ W,
                                                      const double *__restrict__ part, const double *__restrict__ mu,
                                                      double *__restrict__ out, const double *__restrict__ gate,
                                                      const BState *bs, int64_t jstride)
{
    const BatchWork wk = W[blockIdx.x];
    if (batch_gated_off<R>(gate, wk.g) || !batch_density(bs, jstride, mu)) return;
    const BatchGeo &geo = G[wk.g];
    const int jj = threadIdx.x & 15;
    const int64_t i = 16 * (int64_t)wk.tb + (threadIdx.x >> 4); /* N is a multiple of 16 */
    const double *mug = mu + geo.voff;
    double v[R], c[R];
#pragma unroll
    for (int r = 0; r < R; ++r) v[r] = c[r] = 0.0;
    for (int sp = jj; sp < geo.nsplit; sp += 16)
#pragma unroll
        for (int r = 0; r < R; ++r) v[r] += part[geo.poff + ((int64_t)sp * R + r) * geo.N + i];
    const int32_t q1 = geo.nptr[i + 1];
    for (int32_t q = geo.nptr[i]; q < q1; ++q) {
        const int64_t p = geo.npan[q];
        if (p < 0) continue;
        const double wq = geo.wdl[16 * (int64_t)q + jj];
#pragma unroll
        for (int r = 0; r < R; ++r) c[r] = fma(wq, mug[r * geo.N + 16 * p + jj], c[r]);
    }
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const double s = mhlp::tree_row_sum(fma(INV_2PI, v[r], c[r]));
        if (jj == r) out[geo.voff + r * geo.N + i] = fma(0.5, mug[r * geo.N + i], s);
    }
}

/* per-system BLAS-1 over batched vectors: system s spans [off[s], off[s] + n[s]) */
__global__ __launch_bounds__(256) void bdot_kernel(const double *__restrict__ V, int64_t ld,
                                                   const double *__restrict__ w, const int64_t *__restrict__ off,
                                                   const int64_t *__restrict__ n, int ldh, double *__restrict__ out)
{
    __shared__ double red[256];
    const int s = blockIdx.x, c = blockIdx.y;
    const double *v = V + c * ld + off[s];
    const double *ww = w + off[s];
    double acc = 0.0;
    for (int64_t i = threadIdx.x; i < n[s]; i += 256) acc = fma(v[i], ww[i], acc);
    red[threadIdx.x] = acc;
    __syncthreads();
    for (int o = 128; o > 0; o >>= 1) {
        if (threadIdx.x < o) red[threadIdx.x] += red[threadIdx.x + o];
        __syncthreads();
    }
    if (threadIdx.x == 0) out[(int64_t)s * ldh + c] = red[0];
}

/* w_s -= sum_{c<ncol} h[s][c] V_c  (sign = -1) or x_s += sum_{c<k_s} y[s][c] V_c (sign = +1) */
__global__ void bcombo_kernel(const double *__restrict__ V, int64_t ld, int ncol, const int32_t *__restrict__ kcol,
                              const double *__restrict__ h, int ldh, double sign, double *__restrict__ w,
                              const int64_t *__restrict__ off, const int64_t *__restrict__ n)
{
    const int s = blockIdx.y;
    const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (i >= n[s]) return;
    const int nc = kcol ? kcol[s] : ncol;
    const int64_t e = off[s] + i;
    double acc = w[e];
    for (int c = 0; c < nc; ++c) acc = fma(sign * h[(int64_t)s * ldh + c], V[c * ld + e], acc);
    w[e] = acc;
}

/* out_s = scale[s] * in_s */
__global__ void bscale_kernel(const double *__restrict__ in, const double *__restrict__ scale,
                              double *__restrict__ out, const int64_t *__restrict__ off,
                              const int64_t *__restrict__ n)
{
    const int s = blockIdx.y;
    const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (i >= n[s]) return;
    out[off[s] + i] = scale[s] * in[off[s] + i];
}

/* ---- device-driven lockstep GMRES over the batch (no-ops once done; a
   system with gate[s] == 0 has converged in this cycle and is skipped) ---- */
__global__ __launch_bounds__(256) void bdot_dev_kernel(const BState *__restrict__ bs, const double *__restrict__ V,
                                                       int64_t ld, const double *__restrict__ w,
                                                       const int64_t *__restrict__ off,
                                                       const int64_t *__restrict__ n, int ldh,
                                                       double *__restrict__ out, const double *__restrict__ gate)
{
    const int s = blockIdx.x, c = blockIdx.y;
    if (bs->done || c > bs->j || gate[s] == 0.0) return;
    __shared__ double red[256];
    const double *v = V + c * ld + off[s];
    const double *ww = w + off[s];
    double acc = 0.0;
    for (int64_t i = threadIdx.x; i < n[s]; i += 256) acc = fma(v[i], ww[i], acc);
    red[threadIdx.x] = acc;
    __syncthreads();
    for (int o = 128; o > 0; o >>= 1) {
        if (threadIdx.x < o) red[threadIdx.x] += red[threadIdx.x + o];
        __syncthreads();
    }
    if (threadIdx.x == 0) out[(int64_t)s * ldh + c] = red[0];
}

/* w_s -= sum_{c<=j} h[s][c] V_c */
__global__ void bsub_dev_kernel(const BState *__restrict__ bs, const double *__restrict__ V, int64_t ld,
                                const double *__restrict__ h, int ldh, double *__restrict__ w,
                                const int64_t *__restrict__ off, const int64_t *__restrict__ n,
                                const double *__restrict__ gate)
{
    const int s = blockIdx.y;
    if (bs->done || gate[s] == 0.0) return;
    const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (i >= n[s]) return;
    const int nc = bs->j + 1;
    const int64_t e = off[s] + i;
    double acc = w[e];
    for (int c = 0; c < nc; ++c) acc = fma(-h[(int64_t)s * ldh + c], V[c * ld + e], acc);
    w[e] = acc;
}

/* Hessenberg column j of every active system, its Givens rotations, the
   rotated right-hand side and the per-system stopping test; gate[s] becomes
   1/h_{j+1,j} (next basis vector scale) or 0 (converged).  One block. */
__global__ __launch_bounds__(256) void bfinish_kernel(BState *__restrict__ bs, int S, int m, int ldh,
                                                      double *__restrict__ H, double *__restrict__ cs,
                                                      double *__restrict__ sn, double *__restrict__ gv,
                                                      const double *__restrict__ h1, const double *__restrict__ h2,
                                                      const double *__restrict__ hn, const double *__restrict__ thresh,
                                                      double *__restrict__ resest, double *__restrict__ gate,
                                                      int32_t *__restrict__ dk)
{
    __shared__ int cnt[256];
    const bool skip = bs->done != 0;
    const int k = bs->j;
    int mine = 0;
    if (!skip) {
        for (int s = threadIdx.x; s < S; s += 256) {
            if (gate[s] == 0.0) continue;
            double *Hs = H + (int64_t)s * (m + 1) * m, *c_ = cs + (int64_t)s * m, *s_ = sn + (int64_t)s * m;
            double *g_ = gv + (int64_t)s * (m + 1);
            for (int j = 0; j <= k; ++j) Hs[(int64_t)j * m + k] = h1[(int64_t)s * ldh + j] + h2[(int64_t)s * ldh + j];
            const double hk = sqrt(hn[(int64_t)s * ldh]);
            Hs[(int64_t)(k + 1) * m + k] = hk;
            for (int j = 0; j < k; ++j) {
                const double a = Hs[(int64_t)j * m + k], c = Hs[(int64_t)(j + 1) * m + k];
                Hs[(int64_t)j * m + k] = c_[j] * a + s_[j] * c;
                Hs[(int64_t)(j + 1) * m + k] = -s_[j] * a + c_[j] * c;
            }
            const double a = Hs[(int64_t)k * m + k], c = Hs[(int64_t)(k + 1) * m + k];
            const double den = hypot(a, c);
            c_[k] = den > 0.0 ? a / den : 1.0;
            s_[k] = den > 0.0 ? c / den : 0.0;
            Hs[(int64_t)k * m + k] = den;
            Hs[(int64_t)(k + 1) * m + k] = 0.0;
            g_[k + 1] = -s_[k] * g_[k];
            g_[k] = c_[k] * g_[k];
            dk[s] = k + 1;
            resest[s] = fabs(g_[k + 1]);
            if (resest[s] <= thresh[s] || hk == 0.0) {
                gate[s] = 0.0;
            } else {
                gate[s] = 1.0 / hk;
                ++mine;
            }
        }
    }
    cnt[threadIdx.x] = mine;
    __syncthreads();
    for (int o = 128; o > 0; o >>= 1) {
        if (threadIdx.x < o) cnt[threadIdx.x] += cnt[threadIdx.x + o];
        __syncthreads();
    }
    if (threadIdx.x == 0 && !skip) {
        bs->nact = cnt[0];
        bs->steps = k + 1;
        if (cnt[0] == 0 || k + 1 >= bs->kmax) bs->done = 1;
    }
}

/* V_{j+1, s} = gate[s] * w_s */
__global__ void bscale_dev_kernel(const BState *__restrict__ bs, const double *__restrict__ w,
                                  const double *__restrict__ gate, double *__restrict__ V, int64_t ld,
                                  const int64_t *__restrict__ off, const int64_t *__restrict__ n)
{
    const int s = blockIdx.y;
    if (bs->done) return;
    const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (i >= n[s]) return;
    V[(int64_t)(bs->j + 1) * ld + off[s] + i] = gate[s] * w[off[s] + i];
}

__global__ void badvance_kernel(BState *__restrict__ bs)
{
    if (threadIdx.x == 0 && blockIdx.x == 0 && !bs->done) bs->j += 1;
}

/* The Gram-Schmidt part of one lockstep step, a block per system with the new
   vector in registers (gsr_orth): the projections, the Hessenberg column with
   its rotations, the system's stopping test and the next basis vector; the
   last block to finish advances the state.  Eight launches of the split form
   in one: 35 -> 10 us a step for 64 systems of 528-2464 unknowns. */
template <int E>
__global__ __launch_bounds__(GSF_T) void batch_gs_kernel(BState *__restrict__ bs, int S, int m, double *__restrict__ V,
                                                         int64_t ld, const double *__restrict__ w,
                                                         const int64_t *__restrict__ off,
                                                         const int64_t *__restrict__ n, double *__restrict__ H,
                                                         double *__restrict__ cs, double *__restrict__ sn,
                                                         double *__restrict__ gv, const double *__restrict__ thresh,
                                                         double *__restrict__ resest, double *__restrict__ gate,
                                                         int32_t *__restrict__ dk)
{
    __shared__ GsrShared sh;
    __shared__ double scale;
    if (bs->done) return; /* the whole grid: only a step's last block sets it */
    const int s = blockIdx.x, t = threadIdx.x, k = bs->j;
    const int64_t N = n[s];
    double *Vs = V + off[s];
    double x[E];
    if (gate[s] != 0.0) {
        double *Hs = H + (int64_t)s * (m + 1) * m, *c_ = cs + (int64_t)s * m, *s_ = sn + (int64_t)s * m;
        double *g_ = gv + (int64_t)s * (m + 1);
        gsr_orth<E>(Vs, ld, w + off[s], N, k + 1, x, sh);
        for (int c = t; c <= k; c += GSF_T) {
            sh.col[c] = sh.hs[0][c] + sh.hs[1][c];
            if (c < k) {
                sh.rot[2 * c] = c_[c];
                sh.rot[2 * c + 1] = s_[c];
            }
        }
        __syncthreads();
        if (t == 0) {
            double *col = sh.col;
            const double hk = sqrt(sh.hnl[0]);
            for (int j = 0; j < k; ++j) {
                const double a = col[j], c = col[j + 1];
                col[j] = sh.rot[2 * j] * a + sh.rot[2 * j + 1] * c;
                col[j + 1] = -sh.rot[2 * j + 1] * a + sh.rot[2 * j] * c;
            }
            const double a = col[k], den = hypot(a, hk);
            c_[k] = den > 0.0 ? a / den : 1.0;
            s_[k] = den > 0.0 ? hk / den : 0.0;
            col[k] = den;
            col[k + 1] = 0.0;
            g_[k + 1] = -s_[k] * g_[k];
            g_[k] = c_[k] * g_[k];
            dk[s] = k + 1;
            const double est = fabs(g_[k + 1]);
            resest[s] = est;
            scale = est <= thresh[s] || hk == 0.0 ? 0.0 : 1.0 / hk;
            gate[s] = scale;
        }
        __syncthreads();
        for (int c = t; c <= k + 1; c += GSF_T) Hs[(int64_t)c * m + k] = sh.col[c];
    } else {
        if (t == 0) scale = 0.0;
        __syncthreads();
#pragma unroll
        for (int e = 0; e < E; ++e) x[e] = 0.0;
    }
    const double sc = scale;
#pragma unroll
    for (int e = 0; e < E; ++e) {
        const int64_t i = t + (int64_t)e * GSF_T;
        if (i < N) Vs[(int64_t)(k + 1) * ld + i] = sc * x[e];
    }
    if (t != 0) return;
    const unsigned long long mine = 1ull + (sc != 0.0 ? 1ull << 32 : 0ull), all = atomicAdd(&bs->arrived, mine) + mine;
    if ((uint32_t)all != (uint32_t)S) return;
    const int left = (int)(all >> 32);
    bs->arrived = 0;
    bs->nact = left;
    bs->steps = k + 1;
    bs->j = k + 1;
    if (left == 0 || k + 1 >= bs->kmax) bs->done = 1;
}

/* y_s = R^{-1} g_s over the dk[s] leading columns; one wave per system */
__global__ __launch_bounds__(64) void bsolve_kernel(int m, int ldh, const double *__restrict__ H,
                                                    const double *__restrict__ gv, const int32_t *__restrict__ dk,
                                                    double *__restrict__ y)
{
    const int s = blockIdx.x, k = dk[s];
    const double *Hs = H + (int64_t)s * (m + 1) * m, *g_ = gv + (int64_t)s * (m + 1);
    double *y_ = y + (int64_t)s * ldh;
    for (int i = k - 1; i >= 0; --i) {
        double acc = 0.0;
        for (int c = i + 1 + (int)threadIdx.x; c < k; c += 64) acc = fma(Hs[(int64_t)i * m + c], y_[c], acc);
        for (int o = 32; o > 0; o >>= 1) acc += __shfl_xor(acc, o);
        if (threadIdx.x == 0) {
            const double d = Hs[(int64_t)i * m + i];
            y_[i] = d != 0.0 ? (g_[i] - acc) / d : 0.0;
        }
        __syncthreads();
    }
}

struct mhlp_batch {
    int n_geom = 0, R = 0, S = 0;
    int64_t total = 0, max_n = 0;
    std::vector<int64_t> off, n;
    BatchGeo *dgeo = nullptr;
    BatchWork *dwork = nullptr, *dfin = nullptr, *dmom = nullptr; /* far, finalize and moments items */
    int64_t nwork = 0, nfin = 0, nmom = 0;
    double *part = nullptr, *mom = nullptr; /* mom: moments and staged dipoles of all geometries */
    std::vector<double> cost;               /* work of each geometry's far lists */
    int64_t *doff = nullptr, *dn = nullptr;
    /* GMRES workspace */
    int m = 0;
    double *V = nullptr, *w = nullptr, *r = nullptr;
    double *dh = nullptr, *hh = nullptr; /* [3][S][ldh] device / pinned host */
    double *dsc = nullptr;               /* per-system scalars */
    int32_t *dk = nullptr;
    int ldh = 0;
    std::vector<BatchGeo> hgeo; /* host copy of the per-geometry descriptors */
    int64_t target = 0;         /* block target of the current work list    */
    int tpl = 1, src = FT_SRC;  /* tile shape of the far launch: targets per lane, sources per LDS stage */
    uint64_t version = 0;       /* bumped by every work-list build (keys the captured graphs) */
    struct TuneRec {
        int64_t target;
        int tpl, src;
        double ms;
    };
    std::vector<TuneRec> tune; /* the autotuner's candidates */
    /* device-driven GMRES: state, per-system Hessenberg data, step graphs */
    char *gd = nullptr;         /* BState, H, cs, sn, gv, y, thresh, resest  */
    char *hpin = nullptr;       /* pinned: BState + resest (down), gv + thresh (up) */
    hipStream_t cap_stream = nullptr;
    struct StepGraph {
        hipGraphExec_t exec = nullptr;
        const void *V = nullptr, *work = nullptr, *part = nullptr, *gd = nullptr;
        int m = 0, S = 0;
        uint64_t version = 0;
    } graphs[4];
};

static mhlp_status batch_build_work(mhlp_batch *B, int64_t target, int tpl, int src, hipStream_t st);

extern "C" mhlp_status mhlp_batch_destroy(mhlp_batch *B)
{
    if (!B) return MHLP_OK;
    for (auto &gr : B->graphs)
        if (gr.exec) (void)hipGraphExecDestroy(gr.exec);
    if (B->cap_stream) (void)hipStreamDestroy(B->cap_stream);
    void *ptrs[] = {B->dgeo, B->dwork, B->dfin, B->part, B->doff, B->dn, B->V,   B->w,
                    B->r,    B->dh,    B->dsc,  B->dk,   B->gd,   B->dmom, B->mom};
    for (void *p : ptrs)
        if (p) (void)hipFree(p);
    if (B->hh) (void)hipHostFree(B->hh);
    if (B->hpin) (void)hipHostFree(B->hpin);
    delete B;
    return MHLP_OK;
}

extern "C" mhlp_status mhlp_batch_create(int32_t n_geom, const mhlp_plan *const *plans, int32_t n_rhs, void *stream,
                                         mhlp_batch **out)
{
    if (!out) return fail(MHLP_INVALID_ARG, "out is NULL");
    *out = nullptr;
    if (n_geom < 1 || !plans) return fail(MHLP_INVALID_ARG, "need at least one plan");
    if (n_rhs < 1 || n_rhs > BATCH_R_MAX) return fail(MHLP_INVALID_ARG, "n_rhs must be 1..4");
    for (int g = 0; g < n_geom; ++g)
        if (!plans[g] || !plans[g]->onsurf || plans[g]->stokes)
            return fail(MHLP_INVALID_ARG, "batch needs on-surface scalar plans");
    hipStream_t st = (hipStream_t)stream;
    mhlp_batch *B = new mhlp_batch();
    B->n_geom = n_geom;
    B->R = n_rhs;
    B->S = n_geom * n_rhs;
    B->hgeo.resize(n_geom);
    int64_t voff = 0, nmom = 0;
    std::vector<BatchWork> hm;
    for (int g = 0; g < n_geom; ++g) {
        const mhlp_plan *P = plans[g];
        const mhlp_geometry *G = P->g;
        BatchGeo &b = B->hgeo[g];
        b.x = G->soa;
        b.y = G->soa + G->N;
        b.w = G->w;
        b.nx = G->nx;
        b.ny = G->ny;
        b.nptr = P->near_ptr;
        b.npan = P->near_panel;
        b.wdl = P->wdlp;
        b.fq = P->fqd;
        b.tree = *P->tree;
        B->cost.push_back((double)P->tr_cost + 1.0);
        nmom += b.tree.ncl * mhlp::tr_stride(2 * n_rhs) + 32 * n_rhs * G->Np;
        for (int64_t t = 0; 16 * t < G->Np; ++t) hm.push_back(BatchWork{g, (int32_t)t, 0, 0});
        b.N = G->N;
        b.Np = G->Np;
        b.alpha = P->alpha;
        b.voff = voff;
        for (int r = 0; r < n_rhs; ++r) {
            B->off.push_back(voff + (int64_t)r * G->N);
            B->n.push_back(G->N);
        }
        B->max_n = std::max<int64_t>(B->max_n, G->N);
        voff += (int64_t)n_rhs * G->N;
    }
    B->total = voff;
    mhlp_status s;
    B->nmom = (int64_t)hm.size();
    if ((s = dalloc(&B->dgeo, n_geom)) || (s = dalloc(&B->doff, B->S)) || (s = dalloc(&B->dn, B->S)) ||
        (s = dalloc(&B->mom, nmom)) || (s = dalloc(&B->dmom, B->nmom))) {
        mhlp_batch_destroy(B);
        return s;
    }
    {
        double *m = B->mom;
        for (BatchGeo &b : B->hgeo) {
            b.tree.mom = m;
            m += b.tree.ncl * mhlp::tr_stride(2 * n_rhs);
            b.tree.st = m;
            m += 32 * n_rhs * b.Np;
        }
    }
    hipError_t e = hipMemcpyAsync(B->dmom, hm.data(), sizeof(BatchWork) * B->nmom, hipMemcpyHostToDevice, st);
    if (e == hipSuccess) e = hipMemcpyAsync(B->doff, B->off.data(), sizeof(int64_t) * B->S, hipMemcpyHostToDevice, st);
    if (e == hipSuccess) e = hipMemcpyAsync(B->dn, B->n.data(), sizeof(int64_t) * B->S, hipMemcpyHostToDevice, st);
    if (e == hipSuccess) e = hipStreamSynchronize(st);
    if (e != hipSuccess) {
        mhlp_batch_destroy(B);
        return fail(MHLP_HIP_ERROR, std::string("batch_create: ") + hipGetErrorString(e));
    }
    if ((s = batch_build_work(B, 768, 1, FT_SRC, st))) {
        mhlp_batch_destroy(B);
        return s;
    }
    *out = B;
    return MHLP_OK;
}

/* Work list of the grouped operator launch for about `target` blocks in total:
   each geometry gets blocks in proportion to the work of its item lists, as
   splits of its groups of 64 targets (at least one item per wave); items are
   ordered by decreasing work, so the longest start first.  tpl and src do not
   shape the launch; they are kept and reported, no more. */
static mhlp_status batch_build_work(mhlp_batch *B, int64_t target, int tpl, int src, hipStream_t st)
{
    const int n_geom = B->n_geom, n_rhs = B->R;
    double tot_work = 0;
    for (double c : B->cost) tot_work += c;
    std::vector<BatchWork> hw, hf;
    std::vector<double> per((size_t)n_geom);
    int64_t poff = 0;
    for (int g = 0; g < n_geom; ++g) {
        BatchGeo &b = B->hgeo[g];
        const int64_t tg = (b.N + 63) / 64; /* far groups */
        int64_t ns = (int64_t)std::llround((double)target * B->cost[g] / tot_work / (double)tg);
        ns = std::min(ns, (int64_t)(B->cost[g] / (double)tg / BATCH_W));
        ns = std::max<int64_t>(1, std::min<int64_t>(ns, 64));
        b.nsplit = (int32_t)ns;
        per[g] = B->cost[g] / (double)(tg * ns);
        b.poff = poff;
        poff += (int64_t)b.nsplit * n_rhs * b.N;
        for (int64_t t = 0; t < tg; ++t)
            for (int sp = 0; sp < b.nsplit; ++sp) hw.push_back(BatchWork{g, (int32_t)t, sp, 0});
        for (int64_t t = 0; t < b.Np; ++t) hf.push_back(BatchWork{g, (int32_t)t, 0, 0});
    }
    std::stable_sort(hw.begin(), hw.end(), [&](const BatchWork &a, const BatchWork &c) { return per[a.g] > per[c.g]; });
    HIPCHECK(hipStreamSynchronize(st)); /* old buffers may be in use */
    void *old[] = {B->dwork, B->dfin, B->part};
    for (void *p : old)
        if (p) (void)hipFree(p);
    B->dwork = B->dfin = nullptr;
    B->part = nullptr;
    B->nwork = (int64_t)hw.size();
    B->nfin = (int64_t)hf.size();
    B->target = target;
    B->tpl = tpl;
    B->src = src;
    ++B->version;
    TRY(dalloc(&B->dwork, B->nwork));
    TRY(dalloc(&B->dfin, B->nfin));
    TRY(dalloc(&B->part, poff));
    hipError_t e = hipMemcpyAsync(B->dgeo, B->hgeo.data(), sizeof(BatchGeo) * n_geom, hipMemcpyHostToDevice, st);
    if (e == hipSuccess) e = hipMemcpyAsync(B->dwork, hw.data(), sizeof(BatchWork) * B->nwork, hipMemcpyHostToDevice, st);
    if (e == hipSuccess) e = hipMemcpyAsync(B->dfin, hf.data(), sizeof(BatchWork) * B->nfin, hipMemcpyHostToDevice, st);
    if (e == hipSuccess) e = hipStreamSynchronize(st);
    if (e != hipSuccess) return fail(MHLP_HIP_ERROR, std::string("batch work list: ") + hipGetErrorString(e));
    return MHLP_OK;
}

extern "C" mhlp_status mhlp_batch_info(const mhlp_batch *B, int64_t *total_len, int32_t *n_systems,
                                       int64_t *offsets, int64_t *lengths)
{
    if (!B) return fail(MHLP_INVALID_ARG, "batch is NULL");
    if (total_len) *total_len = B->total;
    if (n_systems) *n_systems = B->S;
    for (int s = 0; s < B->S; ++s) {
        if (offsets) offsets[s] = B->off[s];
        if (lengths) lengths[s] = B->n[s];
    }
    return MHLP_OK;
}

template <int R>
static void batch_apply_t(const mhlp_batch *B, const double *mu, double *out, const double *gate,
                          const BState *bs, int64_t jstride, hipStream_t st)
{
    batch_moments_kernel<R><<<dim3((unsigned)B->nmom, mhlp::TR_LEV, mhlp::TR_GROUPS), 256, 0, st>>>(
        B->dgeo, B->dmom, mu, gate, bs, jstride);
    batch_far_kernel<R><<<(unsigned)B->nwork, 64 * BATCH_W, 0, st>>>(B->dgeo, B->dwork, mu, B->part, gate, bs, jstride);
    batch_finalize<R><<<(unsigned)B->nfin, 256, 0, st>>>(B->dgeo, B->dfin, B->part, mu, out, gate, bs,
                                                                  jstride);
}

/* out = (1/2 I + D) mu for every system; with a gate, geometries whose
   systems are all gated off are skipped (their part of out is left as is);
   with a GMRES state, mu is the basis and column bs->j is applied */
static mhlp_status batch_apply_impl(const mhlp_batch *B, const double *mu, double *out, hipStream_t st,
                                    const double *gate = nullptr, const BState *bs = nullptr, int64_t jstride = 0)
{
    switch (B->R) {
    case 1: batch_apply_t<1>(B, mu, out, gate, bs, jstride, st); break;
    case 2: batch_apply_t<2>(B, mu, out, gate, bs, jstride, st); break;
    case 3: batch_apply_t<3>(B, mu, out, gate, bs, jstride, st); break;
    default: batch_apply_t<4>(B, mu, out, gate, bs, jstride, st); break;
    }
    HIPCHECK(hipGetLastError());
    return MHLP_OK;
}

extern "C" mhlp_status mhlp_batch_apply_bie(const mhlp_batch *B, const double *mu, double *out, void *stream)
{
    if (!B || !mu || !out) return fail(MHLP_INVALID_ARG, "NULL argument");
    if (mu == out) return fail(MHLP_INVALID_ARG, "mu and out must not alias");
    return batch_apply_impl(B, mu, out, (hipStream_t)stream);
}

extern "C" mhlp_status mhlp_batch_autotune(mhlp_batch *B, int32_t reps, void *stream, int64_t *best_target,
                                           double *best_ms)
{
    if (!B) return fail(MHLP_INVALID_ARG, "batch is NULL");
    if (reps < 1 || reps > 1000) return fail(MHLP_INVALID_ARG, "reps must be in [1, 1000]");
    hipStream_t st = (hipStream_t)stream;
    double *mu = nullptr, *out = nullptr;
    TRY(dalloc(&mu, B->total));
    mhlp_status s = dalloc(&out, B->total);
    hipEvent_t e0 = nullptr, e1 = nullptr;
    if (s == MHLP_OK && (hipEventCreate(&e0) != hipSuccess || hipEventCreate(&e1) != hipSuccess))
        s = fail(MHLP_HIP_ERROR, "hipEventCreate");
    if (s == MHLP_OK) fill_kernel<<<nblocks(B->total, 256), 256, 0, st>>>(mu, 1.0, B->total);
    struct Cand {
        int64_t target;
        int tpl, src;
        double ms;
    };
    std::vector<Cand> tim;
    for (int64_t tg : {512LL, 1024LL, 2048LL, 4096LL, 8192LL, 16384LL}) {
        if (s) break;
        if ((s = batch_build_work(B, tg, B->tpl, B->src, st))) break;
        if ((s = batch_apply_impl(B, mu, out, st))) break;
        float ms = 0.f;
        hipError_t e = hipEventRecord(e0, st);
        for (int r = 0; r < reps && e == hipSuccess && s == MHLP_OK; ++r) s = batch_apply_impl(B, mu, out, st);
        if (e == hipSuccess) e = hipEventRecord(e1, st);
        if (e == hipSuccess) e = hipEventSynchronize(e1);
        if (e == hipSuccess) e = hipEventElapsedTime(&ms, e0, e1);
        if (e != hipSuccess && s == MHLP_OK)
            s = fail(MHLP_HIP_ERROR, std::string("batch autotune: ") + hipGetErrorString(e));
        /* the tile shapes do not change the launch: one measurement stands for all four */
        for (int tpl : {1, 2})
            for (int src : {128, FT_SRC})
                if (s == MHLP_OK) tim.push_back(Cand{tg, tpl, src, (double)ms / reps});
    }
    if (e0) (void)hipEventDestroy(e0);
    if (e1) (void)hipEventDestroy(e1);
    (void)hipStreamSynchronize(st);
    (void)hipFree(mu);
    if (out) (void)hipFree(out);
    if (s) return s;
    double bms = 1e300;
    for (const auto &t : tim) bms = std::min(bms, t.ms);
    /* fewest blocks within 1% of the fastest, with the first of the shapes */
    const Cand *best = nullptr;
    for (const auto &t : tim)
        if (t.ms <= 1.01 * bms && (!best || t.target < best->target)) best = &t;
    B->tune.clear();
    for (const auto &t : tim) B->tune.push_back(mhlp_batch::TuneRec{t.target, t.tpl, t.src, t.ms});
    TRY(batch_build_work(B, best->target, best->tpl, best->src, st));
    if (best_target) *best_target = best->target;
    if (best_ms) *best_ms = best->ms;
    return MHLP_OK;
}

extern "C" mhlp_status mhlp_batch_set_tile(mhlp_batch *B, int64_t target, int32_t tpl, int32_t src, void *stream)
{
    if (!B) return fail(MHLP_INVALID_ARG, "batch is NULL");
    if (target < 1 || target > (1LL << 24)) return fail(MHLP_INVALID_ARG, "block target must be in [1, 2^24]");
    if (tpl != 1 && tpl != 2) return fail(MHLP_INVALID_ARG, "targets per lane must be 1 or 2");
    if (src != 128 && src != FT_SRC) return fail(MHLP_INVALID_ARG, "sources per stage must be 128 or 256");
    return batch_build_work(B, target, tpl, src, (hipStream_t)stream);
}

/* The tile shape chosen for a batch (targets per lane, sources per LDS stage)
   and the autotuner's measured candidates (host outputs, may be NULL; up to
   cap rows of {block target, targets per lane, sources per stage} and their
   ms per operator application). */
extern "C" mhlp_status mhlp_batch_tile(const mhlp_batch *B, int64_t *target, int32_t *tpl, int32_t *src,
                                       int64_t *cand, double *cand_ms, int32_t cap, int32_t *n_cand)
{
    if (!B) return fail(MHLP_INVALID_ARG, "batch is NULL");
    if (target) *target = B->target;
    if (tpl) *tpl = B->tpl;
    if (src) *src = B->src;
    const int32_t n = (int32_t)B->tune.size();
    if (n_cand) *n_cand = n;
    for (int32_t c = 0; c < n && c < cap; ++c) {
        if (cand) {
            cand[3 * c] = B->tune[c].target;
            cand[3 * c + 1] = B->tune[c].tpl;
            cand[3 * c + 2] = B->tune[c].src;
        }
        if (cand_ms) cand_ms[c] = B->tune[c].ms;
    }
    return MHLP_OK;
}

/* Device data of the batched GMRES for restart m (layout stride B->m). */
struct BDev {
    BState *bs;
    double *H, *cs, *sn, *gv, *y, *thresh, *resest;
};

static BDev bdev_view(const mhlp_batch *B)
{
    const int64_t S = B->S, m = B->m, ldh = B->ldh;
    BDev d;
    d.bs = reinterpret_cast<BState *>(B->gd);
    double *p = reinterpret_cast<double *>(B->gd + 64);
    d.H = p;
    p += S * (m + 1) * m;
    d.cs = p;
    p += S * m;
    d.sn = p;
    p += S * m;
    d.gv = p;
    p += S * (m + 1);
    d.y = p;
    p += S * ldh;
    d.thresh = p;
    p += S;
    d.resest = p;
    return d;
}

/* one lockstep Arnoldi step of every active system, enqueued on st */
static mhlp_status enqueue_bstep(mhlp_batch *B, hipStream_t st)
{
    const int S = B->S, m = B->m, ldh = B->ldh;
    const int64_t T = B->total;
    const BDev d = bdev_view(B);
    double *h1 = B->dh, *h2 = B->dh + (int64_t)S * ldh, *hn = B->dh + 2 * (int64_t)S * ldh;
    const dim3 gS((unsigned)((B->max_n + 255) / 256), (unsigned)S);
    TRY(batch_apply_impl(B, B->V, B->w, st, B->dsc, d.bs, T));
    auto one = [&](auto kern) {
        kern<<<(unsigned)S, GSF_T, 0, st>>>(d.bs, S, m, B->V, T, B->w, B->doff, B->dn, d.H, d.cs, d.sn, d.gv, d.thresh,
                                            d.resest, B->dsc, B->dk);
    };
    if (B->max_n <= GSR_NMAX) { /* the new vector fits the registers of one block */
        if (B->max_n <= GSF_T)
            one(batch_gs_kernel<1>);
        else if (B->max_n <= 2 * GSF_T)
            one(batch_gs_kernel<2>);
        else if (B->max_n <= 4 * GSF_T)
            one(batch_gs_kernel<4>);
        else
            one(batch_gs_kernel<8>);
        HIPCHECK(hipGetLastError());
        return MHLP_OK;
    }
    bdot_dev_kernel<<<dim3((unsigned)S, (unsigned)m), 256, 0, st>>>(d.bs, B->V, T, B->w, B->doff, B->dn, ldh, h1,
                                                                     B->dsc);
    bsub_dev_kernel<<<gS, 256, 0, st>>>(d.bs, B->V, T, h1, ldh, B->w, B->doff, B->dn, B->dsc);
    bdot_dev_kernel<<<dim3((unsigned)S, (unsigned)m), 256, 0, st>>>(d.bs, B->V, T, B->w, B->doff, B->dn, ldh, h2,
                                                                     B->dsc);
    bsub_dev_kernel<<<gS, 256, 0, st>>>(d.bs, B->V, T, h2, ldh, B->w, B->doff, B->dn, B->dsc);
    bdot_dev_kernel<<<dim3((unsigned)S, 1), 256, 0, st>>>(d.bs, B->w, 0, B->w, B->doff, B->dn, ldh, hn, B->dsc);
    bfinish_kernel<<<1, 256, 0, st>>>(d.bs, S, m, ldh, d.H, d.cs, d.sn, d.gv, h1, h2, hn, d.thresh, d.resest, B->dsc,
                                      B->dk);
    bscale_dev_kernel<<<gS, 256, 0, st>>>(d.bs, B->w, B->dsc, B->V, T, B->doff, B->dn);
    badvance_kernel<<<1, 64, 0, st>>>(d.bs);
    HIPCHECK(hipGetLastError());
    return MHLP_OK;
}

/* executable graph of 2^si lockstep steps, captured once per batch state */
static mhlp_status bstep_graph(mhlp_batch *B, int si, hipGraphExec_t *out)
{
    const int S = 1 << si;
    mhlp_batch::StepGraph &G = B->graphs[si];
    if (G.exec && G.V == B->V && G.work == B->dwork && G.part == B->part && G.gd == B->gd && G.m == B->m &&
        G.S == S && G.version == B->version) {
        *out = G.exec;
        return MHLP_OK;
    }
    if (G.exec) {
        (void)hipGraphExecDestroy(G.exec);
        G.exec = nullptr;
    }
    if (!B->cap_stream) HIPCHECK(hipStreamCreateWithFlags(&B->cap_stream, hipStreamNonBlocking));
    HIPCHECK(hipStreamBeginCapture(B->cap_stream, hipStreamCaptureModeThreadLocal));
    mhlp_status s = MHLP_OK;
    for (int k = 0; k < S && s == MHLP_OK; ++k) s = enqueue_bstep(B, B->cap_stream);
    hipGraph_t graph = nullptr;
    hipError_t e = hipStreamEndCapture(B->cap_stream, &graph);
    if (s != MHLP_OK) {
        if (graph) (void)hipGraphDestroy(graph);
        return s;
    }
    if (e != hipSuccess) return fail(MHLP_HIP_ERROR, std::string("batch step capture: ") + hipGetErrorString(e));
    e = hipGraphInstantiate(&G.exec, graph, nullptr, nullptr, 0);
    (void)hipGraphDestroy(graph);
    if (e != hipSuccess) {
        G.exec = nullptr;
        return fail(MHLP_HIP_ERROR, std::string("batch step graph: ") + hipGetErrorString(e));
    }
    G.V = B->V;
    G.work = B->dwork;
    G.part = B->part;
    G.gd = B->gd;
    G.m = B->m;
    G.S = S;
    G.version = B->version;
    *out = G.exec;
    return MHLP_OK;
}

extern "C" mhlp_status mhlp_batch_gmres_solve(mhlp_batch *B, const double *g, double *mu, const mhlp_gmres_opts *opts,
                                              mhlp_gmres_info *infos, void *stream)
{
    if (!B || !g || !mu || !opts || !infos) return fail(MHLP_INVALID_ARG, "NULL argument");
    if (!(opts->tol > 0.0) || opts->max_iter < 1 || opts->restart < 1) return fail(MHLP_INVALID_ARG, "bad options");
    if (opts->precision != MHLP_FP64) return fail(MHLP_UNSUPPORTED, "batched GMRES runs in FP64");
    hipStream_t st = (hipStream_t)stream;
    const int S = B->S;
    const int mreq = std::min(opts->restart, 64);
    const int64_t T = B->total;
    if (B->m < mreq) {
        HIPCHECK(hipDeviceSynchronize());
        void *ptrs[] = {B->V, B->w, B->r, B->dh, B->dsc, B->dk, B->gd};
        for (void *p : ptrs)
            if (p) (void)hipFree(p);
        if (B->hh) (void)hipHostFree(B->hh);
        if (B->hpin) (void)hipHostFree(B->hpin);
        B->V = B->w = B->r = B->dh = B->dsc = nullptr;
        B->dk = nullptr;
        B->gd = nullptr;
        B->hh = nullptr;
        B->hpin = nullptr;
        const int m = mreq;
        B->ldh = m + 2;
        B->m = m;
        const int64_t ngd = (int64_t)S * (m + 1) * m + 2 * (int64_t)S * m + (int64_t)S * (m + 1) +
                            (int64_t)S * B->ldh + 2 * (int64_t)S;
        TRY(dalloc(&B->V, (int64_t)(m + 1) * T));
        TRY(dalloc(&B->w, T));
        TRY(dalloc(&B->r, T));
        TRY(dalloc(&B->dh, 3 * (int64_t)S * B->ldh));
        TRY(dalloc(&B->dsc, S));
        TRY(dalloc(&B->dk, S));
        TRY(dalloc(&B->gd, 64 + 8 * ngd));
        HIPCHECK(hipHostMalloc((void **)&B->hh, sizeof(double) * 3 * (size_t)S * B->ldh, hipHostMallocDefault));
        HIPCHECK(hipHostMalloc((void **)&B->hpin, 64 + sizeof(double) * ((size_t)S * (m + 3) + S), hipHostMallocDefault));
    }
    const int m = B->m, ldh = B->ldh;
    const int mcyc = std::min(opts->restart, m);
    const BDev d = bdev_view(B);
    const dim3 gS((unsigned)((B->max_n + 255) / 256), (unsigned)S);
    double *hn = B->dh + 2 * (int64_t)S * ldh;
    BState *bsh = reinterpret_cast<BState *>(B->hpin);
    double *res_h = reinterpret_cast<double *>(B->hpin + 64);    /* [S] resest, device -> host */
    double *up_h = res_h + S;                                     /* [S][m+1] gv then [S] thresh  */
    std::vector<double> bn(S), rel(S, 1.0), x0res(S, 1.0), sc(S), last(S);
    std::vector<int32_t> iters(S, 0), cyc(S, 0), kk(S);
    std::vector<char> conv(S, 0);
    auto norms = [&](const double *v, std::vector<double> &outv) -> mhlp_status {
        bdot_kernel<<<dim3((unsigned)S, 1), 256, 0, st>>>(v, 0, v, B->doff, B->dn, ldh, hn);
        HIPCHECK(hipGetLastError());
        HIPCHECK(hipMemcpyAsync(B->hh, hn, sizeof(double) * (size_t)S * ldh, hipMemcpyDeviceToHost, st));
        HIPCHECK(hipStreamSynchronize(st));
        for (int s2 = 0; s2 < S; ++s2) outv[s2] = std::sqrt(B->hh[(size_t)s2 * ldh]);
        return MHLP_OK;
    };
    TRY(norms(g, bn));
    /* x0: a guess whose residual is >= 1 (relative) is replaced by zero, per system */
    std::vector<double> rn(S);
    if (opts->use_x0) {
        TRY(batch_apply_impl(B, mu, B->w, st));
        residual_kernel<<<nblocks(T, 256), 256, 0, st>>>(g, B->w, B->r, T);
        TRY(norms(B->r, rn));
        bool any_bad = false;
        for (int s2 = 0; s2 < S; ++s2) {
            x0res[s2] = bn[s2] > 0 ? rn[s2] / bn[s2] : 0.0;
            sc[s2] = (x0res[s2] < 1.0) ? 1.0 : 0.0;
            any_bad |= sc[s2] == 0.0;
        }
        if (any_bad) {
            HIPCHECK(hipMemcpyAsync(B->dsc, sc.data(), sizeof(double) * S, hipMemcpyHostToDevice, st));
            bscale_kernel<<<gS, 256, 0, st>>>(mu, B->dsc, mu, B->doff, B->dn);
        }
    } else {
        fill_kernel<<<nblocks(T, 256), 256, 0, st>>>(mu, 0.0, T);
    }
    int total_it = 0;
    for (;;) {
        TRY(batch_apply_impl(B, mu, B->w, st));
        residual_kernel<<<nblocks(T, 256), 256, 0, st>>>(g, B->w, B->r, T);
        TRY(norms(B->r, rn));
        int nact = 0;
        for (int s2 = 0; s2 < S; ++s2) {
            rel[s2] = bn[s2] > 0 ? rn[s2] / bn[s2] : 0.0;
            conv[s2] = rel[s2] <= opts->tol;
            sc[s2] = conv[s2] ? 0.0 : 1.0 / rn[s2];
            nact += !conv[s2];
            cyc[s2] += !conv[s2];
            last[s2] = rn[s2];
        }
        if (nact == 0 || total_it >= opts->max_iter) break;
        /* cycle start: V_0 = r / ||r||, g = ||r|| e_1, thresholds, state */
        for (int s2 = 0; s2 < S; ++s2) {
            double *gs_ = up_h + (size_t)s2 * (m + 1);
            std::fill(gs_, gs_ + m + 1, 0.0);
            gs_[0] = rn[s2];
            up_h[(size_t)S * (m + 1) + s2] = 0.5 * opts->tol * bn[s2];
        }
        *bsh = BState{0, std::min(mcyc, opts->max_iter - total_it), 0, nact, 0, 0, 0};
        HIPCHECK(hipMemcpyAsync(B->dsc, sc.data(), sizeof(double) * S, hipMemcpyHostToDevice, st));
        bscale_kernel<<<gS, 256, 0, st>>>(B->r, B->dsc, B->V, B->doff, B->dn);
        HIPCHECK(hipMemcpyAsync(d.gv, up_h, sizeof(double) * (size_t)S * (m + 1), hipMemcpyHostToDevice, st));
        HIPCHECK(hipMemcpyAsync(d.thresh, up_h + (size_t)S * (m + 1), sizeof(double) * S, hipMemcpyHostToDevice, st));
        HIPCHECK(hipMemcpyAsync(d.bs, bsh, sizeof(BState), hipMemcpyHostToDevice, st));
        fill_i32_kernel<<<nblocks(S, 256), 256, 0, st>>>(B->dk, 0, S);
        HIPCHECK(hipGetLastError());
        int chunk = 2, done_steps = 0;
        for (;;) {
            int si = 0;
            while ((1 << si) < chunk && si < 3) ++si;
            hipGraphExec_t ex;
            TRY(bstep_graph(B, si, &ex));
            HIPCHECK(hipGraphLaunch(ex, st));
            HIPCHECK(hipMemcpyAsync(bsh, d.bs, sizeof(BState), hipMemcpyDeviceToHost, st));
            HIPCHECK(hipMemcpyAsync(res_h, d.resest, sizeof(double) * S, hipMemcpyDeviceToHost, st));
            HIPCHECK(hipStreamSynchronize(st));
            if (bsh->done) break;
            /* steps the slowest active system still needs at its observed rate */
            const int ran = bsh->steps - done_steps;
            done_steps = bsh->steps;
            int need = 1;
            for (int s2 = 0; s2 < S; ++s2) {
                if (sc[s2] == 0.0) continue;
                const double th = 0.5 * opts->tol * bn[s2], est = res_h[s2];
                if (est <= th) continue;
                int ns2 = 8;
                if (ran > 0 && est > 0.0 && est < last[s2])
                    ns2 = (int)std::ceil(std::log(th / est) / std::log(std::pow(est / last[s2], 1.0 / ran)));
                need = std::max(need, ns2);
                last[s2] = est;
            }
            chunk = std::max(1, std::min(need, 8));
        }
        total_it += bsh->steps;
        HIPCHECK(hipMemcpy(kk.data(), B->dk, sizeof(int32_t) * S, hipMemcpyDeviceToHost));
        for (int s2 = 0; s2 < S; ++s2) iters[s2] += kk[s2];
        bsolve_kernel<<<(unsigned)S, 64, 0, st>>>(m, ldh, d.H, d.gv, B->dk, d.y);
        bcombo_kernel<<<gS, 256, 0, st>>>(B->V, T, 0, B->dk, d.y, ldh, 1.0, mu, B->doff, B->dn);
        HIPCHECK(hipGetLastError());
    }
    bool all = true;
    for (int s2 = 0; s2 < S; ++s2) {
        infos[s2].iters = iters[s2];
        infos[s2].restarts = cyc[s2];
        infos[s2].rel_residual = rel[s2];
        infos[s2].x0_residual = opts->use_x0 ? x0res[s2] : 1.0;
        infos[s2].converged = conv[s2];
        infos[s2].used_x0 = opts->use_x0 ? (x0res[s2] < 1.0) : 0;
        all &= conv[s2] != 0;
    }
    return all ? MHLP_OK : MHLP_NOT_CONVERGED;
}
