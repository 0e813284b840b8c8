/* Far field of the layer potentials by cluster expansions (FP64), for every
   far sum over the panels of a plan.

   Clusters are runs of 1, 2, 4, 8 or 16 consecutive panels (level 0..4, aligned
   at their size).  The field of a cluster's charges q_j and dipoles d_j at y_j,
       sum_j q_j K0(alpha |x - y_j|) + d_j . grad_y K0(alpha |x - y_j|),
   is, by Graf's addition theorem about the cluster's centre c,
       Re sum_{n=0..p} M_n K_n(alpha r) e^{i n theta},   x - c = r e^{i theta},
       M_n = (2 - delta_n0) sum_j q_j B_n(y_j - c),  B_n(d) = I_n(alpha |d|) e^{-i n arg d},
       dipoles: M_n = (2 - delta_n0)(alpha/2) sum_j [conj(d_j) B_{n-1} + d_j B_{n+1}]  (n >= 1),
                M_0 = alpha sum_j Re(d_j B_1).
   A wave of 64 targets takes each panel once: through the largest cluster whose
   expansion of an order up to TR_PMAX reaches rounding at all its targets
   (tree_order_ratio), else directly (the class-table tiles of the far
   kernels).  The lists are built with the plan (tree_lists_kernel); the moments
   of every evaluation come from tree_moments_kernel, which also stages the
   charges and dipoles of the direct part.

   Why this split: a pair costs 55-75 FP64 instructions directly, an order of a
   cluster 10 for both layers and about 50 once per cluster, so a panel of 16
   sources costs about 1100 directly and 130-370 through its own expansion, and
   far clusters hold up to 16 panels.  alpha R <= TR_AMAX keeps the terms of the
   expansion within e^{2 alpha R} of its value (wider clusters would lose digits
   to cancellation, and need more orders than they have panels). */
#pragma once

namespace mhlp {

constexpr int TR_LEV = 5;                    /* cluster levels: 1, 2, 4, 8, 16 panels */
constexpr int TR_PMIN = 8, TR_PSTEP = 2, TR_NP = 13, TR_PMAX = TR_PMIN + TR_PSTEP * (TR_NP - 1);
constexpr int TR_GRAD = 2;                   /* orders a gradient takes beyond the potential's */
constexpr int TR_ROWS = TR_PMAX + TR_GRAD + 1; /* orders of a moment table */
constexpr int TR_RM = 16;                    /* distances kept per cluster: TR_NP orders, then (last) the underflow's,
                                                or the radius in a stresslet plan */
/* doubles of a cluster's moment table: rows of nv values, padded to the 32 doubles of a row load */
constexpr int tr_stride(int nv) { return (TR_ROWS * nv + 31) / 32 * 32; }
constexpr double TR_AMIN = 1e-6, TR_AMAX = 2.0; /* alpha R of an expansion (below: K_n, I_n leave the range of a double) */
constexpr double TR_ZZERO = 746.0;           /* e^{-z} is exactly 0 in double from here on (also scaled by 2^-1074) */
constexpr double TR_EPS = 0x1p-54;           /* truncation of an expansion, relative to its smallest pair */

struct TreeDev {
    int64_t Np = 0;
    int nlev = 0;
    int64_t off[TR_LEV] = {0, 0, 0, 0, 0};   /* first cluster of each level */
    int64_t ncl = 0;
    int stokes = 0;                          /* stresslet lists (tree_stokes_order) */
    double *flux = nullptr;                  /* on-surface stresslet: [Np] sums of w mu.n */
    int cut = 0;                             /* a direct item is 2^cut units of work (16/2^cut sources each) */
    double *cc = nullptr;                    /* [ncl][2] centres */
    double *rmin = nullptr;                  /* [ncl][TR_RM]: distance from which order TR_PMIN + TR_PSTEP k serves
                                                (k < TR_NP; INFINITY: never); last: from which every pair underflows */
    double *mom = nullptr;                   /* [ncl][tr_stride]: rows of the coefficients of K_n cos n theta
                                                and K_n sin n theta per field (stresslet: then of r^-n) */
    double *small = nullptr;                 /* stresslet lists with TR_SMALL items: rows of their powers' coefficients,
                                                [ncl][tr_stride(4 or, for gradients, 8)] */
    double *st = nullptr;                    /* staged sources [Np][3][16]: w sigma, alpha w mu n_x, alpha w mu n_y */
    uint2 *items = nullptr;                  /* the groups' lists: direct items from the front, expansions from the back */
    longlong2 *at = nullptr;                 /* [groups]: begin and end of a group's list */
    int2 *cnt = nullptr;                     /* [groups]: numbers of direct items and expansions */
    double *part = nullptr;                  /* [groups][blocks per group][fields][64] sums of split groups */
    double *base = nullptr;                  /* [groups][fields][64] sums of the items always summed (TREE_NEAREST) */
    float *room = nullptr;                   /* [groups][fields]: log2 of what an item may then add without showing */
    uint32_t *arrived = nullptr;             /* [groups]: blocks of split groups that are through, counted round and round */
    unsigned long long *cost = nullptr;      /* total work of the groups (tree_cost); [1]: the largest spread of
                                                the z classes of a group's items (TR_ZSTEP), of a stresslet plan whether
                                                it has TR_SMALL items; [2]: all items; [3]: whether there are expansions */
    float *lb = nullptr;                     /* [ncl] log2 of the sum of |charges| and |dipoles|, rounded up */
    int *znear = nullptr;                    /* [groups] smallest z class of the items */
    int expands = 1;                         /* some item is (while the lists are built: may be) an expansion; else the
                                                moments kernel only stages, if it runs at all */
    int skip = 0;                            /* far items are held against the near ones' sum (far_tree_kernel) */
    int32_t *order = nullptr;                /* [groups] launch order: the groups with the most work first */
};

/* item: x = cluster, y = piece + 1 (bits 0-4) | order (bits 8-13) | flags */
constexpr uint32_t TR_NEAR = 1u << 16; /* direct: some target of the wave lists the panel */
constexpr uint32_t TR_ZERO = 1u << 17; /* every pair underflows to zero: only non-finite densities matter */
constexpr uint32_t TR_LAP = 1u << 18;  /* stresslet: the K part of every pair is below rounding */
constexpr uint32_t TR_SMALL = 1u << 19; /* stresslet: some pair has z < TR_SZ, singular parts with the powers */
/* bits 24-31: the z class, z >= TR_ZSTEP times it for every pair of the item */
constexpr double TR_ZSTEP = 4.0;
constexpr int TR_ZNEAR = 3;            /* classes from a group's smallest one that are always summed */
constexpr int TR_ZSKIP = 40;           /* spread of classes (z: 160) from which a plan looks for items to leave out; below,
                                          hardly any can be (both layers, 109,314 targets: alpha = 50, spread 33: 211 us
                                          without, 216 with; alpha = 100, spread 65: 370, 233) */
__host__ __device__ inline uint32_t tree_zclass(double z) { return z > 0.0 ? (uint32_t)fmin(z * (1.0 / TR_ZSTEP), 255.0) << 24 : 0u; }

/* Stresslet double layer by clusters.  With U = u_1 + i u_2, x - y = r e^{i theta},
   sigma = (m_1 + i m_2)(n_1 + i n_2)/2, tau = m.n (m = w mu) and O_k = K_k(alpha r) e^{i k theta},
   the closed forms of T1..T3 (App. B) are
     2 pi U = conj(sigma) [8/(alpha^2 conj(x - y)^3) - alpha O_3] + sigma alpha O_{-1} + tau/conj(x - y):
   derivatives of K0 and of log r, each of which has its expansion about the
   cluster's centre (Graf's theorem; powers of 1/conj(x - c)).  The two parts
   in brackets cancel like z^2/8 for small z.  Below alpha (r - R) = TR_SZ the
   singular part S_n = (n-1)!/2 (2/z)^n of every K_n, n >= 1, therefore goes with
   the powers: K_n - S_n falls by z^2 against K_n, follows K_n's recurrence
   stably (K_{n+1} - S_{n+1} = K_{n-1} + 2n/z (K_n - S_n)), and the powers'
   coefficients with it are formed without the cancelling parts (TreeSmall).
   From TR_SLAP on the K part is below rounding against the other's 1/r and left
   out (K_3(42) = 1e-19), for clusters of any alpha R.  Order: the terms of the bracket differ by the
   factor z^2/(4 n) once n > z^2/4, so the neglected terms are below
   n t^{n-3}/r in every regime (t = R/r). */
constexpr double TR_SZ = 2.0, TR_SLAP = 42.0, TR_SAMAX = 1e7;
constexpr int TR_SNP = 12; /* orders 8..30: the gradient takes TR_SGRAD more */
constexpr int TR_SGRAD = 4;

/* Truncation of an order-p expansion with alpha R = a at distance t R from the
   centre: bound of sum_{n>p} alpha (I_{n-1} + I_{n+1})(a) K_n(a t), the
   neglected field of a unit dipole on the cluster's rim (a charge's is
   smaller), over alpha K_1(a t + a), that dipole's smallest field.
   I_p(a) <= (a/2)^p/p! e^{a^2/(4(p+1))}; K_{p+1}/K_1 by the upward ratios;
   K_1(b)/K_1(b + a) <= e^a (1 + a/b). */
__host__ __device__ inline float tree_truncation(int p, float a, float t)
{
    const float b = a * t;
    float prod = 1.0f, h = 2.0f / b + 1.0f;
    for (int n = 1; n <= p; ++n) {
        prod *= (0.5f * a / (float)n) * h;
        h = (float)(2 * (n + 1)) / b + 1.0f / h;
    }
    return prod * expf(a + 0.25f * a * a / (float)(p + 1)) * (1.0f + 1.0f / t) / (1.0f - 1.0f / t);
}

/* the stresslet's t = r/R from which order p serves */
__host__ __device__ inline double tree_stokes_ratio(int p)
{
    double t = pow(TR_EPS / (p + 2), 1.0 / (p - 2)); /* the bound without its 1/(1 - t)^2, then with it */
    for (int k = 0; k < 3; ++k) t = pow(TR_EPS * (1.0 - t) * (1.0 - t) / (p + 2), 1.0 / (p - 2));
    return 1.0 / t;
}

/* the smallest t = r/R (to 2%, rounded up) from which order p serves; single
   precision is enough for a bound */
__host__ __device__ inline double tree_order_ratio(int p, double alphaR, double amax = TR_AMAX)
{
    constexpr float TMIN = 1.5f, TMAX = 300.0f, EPS = (float)(0.999 * TR_EPS);
    const float a = (float)alphaR;
    if (!(alphaR >= TR_AMIN && alphaR <= amax) || !(tree_truncation(p, a, TMAX) <= EPS)) return INFINITY;
    float lo = logf(TMIN), hi = logf(TMAX);
    for (int k = 0; k < 8; ++k) {
        const float mid = 0.5f * (lo + hi);
        if (tree_truncation(p, a, expf(mid)) <= EPS)
            hi = mid;
        else
            lo = mid;
    }
    return (double)expf(hi) * (1.0 + 1e-5);
}

__device__ __forceinline__ float tr_dpp_f(float v, float old, int sel)
{
    const int o = __float_as_int(old), i = __float_as_int(v);
    int r;
    switch (sel) {
    case 0: r = __builtin_amdgcn_update_dpp(o, i, 0x111, 0xf, 0xf, false); break;
    case 1: r = __builtin_amdgcn_update_dpp(o, i, 0x112, 0xf, 0xf, false); break;
    case 2: r = __builtin_amdgcn_update_dpp(o, i, 0x114, 0xf, 0xf, false); break;
    case 3: r = __builtin_amdgcn_update_dpp(o, i, 0x118, 0xf, 0xf, false); break;
    case 4: r = __builtin_amdgcn_update_dpp(o, i, 0x142, 0xa, 0xf, false); break;
    default: r = __builtin_amdgcn_update_dpp(o, i, 0x143, 0xc, 0xf, false); break;
    }
    return __int_as_float(r);
}
/* smallest and largest value over the wave's 64 lanes (NaN lanes do not count) */
__device__ __forceinline__ float wave_min_f(float v)
{
#pragma unroll
    for (int k = 0; k < 6; ++k) v = fminf(v, tr_dpp_f(v, INFINITY, k));
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 63));
}
__device__ __forceinline__ float wave_max_f(float v)
{
#pragma unroll
    for (int k = 0; k < 6; ++k) v = fmaxf(v, tr_dpp_f(v, -INFINITY, k));
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 63));
}

__device__ __forceinline__ int tree_level_of(const TreeDev &T, int64_t c)
{
    int k = 0;
    while (k + 1 < T.nlev && c >= T.off[k + 1]) ++k;
    return k;
}

__device__ __forceinline__ void tree_panels_of(const TreeDev &T, int64_t c, int64_t &p0, int64_t &p1)
{
    const int k = tree_level_of(T, c);
    p0 = (c - T.off[k]) << k;
    p1 = min(T.Np, p0 + (1 << k));
}

/* plan time: centre (of the bounding box), and the distances rmin of each
   cluster; one wave per cluster.  A cluster is far enough from every target
   that could list one of its panels: a listed panel has a node within
   near_factor h, so r >= R + near_factor max h rules it out. */
__global__ __launch_bounds__(256) void tree_clusters_kernel(TreeDev T, const double *__restrict__ x,
                                                            const double *__restrict__ y,
                                                            const double *__restrict__ ph, double alpha,
                                                            double near_factor)
{
    const int64_t c = blockIdx.x * (int64_t)4 + (threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    if (c >= T.ncl) return;
    const int k = tree_level_of(T, c);
    const int64_t p0 = (c - T.off[k]) << k, p1 = min(T.Np, p0 + (1 << k));
    double xl = INFINITY, xh = -INFINITY, yl = INFINITY, yh = -INFINITY, h = 0.0;
    for (int64_t j = 16 * p0 + lane; j < 16 * p1; j += 64) {
        xl = fmin(xl, x[j]), xh = fmax(xh, x[j]);
        yl = fmin(yl, y[j]), yh = fmax(yh, y[j]);
        h = fmax(h, ph[j >> 4]);
    }
    for (int o = 32; o > 0; o >>= 1) {
        xl = fmin(xl, __shfl_xor(xl, o)), xh = fmax(xh, __shfl_xor(xh, o));
        yl = fmin(yl, __shfl_xor(yl, o)), yh = fmax(yh, __shfl_xor(yh, o));
        h = fmax(h, __shfl_xor(h, o));
    }
    const double cx = 0.5 * (xl + xh), cy = 0.5 * (yl + yh);
    double R = 0.0;
    for (int64_t j = 16 * p0 + lane; j < 16 * p1; j += 64) R = fmax(R, hypot(x[j] - cx, y[j] - cy));
    for (int o = 32; o > 0; o >>= 1) R = fmax(R, __shfl_xor(R, o));
    R *= 1.0 + 1e-12;
    if (lane == 0) {
        T.cc[2 * c] = cx;
        T.cc[2 * c + 1] = cy;
    }
    if (lane < TR_RM) {
        const double clear = R + near_factor * h * (1.0 + 1e-12);
        double v;
        if (T.stokes)
            v = lane < TR_SNP ? fmax(R * tree_stokes_ratio(TR_PMIN + TR_PSTEP * lane), clear)
                              : (lane < TR_RM - 1 ? INFINITY : R);
        else if (lane < TR_NP)
            v = fmax(R * tree_order_ratio(TR_PMIN + TR_PSTEP * lane, alpha * R), clear);
        else
            v = fmax(R + TR_ZZERO * (1.0 + 1e-12) / alpha, clear);
        T.rmin[TR_RM * c + lane] = v;
    }
}

/* the piece class of z in [zlo, zhi] (0: z <= 2, piece + 1, KQ_NP + 1: per-pair) */
__device__ __forceinline__ int tree_piece(double zlo, double zhi)
{
    int lo = 0, hi = 0;
    for (int b = 0; b < KQ_NB; ++b) {
        lo += zlo > KQ_B[b] ? 1 : 0;
        hi += zhi > KQ_B[b] ? 1 : 0;
    }
    if (lo == hi) return lo;
    if (lo >= 1 && hi == lo + 1 && lo <= KQ_NB - 1) return KQ_NB + lo;
    return KQ_NP + 1;
}

/* plan time: the items of each group of 64 targets, one wave per group and run
   of 16 panels (the widest cluster), of the groups g0 on: into 16 slots of tmp
   per run, direct items from the front, expansions from the back, and their
   numbers and z classes into runs.  Panels are visited in order; at each, the
   largest aligned cluster is tried first, then its halves.  A wave per group
   alone left a plan of few groups waiting: 1024 panels all direct, 313 groups,
   2 ms. */
constexpr int TR_RUN = 1 << (TR_LEV - 1);
__host__ __device__ inline int tree_nrun(int64_t Np) { return (int)((Np + TR_RUN - 1) / TR_RUN); }
__device__ __forceinline__ uint32_t tree_run_word(int nd, int nf, int zlo, int zhi, bool expands)
{
    return (uint32_t)(nd | nf << 5 | zlo << 10 | zhi << 18) | (expands ? 1u << 26 : 0u);
}
__global__ __launch_bounds__(256) void tree_lists_kernel(TreeDev T, const double *__restrict__ tx,
                                                         const double *__restrict__ ty, int64_t M,
                                                         const double *__restrict__ sx, const double *__restrict__ sy,
                                                         double alpha, const int32_t *__restrict__ nptr,
                                                         const int32_t *__restrict__ npan, int64_t g0, int64_t ng,
                                                         uint2 *__restrict__ tmp, uint32_t *__restrict__ runs)
{
    const int64_t u = blockIdx.x * (int64_t)4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lane = threadIdx.x & 63, nrun = tree_nrun(T.Np);
    if (u >= ng * nrun) return;
    const int64_t run = u % nrun, i = min(64 * (g0 + u / nrun) + lane, M - 1);
    const double x = tx[i], y = ty[i];
    const int32_t k0 = nptr[i], k1 = nptr[i + 1];
    uint2 *items = tmp + u * TR_RUN;
    int nd = 0, nf = 0, zlo = 255, zhi = 0;
    bool expands = false;
    for (int64_t p = TR_RUN * run, pe = min(T.Np, p + TR_RUN); p < pe;) {
        int k = min(T.nlev - 1, __builtin_ctz((uint32_t)p | TR_RUN));
        for (;; --k) {
            const int64_t c = T.off[k] + (p >> k);
            const double dx = x - T.cc[2 * c], dy = y - T.cc[2 * c + 1], r = sqrt(fma(dx, dx, dy * dy));
            /* extreme distances, widened past the rounding to float */
            const double rlo = (double)wave_min_f((float)r) * (1.0 - 3e-7);
            const double rhi = (double)wave_max_f((float)r) * (1.0 + 3e-7);
            const double *rm = T.rmin + TR_RM * c;
            uint32_t y_ = 0xffffffffu;
            bool expand = T.expands, lap = false, small = false;
            if (T.stokes) {
                const double R = rm[TR_RM - 1], a = alpha * R, zc = alpha * (rlo - R);
                lap = zc >= TR_SLAP;
                small = zc < TR_SZ;
                expand = expand && a >= TR_AMIN && a <= (lap ? TR_SAMAX : TR_AMAX);
            }
            if (!T.stokes && rlo >= rm[TR_RM - 1]) {
                y_ = TR_ZERO;
            } else if (expand) {
                for (int q = TR_NP - 1 - T.stokes; /* the stresslet has one order fewer */ q >= 0 && rlo >= rm[q]; --q) /* rm falls with the order */
                    y_ = (uint32_t)(TR_PMIN + TR_PSTEP * q) << 8;
                if (y_ != 0xffffffffu) y_ |= (uint32_t)tree_piece(alpha * rlo, alpha * rhi) | (lap ? TR_LAP : small ? TR_SMALL : 0u);
            }
            if (y_ != 0xffffffffu) {
                if (!T.stokes && y_ != TR_ZERO) {
                    /* rm[0] and up exceed the radius: R <= rm of the highest order / 1.5 */
                    const uint32_t zc = tree_zclass(alpha * (rlo - rm[TR_NP - 1] * (1.0 / 1.5)) * (1.0 - 1e-12));
                    zlo = min(zlo, (int)(zc >> 24));
                    zhi = max(zhi, (int)(zc >> 24));
                    y_ |= zc;
                } else if (T.stokes && small) {
                    zlo = 0, zhi = 1; /* no z classes here: the plan has such items */
                }
                expands = expands || y_ != TR_ZERO;
                if (lane == 0) items[TR_RUN - 1 - nf] = make_uint2((uint32_t)c, y_);
                ++nf;
                break;
            }
            if (k > 0) continue;
            /* direct: the piece of the targets that do not list the panel */
            bool listed = false;
            for (int32_t q = k0; q < k1; ++q) listed = listed || npan[q] == (int32_t)p;
            const bool any = __ballot(listed) != 0;
            if (__ballot(!listed) != 0) {
                double r2lo = INFINITY, r2hi = 0.0;
                for (int j = 0; j < 16; ++j) {
                    const double ex = x - sx[16 * p + j], ey = y - sy[16 * p + j];
                    const double r2 = fma(ex, ex, ey * ey);
                    r2lo = fmin(r2lo, r2);
                    r2hi = fmax(r2hi, r2);
                }
                const double dlo = (double)wave_min_f(listed ? INFINITY : (float)sqrt(r2lo)) * (1.0 - 3e-7);
                const double dhi = (double)wave_max_f(listed ? -INFINITY : (float)sqrt(r2hi)) * (1.0 + 3e-7);
                const uint32_t zc = tree_zclass(alpha * dlo * (1.0 - 1e-12));
                if (!T.stokes) {
                    zlo = min(zlo, (int)(zc >> 24));
                    zhi = max(zhi, (int)(zc >> 24));
                }
                if (lane == 0)
                    items[nd] = make_uint2((uint32_t)c, (uint32_t)tree_piece(alpha * dlo, alpha * dhi) |
                                                            (any ? TR_NEAR : 0u) | zc);
                ++nd;
            }
            break;
        }
        p += (int64_t)1 << k;
    }
    if (lane == 0) runs[u] = tree_run_word(nd, nf, zlo, zhi, expands);
}

/* plan time: a group's counts and z classes from its runs', one wave per group */
__global__ __launch_bounds__(64) void tree_count_kernel(TreeDev T, int64_t g0, const uint32_t *__restrict__ runs)
{
    const int lane = threadIdx.x, nrun = tree_nrun(T.Np);
    const int64_t g = g0 + blockIdx.x;
    const uint32_t *w = runs + blockIdx.x * (int64_t)nrun;
    int nd = 0, nf = 0, zlo = 255, zhi = 0;
    bool expands = false;
    for (int r = lane; r < nrun; r += 64) {
        const uint32_t v = w[r];
        expands = expands || v >> 26;
        nd += v & 31;
        nf += (v >> 5) & 31;
        zlo = min(zlo, (int)((v >> 10) & 255));
        zhi = max(zhi, (int)((v >> 18) & 255));
    }
    for (int o = 32; o > 0; o >>= 1) {
        nd += __shfl_xor(nd, o), nf += __shfl_xor(nf, o);
        zlo = min(zlo, __shfl_xor(zlo, o)), zhi = max(zhi, __shfl_xor(zhi, o));
    }
    expands = __ballot(expands) != 0;
    if (lane != 0) return;
    if (expands) T.cost[3] = 1; /* all that write it write this */
    T.cnt[g] = make_int2(nd, nf);
    T.znear[g] = zlo;
    if (zhi > zlo) atomicMax(T.cost + 1, (unsigned long long)(zhi - zlo));
}

/* plan time: the runs' items to their places in the groups' lists, one wave per
   group, a lane per run */
__global__ __launch_bounds__(64) void tree_fill_kernel(TreeDev T, int64_t g0, const uint2 *__restrict__ tmp,
                                                       const uint32_t *__restrict__ runs)
{
    const int lane = threadIdx.x, nrun = tree_nrun(T.Np);
    const int64_t u0 = blockIdx.x * (int64_t)nrun;
    const longlong2 at = T.at[g0 + blockIdx.x];
    int64_t front = at.x, back = at.y;
    for (int r0 = 0; r0 < nrun; r0 += 64) {
        const int r = r0 + lane;
        const uint32_t v = r < nrun ? runs[u0 + r] : 0u;
        const uint32_t mine = (v & 31) | ((v >> 5) & 31) << 16; /* at most 1024 of either in 64 runs */
        uint32_t inc = mine;
        for (int o = 1; o < 64; o <<= 1) {
            const uint32_t q = __shfl_up(inc, o);
            if (lane >= o) inc += q;
        }
        const uint32_t all = __shfl(inc, 63), before = inc - mine;
        const uint2 *src = tmp + (u0 + r) * TR_RUN;
        for (int k = 0; k < (int)(mine & 0xffff); ++k) T.items[front + (before & 0xffff) + k] = src[k];
        for (int k = 0; k < (int)(mine >> 16); ++k) T.items[back - 1 - (before >> 16) - k] = src[TR_RUN - 1 - k];
        front += all & 0xffff;
        back -= all >> 16;
    }
}

/* plan time, where the lists are not to be had: one list for all groups, every
   panel direct and per pair */
__global__ void tree_direct_kernel(TreeDev T, int64_t G)
{
    const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (i < T.Np) T.items[i] = make_uint2((uint32_t)i, (uint32_t)(KQ_NP + 1) | TR_NEAR);
    if (i >= G) return;
    T.at[i] = make_longlong2(0, T.Np);
    T.cnt[i] = make_int2((int)T.Np, 0);
    T.znear[i] = 0;
    T.order[i] = (int32_t)i;
}


/* work of a group in expansions (a direct item costs about three) */
__device__ __forceinline__ int tree_cost(int2 cnt) { return 3 * cnt.x + cnt.y; }

/* plan time: the groups by falling work, its sum, and the places of their lists;
   one block, a counting sort: blocks start in this order, so the groups next to
   the curve, with up to five times the work of the others, do not start last */
constexpr int TR_BINS = 1024;
__global__ __launch_bounds__(1024) void tree_order_kernel(TreeDev T, int64_t G)
{
    __shared__ int32_t pos[TR_BINS];
    __shared__ unsigned long long start[1024];
    __shared__ unsigned long long total;
    auto bin = [&](int64_t g) { return TR_BINS - 1 - min(TR_BINS - 1, tree_cost(T.cnt[g])); };
    const int t = threadIdx.x;
    pos[t] = 0;
    if (t == 0) total = 0;
    __syncthreads();
    unsigned long long sum = 0;
    for (int64_t g = t; g < G; g += 1024) {
        atomicAdd(&pos[bin(g)], 1);
        sum += (unsigned long long)tree_cost(T.cnt[g]);
    }
    atomicAdd(&total, sum);
    __syncthreads();
    if (t == 0) *T.cost = total;
    for (int o = 1; o < TR_BINS; o <<= 1) {
        const int32_t v = t >= o ? pos[t - o] : 0;
        __syncthreads();
        pos[t] += v;
        __syncthreads();
    }
    const int32_t before = t ? pos[t - 1] : 0;
    __syncthreads();
    pos[t] = before;
    __syncthreads();
    for (int64_t g = t; g < G; g += 1024) T.order[atomicAdd(&pos[bin(g)], 1)] = (int32_t)g;
    /* places: a thread takes a run of groups */
    const int64_t per = (G + 1023) / 1024, ga = min(G, t * per), gb = min(G, ga + per);
    unsigned long long n = 0;
    for (int64_t g = ga; g < gb; ++g) n += (unsigned long long)(T.cnt[g].x + T.cnt[g].y);
    unsigned long long inc = n;
    for (int o = 1; o < 1024; o <<= 1) {
        start[t] = inc;
        __syncthreads();
        if (t >= o) inc += start[t - o];
        __syncthreads();
    }
    if (t == 1023) T.cost[2] = inc;
    inc -= n;
    for (int64_t g = ga; g < gb; ++g) {
        const unsigned long long end = inc + (unsigned long long)(T.cnt[g].x + T.cnt[g].y);
        T.at[g] = make_longlong2((long long)inc, (long long)end);
        inc = end;
    }
}

/* ------------------------------------------------------------------------ */
/* moments of one evaluation                                                 */
/* ------------------------------------------------------------------------ */
/* A block takes 256 sources (16 panels) at one level (blockIdx.y) and TR_NG
   orders (blockIdx.z).  With w = (alpha/2) conj(y - c) and q = |w|^2,
   B_n = w^n/n! S_n(q), S_n = sum_k q^k/(k! (n+1)..(n+k)), from the backward
   recurrence S_{n-1} = S_n + q/(n(n+1)) S_{n+1} (all terms positive: stable)
   started by the series; no root, division or angle per source.  The sources
   of a panel are added through LDS in a fixed order, panels of a cluster by a
   fixed tree.  Latency bound (config 2: 240 blocks, 14 MFLOP): the split over
   orders keeps a block at three short rounds. */
constexpr int TR_NG = 12, TR_GROUPS = (TR_ROWS + TR_NG - 1) / TR_NG;
constexpr int TR_PAD = 17; /* LDS row of a panel's 16 sources */

template <int N0, int CNT>
__device__ __forceinline__ void tree_regular(double wr, double wi, double q, double (&br)[CNT], double (&bi)[CNT])
{
    /* B_n, n = N0 .. N0 + CNT - 1 */
    constexpr int top = N0 + CNT - 1;
    double s1 = 1.0, s0 = 1.0; /* S_{top+1}, S_top by Horner, 10 terms (q <= 1) */
#pragma unroll
    for (int k = 10; k >= 1; --k) {
        s1 = fma(q * (1.0 / ((double)k * (top + 1 + k))), s1, 1.0);
        s0 = fma(q * (1.0 / ((double)k * (top + k))), s0, 1.0);
    }
#pragma unroll
    for (int n = top; n >= N0; --n) {
        br[n - N0] = s0;
        if (n > 0) {
            const double t = fma(q * (1.0 / ((double)n * (n + 1))), s1, s0);
            s1 = s0;
            s0 = t;
        }
    }
    double pr = 1.0, pi = 0.0;
#pragma unroll
    for (int n = 1; n <= top; ++n) {
        if (n - 1 >= N0) {
            bi[n - 1 - N0] = pi * br[n - 1 - N0];
            br[n - 1 - N0] *= pr;
        }
        const double a = wr * (1.0 / n), b = wi * (1.0 / n);
        const double t = fma(pr, a, -pi * b);
        pi = fma(pr, b, pi * a);
        pr = t;
    }
    bi[CNT - 1] = pi * br[CNT - 1];
    br[CNT - 1] *= pr;
}

/* S_n and S_n - 1 of B_n = w^n/n! S_n, n = N0 .. N0 + CNT - 1, as tree_regular
   forms S_n; all terms positive */
template <int N0, int CNT>
__device__ __forceinline__ void tree_regular_series(double q, double (&s)[CNT], double (&d)[CNT])
{
    constexpr int top = N0 + CNT - 1;
    double u1 = 1.0, u0 = 1.0;
#pragma unroll
    for (int k = 10; k >= 2; --k) {
        u1 = fma(q * (1.0 / ((double)k * (top + 1 + k))), u1, 1.0);
        u0 = fma(q * (1.0 / ((double)k * (top + k))), u0, 1.0);
    }
    double s1 = fma(q * (1.0 / (top + 2)), u1, 1.0); /* S_{top+1} */
    double d0 = q * (1.0 / (top + 1)) * u0;
#pragma unroll
    for (int n = top; n >= N0; --n) {
        d[n - N0] = d0;
        s[n - N0] = 1.0 + d0;
        if (n > 0) {
            d0 = fma(q * (1.0 / ((double)n * (n + 1))), s1, d0);
            s1 = s[n - N0];
        }
    }
}

/* B_n is kept for n = N0 - H .. N0 + TR_NG - 1 + H: the potential of a dipole
   takes the neighbours of order n (H = 1), its gradient the next ones too */
template <bool GRAD, int Z>
struct TreeB {
    static constexpr int H = GRAD ? 2 : 1, N0 = Z * TR_NG, LO = N0 < H ? 0 : N0 - H, CNT = N0 + TR_NG + H - LO;
    double br[CNT], bi[CNT];
    /* M_n (n >= 0, without the factor 2 of n > 0) of a unit charge, and of the dipole (ex, ey)/alpha */
    template <int N>
    __device__ __forceinline__ void dipole(double ex, double ey, double &re, double &im) const
    {
        constexpr int b = N - LO;
        if constexpr (N == 0) {
            re = fma(ex, br[1], -ey * bi[1]);
            im = 0.0;
        } else {
            re = 0.5 * fma(ex, br[b - 1] + br[b + 1], ey * (bi[b - 1] - bi[b + 1]));
            im = 0.5 * fma(ex, bi[b - 1] + bi[b + 1], ey * (br[b + 1] - br[b - 1]));
        }
    }
};

/* row n of one layer: the potential's (2 Re M, -2 Im M), or the same of its x
   and y derivatives: (d_x + i d_y) sum_n M_n K_n e^{i n theta} =
   -alpha sum_n M_n K_{n+1} e^{i (n+1) theta} over all n, M_{-n} = conj M_n. */
template <bool GRAD, int N, class M>
__device__ __forceinline__ void tree_row_values(const M &m, double alpha, double (*v)[16 * TR_PAD], int at)
{
    double a, b;
    if constexpr (!GRAD) {
        m.template at<N>(a, b);
        v[0][at] = N == 0 ? a : 2.0 * a;
        v[1][at] = N == 0 ? 0.0 : -2.0 * b;
    } else {
        double c, d;
        m.template at<N + 1>(c, d);
        if constexpr (N == 0) {
            v[0][at] = -alpha * c;
            v[1][at] = 0.0;
            v[2][at] = alpha * d;
            v[3][at] = 0.0;
        } else {
            m.template at<N - 1>(a, b);
            v[0][at] = -alpha * (a + c);
            v[1][at] = alpha * (b + d);
            v[2][at] = -alpha * (b - d);
            v[3][at] = -alpha * (a - c);
        }
    }
}

template <class B>
struct TreeCharge {
    const B &b;
    double q;
    template <int N>
    __device__ __forceinline__ void at(double &re, double &im) const
    {
        re = q * b.br[N - B::LO];
        im = q * b.bi[N - B::LO];
    }
};
template <class B>
struct TreeDipole {
    const B &b;
    double ex, ey;
    template <int N>
    __device__ __forceinline__ void at(double &re, double &im) const
    {
        b.template dipole<N>(ex, ey, re, im);
    }
};

template <bool SLP, bool DLP, bool GRAD, int Z, int R, class B>
__device__ __forceinline__ void tree_moments_rounds(const TreeDev &T, int k, int64_t p0, const B &b, double alpha,
                                                    double q, double ex, double ey, double (*buf)[16 * TR_PAD])
{
    constexpr int NL = GRAD ? 4 : 2, NV = NL * ((SLP ? 1 : 0) + (DLP ? 1 : 0)), RO = NV > 4 ? 2 : 4; /* orders a round */
    constexpr int N = Z * TR_NG + R;
    if constexpr (R < TR_NG && N < TR_ROWS) {
        const int t = threadIdx.x, at = (t >> 4) * TR_PAD + (t & 15), pp = t & 15;
        const TreeCharge<B> mc{b, q};
        const TreeDipole<B> md{b, ex, ey};
        double(*bd)[16 * TR_PAD] = buf + (SLP ? NL : 0);
        if (SLP) tree_row_values<GRAD, N>(mc, alpha, buf, at);
        if (DLP) tree_row_values<GRAD, N>(md, alpha, bd, at);
        if (SLP) tree_row_values<GRAD, N + 1>(mc, alpha, buf + NV, at);
        if (DLP) tree_row_values<GRAD, N + 1>(md, alpha, bd + NV, at);
        if constexpr (RO > 2) {
            if (SLP) tree_row_values<GRAD, N + 2>(mc, alpha, buf + 2 * NV, at);
            if (DLP) tree_row_values<GRAD, N + 2>(md, alpha, bd + 2 * NV, at);
            if (SLP) tree_row_values<GRAD, N + 3>(mc, alpha, buf + 3 * NV, at);
            if (DLP) tree_row_values<GRAD, N + 3>(md, alpha, bd + 3 * NV, at);
        }
        __syncthreads();
        const int cb = t >> 4;
        if (cb < RO * NV) {
            const double *row = buf[cb] + pp * TR_PAD;
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
            if ((pp & ((1 << k) - 1)) == 0 && p < T.Np && n < TR_ROWS)
                T.mom[(T.off[k] + (p >> k)) * tr_stride(NV) + n * NV + cb % NV] = s;
        }
        __syncthreads();
        tree_moments_rounds<SLP, DLP, GRAD, Z, R + RO>(T, k, p0, b, alpha, q, ex, ey, buf);
    }
}

template <bool SLP, bool DLP, bool GRAD, int Z>
__device__ __forceinline__ void tree_moments_body(const FarArgs &A, const TreeDev &T, const double *mu,
                                                  double (*buf)[16 * TR_PAD])
{
    const int k = blockIdx.y, t = threadIdx.x;
    const int64_t p0 = (int64_t)blockIdx.x * 16, j = 16 * p0 + t;
    const bool have = j < A.N;
    const int64_t js = have ? j : A.N - 1, ps = js >> 4;
    const int64_t c = T.off[k] + (ps >> k);
    const double dx = A.sx[js] - T.cc[2 * c], dy = A.sy[js] - T.cc[2 * c + 1];
    const double wj = have ? A.sw[js] : 0.0;
    double q = 0.0, ex = 0.0, ey = 0.0;
    if (SLP) q = have ? wj * A.sigma[js] : 0.0;
    if (DLP) {
        const double m = have ? (A.alpha * wj) * mu[js] : 0.0; /* alpha goes with the dipole */
        ex = m * A.snx[js];
        ey = m * A.sny[js];
    }
    if (Z == 0 && k == 0 && have) {
        double *s = T.st + (j >> 4) * 48 + (j & 15);
        if (SLP) s[0] = GRAD ? A.alpha * q : q; /* a gradient pair evaluates K1(z)/r of both */
        if (DLP) {
            s[16] = ex;
            s[32] = ey;
        }
    }
    if (Z == 0 && T.skip) {
        /* bound of a cluster's charges, for far_tree_kernel */
        double sum = (SLP ? fabs(q) : 0.0) + (DLP ? fabs(ex) + fabs(ey) : 0.0);
        for (int o = 1; o < 16; o <<= 1) sum += __shfl_xor(sum, o);
        if ((t & 15) == 0) buf[0][t >> 4] = sum;
        __syncthreads();
        const int64_t p = p0 + t;
        if (t < 16 && (t & ((1 << k) - 1)) == 0 && p < T.Np) {
            double b = 0.0;
            for (int u = t; u < t + (1 << k) && p0 + u < T.Np; ++u) b += buf[0][u];
            T.lb[T.off[k] + (p >> k)] = (float)log2(b) + 0.01f;
        }
        __syncthreads();
    }
    if (!T.expands) return;
    /* clusters too wide to expand (the same test as tree_order_ratio through rmin) */
    const bool live = T.rmin[TR_RM * c + TR_NP - 1] < INFINITY;
    if (__syncthreads_or(live ? 1 : 0) == 0) return;
    const double ah = 0.5 * A.alpha, wr = live ? ah * dx : 0.0, wi = live ? -ah * dy : 0.0;
    TreeB<GRAD, Z> b;
    tree_regular<TreeB<GRAD, Z>::LO, TreeB<GRAD, Z>::CNT>(wr, wi, fma(wr, wr, wi * wi), b.br, b.bi);
    tree_moments_rounds<SLP, DLP, GRAD, Z, 0>(T, k, p0, b, A.alpha, q, ex, ey, buf);
}

/* rows of the stresslet: per complex field (the velocity; with GRAD its x and
   y derivatives) the coefficients of K_n cos and K_n sin of its real and
   imaginary part, then Re and Im of the power (2/z)^n e^{i n theta} (GRAD: of
   the x derivative; the y derivative's is -i times it). */
template <bool GRAD, int Z>
struct TreeS {
    static constexpr int H = GRAD ? 4 : 3, N0 = Z * TR_NG, LO = N0 < H ? 0 : N0 - H, CNT = N0 + TR_NG + H - LO;
    double br[CNT], bi[CNT], pr[CNT], pi[CNT]; /* B_n and w^n */
    cplx sg;                                   /* alpha sigma */
    double tau, alpha;
    template <int N>
    __device__ __forceinline__ cplx b() const
    {
        return mk(br[N - LO], bi[N - LO]);
    }
    template <int N>
    __device__ __forceinline__ cplx w() const
    {
        return mk(pr[N - LO], pi[N - LO]);
    }
    /* coefficient of O_K: -conj(sigma) R_{3-K} + sigma R_{-1-K} (times alpha), R_{-n} = B_n = conj R_n */
    template <int K>
    __device__ __forceinline__ cplx c() const
    {
        if constexpr (K >= 3) return sg * b<K + 1>() - conj(sg) * b<K - 3>();
        else if constexpr (K >= 0) return sg * b<K + 1>() - conj(sg * b<3 - K>());
        else return sg * conj(b<-K - 1>()) - conj(sg * b<3 - K>());
    }
    /* coefficient of (2/z)^N e^{i N theta} */
    template <int N>
    __device__ __forceinline__ cplx l() const
    {
        if constexpr (N < 1) return mk(0.0, 0.0);
        else {
            cplx v = (0.5 * alpha * tau) * w<N - 1>();
            if constexpr (N >= 3) v = v + (0.5 * (N - 1) * (N - 2)) * (conj(sg) * w<N - 3>());
            return v;
        }
    }
    template <int N>
    __device__ __forceinline__ void row(double (*v)[16 * TR_PAD], int at) const
    {
        if constexpr (!GRAD) {
            put<N>(c<N>(), c<-N>(), v, at);
            const cplx p = l<N>();
            v[4][at] = p.re;
            v[5][at] = p.im;
        } else {
            /* d_x: -(alpha/2)(C_{k-1} + C_{k+1}), d_y: (i alpha/2)(C_{k-1} - C_{k+1}) */
            const double ah = 0.5 * alpha;
            const cplx a = c<N - 1>(), b_ = c<N + 1>(), d = c<-N - 1>(), e = c<1 - N>();
            put<N>(-ah * (a + b_), -ah * (d + e), v, at);
            const cplx yp = ah * (a - b_), ym = ah * (d - e);
            put<N>(mk(-yp.im, yp.re), mk(-ym.im, ym.re), v + 4, at);
            const cplx p = (-ah * (N - 1)) * l<N - 1>();
            v[8][at] = p.re;
            v[9][at] = p.im;
        }
    }
    template <int N>
    static __device__ __forceinline__ void put(cplx p, cplx m, double (*v)[16 * TR_PAD], int at)
    {
        const bool z = N == 0; /* K_0: one coefficient */
        v[0][at] = z ? p.re : p.re + m.re;
        v[1][at] = z ? 0.0 : m.im - p.im;
        v[2][at] = z ? p.im : p.im + m.im;
        v[3][at] = z ? 0.0 : p.re - m.re;
    }
};

/* The powers' rows of TR_SMALL items: 4 values (8 with GRAD: the x and y
   derivatives) in the K part's layout, of
     l~_k = l_k + (k-1)!/2 c_k  at (2/z)^k e^{i k theta},
     (k-1)!/2 c_{-k}            at (2/z)^k e^{-i k theta}   (k >= 1)
   with c and l as in TreeS.  The parts of l_k and c_k that cancel leave S_n - 1
   of the regular functions B_n = w^n/n! S_n; all factorials are ratios of near
   ones. */
template <bool GRAD, int Z>
struct TreeSmall {
    static constexpr int H = GRAD ? 4 : 3, N0 = Z * TR_NG, LO = N0 < H ? 0 : N0 - H, CNT = N0 + TR_NG + H - LO;
    double s[CNT], d[CNT], pr[CNT], pi[CNT]; /* S_n, S_n - 1 and w^n */
    cplx sg;                                 /* alpha sigma */
    double tau, alpha;
    template <int N>
    __device__ __forceinline__ cplx w() const
    {
        return mk(pr[N - LO], pi[N - LO]);
    }
    /* w^N S_N / D */
    template <int N>
    __device__ __forceinline__ cplx ws(double D) const
    {
        return (s[N - LO] * (1.0 / D)) * w<N>();
    }
    /* l~_K */
    template <int K>
    __device__ __forceinline__ cplx l() const
    {
        if constexpr (K < 1) return mk(0.0, 0.0);
        else {
            cplx v = (0.5 * alpha * tau) * w<K - 1>() + 0.5 * (sg * ws<K + 1>((double)K * (K + 1)));
            if constexpr (K >= 3) v = v - (0.5 * (K - 1) * (K - 2) * d[K - 3 - LO]) * (conj(sg) * w<K - 3>());
            else v = v - 0.5 * conj(sg * ws<3 - K>(K == 1 ? 2.0 : 1.0));
            return v;
        }
    }
    /* (K-1)!/2 c_{-K} */
    template <int K>
    __device__ __forceinline__ cplx m() const
    {
        return 0.5 * (sg * conj(ws<K - 1>(1.0))) - 0.5 * conj(sg * ws<K + 3>((double)K * (K + 1) * (K + 2) * (K + 3)));
    }
    /* c_0 / 2 */
    __device__ __forceinline__ cplx c0() const { return 0.5 * (sg * ws<1>(1.0)) - 0.5 * conj(sg * ws<3>(6.0)); }
    template <int N>
    __device__ __forceinline__ void row(double (*v)[16 * TR_PAD], int at) const
    {
        if constexpr (N == 0) {
            for (int k = 0; k < (GRAD ? 8 : 4); ++k) v[k][at] = 0.0;
        } else if constexpr (!GRAD) {
            TreeS<false, Z>::template put<N>(l<N>(), m<N>(), v, at);
        } else {
            /* d_x: -(alpha/2)(C_{k-1} + C_{k+1}), d_y: (i alpha/2)(C_{k-1} - C_{k+1}), each times (N-1)!/2, with
               (N-1) l_{N-1} in the upper ones */
            const double ah = 0.5 * alpha;
            cplx up, uq, lp, lq; /* of e^{i N theta}: neighbours N - 1 and N + 1; of e^{-i N theta}: -N - 1 and 1 - N */
            if constexpr (N == 1) {
                up = c0();
                uq = 0.5 * (sg * ws<3>(6.0)) - 0.5 * conj(sg * ws<1>(1.0));
                lq = up;
            } else {
                up = (double)(N - 1) * l<N - 1>();
                uq = 0.5 * (sg * ws<N + 2>((double)N * (N + 1) * (N + 2))) -
                     (0.5 * (N - 1)) * (conj(sg) * ws<N - 2>(1.0));
                lq = (0.5 * (N - 1)) * (sg * conj(ws<N - 2>(1.0))) -
                     0.5 * conj(sg * ws<N + 2>((double)N * (N + 1) * (N + 2)));
            }
            lp = 0.5 * (sg * conj(ws<N>((double)N))) -
                 0.5 * conj(sg * ws<N + 4>((double)N * (N + 1) * (N + 2) * (N + 3) * (N + 4)));
            TreeS<true, Z>::template put<N>(-ah * (up + uq), -ah * (lp + lq), v, at);
            const cplx yp = ah * (up - uq), ym = ah * (lp - lq);
            TreeS<true, Z>::template put<N>(mk(-yp.im, yp.re), mk(-ym.im, ym.re), v + 4, at);
        }
    }
};

/* sums of the rows of B (NV values each, RO rows a round) over the sources of each
   cluster, into mom.  Bound by the latency of its rounds: two rows a round took
   9.0 us at 64 panels, four 8.3 (GRAD: two instead of one) */
template <int NV, int RO, int Z, int R, class B>
__device__ __forceinline__ void tree_stokes_rounds(const TreeDev &T, double *mom, int k, int64_t p0, const B &b,
                                                   double (*buf)[16 * TR_PAD])
{
    constexpr int N = Z * TR_NG + R;
    if constexpr (R < TR_NG && N < TR_ROWS) {
        const int t = threadIdx.x, at = (t >> 4) * TR_PAD + (t & 15), pp = t & 15, cb = t >> 4;
        b.template row<N>(buf, at);
        b.template row<N + 1>(buf + NV, at);
        if constexpr (RO > 2) {
            b.template row<N + 2>(buf + 2 * NV, at);
            b.template row<N + 3>(buf + 3 * NV, at);
        }
        __syncthreads();
#pragma unroll
        for (int c0 = 0; c0 < RO * NV; c0 += 16) {
            const int c = c0 + cb;
            if (c >= RO * NV) continue;
            const double *row = buf[c] + pp * TR_PAD;
            double s0 = 0.0, s1 = 0.0;
#pragma unroll
            for (int l = 0; l < 16; l += 2) {
                s0 += row[l];
                s1 += row[l + 1];
            }
            double s = s0 + s1;
            for (int o = 1; o < (1 << k); o <<= 1) s += __shfl_xor(s, o);
            const int n = N + c / NV;
            const int64_t p = p0 + pp;
            if ((pp & ((1 << k) - 1)) == 0 && p < T.Np && n < TR_ROWS)
                mom[(T.off[k] + (p >> k)) * tr_stride(NV) + n * NV + c % NV] = s;
        }
        __syncthreads();
        tree_stokes_rounds<NV, RO, Z, R + RO>(T, mom, k, p0, b, buf);
    }
}

template <bool GRAD, int Z, bool SMALL>
__device__ __forceinline__ void tree_stokes_body(const FarArgs &A, const TreeDev &T, const double *mu,
                                                 double (*buf)[16 * TR_PAD])
{
    const int k = blockIdx.y, t = threadIdx.x;
    const int64_t p0 = (int64_t)blockIdx.x * 16, j = 16 * p0 + t;
    const bool have = j < A.N;
    const int64_t js = have ? j : A.N - 1;
    const int64_t c = T.off[k] + ((js >> 4) >> k);
    const double dx = A.sx[js] - T.cc[2 * c], dy = A.sy[js] - T.cc[2 * c + 1];
    const double wj = have ? A.sw[js] : 0.0, nx = A.snx[js], ny = A.sny[js];
    const double m1 = have ? wj * mu[js] : 0.0, m2 = have ? wj * mu[A.N + js] : 0.0;
    typename std::conditional<SMALL, TreeSmall<GRAD, Z>, TreeS<GRAD, Z>>::type b;
    b.alpha = A.alpha;
    b.tau = fma(m1, nx, m2 * ny);
    b.sg = (0.5 * A.alpha) * (mk(m1, m2) * mk(nx, ny));
    if (Z == 0 && k == 0 && !SMALL) {
        if (have) {
            double *s = T.st + (j >> 4) * 48 + (j & 15);
            s[0] = m1;
            s[16] = m2;
        }
        if (T.flux) {
            double f = b.tau;
            for (int o = 1; o < 16; o <<= 1) f += __shfl_xor(f, o);
            if ((t & 15) == 0 && have) T.flux[j >> 4] = f;
        }
    }
    if (!T.expands) return;
    const double ah = 0.5 * A.alpha, wr = ah * dx, wi = -ah * dy, q2 = fma(wr, wr, wi * wi);
    if constexpr (SMALL)
        tree_regular_series<TreeS<GRAD, Z>::LO, TreeS<GRAD, Z>::CNT>(q2, b.s, b.d);
    else
        tree_regular<TreeS<GRAD, Z>::LO, TreeS<GRAD, Z>::CNT>(wr, wi, q2, b.br, b.bi);
    double pr = 1.0, pi = 0.0;
#pragma unroll
    for (int n = 0; n < TreeS<GRAD, Z>::LO + TreeS<GRAD, Z>::CNT; ++n) {
        if (n >= TreeS<GRAD, Z>::LO) {
            b.pr[n - TreeS<GRAD, Z>::LO] = pr;
            b.pi[n - TreeS<GRAD, Z>::LO] = pi;
        }
        const double q = fma(pr, wr, -pi * wi);
        pi = fma(pr, wi, pi * wr);
        pr = q;
    }
    tree_stokes_rounds<SMALL ? (GRAD ? 8 : 4) : (GRAD ? 10 : 6), GRAD ? 2 : 4, Z, 0>(T, SMALL ? T.small : T.mom, k, p0, b, buf);
}

template <bool GRAD>
__global__ __launch_bounds__(256) void tree_stokes_kernel(FarArgs A, TreeDev T)
{
    __shared__ double buf[24][16 * TR_PAD];
    const double *mu;
    if (!far_density(A, mu)) return;
    switch (blockIdx.z) { /* from TR_GROUPS on the rows of TR_SMALL items */
    case 0: tree_stokes_body<GRAD, 0, false>(A, T, mu, buf); break;
    case 1: tree_stokes_body<GRAD, 1, false>(A, T, mu, buf); break;
    case 2: tree_stokes_body<GRAD, 2, false>(A, T, mu, buf); break;
    case 3: tree_stokes_body<GRAD, 0, true>(A, T, mu, buf); break;
    case 4: tree_stokes_body<GRAD, 1, true>(A, T, mu, buf); break;
    default: tree_stokes_body<GRAD, 2, true>(A, T, mu, buf); break;
    }
}

template <bool SLP, bool DLP, bool GRAD>
__global__ __launch_bounds__(256) void tree_moments_kernel(FarArgs A, TreeDev T)
{
    constexpr int NV = (GRAD ? 4 : 2) * ((SLP ? 1 : 0) + (DLP ? 1 : 0));
    __shared__ double buf[(NV > 4 ? 2 : 4) * NV][16 * TR_PAD];
    const double *mu;
    if (!far_density(A, mu)) return;
    switch (blockIdx.z) {
    case 0: tree_moments_body<SLP, DLP, GRAD, 0>(A, T, mu, buf); break;
    case 1: tree_moments_body<SLP, DLP, GRAD, 1>(A, T, mu, buf); break;
    default: tree_moments_body<SLP, DLP, GRAD, 2>(A, T, mu, buf); break;
    }
}
static_assert(TR_GROUPS == 3, "tree_moments_kernel has a case for each group of orders");

/* ------------------------------------------------------------------------ */
/* evaluation                                                                */
/* ------------------------------------------------------------------------ */
/* K0, K1 at distance^2 r2 in piece PC (-1: z <= 2; KQ_NP: per-lane), and 1/r */
template <int PC>
__device__ __forceinline__ void tree_k01(const FarConst &fc, const double *fq, double r2, double &ri, double &k0,
                                         double &k1)
{
    constexpr int K = PC < 0 || PC >= KQ_NP ? 0 : PC;
    const FarTab T = far_table();
    if constexpr (PC >= 0 && PC < KQ_NP) {
        double qa, qk, d;
        fine_q<K>(fq, qa, qk);
        ri = lean_rsq(r2);
        const double z = fc.a * (r2 * ri);
        const double e = lean_exp_neg(T, z) * lean_rsq(z);
        k0 = e * far_piece_fine<true, true, K>(T, qa, qk, ri, d);
        k1 = e * d;
    } else {
        K01 o, o2;
        if constexpr (PC < 0)
            o = k01_far_small<true, true, true>(T, r2, fc);
        else
            k01_far2<true, true, true, true>(T, fc, r2, r2, o, o2);
        ri = lean_rsq(r2);
        k0 = o.k0;
        k1 = o.ak1r * (r2 * ri);
    }
}

__device__ __forceinline__ void tree_k01_pc(int pc, const FarConst &fc, const double *fq, double r2, double &ri,
                                            double &k0, double &k1)
{
    switch (pc) {
#define MHLP_TREE_PC(PCV) \
    case PCV: tree_k01<PCV>(fc, fq, r2, ri, k0, k1); break;
        MHLP_PC_CASES(MHLP_TREE_PC)
#undef MHLP_TREE_PC
    default: tree_k01<KQ_NP>(fc, fq, r2, ri, k0, k1);
    }
}

/* f0 += a s0, f1 += b s1 with a, b the values AT, AT + 1 (AT even; SWAP: b, a) of
   the moment table.  The table sits 32 doubles to a register quadruple, two
   per lane and repeated in every row of 16 lanes, and reaches the FMA as its
   row-broadcast operand.  A register that the VALU has just written may not be
   read so before two wait states: the s_nop covers any copy the compiler puts
   in front. */
template <int AT, bool SWAP = false>
__device__ __forceinline__ void fmac_pair(double &f0, double &f1, const double2 *m, double s0, double s1)
{
    static_assert(AT % 2 == 0, "both values lie in one lane");
    const double a = SWAP ? m[AT / 32].y : m[AT / 32].x, b = SWAP ? m[AT / 32].x : m[AT / 32].y;
    asm("s_nop 1\n\t"
        "v_fmac_f64_dpp %0, %2, %4 row_newbcast:%6 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %1, %3, %5 row_newbcast:%6 row_mask:0xf bank_mask:0xf"
        : "+&v"(f0), "+&v"(f1)
        : "v"(a), "v"(b), "v"(s0), "v"(s1), "n"((AT % 32) / 2));
}

/* two fields of a row in one go */
template <int AT>
__device__ __forceinline__ void fmac_quad(double &f0, double &f1, double &g0, double &g1, const double2 *m, double s0,
                                          double s1)
{
    static_assert(AT % 2 == 0 && AT % 32 != 30, "the four values lie in neighbouring lanes");
    asm("s_nop 1\n\t"
        "v_fmac_f64_dpp %0, %4, %6 row_newbcast:%8 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %1, %5, %7 row_newbcast:%8 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %2, %4, %6 row_newbcast:%9 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %3, %5, %7 row_newbcast:%9 row_mask:0xf bank_mask:0xf"
        : "+&v"(f0), "+&v"(f1), "+&v"(g0), "+&v"(g1)
        : "v"(m[AT / 32].x), "v"(m[AT / 32].y), "v"(s0), "v"(s1), "n"((AT % 32) / 2), "n"((AT % 32) / 2 + 1));
}

template <int NF, int N, int F>
__device__ __forceinline__ void tree_row(const double2 *m, double kc, double ks, double (&f0)[NF], double (&f1)[NF])
{
    if constexpr (F + 1 < NF && (N * 2 * NF + 2 * F) % 32 != 30) {
        fmac_quad<N * 2 * NF + 2 * F>(f0[F], f1[F], f0[F + 1], f1[F + 1], m, kc, ks);
        tree_row<NF, N, F + 2>(m, kc, ks, f0, f1);
    } else if constexpr (F < NF) {
        fmac_pair<N * 2 * NF + 2 * F>(f0[F], f1[F], m, kc, ks);
        tree_row<NF, N, F + 1>(m, kc, ks, f0, f1);
    }
}

/* orders N, N + 1 and on to `order` (even) */
template <int NF, int N>
__device__ __forceinline__ void tree_rows(int order, const double2 *m, double c2, double h, double b, double km,
                                          double k, double cp, double cn, double sp, double sn, double (&f0)[NF],
                                          double (&f1)[NF])
{
    if constexpr (N + 1 < TR_ROWS) {
        if (N > order) return;
        tree_row<NF, N, 0>(m, k * cn, k * sn, f0, f1);
        km = fma(b, k, km);
        cp = fma(c2, cn, -cp);
        sp = fma(c2, sn, -sp);
        b += h;
        tree_row<NF, N + 1, 0>(m, km * cp, km * sp, f0, f1);
        k = fma(b, km, k);
        cn = fma(c2, cp, -cn);
        sn = fma(c2, sp, -sn);
        tree_rows<NF, N + 2>(order, m, c2, h, b + h, km, k, cp, cn, sp, sn, f0, f1);
    }
}

/* NF fields of one cluster expansion at the lane's target.  K_n
   by the upward recurrence (stable), cos and sin of n theta by theirs; the
   n-th term falls like (R/r)^n, so the growth of their rounding with n does not
   show.  The moments are loaded whole (a row of 16 lanes holds 32 doubles per
   load) while K0 and K1 are formed: reading them order by order through the
   scalar cache left the kernel waiting (its 16 KB serve two CUs). */
template <int NF>
__device__ __forceinline__ void tree_expand(const double *fq, const TreeDev &T, uint32_t c,
                                            int pc, int order, double x, double y, double (&f0)[NF])
{
    constexpr int NL = tr_stride(2 * NF) / 32;
    const double2 *mp = (const double2 *)(T.mom + (int64_t)c * tr_stride(2 * NF)) + (threadIdx.x & 15);
    double2 m[NL];
#pragma unroll
    for (int l = 0; l < NL; ++l) m[l] = mp[16 * l];
    const MHLP_CAS double *cc = (const MHLP_CAS double *)T.cc + 2 * (int64_t)c;
    const FarConst fc = far_const_of(fq);
    const double ex = x - cc[0], ey = y - cc[1];
    double ri, k0, k1;
    tree_k01_pc(pc, fc, fq, fma(ex, ex, ey * ey), ri, k0, k1);
    const double ct = ex * ri, st = ey * ri, h = 2.0 * fc.ia * ri;
    double f1[NF];
#pragma unroll
    for (int f = 0; f < NF; ++f) f0[f] = f1[f] = 0.0;
    tree_row<NF, 0, 0>(m, k0, 0.0, f0, f1);
    tree_rows<NF, 1>(order, m, 2.0 * ct, h, h, k0, k1, 1.0, ct, 0.0, st, f0, f1);
#pragma unroll
    for (int f = 0; f < NF; ++f) f0[f] += f1[f];
}

/* orders N and on of a stresslet expansion: NC complex fields (1: velocity, 2:
   its x and y derivatives) of the K part in f0, f1 (as tree_rows), the power
   part's four products in g.  LAP: the power part alone. */
template <int NC, bool LAP, int N>
__device__ __forceinline__ void tree_stokes_rows(int order, const double2 *m, double c2, double h, double b, double km,
                                                 double k, double cp, double cn, double sp, double sn, double rho,
                                                 double (&f0)[2 * NC], double (&f1)[2 * NC], double (&g)[4])
{
    constexpr int NV = 4 * NC + 2;
    if constexpr (N < TR_ROWS) {
        if (N > order) return;
        const double rc = rho * cn, rs = rho * sn;
        fmac_pair<N * NV + 4 * NC>(g[0], g[1], m, rc, rs);
        fmac_pair<N * NV + 4 * NC, true>(g[2], g[3], m, rc, rs);
        double kn = 0.0;
        if constexpr (!LAP) {
            const double kc = k * cn, ks = k * sn;
            fmac_pair<N * NV>(f0[0], f1[0], m, kc, ks);
            fmac_pair<N * NV + 2>(f0[1], f1[1], m, kc, ks);
            if constexpr (NC == 2) {
                fmac_pair<N * NV + 4>(f0[2], f1[2], m, kc, ks);
                fmac_pair<N * NV + 6>(f0[3], f1[3], m, kc, ks);
            }
            kn = fma(b, k, km);
        }
        tree_stokes_rows<NC, LAP, N + 1>(order, m, c2, h, b + h, k, kn, cn, fma(c2, cn, -cp), sn, fma(c2, sn, -sp),
                                         rho * h, f0, f1, g);
    }
}

/* orders N and on of a TR_SMALL item: K_n - S_n (kt, the next one in kt1) with the
   K part's rows in m, the powers with theirs in ms, into the same sums */
template <int NC, int N>
__device__ __forceinline__ void tree_small_rows(int order, const double2 *m, const double2 *ms, double c2, double h,
                                                double b, double k, double k1, double kt, double kt1, double cp,
                                                double cn, double sp, double sn, double rho, double (&f0)[2 * NC],
                                                double (&f1)[2 * NC])
{
    constexpr int NV = 4 * NC + 2, NS = 4 * NC;
    if constexpr (N < TR_ROWS) {
        if (N > order) return;
        const double kc = kt * cn, ks = kt * sn, rc = rho * cn, rs = rho * sn;
        fmac_pair<N * NV>(f0[0], f1[0], m, kc, ks);
        fmac_pair<N * NV + 2>(f0[1], f1[1], m, kc, ks);
        fmac_pair<N * NS>(f0[0], f1[0], ms, rc, rs);
        fmac_pair<N * NS + 2>(f0[1], f1[1], ms, rc, rs);
        if constexpr (NC == 2) {
            fmac_pair<N * NV + 4>(f0[2], f1[2], m, kc, ks);
            fmac_pair<N * NV + 6>(f0[3], f1[3], m, kc, ks);
            fmac_pair<N * NS + 4>(f0[2], f1[2], ms, rc, rs);
            fmac_pair<N * NS + 6>(f0[3], f1[3], ms, rc, rs);
        }
        /* k, k1: K_N and K_{N+1}; b: 2 (N + 1)/z */
        tree_small_rows<NC, N + 1>(order, m, ms, c2, h, b + h, k1, fma(b, k1, k), kt1, fma(b, kt1, k), cn,
                                   fma(c2, cn, -cp), sn, fma(c2, sn, -sp), rho * h, f0, f1);
    }
}

/* K_0, K_1, K_1 - 1/z and K_2 - 2/z^2 at distance^2 r2.  z <= 2: from the fitted
   smooth parts T1, T3 of the stresslet, z K_1 - 1 = 2 pi z^2 T3 and
   K_2 - 2/z^2 = -1/2 - pi z^2 (T1 + T3), where nothing cancels. */
__device__ __forceinline__ void tree_k_small(const double *fq, double r2, double &ri, double &k0, double &k1, double &kt1,
                                             double &kt2)
{
    const FarTab T = far_table();
    const FarConst fc = far_const_of(fq);
    ri = lean_rsq(r2);
    const double z = fc.a * (r2 * ri), zi = fc.ia * ri, q = fc.a2q * r2;
    if (q <= 1.0) {
        const double lz = fma(0.5, lean_log01(T, q), LN2);
        const double t1 = fma(hornerc<14>(T->stk[3], q), lz, hornerc<14>(T->stk[0], q));
        const double t3 = fma(hornerc<14>(T->stk[5], q), lz, hornerc<14>(T->stk[2], q));
        kt1 = (2.0 * PI * z) * t3;
        kt2 = fma(-PI * (z * z), t1 + t3, -0.5);
        k0 = fma(-4.0 * PI, t3, kt2);
        k1 = zi + kt1;
    } else {
        K01 o, o2;
        k01_far2<true, true, true, true>(T, fc, r2, r2, o, o2);
        k0 = o.k0;
        k1 = o.ak1r * (r2 * ri);
        kt1 = k1 - zi;
        kt2 = fma(2.0 * zi, kt1, k0);
    }
}

template <int NC>
__device__ __forceinline__ void tree_expand_small(const double *fq, const TreeDev &T, uint32_t c, int order, double x,
                                                  double y, double (&f0)[2 * NC])
{
    constexpr int NV = 4 * NC + 2, NS = 4 * NC, NL = tr_stride(NV) / 32, NLS = tr_stride(NS) / 32;
    const double2 *mp = (const double2 *)(T.mom + (int64_t)c * tr_stride(NV)) + (threadIdx.x & 15);
    const double2 *sp = (const double2 *)(T.small + (int64_t)c * tr_stride(NS)) + (threadIdx.x & 15);
    double2 m[NL], ms[NLS];
#pragma unroll
    for (int l = 0; l < NL; ++l) m[l] = mp[16 * l];
#pragma unroll
    for (int l = 0; l < NLS; ++l) ms[l] = sp[16 * l];
    const MHLP_CAS double *cc = (const MHLP_CAS double *)T.cc + 2 * (int64_t)c;
    const double ex = x - cc[0], ey = y - cc[1];
    double ri, k0, k1, kt1, kt2;
    tree_k_small(fq, fma(ex, ex, ey * ey), ri, k0, k1, kt1, kt2);
    const double ct = ex * ri, h = 2.0 * far_const_of(fq).ia * ri;
    double f1[2 * NC];
#pragma unroll
    for (int n = 0; n < 2 * NC; ++n) f0[n] = f1[n] = 0.0;
    fmac_pair<0>(f0[0], f1[0], m, k0, 0.0);
    fmac_pair<2>(f0[1], f1[1], m, k0, 0.0);
    if constexpr (NC == 2) {
        fmac_pair<4>(f0[2], f1[2], m, k0, 0.0);
        fmac_pair<6>(f0[3], f1[3], m, k0, 0.0);
    }
    tree_small_rows<NC, 1>(order, m, ms, 2.0 * ct, h, 2.0 * h, k1, fma(h, k1, k0), kt1, kt2, 1.0, ct, 0.0, ey * ri, h, f0,
                           f1);
#pragma unroll
    for (int n = 0; n < 2 * NC; ++n) f0[n] += f1[n];
    if constexpr (NC == 2) { /* x derivatives of u_1, u_2, then y: to d_1 u_1, d_2 u_1, d_1 u_2, d_2 u_2 */
        const double t = f0[1];
        f0[1] = f0[2];
        f0[2] = t;
    }
}

/* a cluster's stresslet field (NC = 1: u_1, u_2) or its gradient (NC = 2:
   d_1 u_1, d_2 u_1, d_1 u_2, d_2 u_2), times 2 pi */
template <int NC>
__device__ __forceinline__ void tree_expand_stokes(const double *fq, const TreeDev &T, uint32_t c,
                                                   uint32_t fl, int order, double x, double y, double (&f)[2 * NC])
{
    constexpr int NV = 4 * NC + 2, NL = tr_stride(NV) / 32;
    const double2 *mp = (const double2 *)(T.mom + (int64_t)c * tr_stride(NV)) + (threadIdx.x & 15);
    double2 m[NL];
#pragma unroll
    for (int l = 0; l < NL; ++l) m[l] = mp[16 * l];
    const MHLP_CAS double *cc = (const MHLP_CAS double *)T.cc + 2 * (int64_t)c;
    const FarConst fc = far_const_of(fq);
    const double ex = x - cc[0], ey = y - cc[1], r2 = fma(ex, ex, ey * ey);
    double f0[2 * NC], f1[2 * NC], g[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int n = 0; n < 2 * NC; ++n) f0[n] = f1[n] = 0.0;
    if (fl & TR_LAP) {
        const double ri = lean_rsq(r2), ct = ex * ri, h = 2.0 * fc.ia * ri;
        tree_stokes_rows<NC, true, 1>(order, m, 2.0 * ct, h, 0.0, 0.0, 0.0, 1.0, ct, 0.0, ey * ri, h, f0, f1, g);
    } else {
        double ri, k0, k1;
        tree_k01_pc((int)(fl & 31) - 1, fc, fq, r2, ri, k0, k1);
        const double ct = ex * ri, h = 2.0 * fc.ia * ri;
        /* row 0 has no sine: its second values are zero */
        fmac_pair<0>(f0[0], f1[0], m, k0, 0.0);
        fmac_pair<2>(f0[1], f1[1], m, k0, 0.0);
        if constexpr (NC == 2) {
            fmac_pair<4>(f0[2], f1[2], m, k0, 0.0);
            fmac_pair<6>(f0[3], f1[3], m, k0, 0.0);
        }
        tree_stokes_rows<NC, false, 1>(order, m, 2.0 * ct, h, h, k0, k1, 1.0, ct, 0.0, ey * ri, h, f0, f1, g);
    }
    const double gr = g[0] - g[1], gi = g[2] + g[3];
    if constexpr (NC == 1) {
        f[0] = f0[0] + f1[0] + gr;
        f[1] = f0[1] + f1[1] + gi;
    } else {
        f[0] = f0[0] + f1[0] + gr;
        f[2] = f0[1] + f1[1] + gi;
        f[1] = f0[2] + f1[2] + gi;
        f[3] = f0[3] + f1[3] - gr;
    }
}

/* the density that far_density gives, from scalar registers */
__device__ __forceinline__ const double *tree_density(const FarArgs &A)
{
    return A.gs ? A.mu + (int64_t)__builtin_amdgcn_readfirstlane(A.gs->j) * A.jstride : A.mu;
}

/* Charges and dipoles of panel p for the direct pairs: staged by the moments
   kernel, or, RAW, formed where they are read, with the same roundings (small
   plans without expansions: a launch less; 1 to 4 multiplications a source and
   lane more).  GRAD: the charges carry alpha. */
template <bool SLP, bool DLP, bool GRAD, bool RAW>
struct TreeSrc {
    const MHLP_CAS double *st, *w, *sg, *mu, *nx, *ny;
    double alpha;
    __device__ __forceinline__ TreeSrc(const FarArgs &A, const TreeDev &D, int64_t p)
    {
        if constexpr (RAW) {
            w = (const MHLP_CAS double *)A.sw + 16 * p;
            sg = (const MHLP_CAS double *)A.sigma + 16 * p;
            if (DLP) mu = (const MHLP_CAS double *)tree_density(A) + 16 * p;
            nx = (const MHLP_CAS double *)A.snx + 16 * p;
            ny = (const MHLP_CAS double *)A.sny + 16 * p;
            alpha = A.alpha;
        } else {
            st = (const MHLP_CAS double *)D.st + 48 * p;
        }
    }
    __device__ __forceinline__ double q(int s) const
    {
        if constexpr (!RAW) return st[s];
        else if constexpr (GRAD) return alpha * (w[s] * sg[s]);
        else return w[s] * sg[s];
    }
    __device__ __forceinline__ void d(int s, double &dx, double &dy) const
    {
        if constexpr (!RAW) {
            dx = st[16 + s];
            dy = st[32 + s];
        } else {
            const double m = (alpha * w[s]) * mu[s];
            dx = m * nx[s];
            dy = m * ny[s];
        }
    }
};

/* whether a charge or dipole of the cluster is infinite or NaN */
template <bool SLP, bool DLP, bool RAW>
__device__ __forceinline__ bool tree_bad(const FarArgs &A, const TreeDev &T, int64_t p0, int64_t p1)
{
    double s = 0.0;
    for (int64_t j = 16 * p0 + (threadIdx.x & 63); j < 16 * p1; j += 64) {
        if constexpr (RAW) {
            if (SLP) s = fma(0.0, A.sw[j] * A.sigma[j], s);
            if (DLP) {
                const double m = (A.alpha * A.sw[j]) * tree_density(A)[j];
                s = fma(0.0, m * A.snx[j], fma(0.0, m * A.sny[j], s));
            }
        } else {
            const double *q = T.st + (j >> 4) * 48 + (j & 15);
            if (SLP) s = fma(0.0, q[0], s);
            if (DLP) s = fma(0.0, q[16], fma(0.0, q[32], s));
        }
    }
    return __ballot(!(s == 0.0)) != 0;
}

/* What a far sum evaluates.  NF fields, EXTRA orders beyond the list's, blocks
   of up to WMAX waves;
   panel<PC>: staged sources s0..s1-1 of panel p against the lane's target in
   piece PC (-1: z <= 2; KQ_NP: per pair), added to f (sources come through the
   scalar cache, two at a time); near: the correction of node jj of the listed
   pair q; store: field f of target i, common what every store of a wave shares.  The sums
   carry no 1/(2 pi) until they leave the wave. */
template <bool SLP, bool DLP, bool RAW = false>
struct TreePot {
    static constexpr int NF = (SLP ? 1 : 0) + (DLP ? 1 : 0), EXTRA = 0, WMAX = 16;
    static constexpr bool SKIP = !RAW; /* tree_moments_kernel leaves the bounds that takes */
    template <int PC>
    static __device__ __forceinline__ void panel(const FarArgs &A, const TreeDev &D, int64_t p,
                                                 int s0, int s1, double x, double y, double (&f)[NF])
    {
        constexpr int K = PC < 0 || PC >= KQ_NP ? 0 : PC;
        const MHLP_CAS double *sx = (const MHLP_CAS double *)A.sx + 16 * p;
        const MHLP_CAS double *sy = (const MHLP_CAS double *)A.sy + 16 * p;
        const TreeSrc<SLP, DLP, false, RAW> src(A, D, p);
        FarTab T = far_table();
        const FarConst fc = far_const_of(A.fq);
        double qa, qk;
        fine_q<K>(A.fq, qa, qk);
#pragma unroll 1
        for (int s = s0; s < s1; s += 2) {
            if (PC < 0 || PC >= KQ_NP) T = far_table(); /* their coefficients exceed the scalar registers */
            const double ex0 = x - sx[s], ey0 = y - sy[s];
            const double ex1 = x - sx[s + 1], ey1 = y - sy[s + 1];
            const double r20 = fma(ex0, ex0, ey0 * ey0), r21 = fma(ex1, ex1, ey1 * ey1);
            K01 o0, o1;
            if constexpr (PC >= KQ_NP)
                k01_far2<SLP, DLP, true, true>(T, fc, r20, r21, o0, o1);
            else
                k01_far2_fixed<SLP, DLP, PC>(T, fc, qa, qk, r20, r21, o0, o1);
            if (SLP) f[0] = fma(o1.k0, src.q(s + 1), fma(o0.k0, src.q(s), f[0]));
            if (DLP) {
                double dx0, dy0, dx1, dy1;
                src.d(s, dx0, dy0);
                src.d(s + 1, dx1, dy1);
                f[NF - 1] = fma(o1.ak1r, fma(ex1, dx1, ey1 * dy1), fma(o0.ak1r, fma(ex0, dx0, ey0 * dy0), f[NF - 1]));
            }
        }
    }
    static __device__ __forceinline__ void near(const FarArgs &A, const double *mu, int64_t q, int64_t p, int jj,
                                                double (&n)[NF])
    {
        if (SLP) n[0] = fma(A.wsl[16 * q + jj], A.sigma[16 * p + jj], n[0]);
        if (DLP) n[NF - 1] = fma(A.wdl[16 * q + jj], mu[16 * p + jj], n[NF - 1]);
    }
    static __device__ __forceinline__ void store(const FarArgs &A, double, const double *mu, int64_t i, int f,
                                                 double v)
    {
        const int64_t o = A.perm ? (int64_t)A.perm[i] : i;
        if (SLP && f == 0) {
            A.us[o] = v;
        } else {
            if (A.half_term != 0.0) v = fma(A.half_term, mu[i], v);
            A.ud[o] = v;
        }
    }
    static __device__ __forceinline__ bool bad(const FarArgs &A, const TreeDev &T, int64_t p0, int64_t p1)
    {
        return tree_bad<SLP, DLP, RAW>(A, T, p0, p1);
    }
    static __device__ __forceinline__ double common(const FarArgs &, const TreeDev &) { return 0.0; }
    static __device__ __forceinline__ void expand(const double *fq, const TreeDev &T, uint32_t c,
                                                  uint32_t fl, double x, double y, double (&f)[NF])
    {
        tree_expand<NF>(fq, T, c, (int)(fl & 31) - 1, ((int)(fl >> 8) & 63) + EXTRA, x, y, f);
    }
};

/* the target gradients: d_x S, d_y S, d_x D, d_y D (without the absent layer's) */
template <bool SLP, bool DLP, bool RAW = false>
struct TreeGrad {
    static constexpr int NF = (SLP ? 2 : 0) + (DLP ? 2 : 0), EXTRA = TR_GRAD, WMAX = 16;
    static constexpr bool SKIP = false;
    template <int PC>
    static __device__ __forceinline__ void panel(const FarArgs &A, const TreeDev &D, int64_t p,
                                                 int s0, int s1, double x, double y, double (&f)[NF])
    {
        constexpr int K = PC < 0 || PC >= KQ_NP ? 0 : PC;
        const MHLP_CAS double *sx = (const MHLP_CAS double *)A.sx + 16 * p;
        const MHLP_CAS double *sy = (const MHLP_CAS double *)A.sy + 16 * p;
        const TreeSrc<SLP, DLP, true, RAW> src(A, D, p);
        FarTab T = far_table();
        const FarConst fc = far_const_of(A.fq);
        double qa, qk;
        fine_q<K>(A.fq, qa, qk);
#pragma unroll 1
        for (int s = s0; s < s1; s += 2) {
            if (PC < 0 || PC >= KQ_NP) T = far_table(); /* their coefficients exceed the scalar registers */
            const double ex0 = x - sx[s], ey0 = y - sy[s];
            const double ex1 = x - sx[s + 1], ey1 = y - sy[s + 1];
            const double r20 = fma(ex0, ex0, ey0 * ey0), r21 = fma(ex1, ex1, ey1 * ey1);
            K01 o0, o1; /* ak1r holds K1(z)/r; the staged charges and dipoles carry alpha */
            if constexpr (PC >= KQ_NP)
                k01_far2<DLP, true, true, true>(T, fc, r20, r21, o0, o1);
            else
                k01_far2_fixed<DLP, true, PC>(T, fc, qa, qk, r20, r21, o0, o1);
            if (SLP) {
                const double c0 = o0.ak1r * src.q(s), c1 = o1.ak1r * src.q(s + 1);
                f[0] = fma(-c1, ex1, fma(-c0, ex0, f[0]));
                f[1] = fma(-c1, ey1, fma(-c0, ey0, f[1]));
            }
            if (DLP) {
                /* (alpha^2 K0 + 2 alpha K1/r) (x-y).d / r^2, alpha from the dipole */
                double dx0, dy0, dx1, dy1;
                src.d(s, dx0, dy0);
                src.d(s + 1, dx1, dy1);
                const double n0 = fma(ex0, dx0, ey0 * dy0);
                const double n1 = fma(ex1, dx1, ey1 * dy1);
                const double b0 = n0 * fma(A.alpha, o0.k0, 2.0 * o0.ak1r) * o0.ri2;
                const double b1 = n1 * fma(A.alpha, o1.k0, 2.0 * o1.ak1r) * o1.ri2;
                double &gx = f[NF - 2], &gy = f[NF - 1];
                gx = fma(-b1, ex1, fma(o1.ak1r, dx1, fma(-b0, ex0, fma(o0.ak1r, dx0, gx))));
                gy = fma(-b1, ey1, fma(o1.ak1r, dy1, fma(-b0, ey0, fma(o0.ak1r, dy0, gy))));
            }
        }
    }
    static __device__ __forceinline__ void near(const FarArgs &A, const double *mu, int64_t q, int64_t p, int jj,
                                                double (&n)[NF])
    {
        const int64_t o = 16 * q + jj, block = 16 * A.nnz;
        if (SLP) {
            const double sg = A.sigma[16 * p + jj];
            n[0] = fma(A.wg[o], sg, n[0]);
            n[1] = fma(A.wg[block + o], sg, n[1]);
        }
        if (DLP) {
            const double m = mu[16 * p + jj];
            n[NF - 2] = fma(A.wg[2 * block + o], m, n[NF - 2]);
            n[NF - 1] = fma(A.wg[3 * block + o], m, n[NF - 1]);
        }
    }
    static __device__ __forceinline__ void store(const FarArgs &A, double, const double *, int64_t i, int f,
                                                 double v)
    {
        A.gout[SLP ? f : f + 2][A.perm ? (int64_t)A.perm[i] : i] = v;
    }
    static __device__ __forceinline__ bool bad(const FarArgs &A, const TreeDev &T, int64_t p0, int64_t p1)
    {
        return tree_bad<SLP, DLP, RAW>(A, T, p0, p1);
    }
    static __device__ __forceinline__ double common(const FarArgs &, const TreeDev &) { return 0.0; }
    static __device__ __forceinline__ void expand(const double *fq, const TreeDev &T, uint32_t c,
                                                  uint32_t fl, double x, double y, double (&f)[NF])
    {
        tree_expand<NF>(fq, T, c, (int)(fl & 31) - 1, ((int)(fl >> 8) & 63) + EXTRA, x, y, f);
    }
};

/* the stresslet double layer, and with GRAD its target gradient; SMALL: for plans
   with TR_SMALL items (their rows take registers that the others need not pay for);
   RAW as in TreeSrc */
template <bool GRAD, bool SMALL, bool RAW = false>
struct TreeStokes {
    /* the gradient and SMALL need more than the 128 registers of a 16-wave block */
    static constexpr int NF = GRAD ? 4 : 2, WMAX = GRAD || SMALL ? 8 : 16;
    static constexpr bool SKIP = false;
    template <int PC>
    static __device__ __forceinline__ void panel(const FarArgs &A, const TreeDev &D, int64_t p,
                                                 int s0, int s1, double x, double y, double (&f)[NF])
    {
        constexpr int K = PC < 0 || PC >= KQ_NP ? 0 : PC;
        const MHLP_CAS double *sx = (const MHLP_CAS double *)A.sx + 16 * p;
        const MHLP_CAS double *sy = (const MHLP_CAS double *)A.sy + 16 * p;
        const MHLP_CAS double *snx = (const MHLP_CAS double *)A.snx + 16 * p;
        const MHLP_CAS double *sny = (const MHLP_CAS double *)A.sny + 16 * p;
        const MHLP_CAS double *st = (const MHLP_CAS double *)D.st + 48 * p;
        const MHLP_CAS double *w = (const MHLP_CAS double *)A.sw + 16 * p;
        const MHLP_CAS double *mu = (const MHLP_CAS double *)tree_density(A) + 16 * p;
        FarTab T = far_table();
        const FarConst fc = far_const_of(A.fq);
        double qa, qk, al2, ial2;
        far_squares_of(A.fq, al2, ial2);
        fine_q<K>(A.fq, qa, qk);
        double a[NF];
#pragma unroll
        for (int n = 0; n < NF; ++n) a[n] = 0.0;
#pragma unroll 1
        for (int s = s0; s < s1; s += 2) {
            if (PC < 0 || PC >= KQ_NP) T = far_table(); /* their coefficients exceed the scalar registers */
            const double ex[2] = {x - sx[s], x - sx[s + 1]}, ey[2] = {y - sy[s], y - sy[s + 1]};
            const double r20 = fma(ex[0], ex[0], ey[0] * ey[0]), r21 = fma(ex[1], ex[1], ey[1] * ey[1]);
            double Ak[2][3], Bk[2][3];
            if constexpr (GRAD)
                stk_far2_ab_pc<PC>(T, fc, qa, qk, al2, ial2, r20, r21, Ak[0], Bk[0], Ak[1], Bk[1]);
            else
                stk_far2_pc<PC>(T, fc, qa, qk, al2, ial2, r20, r21, Ak[0], Ak[1]);
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                const double nx = snx[s + u], ny = sny[s + u];
                const double m1 = RAW ? w[s + u] * mu[s + u] : st[s + u];
                const double m2 = RAW ? w[s + u] * mu[A.N + s + u] : st[16 + s + u];
                const double *A_ = Ak[u];
                const double rn = fma(ex[u], nx, ey[u] * ny);
                const double rm = fma(ex[u], m1, ey[u] * m2);
                const double nm = fma(nx, m1, ny * m2);
                if constexpr (!GRAD) {
                    const double c = fma(A_[1] * rm, rn, A_[2] * nm);
                    a[0] -= fma(A_[0], fma(nx, rm, fma(ex[u], nm, m1 * rn)), c * ex[u]);
                    a[1] -= fma(A_[0], fma(ny, rm, fma(ey[u], nm, m2 * rn)), c * ey[u]);
                } else {
                    const double *b = Bk[u];
                    const double sr = fma(b[1] * rn, rm, (b[0] + b[2]) * nm);
                    const double p1 = fma(b[0], fma(nx, rm, m1 * rn), ex[u] * sr);
                    const double p2 = fma(b[0], fma(ny, rm, m2 * rn), ey[u] * sr);
                    const double a1 = fma(A_[0], m1, A_[1] * rm * ex[u]), a2 = fma(A_[0], m2, A_[1] * rm * ey[u]);
                    const double c1 = fma(A_[0], nx, A_[1] * rn * ex[u]), c2 = fma(A_[0], ny, A_[1] * rn * ey[u]);
                    const double d = fma(A_[0] + A_[2], nm, A_[1] * rn * rm);
                    a[0] -= fma(ex[u], p1, fma(nx, a1, fma(m1, c1, d)));
                    a[1] -= fma(ey[u], p1, fma(ny, a1, m2 * c1));
                    a[2] -= fma(ex[u], p2, fma(nx, a2, m1 * c2));
                    a[3] -= fma(ey[u], p2, fma(ny, a2, fma(m2, c2, d)));
                }
            }
        }
#pragma unroll
        for (int n = 0; n < NF; ++n) f[n] = fma(2.0 * PI, a[n], f[n]);
    }
    static __device__ __forceinline__ void expand(const double *fq, const TreeDev &T, uint32_t c,
                                                  uint32_t fl, double x, double y, double (&f)[NF])
    {
        const int order = ((int)(fl >> 8) & 63) + (GRAD ? TR_SGRAD : 0);
        if (SMALL && fl & TR_SMALL)
            tree_expand_small<NF / 2>(fq, T, c, order, x, y, f);
        else
            tree_expand_stokes<NF / 2>(fq, T, c, fl, order, x, y, f);
    }
    static __device__ __forceinline__ void near(const FarArgs &A, const double *mu, int64_t q, int64_t p, int jj,
                                                double (&n)[NF])
    {
        /* blocks of [nnz][16]: D11 D12 D21 D22, or d_l u_i per mu_j at (2 i + l) 2 + j */
        const double m1 = mu[16 * p + jj], m2 = mu[A.N + 16 * p + jj];
        const int64_t block = 16 * A.nnz;
        const double *w = A.wg + 16 * q + jj;
#pragma unroll
        for (int k = 0; k < NF; ++k) n[k] = fma(w[2 * k * block], m1, fma(w[(2 * k + 1) * block], m2, n[k]));
    }
    /* sum of the panels' fluxes over |Gamma|, the same in every lane of the (whole) wave */
    static __device__ __forceinline__ double common(const FarArgs &A, const TreeDev &T)
    {
        if (GRAD || A.half_term == 0.0) return 0.0;
        double s = 0.0;
        for (int64_t p = threadIdx.x & 63; p < T.Np; p += 64) s += T.flux[p];
        return wave_sum_dpp(s) * A.inv_len;
    }
    static __device__ __forceinline__ void store(const FarArgs &A, double flux, const double *mu, int64_t i, int f,
                                                 double v)
    {
        /* on-surface operator: + 1/2 mu + n flux/|Gamma| */
        if (!GRAD && A.half_term != 0.0) v = fma(A.half_term, mu[f * A.N + i], fma((f ? A.sny : A.snx)[i], flux, v));
        A.gout[f][A.perm ? (int64_t)A.perm[i] : i] = v;
    }
    static __device__ __forceinline__ bool bad(const FarArgs &, const TreeDev &, int64_t, int64_t) { return false; }
};

template <class Op, class Args>
__device__ __forceinline__ void tree_panel(int pc, const Args &A, const TreeDev &T, int64_t p,
                                           int s0, int s1, double x, double y, double (&f)[Op::NF])
{
    switch (pc) {
#define MHLP_TREE_PANEL(PCV) \
    case PCV: Op::template panel<PCV>(A, T, p, s0, s1, x, y, f); break;
        MHLP_PC_CASES(MHLP_TREE_PANEL)
#undef MHLP_TREE_PANEL
    default: Op::template panel<KQ_NP>(A, T, p, s0, s1, x, y, f);
    }
}


/* sum over the 16 lanes of a row, in all of them */
__device__ __forceinline__ double tree_row_sum(double v)
{
#define MHLP_ROR(N)                                                                                                  \
    v += __hiloint2double(__builtin_amdgcn_update_dpp(0, __double2hiint(v), 0x120 + N, 0xf, 0xf, true),              \
                          __builtin_amdgcn_update_dpp(0, __double2loint(v), 0x120 + N, 0xf, 0xf, true));
    MHLP_ROR(8) MHLP_ROR(4) MHLP_ROR(2) MHLP_ROR(1)
#undef MHLP_ROR
    return v;
}

/* One block per group of 64 targets (lane = target), in the order of the
   groups' work; the waves of the gridDim.y blocks of a group share its items:
   direct ones in units of 16 / 2^cut sources in turn, expansions in equal
   runs, starting from the other end, so that no wave gets more than its share
   of both, and the near corrections by node.  The wave sums are added
   in wave order; with several blocks a group each leaves them
   in its slot, and the last one to arrive adds the slots in order: a launch of
   its own for that took 4 us (64 targets, 256 sources: 15 -> 11 us a call in
   all).  A cluster whose expansion is not finite (an infinite or NaN
   density), or whose pairs all underflow with such a density, is summed
   directly, pair by pair.

   Bound by VALU FP64 (109,314 targets, 4096 sources, alpha = 5: 15.6e3
   instructions per group against 304e3 for the direct sum of all pairs, 66 us
   against 1.07 ms; alpha = 500, all pairs direct: within 5% of the issue rate before items were
   left out).
   Far items that cannot show (plans with a large spread of z; off the curve one
   block a group makes both passes, on it, where groups are few, each pass is a
   launch of split groups): the items of the TR_ZNEAR + 1 nearest z classes are summed first;
   with the smallest |u| of the group's targets so far in hand, an item is left
   out when the bound of its charges times e^-z stays below 2^-55 |u| over the
   number of items, so that all that is left out stays below 2^-55 of the nearest
   classes' sum at every target, whose own rounding is larger.  Where that sum
   is small (cancellation) or not finite, the item is summed.
   109,314 x 4096, alpha = 100 / 200 / 500 / 1000, both layers: 370 / 964 / 735 /
   272 -> 233 / 365 / 239 / 142 us.
   Waves per group (tree_shape): four for many groups; up to 512 for few, where
   the longest wave (a direct panel in one wave takes about 20 us) sets the time. */
enum TreePass { TREE_ALL, TREE_BOTH, TREE_NEAREST, TREE_REST }; /* every item; those that show: in two passes, or the first, the second */

template <class Op, TreePass PASS>
__global__ __launch_bounds__(64 * Op::WMAX) void far_tree_kernel(FarArgs A, TreeDev T)
{
    constexpr int NF = Op::NF;
    constexpr bool SKIP = PASS != TREE_ALL;
    __shared__ double red[NF][Op::WMAX][64];
    const double *mu;
    if (!far_density(A, mu)) return;
    const int lane = threadIdx.x & 63, waves = blockDim.x >> 6;
    int W = waves; /* sums of a field in red */
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t g = T.order[blockIdx.x];
    const int64_t i = 64 * g + lane;
    const bool valid = i < A.M;
    const int64_t iv = valid ? i : A.M - 1; /* lanes past the last target repeat it, as in the lists */
    const double x = A.tx[iv], y = A.ty[iv];
    const int32_t k0 = A.nptr[iv], k1 = A.nptr[iv + 1];
    const int NW = W * gridDim.y, wg = w * gridDim.y + blockIdx.y;
    const int2 cnt = T.cnt[g];
    const longlong2 at = T.at[g];
    const uint2 *items = T.items + at.x, *back = T.items + at.y - 1;
    double acc[NF];
#pragma unroll
    for (int f = 0; f < NF; ++f) acc[f] = 0.0;
    /* the wave's sums, with its share of the near corrections, into LDS */
    auto put = [&]() {
        double nr[NF];
#pragma unroll
        for (int f = 0; f < NF; ++f) nr[f] = 0.0;
        if (PASS != TREE_REST && wg < 16)
            for (int32_t q = k0; q < k1; ++q) {
                const int64_t p = A.npan[q];
                if (p < 0) continue;
                for (int jj = wg; jj < 16; jj += NW) Op::near(A, mu, q, p, jj, nr);
            }
#pragma unroll
        for (int f = 0; f < NF; ++f) red[f][w][lane] = fma(INV_2PI, acc[f], nr[f]);
    };
    const int nsrc = 16 >> T.cut;
    const uint32_t znear = SKIP ? (uint32_t)(T.znear[g] + TR_ZNEAR) : 255u;
    float room = -INFINITY;
    /* log2 of what an item may add to field sums s of the group's targets without showing */
    auto room_of = [&](double s) {
        s = __builtin_isfinite(s) ? fabs(s) : 0.0; /* beside a NaN or an infinity nothing is left out */
        for (int o = 32; o > 0; o >>= 1) s = fmin(s, __shfl_xor(s, o));
        return (float)log2(s) - 55.0f - log2f((float)(cnt.x + cnt.y));
    };
    if constexpr (PASS == TREE_REST) {
        room = INFINITY;
        for (int f = 0; f < NF; ++f) room = fminf(room, T.room[g * NF + f]);
        room = __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(room)));
    }
#pragma unroll 1
    for (int pass = PASS == TREE_REST; pass < (PASS == TREE_BOTH || PASS == TREE_REST ? 2 : 1); ++pass) {
        if (PASS == TREE_BOTH && pass == 1) {
            put();
            __syncthreads();
            room = INFINITY;
#pragma unroll
            for (int f = 0; f < NF; ++f) {
                double s = 0.0;
                for (int v = 0; v < W; ++v) s += red[f][v][lane];
                room = fminf(room, room_of(s));
            }
            room = __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(room)));
            __syncthreads();
        }
        auto direct_item = [&](int k, uint32_t p, uint32_t fl) {
            const int s0 = (k & ((1 << T.cut) - 1)) * nsrc;
            bool listed = false;
            if (fl & TR_NEAR)
                for (int32_t q = k0; q < k1; ++q) listed = listed || A.npan[q] == (int32_t)p;
            if (listed) return;
            double f[NF];
#pragma unroll
            for (int n = 0; n < NF; ++n) f[n] = 0.0;
            tree_panel<Op>((int)(fl & 31) - 1, A, T, p, s0, s0 + nsrc, x, y, f);
#pragma unroll
            for (int n = 0; n < NF; ++n) acc[n] += f[n];
        };
        auto far_item = [&](uint32_t c, uint32_t fl) {
            double f[NF];
            bool direct = false;
            if (fl & TR_ZERO) {
#pragma unroll
                for (int n = 0; n < NF; ++n) f[n] = 0.0;
                int64_t p0, p1;
                tree_panels_of(T, c, p0, p1);
                direct = Op::bad(A, T, p0, p1);
            } else {
                Op::expand(A.fq, T, c, fl, x, y, f);
                bool fin = true;
#pragma unroll
                for (int n = 0; n < NF; ++n) fin = fin && __builtin_isfinite(f[n]);
                direct = __ballot(!fin) != 0;
            }
            if (direct) {
#pragma unroll
                for (int n = 0; n < NF; ++n) f[n] = 0.0;
                int64_t p0, p1;
                tree_panels_of(T, c, p0, p1);
                for (int64_t p = p0; p < p1; ++p) Op::template panel<KQ_NP>(A, T, p, 0, 16, x, y, f);
            }
#pragma unroll
            for (int n = 0; n < NF; ++n) acc[n] += f[n];
        };
        const int ndir = cnt.x << T.cut;
        const int fb = cnt.y * (NW - 1 - wg) / NW, fe = cnt.y * (NW - wg) / NW;
        if constexpr (SKIP) {
            /* a lane's item; false: left to the other pass, or too small to show: K1(z) <= e^-z from z = 4 on */
            auto take = [&](uint2 it) {
                const uint32_t zc = it.y >> 24;
                if (pass == 0) return zc <= znear;
                if (zc <= znear) return false;
                return zc == 0 || !(T.lb[it.x] - (float)(TR_ZSTEP * 1.4426950) * (float)zc <= room);
            };
            /* the wave's items come 64 at a time, one a lane */
            for (int kb = wg; kb < ndir; kb += 64 * NW) {
                const int kl = kb + lane * NW;
                const uint2 it = items[min(kl, ndir - 1) >> T.cut];
                for (uint64_t todo = __ballot(kl < ndir && take(it)); todo; todo &= todo - 1) {
                    const int b = __builtin_ctzll(todo);
                    direct_item(kb + b * NW, __builtin_amdgcn_readlane(it.x, b), __builtin_amdgcn_readlane(it.y, b));
                }
            }
            for (int kb = fb; kb < fe; kb += 64) {
                const uint2 it = back[-min(kb + lane, fe - 1)];
                for (uint64_t todo = __ballot(kb + lane < fe && take(it)); todo; todo &= todo - 1) {
                    const int b = __builtin_ctzll(todo);
                    far_item(__builtin_amdgcn_readlane(it.x, b), __builtin_amdgcn_readlane(it.y, b));
                }
            }
        } else {
            for (int k = wg; k < ndir; k += NW) {
                const uint2 it = items[k >> T.cut];
                direct_item(k, __builtin_amdgcn_readfirstlane(it.x), __builtin_amdgcn_readfirstlane(it.y));
            }
            for (int k = fb; k < fe; ++k) {
                const uint2 it = back[-k];
                far_item(__builtin_amdgcn_readfirstlane(it.x), __builtin_amdgcn_readfirstlane(it.y));
            }
        }
    }
    put();
    const int split = gridDim.y;
    if (split > 1) {
        __shared__ bool last;
        __syncthreads();
        double *part = T.part + g * split * NF * 64 + lane;
        for (int f = w; f < NF; f += W) {
            double s = 0.0;
            for (int v = 0; v < W; ++v) s += red[f][v][lane];
            __hip_atomic_store(part + (blockIdx.y * NF + f) * 64, s, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        /* the slots go through device-scope stores, which reach the memory that
           all XCDs share; they have arrived once they are waited for */
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
        if (threadIdx.x == 0) last = atomicInc(T.arrived + g, (uint32_t)split - 1) == (uint32_t)split - 1;
        __syncthreads();
        if (!last) return;
        /* the waves share the slots of the fields, as many sums for a field
           whatever NF, so that one alone gets the bits it has beside others */
        const int H = W > 1 ? W / 2 : 1;
        for (int t = w; t < NF * H; t += W) {
            const int f = t % NF, h = t / NF;
            double s = 0.0;
#pragma unroll 4
            for (int k = h; k < split; k += H)
                s += __hip_atomic_load(part + (k * NF + f) * 64, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            red[f][h][lane] = s;
        }
        W = H;
    }
    if constexpr (PASS == TREE_NEAREST) {
        __syncthreads();
        for (int f = w; f < NF; f += waves) {
            double s = 0.0;
            for (int v = 0; v < W; ++v) s += red[f][v][lane];
            T.base[(g * NF + f) * 64 + lane] = s;
            const float r = room_of(s);
            if (lane == 0) T.room[g * NF + f] = r;
        }
        return;
    }
    const double cm = Op::common(A, T); /* every lane takes part */
    __syncthreads();
    if (!valid) return;
    for (int f = w; f < NF; f += waves) {
        double s = 0.0;
        for (int v = 0; v < W; ++v) s += red[f][v][lane];
        if constexpr (PASS == TREE_REST) s += T.base[(g * NF + f) * 64 + lane];
        Op::store(A, cm, mu, i, f, s);
    }
}

} // namespace mhlp
