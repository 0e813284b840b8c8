/* The FP64 volume sum by cluster expansions, built anew for every call: the
   points are sorted along a Hilbert curve into panels of 16, runs of 1-16 panels
   are the clusters of tree.h (their moments and expansions are the single
   layer's), and a block per 64 sorted points lists in LDS, 256 runs of 16 panels
   at a time, what it takes through an expansion and what pair by pair. */
#pragma once

namespace mhlp {

constexpr int VT_TILES = 128;  /* tiles of the sort at most */
constexpr int VT_BOXES = 64;   /* partial bounding boxes */
constexpr int VT_BATCH = 256;  /* runs of 16 panels listed at a time */
constexpr int VT_BINS = 64;    /* bins of alpha R, three to an octave from 2^-20 on */
constexpr int VT_BITS = 11;    /* bits a sort pass takes at most (at least 7) */
/* alpha R of an expansion here: its terms reach e^{2 alpha R} of its value, and
   up to 3 the error stays below that of the plain sum's 10^4 and more roundings
   (65,536 points, alpha = 20: 3e-16 at 2, 4e-16 at 3, plain 7e-15) */
constexpr double VT_AMAX = 3.0;

struct VolSetup {
    double fq[FINE_SCALES];
    float ratio[VT_BINS][TR_NP]; /* tree_order_ratio, the larger of the bin's ends, a percent up */
};

struct VolTree {
    const double *x, *y, *w, *f; /* the caller's points */
    int64_t n;
    int bits;                    /* of a coordinate in the key, and of a sort pass */
    int tile, ntile;             /* points per tile of the sort (a multiple of 64) */
    double alpha, h;
    double *box;                 /* [VT_BOXES][4] partial bounding boxes */
    double *selfc;               /* Wcell / h^2, Wcell */
    VolSetup *setup;
    uint32_t *key[2], *idx[2];   /* [n] */
    uint32_t *hist;              /* [ntile][2^bits] */
    double *xs, *ys, *ws, *fs;   /* sorted, padded to whole panels by the last point with weight 0 */
    double *cbox;                /* [ncl][4] */
    double *u;
};

/* Integral of K0(alpha |x|)/(2 pi) over the h x h cell centred at the origin:
   (1/2pi) 8 int_0^{pi/4} (1 - a K1(a))/alpha^2 dtheta, a = alpha h/(2 cos theta)
   (from int_0^R K0(alpha s) s ds = (1 - alpha R K1(alpha R))/alpha^2);
   composite 32-point Gauss-Legendre on 8 pieces, a node per thread of a block
   of 256, added by a fixed tree: 6 us (398 us on one thread).  The value is
   valid in thread 0. */
__device__ __forceinline__ double self_cell(double alpha, double h, double *red)
{
    const int t = threadIdx.x;
    const double L = 0.25 * PI;
    const double a0 = L * (t >> 5) / 8.0, a1 = L * ((t >> 5) + 1) / 8.0;
    const double mid = 0.5 * (a0 + a1), half = 0.5 * (a1 - a0);
    const double R = 0.5 * h / cos(mid + half * GL32_T[t & 31]);
    const K01 o = k01_fp64<false, true>(R * R, alpha, 0.25 * alpha * alpha, 4.0 / alpha);
    /* o.ak1r = alpha K1(alpha R)/R  =>  alpha R K1 = o.ak1r R^2 */
    red[t] = GL32_W[t & 31] * half * (1.0 - o.ak1r * R * R) / (alpha * alpha);
    __syncthreads();
    for (int s = 128; s > 0; s >>= 1) {
        if (t < s) red[t] += red[t + s];
        __syncthreads();
    }
    return 8.0 * red[0] * INV_2PI;
}

__global__ __launch_bounds__(256) void self_cell_kernel(double alpha, double h, double *out_per_h2, double *out)
{
    __shared__ double red[256];
    const double wc = self_cell(alpha, h, red);
    if (threadIdx.x != 0) return;
    if (out) out[0] = wc;
    if (out_per_h2) out_per_h2[0] = wc / (h * h);
}

/* partial bounding boxes (NaN coordinates do not count); the last block keeps
   the setup and forms the self-cell weight */
__global__ __launch_bounds__(256) void vol_box_kernel(VolTree V, VolSetup S)
{
    __shared__ double red[4][256];
    const int t = threadIdx.x;
    if (blockIdx.x == VT_BOXES) {
        for (int k = t; k < FINE_SCALES; k += 256) V.setup->fq[k] = S.fq[k];
        for (int k = t; k < VT_BINS * TR_NP; k += 256) (&V.setup->ratio[0][0])[k] = (&S.ratio[0][0])[k];
        const double wc = self_cell(V.alpha, V.h, red[0]);
        if (t == 0) {
            V.selfc[0] = wc / (V.h * V.h);
            V.selfc[1] = wc;
        }
        return;
    }
    double b[4] = {INFINITY, -INFINITY, INFINITY, -INFINITY};
    for (int64_t i = blockIdx.x * (int64_t)256 + t; i < V.n; i += 256 * VT_BOXES) {
        b[0] = fmin(b[0], V.x[i]), b[1] = fmax(b[1], V.x[i]);
        b[2] = fmin(b[2], V.y[i]), b[3] = fmax(b[3], V.y[i]);
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) red[k][t] = b[k];
    __syncthreads();
    for (int s = 128; s > 0; s >>= 1) {
        if (t < s)
#pragma unroll
            for (int k = 0; k < 4; ++k)
                red[k][t] = k & 1 ? fmax(red[k][t], red[k][t + s]) : fmin(red[k][t], red[k][t + s]);
        __syncthreads();
    }
    if (t < 4) V.box[4 * blockIdx.x + t] = red[t][0];
}

/* place of a cell along the Hilbert curve (the well-known iteration over the
   bits from the top that takes a quadrant's two bits, then undoes its
   reflection and transposition): unlike Morton order its runs of any
   start and length are connected, so panels and clusters stay compact whatever
   the grid (the figures are at vol_far_kernel) */
__device__ __forceinline__ uint32_t vol_curve(uint32_t x, uint32_t y, int bits)
{
    uint32_t d = 0;
    for (int b = bits - 1; b >= 0; --b) {
        const uint32_t rx = (x >> b) & 1u, ry = (y >> b) & 1u;
        d = d << 2 | ((3u * rx) ^ ry);
        if (ry == 0) { /* the quadrant's curve runs transposed, from the other end when rx */
            const uint32_t m = rx ? (1u << b) - 1u : 0u;
            const uint32_t s = x ^ m;
            x = y ^ m;
            y = s;
        }
    }
    return d;
}

/* digit counts of a tile, one wave; pass 0 forms the keys (a square cell
   of the bounding box; coordinates that are not finite land in some cell) */
template <int PASS>
__global__ __launch_bounds__(64) void vol_hist_kernel(VolTree V)
{
    __shared__ uint32_t cnt[1 << VT_BITS];
    const int lane = threadIdx.x, nb = 1 << V.bits;
    for (int b = lane; b < nb; b += 64) cnt[b] = 0;
    double x0 = 0.0, y0 = 0.0, sc = 0.0;
    if (PASS == 0) {
        double b[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            b[k] = V.box[4 * lane + k];
            for (int o = 32; o > 0; o >>= 1) b[k] = k & 1 ? fmax(b[k], __shfl_xor(b[k], o)) : fmin(b[k], __shfl_xor(b[k], o));
        }
        x0 = b[0];
        y0 = b[2];
        const double side = fmax(b[1] - b[0], b[3] - b[2]);
        sc = side > 0.0 ? nb / side : 0.0;
    }
    __syncthreads();
    const int64_t i0 = (int64_t)blockIdx.x * V.tile, i1 = min(V.n, i0 + V.tile);
    for (int64_t i = i0 + lane; i < i1; i += 64) {
        uint32_t key;
        if (PASS == 0) {
            const double fx = (V.x[i] - x0) * sc, fy = (V.y[i] - y0) * sc;
            const uint32_t qx = fx > 0.0 ? (uint32_t)fmin(fx, nb - 1.0) : 0u;
            const uint32_t qy = fy > 0.0 ? (uint32_t)fmin(fy, nb - 1.0) : 0u;
            key = vol_curve(qx, qy, V.bits);
            V.key[0][i] = key;
        } else {
            key = V.key[1][i] >> V.bits;
        }
        atomicAdd(&cnt[key & (nb - 1)], 1u);
    }
    __syncthreads();
    for (int b = lane; b < nb; b += 64) V.hist[(int64_t)blockIdx.x * nb + b] = cnt[b];
}

/* counts to first positions, digits outermost; one block.  A thread takes four
   neighbouring digits of every GR-th run of tiles, so that the counts come in
   a few wide loads at once: 15 -> 6 us for 128 tiles of 512 digits. */
__global__ __launch_bounds__(1024) void vol_scan_kernel(VolTree V)
{
    __shared__ uint4 part[1024];
    __shared__ uint32_t wsum[16];
    const int t = threadIdx.x, C = 1 << (V.bits - 2), GR = 1024 / C; /* 7 <= bits <= 11 */
    const int col = t & (C - 1), gr = t / C, per = (V.ntile + GR - 1) / GR;
    const int k0 = min(V.ntile, gr * per), k1 = min(V.ntile, k0 + per);
    uint4 *h = (uint4 *)V.hist + col;
    uint4 s = make_uint4(0, 0, 0, 0);
#pragma unroll 16
    for (int k = k0; k < k1; ++k) {
        const uint4 v = h[(int64_t)k * C];
        s.x += v.x, s.y += v.y, s.z += v.z, s.w += v.w;
    }
    part[t] = s;
    __syncthreads();
    uint4 before = make_uint4(0, 0, 0, 0), tot = before; /* of the digits: earlier tiles, all tiles */
    for (int q = 0; q < GR; ++q) {
        const uint4 v = part[q * C + col];
        if (q < gr) before.x += v.x, before.y += v.y, before.z += v.z, before.w += v.w;
        tot.x += v.x, tot.y += v.y, tot.z += v.z, tot.w += v.w;
    }
    const uint32_t mine = gr == 0 ? tot.x + tot.y + tot.z + tot.w : 0u;
    uint32_t inc = mine;
    for (int o = 1; o < 64; o <<= 1) {
        const uint32_t v = __shfl_up(inc, o);
        if ((t & 63) >= o) inc += v;
    }
    if ((t & 63) == 63) wsum[t >> 6] = inc;
    __syncthreads();
    uint32_t at = inc - mine;
    for (int k = 0; k < (t >> 6); ++k) at += wsum[k];
    __syncthreads();
    if (gr == 0) part[col].x = at;
    __syncthreads();
    at = part[col].x;
    uint4 run = make_uint4(at + before.x, at + tot.x + before.y, at + tot.x + tot.y + before.z,
                           at + tot.x + tot.y + tot.z + before.w);
#pragma unroll 16
    for (int k = k0; k < k1; ++k) {
        const uint4 v = h[(int64_t)k * C];
        h[(int64_t)k * C] = run;
        run.x += v.x, run.y += v.y, run.z += v.z, run.w += v.w;
    }
}

/* stable scatter of a tile by its digit, one wave: lanes of equal digit take
   consecutive places in lane order.  Eight rounds' loads are in flight at a
   time.  Pass 1 moves the points themselves. */
template <int PASS>
__global__ __launch_bounds__(64) void vol_scatter_kernel(VolTree V)
{
    constexpr int U = 8;
    __shared__ uint32_t at[1 << VT_BITS];
    const int lane = threadIdx.x, nb = 1 << V.bits;
    for (int b = lane; b < nb; b += 64) at[b] = V.hist[(int64_t)blockIdx.x * nb + b];
    __syncthreads();
    const int64_t i0 = (int64_t)blockIdx.x * V.tile, i1 = min(V.n, i0 + V.tile);
    for (int64_t r = i0; r < i1; r += 64 * U) {
        uint32_t key[U], src[U];
        double x[U], y[U], w[U], f[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t i = min(r + 64 * u + lane, i1 - 1);
            key[u] = V.key[PASS][i];
            src[u] = PASS == 0 ? (uint32_t)i : V.idx[1][i];
        }
        if (PASS == 1)
#pragma unroll
            for (int u = 0; u < U; ++u) x[u] = V.x[src[u]], y[u] = V.y[src[u]], w[u] = V.w[src[u]], f[u] = V.f[src[u]];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const bool have = r + 64 * u + lane < i1;
            const uint32_t d = (PASS == 0 ? key[u] : key[u] >> V.bits) & (nb - 1);
            uint64_t same = __ballot(have);
            for (int b = 0; b < V.bits; ++b) {
                const uint64_t m = __ballot((d >> b) & 1);
                same &= (d >> b) & 1 ? m : ~m;
            }
            const int rank = __popcll(same & ((1ull << lane) - 1ull));
            const uint32_t pos = have ? at[d] + rank : 0u;
            __syncthreads();
            if (have && rank == 0) at[d] += (uint32_t)__popcll(same);
            __syncthreads();
            if (!have) continue;
            if (PASS == 0) {
                V.key[1][pos] = key[u];
                V.idx[1][pos] = src[u];
            } else {
                V.idx[0][pos] = src[u];
                V.xs[pos] = x[u];
                V.ys[pos] = y[u];
                V.ws[pos] = w[u];
                V.fs[pos] = f[u];
                if (pos == V.n - 1)
                    for (int64_t k = V.n; k & 15; ++k) {
                        V.xs[k] = x[u];
                        V.ys[k] = y[u];
                        V.ws[k] = V.fs[k] = 0.0;
                    }
            }
        }
    }
}

/* centre, box and distances of each cluster, one wave per cluster.  A distance
   that never serves is NaN, which no comparison passes, not even that of an
   infinite distance.  A point that is not finite keeps its clusters from every
   expansion and from being left out, and makes their boxes unbounded; a charge
   that is not finite keeps them from being left out where all pairs underflow. */
__global__ __launch_bounds__(256) void vol_clusters_kernel(VolTree V, TreeDev T)
{
    const int64_t c = blockIdx.x * (int64_t)4 + (threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    if (c >= T.ncl) return;
    const int k = tree_level_of(T, c);
    const int64_t p0 = (c - T.off[k]) << k, p1 = min(T.Np, p0 + (1 << k));
    double xl = INFINITY, xh = -INFINITY, yl = INFINITY, yh = -INFINITY;
    bool bad = false, badq = false;
    for (int64_t j = 16 * p0 + lane; j < 16 * p1; j += 64) {
        const double x = V.xs[j], y = V.ys[j];
        xl = fmin(xl, x), xh = fmax(xh, x);
        yl = fmin(yl, y), yh = fmax(yh, y);
        bad = bad || !__builtin_isfinite(x) || !__builtin_isfinite(y);
        badq = badq || !__builtin_isfinite(V.ws[j] * V.fs[j]);
    }
    bad = __ballot(bad) != 0;
    badq = __ballot(badq) != 0;
    for (int o = 32; o > 0; o >>= 1) {
        xl = fmin(xl, __shfl_xor(xl, o)), xh = fmax(xh, __shfl_xor(xh, o));
        yl = fmin(yl, __shfl_xor(yl, o)), yh = fmax(yh, __shfl_xor(yh, o));
    }
    const double cx = 0.5 * xl + 0.5 * xh, cy = 0.5 * yl + 0.5 * yh;
    double R = 0.0;
    for (int64_t j = 16 * p0 + lane; j < 16 * p1; j += 64) R = fmax(R, hypot(V.xs[j] - cx, V.ys[j] - cy));
    for (int o = 32; o > 0; o >>= 1) R = fmax(R, __shfl_xor(R, o));
    R *= 1.0 + 1e-12;
    bad = bad || !__builtin_isfinite(R); /* finite points may lie further apart than a double holds */
    const double a = V.alpha * R;
    if (lane < 2) T.cc[2 * c + lane] = lane ? cy : cx;
    if (lane < 4) V.cbox[4 * c + lane] = bad ? (lane & 1 ? INFINITY : -INFINITY) : lane == 0 ? xl : lane == 1 ? xh : lane == 2 ? yl : yh;
    if (lane < TR_RM) {
        double v = __builtin_nan("");
        if (!bad && lane == TR_RM - 1 && !badq) v = R + TR_ZZERO * (1.0 + 1e-12) / V.alpha;
        if (!bad && lane < TR_NP && a >= TR_AMIN && a <= VT_AMAX) {
            const int bin = (int)(3.0f * (log2f((float)a) + 20.0f));
            v = R * (double)V.setup->ratio[max(0, min(VT_BINS - 1, bin))][lane];
        }
        T.rmin[TR_RM * c + lane] = v;
    }
}

/* pairs of a panel that may hold the lane's own point: coincident points are left out */
__device__ __forceinline__ double vol_self_panel(const FarArgs &A, const TreeDev &D, int64_t p, int s0, int s1,
                                                 double x, double y)
{
    const FarConst fc = far_const_of(A.fq);
    const MHLP_CAS double *sx = (const MHLP_CAS double *)A.sx + 16 * p;
    const MHLP_CAS double *sy = (const MHLP_CAS double *)A.sy + 16 * p;
    const MHLP_CAS double *st = (const MHLP_CAS double *)D.st + 48 * p;
    double f = 0.0;
#pragma unroll 1
    for (int s = s0; s < s1; s += 2) {
        const FarTab T = far_table();
        const double ex0 = x - sx[s], ey0 = y - sy[s], ex1 = x - sx[s + 1], ey1 = y - sy[s + 1];
        double r20 = fma(ex0, ex0, ey0 * ey0), r21 = fma(ex1, ex1, ey1 * ey1);
        const bool self0 = r20 == 0.0, self1 = r21 == 0.0;
        r20 = self0 ? 1.0 : r20;
        r21 = self1 ? 1.0 : r21;
        K01 o0, o1;
        k01_far2<true, false, false>(T, fc, r20, r21, o0, o1);
        f = fma(self1 ? 0.0 : o1.k0, st[s + 1], fma(self0 ? 0.0 : o0.k0, st[s], f));
    }
    return f;
}

/* item: panel of the batch (bits 0-11) | level (12-14) | order's index (15-18) | piece + 1 (19-23) | flags */
constexpr uint32_t VT_FAR = 1u << 24, VT_SELF = 1u << 25;

/* what the points in box b take of the run `top` of 16 panels, in order */
template <class F>
__device__ __forceinline__ void vol_descend(const VolTree &V, const TreeDev &T, const double (&b)[4], int64_t top,
                                            int64_t base, F emit)
{
    const int64_t pe = min(T.Np, 16 * top + 16);
    for (int64_t p = 16 * top; p < pe;) {
        int k = min(T.nlev - 1, __builtin_ctz((uint32_t)p | 16u));
        for (;; --k) {
            const int64_t c = T.off[k] + (p >> k);
            const double cx = T.cc[2 * c], cy = T.cc[2 * c + 1];
            const double dx = fmax(fmax(b[0] - cx, cx - b[1]), 0.0), dy = fmax(fmax(b[2] - cy, cy - b[3]), 0.0);
            const double rlo = sqrt(fma(dx, dx, dy * dy)) * (1.0 - 1e-12);
            const double2 *rm = (const double2 *)(T.rmin + TR_RM * c); /* falls with the order */
            double2 v[TR_RM / 2];
#pragma unroll
            for (int q = 0; q < TR_RM / 2; ++q) v[q] = rm[q];
            if (rlo >= v[TR_RM / 2 - 1].y) break; /* every pair is zero */
            const uint32_t at = (uint32_t)(p - base) | (uint32_t)k << 12;
            uint32_t q = 0;
#pragma unroll
            for (int l = 0; l < TR_NP; ++l) q += rlo >= (l & 1 ? v[l / 2].y : v[l / 2].x) ? 0u : 1u;
            if (q < TR_NP) {
                const double ex = fmax(b[1] - cx, cx - b[0]), ey = fmax(b[3] - cy, cy - b[2]);
                const double rhi = sqrt(fma(ex, ex, ey * ey)) * (1.0 + 1e-12);
                emit(at | q << 15 | (uint32_t)tree_piece(V.alpha * rlo, V.alpha * rhi) << 19 | VT_FAR);
                break;
            }
            if (k > 0) continue;
            const double *pb = V.cbox + 4 * c;
            const double gx = fmax(fmax(b[0] - pb[1], pb[0] - b[1]), 0.0), gy = fmax(fmax(b[2] - pb[3], pb[2] - b[3]), 0.0);
            const double hx = fmax(b[1] - pb[0], pb[1] - b[0]), hy = fmax(b[3] - pb[2], pb[3] - b[2]);
            const double dlo = sqrt(fma(gx, gx, gy * gy)) * (1.0 - 1e-12), dhi = sqrt(fma(hx, hx, hy * hy)) * (1.0 + 1e-12);
            if (dlo > 0.0)
                emit(at | (uint32_t)tree_piece(V.alpha * dlo, V.alpha * dhi) << 19);
            else
                emit(at | VT_SELF);
            break;
        }
        p += (int64_t)1 << k;
    }
}

/* The sums of one group of 64 sorted points.  256 threads list the items of 256
   runs of 16 panels (placed by a scan, so that their order is fixed), then the
   block's waves share them.  Bound by VALU FP64: 65,536 grid points at
   alpha = 20 take 215e3 instructions a group (about 360 expansions of order 27,
   32 panels directly) against 3.5e6 for all pairs, 560 us against 10.4 ms; at
   alpha = 500 all is direct (4.5 ms, in the pieces of the panels' distances).
   In Morton order 182 x 182 points took 1.1 ms, here 0.6. */
__global__ __launch_bounds__(1024) void vol_far_kernel(VolTree V, FarArgs A, TreeDev T)
{
    __shared__ uint32_t items[16 * VT_BATCH];
    __shared__ __align__(8) uint32_t found[16][VT_BATCH]; /* at the end the waves' sums (32 KB in all: four blocks a CU) */
    double(*red)[64] = reinterpret_cast<double(*)[64]>(&found[0][0]);
    __shared__ uint32_t wtot[VT_BATCH / 64];
    const int t = threadIdx.x, lane = t & 63, W = blockDim.x >> 6;
    const int w = __builtin_amdgcn_readfirstlane(t >> 6);
    const int64_t g = blockIdx.x, i = 64 * g + lane;
    const int64_t iv = min(i, V.n - 1);
    const double x = V.xs[iv], y = V.ys[iv];
    double b[4];
    {
        const int64_t c = T.off[2] + g; /* a group is a level-2 cluster */
#pragma unroll
        for (int k = 0; k < 4; ++k) b[k] = V.cbox[4 * c + k];
    }
    const int64_t ntop = (T.Np + 15) >> 4;
    double acc = 0.0;
    for (int64_t t0 = 0; t0 < ntop; t0 += VT_BATCH) {
        const int64_t base = 16 * t0, top = t0 + t;
        const bool mine = t < VT_BATCH && top < ntop;
        uint32_t cnt = 0, inc; /* direct items, expansions << 16 (at most 16 in all) */
        if (mine)
            vol_descend(V, T, b, top, base, [&](uint32_t it) {
                found[(cnt & 0xffffu) + (cnt >> 16)][t] = it;
                cnt += it & VT_FAR ? 0x10000u : 1u;
            });
        inc = cnt;
        for (int o = 1; o < 64; o <<= 1) {
            const uint32_t v = __shfl_up(inc, o);
            if (lane >= o) inc += v;
        }
        __syncthreads(); /* the waves are through with the last batch */
        if (t < VT_BATCH && lane == 63) wtot[w] = inc;
        __syncthreads();
        uint32_t total = 0, before = inc - cnt;
#pragma unroll
        for (int k = 0; k < VT_BATCH / 64; ++k) {
            if (k < w) before += wtot[k];
            total += wtot[k];
        }
        if (mine) {
            uint32_t nd = before & 0xffffu, nf = before >> 16;
            for (uint32_t k = 0; k < (cnt & 0xffffu) + (cnt >> 16); ++k) {
                const uint32_t it = found[k][t];
                if (it & VT_FAR)
                    items[16 * VT_BATCH - 1 - nf++] = it;
                else
                    items[nd++] = it;
            }
        }
        __syncthreads(); /* the items are in place, and nothing reads `found` any more */
        const int nd = __builtin_amdgcn_readfirstlane(total & 0xffffu), nf = __builtin_amdgcn_readfirstlane(total >> 16);
        for (int k = w; k < 2 * nd; k += W) {
            const uint32_t it = __builtin_amdgcn_readfirstlane(items[k >> 1]);
            const int64_t p = base + (it & 0xfffu);
            const int s0 = 8 * (k & 1);
            double f[1] = {0.0};
            if (it & VT_SELF)
                f[0] = vol_self_panel(A, T, p, s0, s0 + 8, x, y);
            else
                tree_panel<TreePot<true, false>>((int)((it >> 19) & 31) - 1, A, T, p, s0, s0 + 8, x, y, f);
            acc += f[0];
        }
        const int fb = nf * (W - 1 - w) / W, fe = nf * (W - w) / W;
        for (int k = fb; k < fe; ++k) {
            const uint32_t it = __builtin_amdgcn_readfirstlane(items[16 * VT_BATCH - 1 - k]);
            const int lev = (it >> 12) & 7;
            const int64_t p0 = base + (it & 0xfffu);
            double f[1];
            tree_expand<1>(A.fq, T, (uint32_t)(T.off[lev] + (p0 >> lev)), (int)((it >> 19) & 31) - 1,
                           TR_PMIN + TR_PSTEP * (int)((it >> 15) & 15), x, y, f);
            if (__ballot(!__builtin_isfinite(f[0])) != 0) {
                f[0] = 0.0;
                const int64_t p1 = min(T.Np, p0 + (1 << lev));
                for (int64_t p = p0; p < p1; ++p) TreePot<true, false>::panel<KQ_NP>(A, T, p, 0, 16, x, y, f);
            }
            acc += f[0];
        }
    }
    red[w][lane] = acc;
    __syncthreads();
    if (w != 0 || i >= V.n) return;
    double s = 0.0;
    for (int v = 0; v < W; ++v) s += red[v][lane];
    V.u[V.idx[0][i]] = fma(INV_2PI, s, V.selfc[0] * V.ws[i] * V.fs[i]);
}

} // namespace mhlp
