/* Particular solution of the modified Stokes equations on a periodic box
   (Sec. 2.1, the periodic stokeslet multiplier; Sec. 3.1.2, grid transforms and
   type-2 sums at the boundary nodes), FP64.

   Box [x0, x0 + Lb) x [y0, y0 + Lb), grid x_a = x0 + a Lb/M, y_b = y0 + b Lb/M,
   fields stored [b][a] (row = y).  Coefficients F^(k) = (1/M^2) sum F e^{-i k.(x - x0)},
   k = (2 pi/Lb)(k1, k2), k1, k2 in [-M/2, M/2) in FFT order; Nyquist coefficients are
   zeroed in every result.
     u^_j = S^_jl F^_l,  S^_jl = (delta_jl - k_j k_l/|k|^2)/(alpha^2 + |k|^2),  S^(0) = I/alpha^2,
     d u_j/d x_m  <-  i k_m u^_j,   u_j(x) = sum_k u^_j(k) e^{i k.(x - x0)} at points.
   FFTs: Stockham with eight elements of a line in the registers of a thread,
   radix 8 (the last stage 2, 4 or 8), LDS only between the stages; twiddles
   e^{-2 pi i j/M} from a host table.  Spectra are stored transposed, [k1][k2],
   so that the y transforms, the multiplier between them and their inverses run
   along contiguous lines in one kernel; the x transforms take FFT_ROWS rows per
   block, which makes their transposed accesses 64 bytes wide.  Real fields are
   read and written as such.  512^2 with gradients and 1024 points: 14 launches
   and 277 us with radix-2 lines, one read and one write of LDS per radix-2
   stage and separate packing kernels, against 6 launches and 85 us (bound by
   latency: a thread's line waits for its loads, twiddles and barriers in turn). */
#pragma once

namespace mhlp {

constexpr int FFT_ROWS = 4;  /* rows per block of the x transforms (fewer from 1024 on) */
constexpr int FFT_T = 256;   /* threads of a block at most */

__host__ __device__ constexpr int fft_rows(int M) { return M > 512 ? (M > 1024 ? 1 : 2) : FFT_ROWS; }
__host__ __device__ constexpr int fft_pad(int i) { return i + (i >> 3); } /* strides of 8 hit all banks */
__host__ __device__ constexpr int fft_line_lds(int M) { return fft_pad(M) + 1; }

__device__ __forceinline__ void fft_dft4(cplx &a, cplx &b, cplx &c, cplx &d)
{
    const cplx t0 = a + c, t1 = a - c, t2 = b + d, t = b - d, t3 = mk(t.im, -t.re);
    a = t0 + t2;
    b = t1 + t3;
    c = t0 - t2;
    d = t1 - t3;
}

__device__ __forceinline__ void fft_dft8(cplx (&v)[8])
{
    constexpr double H = 0.70710678118654752440;
    fft_dft4(v[0], v[2], v[4], v[6]);
    fft_dft4(v[1], v[3], v[5], v[7]);
    const cplx o1 = mk(H * (v[3].re + v[3].im), H * (v[3].im - v[3].re));
    const cplx o2 = mk(v[5].im, -v[5].re);
    const cplx o3 = mk(H * (v[7].im - v[7].re), -H * (v[7].re + v[7].im));
    const cplx e0 = v[0], e1 = v[2], e2 = v[4], e3 = v[6], o0 = v[1];
    v[0] = e0 + o0, v[4] = e0 - o0;
    v[1] = e1 + o1, v[5] = e1 - o1;
    v[2] = e2 + o2, v[6] = e2 - o2;
    v[3] = e3 + o3, v[7] = e3 - o3;
}

/* One stage of radix R = 2^LR behind stages of total radix 2^ls on a line of
   2^lg elements: slot s holds element j + s 2^lg/8; the 8/R butterflies take
   the slots b + q 8/R. */
template <int LR>
__device__ __forceinline__ void fft_stage(cplx (&v)[8], int lg, int ls, int j, const cplx *__restrict__ tw)
{
    constexpr int R = 1 << LR, NB = 8 >> LR;
    const int M = 1 << lg, T = M >> 3;
    if (ls > 0) {
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            const int k = (j + b * T) & ((1 << ls) - 1);
#pragma unroll
            for (int q = 1; q < R; ++q) {
                const int e = (q * k) << (lg - ls - LR);
                cplx w = tw[e & (M / 2 - 1)];
                if (e & (M / 2)) w = -w;
                v[b + q * NB] = v[b + q * NB] * w;
            }
        }
    }
    if constexpr (LR == 3) {
        fft_dft8(v);
    } else if constexpr (LR == 2) {
#pragma unroll
        for (int b = 0; b < NB; ++b) fft_dft4(v[b], v[b + NB], v[b + 2 * NB], v[b + 3 * NB]);
    } else {
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            const cplx t = v[b] - v[b + NB];
            v[b] = v[b] + v[b + NB];
            v[b + NB] = t;
        }
    }
}

/* FFT (unnormalised) of a line of M = 2^lg >= 16 elements by M/8 threads of a
   block that all call it: slot s of thread j is element j + s M/8 before and
   after; sh: the line's LDS (fft_line_lds).  inverse: positive exponents, by
   swapping real and imaginary parts. */
__device__ __forceinline__ void fft_line(cplx (&v)[8], cplx *sh, int lg, int j, const cplx *__restrict__ tw, bool inverse)
{
    const int T = 1 << (lg - 3);
    if (inverse)
#pragma unroll
        for (int s = 0; s < 8; ++s) v[s] = mk(v[s].im, v[s].re);
    for (int ls = 0; ls < lg;) {
        const int lr = min(3, lg - ls);
        if (lr == 3)
            fft_stage<3>(v, lg, ls, j, tw);
        else if (lr == 2)
            fft_stage<2>(v, lg, ls, j, tw);
        else
            fft_stage<1>(v, lg, ls, j, tw);
        if (ls + lr < lg) { /* never the last stage, so lr == 3 */
            const int k = j & ((1 << ls) - 1);
            __syncthreads();
#pragma unroll
            for (int q = 0; q < 8; ++q) sh[fft_pad(((j - k) << 3) + k + (q << ls))] = v[q];
            __syncthreads();
#pragma unroll
            for (int s = 0; s < 8; ++s) v[s] = sh[fft_pad(j + s * T)];
        }
        ls += lr;
    }
    if (inverse)
#pragma unroll
        for (int s = 0; s < 8; ++s) v[s] = mk(v[s].im, v[s].re);
}

/* x transform of real fields f[field][row][M] to spec[field][k1][row]; grid (M/rows, fields) */
__global__ __launch_bounds__(FFT_T) void fft_rows_load_kernel(const double *__restrict__ f, int lg,
                                                              const cplx *__restrict__ tw, cplx *__restrict__ spec)
{
    extern __shared__ cplx fsh[];
    const int M = 1 << lg, L = fft_rows(M), T = M >> 3, l = threadIdx.x % L, j = threadIdx.x / L;
    const int64_t MM = (int64_t)M * M, row = (int64_t)blockIdx.x * L + l;
    const double *in = f + blockIdx.y * MM + row * M;
    cplx v[8];
#pragma unroll
    for (int s = 0; s < 8; ++s) v[s] = mk(in[j + s * T], 0.0);
    fft_line(v, fsh + l * fft_line_lds(M), lg, j, tw, false);
    cplx *out = spec + blockIdx.y * MM + row;
#pragma unroll
    for (int s = 0; s < 8; ++s) out[(int64_t)(j + s * T) * M] = v[s];
}

/* inverse x transform of spectra in[field][k1][row], real parts to out[field][row][M],
   from field 2 on to out2; PADDED: k1 runs over M/2 coefficients in FFT order, the
   others are zero; grid (rows of a field / rows per block, fields from f0 on) */
template <bool PADDED>
__global__ __launch_bounds__(FFT_T) void fft_rows_store_kernel(const cplx *__restrict__ in, int lg, int64_t in_field,
                                                               const cplx *__restrict__ tw, int f0,
                                                               double *__restrict__ out, double *__restrict__ out2)
{
    extern __shared__ cplx fsh[];
    const int M = 1 << lg, L = fft_rows(M), T = M >> 3, l = threadIdx.x % L, j = threadIdx.x / L;
    const int field = f0 + blockIdx.y;
    const int64_t MM = (int64_t)M * M, row = (int64_t)blockIdx.x * L + l;
    const cplx *src = in + field * in_field + row;
    cplx v[8];
#pragma unroll
    for (int s = 0; s < 8; ++s) {
        if (PADDED && s >= 2 && s < 6)
            v[s] = mk(0.0, 0.0);
        else
            v[s] = src[(int64_t)(j + (PADDED && s >= 6 ? s - 4 : s) * T) * M];
    }
    fft_line(v, fsh + l * fft_line_lds(M), lg, j, tw, true);
    double *dst = (field < 2 ? out + field * MM : out2 + (field - 2) * MM) + row * M;
#pragma unroll
    for (int s = 0; s < 8; ++s) dst[j + s * T] = v[s].re;
}

/* One line k1 of the y direction: forward transforms of both forcing components
   (spec[comp][k1][row]), the multiplier, and the inverse y transforms of the
   requested fields into uh[field][k1][row]: fields 0, 1 the solution, 2..5
   i k_x u^_1, i k_y u^_1, i k_x u^_2, i k_y u^_2 (f0 and f1: the first field and
   the end, both even).  The block's groups of M/8 threads all form the forward
   part and share the fields two by two.  coef: the solution's coefficients take
   the forcing's place in spec. */
__global__ __launch_bounds__(FFT_T) void fft_solve_kernel(cplx *spec, int lg, const cplx *__restrict__ tw, double Lb,
                                                          double alpha, int f0, int f1, bool coef,
                                                          cplx *__restrict__ uh)
{
    extern __shared__ cplx fsh[];
    const int M = 1 << lg, T = M >> 3, j = threadIdx.x % T, g = threadIdx.x / T, G = blockDim.x / T;
    const int64_t MM = (int64_t)M * M;
    const int c = blockIdx.x;
    cplx *line = spec + (int64_t)c * M;
    cplx *sh = fsh + g * fft_line_lds(M);
    cplx u1[8], u2[8];
#pragma unroll
    for (int s = 0; s < 8; ++s) {
        u1[s] = line[j + s * T];
        u2[s] = line[MM + j + s * T];
    }
    fft_line(u1, sh, lg, j, tw, false);
    fft_line(u2, sh, lg, j, tw, false);
    const double w = 2.0 * PI / Lb, inv = 1.0 / ((double)M * (double)M);
    const double k1 = w * (c < M / 2 ? c : c - M);
#pragma unroll
    for (int s = 0; s < 8; ++s) {
        const int r = j + s * T;
        const double k2 = w * (r < M / 2 ? r : r - M);
        const cplx f1_ = inv * u1[s], f2_ = inv * u2[s];
        const double kk = k1 * k1 + k2 * k2, den = 1.0 / (alpha * alpha + kk);
        if (r == M / 2 || c == M / 2) {
            u1[s] = u2[s] = mk(0.0, 0.0);
        } else if (kk > 0.0) {
            const double ikk = 1.0 / kk;
            const double p11 = 1.0 - k1 * k1 * ikk, p22 = 1.0 - k2 * k2 * ikk, p12 = -k1 * k2 * ikk;
            u1[s] = den * (p11 * f1_ + p12 * f2_);
            u2[s] = den * (p12 * f1_ + p22 * f2_);
        } else {
            u1[s] = den * f1_;
            u2[s] = den * f2_;
        }
    }
    if (coef && g == 0) /* every group has read the line before fft_line's first barrier */
#pragma unroll
        for (int s = 0; s < 8; ++s) {
            line[j + s * T] = u1[s];
            line[MM + j + s * T] = u2[s];
        }
    /* a group past the end repeats the last pair, so that all meet at the barriers */
    for (int f = f0; f < f1; f += 2 * G) {
        const int p = min(f + 2 * g, f1 - 2);
#pragma unroll 1
        for (int h = 0; h < 2; ++h) {
            cplx v[8];
#pragma unroll
            for (int s = 0; s < 8; ++s) {
                const int r = j + s * T;
                const double k2 = w * (r < M / 2 ? r : r - M);
                const cplx a = u1[s], b = u2[s]; /* selected by value: the arrays stay in registers */
                const bool second = p == 0 ? h != 0 : p == 4;
                const double re = second ? b.re : a.re, im = second ? b.im : a.im, kx = h ? k2 : k1;
                v[s] = p == 0 ? mk(re, im) : mk(-kx * im, kx * re);
            }
            fft_line(v, sh, lg, j, tw, true);
            if (f + 2 * g < f1)
#pragma unroll
                for (int s = 0; s < 8; ++s) uh[(p + h) * MM + (int64_t)c * M + j + s * T] = v[s];
        }
    }
}

/* type-2 sums of u^_1, u^_2 ([comp][k1][k2]) at points: block (point chunk, row chunk of FT2_R
   rows); columns in tiles of FT2_C staged in LDS; per thread e^{i k1 x'} by
   recurrence re-anchored with sincos at every tile, one accumulator per row;
   partial[chunk][comp][point] */
constexpr int FT2_R = 8, FT2_C = 32, FT2_T = 256;

__global__ __launch_bounds__(FT2_T) void type2_points_kernel(const cplx *__restrict__ Uh, int M, double Lb,
                                                             double x0, double y0, const double *__restrict__ px,
                                                             const double *__restrict__ py, int64_t n,
                                                             double *__restrict__ partial)
{
    __shared__ cplx tile[2][FT2_R][FT2_C];
    const int64_t MM = (int64_t)M * M;
    const int64_t i = blockIdx.x * (int64_t)FT2_T + threadIdx.x;
    const bool valid = i < n;
    const int r0 = blockIdx.y * FT2_R;
    const double w = 2.0 * PI / Lb;
    const double xr = valid ? px[i] - x0 : 0.0, yr = valid ? py[i] - y0 : 0.0;
    double sr, cr;
    sincos(w * xr, &sr, &cr);
    const cplx ex1 = mk(cr, sr);
    cplx acc1[FT2_R], acc2[FT2_R];
#pragma unroll
    for (int q = 0; q < FT2_R; ++q) acc1[q] = acc2[q] = mk(0.0, 0.0);
    for (int c0 = 0; c0 < M; c0 += FT2_C) {
        const int nc = min(FT2_C, M);
        __syncthreads();
        for (int t = threadIdx.x; t < 2 * FT2_R * nc; t += FT2_T) {
            const int comp = t / (FT2_R * nc), rem = t % (FT2_R * nc), q = rem / nc, cc = rem % nc;
            tile[comp][q][cc] = Uh[comp * MM + (int64_t)(c0 + cc) * M + r0 + q];
        }
        __syncthreads();
        /* e^{i k1 x'} at the tile's first column, exactly */
        const int cs = c0 < M / 2 ? c0 : c0 - M;
        double s0, c0v;
        sincos(w * cs * xr, &s0, &c0v);
        cplx e = mk(c0v, s0);
        for (int cc = 0; cc < nc; ++cc) {
            if (cc > 0) {
                const int cg = c0 + cc;
                if (cg == M / 2) { /* the negative frequencies start here */
                    double s1, c1;
                    sincos(w * (double)(cg - M) * xr, &s1, &c1);
                    e = mk(c1, s1);
                } else {
                    e = e * ex1;
                }
            }
#pragma unroll
            for (int q = 0; q < FT2_R; ++q) {
                acc1[q] = acc1[q] + tile[0][q][cc] * e;
                acc2[q] = acc2[q] + tile[1][q][cc] * e;
            }
        }
    }
    if (!valid) return;
    double s1 = 0.0, s2 = 0.0;
#pragma unroll
    for (int q = 0; q < FT2_R; ++q) {
        const int r = r0 + q;
        const int ks = r < M / 2 ? r : r - M;
        double sy, cy;
        sincos(w * ks * yr, &sy, &cy);
        const cplx ey = mk(cy, sy);
        s1 += (acc1[q] * ey).re;
        s2 += (acc2[q] * ey).re;
    }
    partial[((int64_t)blockIdx.y * 2 + 0) * n + i] = s1;
    partial[((int64_t)blockIdx.y * 2 + 1) * n + i] = s2;
}

__global__ void type2_reduce_kernel(const double *__restrict__ partial, int nchunk, int64_t n, double *__restrict__ up)
{
    const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (i >= n) return;
    double s1 = 0.0, s2 = 0.0;
    for (int k = 0; k < nchunk; ++k) {
        s1 += partial[((int64_t)k * 2 + 0) * n + i];
        s2 += partial[((int64_t)k * 2 + 1) * n + i];
    }
    up[i] = s1;
    up[n + i] = s2;
}

/* ---- type-2 sums at points by a non-uniform FFT (spreading kernel) ----
   The exponential-of-semicircle kernel phi(z) = exp(beta (sqrt(1 - z^2) - 1)),
   |z| < 1, spans NU_W points of a fine grid of Mf = 2M points (spacing hf):
     b(y_l) = sum_k c(k) e^{i k (y_l - x0)},  c(k) = u^(k) hf^2 / (psi^(k1) psi^(k2)),
     u(x) ~ sum_{l near x} b(y_l) phi_h(x1 - y_l1) phi_h(x2 - y_l2),
   psi^ the Fourier transform of phi_h(x) = phi(2x/(NU_W hf)) (Poisson summation;
   the 2x oversampling and the kernel's decay keep the aliased terms ~1e-14 of
   sum |u^|).  b comes from an inverse FFT of size Mf of the zero-padded c. */
constexpr int NU_W = 14;
constexpr double NU_BETA = 2.30 * NU_W;

/* inverse y transform of c = u^ corr(k1) corr(k2), zero-padded to Mf = 2M: line k1 of
   coef[comp][k1][k2] to fine[comp][k1][y_l]; corr[j] = hf / psi^(k_j) in coarse FFT
   order; grid (M, 2), Mf/8 threads */
__global__ __launch_bounds__(FFT_T) void nufft_lines_kernel(const cplx *__restrict__ coef, int lgf,
                                                            const double *__restrict__ corr,
                                                            const cplx *__restrict__ twf, cplx *__restrict__ fine)
{
    extern __shared__ cplx fsh[];
    const int Mf = 1 << lgf, M = Mf / 2, T = Mf >> 3, j = threadIdx.x;
    const int64_t c = blockIdx.x, field = blockIdx.y;
    const cplx *in = coef + field * M * M + c * M;
    const double cc = corr[c];
    cplx v[8];
#pragma unroll
    for (int s = 0; s < 8; ++s) {
        v[s] = mk(0.0, 0.0);
        if (s < 2 || s >= 6) {
            const int r = j + (s < 2 ? s : s - 4) * T; /* M/2 = 2 T coefficients at either end */
            v[s] = (corr[r] * cc) * in[r];
        }
    }
    fft_line(v, fsh, lgf, j, twf, true);
    cplx *out = fine + (field * M + c) * Mf;
#pragma unroll
    for (int s = 0; s < 8; ++s) out[j + s * T] = v[s];
}

__device__ __forceinline__ double nu_phi(double z)
{
    const double q = 1.0 - z * z;
    return q > 0.0 ? exp(NU_BETA * (sqrt(q) - 1.0)) : 0.0;
}

/* u at the points from the fine-grid values b [2][Mf][Mf], NU_W x NU_W stencil: a
   row of 16 lanes per point, lane a its column a of the stencil (42 -> 5 us for
   1024 points with a thread each, whose 28 exponentials and 392 loads came one
   after the other).  The blocks fill rows of
   NU_ROW: a dimension of a launch holds fewer than 2^32 threads. */
constexpr int NU_ROW = 1 << 20;
__global__ __launch_bounds__(256) void nufft_interp_kernel(const double *__restrict__ fine, int Mf, double hf, double x0,
                                                           double y0, const double *__restrict__ px,
                                                           const double *__restrict__ py, int64_t n,
                                                           double *__restrict__ up)
{
    const int64_t p = (blockIdx.y * (int64_t)gridDim.x + blockIdx.x) * 16 + (threadIdx.x >> 4);
    const int64_t i = min(p, n - 1); /* rows past the end repeat the last point */
    const int a = threadIdx.x & 15, row = threadIdx.x & 48;
    const double xf = (px[i] - x0) / hf, yf = (py[i] - y0) / hf;
    const int ix0 = (int)floor(xf) - NU_W / 2 + 1, iy0 = (int)floor(yf) - NU_W / 2 + 1;
    const double wx = a < NU_W ? nu_phi((xf - (ix0 + a)) * (2.0 / NU_W)) : 0.0;
    const double wy = a < NU_W ? nu_phi((yf - (iy0 + a)) * (2.0 / NU_W)) : 0.0;
    const int64_t MMf = (int64_t)Mf * Mf;
    const int cx = ((ix0 + (a < NU_W ? a : 0)) % Mf + Mf) % Mf; /* idle lanes read column 0 with weight 0 */
    double s1 = 0.0, s2 = 0.0;
#pragma unroll
    for (int b = 0; b < NU_W; ++b) {
        const int ry = ((iy0 + b) % Mf + Mf) % Mf;
        const int64_t o = (int64_t)ry * Mf + cx;
        const double wb = __shfl(wy, row + b);
        s1 = fma(wb, fine[o], s1);
        s2 = fma(wb, fine[MMf + o], s2);
    }
    s1 *= wx;
    s2 *= wx;
    for (int o = 8; o > 0; o >>= 1) {
        s1 += __shfl_xor(s1, o);
        s2 += __shfl_xor(s2, o);
    }
    if (p < n && a == 0) {
        up[i] = s1;
        up[n + i] = s2;
    }
}

/* (u.grad) u from u [2][n] and its gradient g [4][n] (du1/dx, du1/dy, du2/dx, du2/dy) */
__global__ void advect_kernel(const double *__restrict__ u, const double *__restrict__ g, int64_t n,
                              double *__restrict__ out)
{
    const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (i >= n) return;
    const double u1 = u[i], u2 = u[n + i];
    out[i] = fma(u1, g[i], u2 * g[n + i]);
    out[n + i] = fma(u1, g[2 * n + i], u2 * g[3 * n + i]);
}

/* out = sum_{k < nterm} c_k x_k over n elements (terms added in order) */
constexpr int LC_MAX = 16;
struct LinComb {
    const double *x[LC_MAX];
    double c[LC_MAX];
    int nterm;
};

__global__ void lincomb_kernel(LinComb T, int64_t n, double *__restrict__ out)
{
    const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (i >= n) return;
    double s = T.c[0] * T.x[0][i];
    for (int k = 1; k < T.nterm; ++k) s = fma(T.c[k], T.x[k][i], s);
    out[i] = s;
}

} // namespace mhlp
