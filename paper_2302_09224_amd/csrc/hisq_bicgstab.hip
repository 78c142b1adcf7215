// hisq_bicgstab.hip -- mixed-precision BiCGStab(l) (Sec. 6.1; the method of
// Sleijpen and Fokkema) for the whole-lattice HISQ operator M = 2m + D.
//
// The Krylov vectors r_0..r_l, u_0..u_l and the shadow residual live in the
// sloppy triplet's storage format; the solution is accumulated in FP64 at
// every update (Sec. 3.1 item 1).  Reliable updates (Sec. 3, delta): when the
// iterated |r_0| drops by delta below its maximum since the last update (or
// meets the target), r = b - M x is computed with the FP64 operator and
// replaces r_0.  Every scalar (rho, alpha, beta, tau, sigma, gamma, omega) is
// formed on the device, by every block of the kernel that needs it first, from
// the block partials of the kernel before (fixed order, so all blocks agree);
// the first block records it.  A whole cycle (l BiCG steps and the
// minimal-residual step) is enqueued without the host and replayed as a captured
// hipGraph: 5 l + 2 launches,
//   per step j:  u_i = r_i - beta u_i (all i <= j); u_{j+1} = M u_j with <r~, u_{j+1}>;
//                r_i -= alpha u_{i+1} (all i <= j), x += alpha u_0; r_{j+1} = M r_j with
//                <r~, r_{j+1}>
//   l passes of the modified Gram-Schmidt (row i: r_j -= tau_{i-1,j} r_{i-1} for j >= i, and
//   the dot products with r_i in the same pass), the closing updates, the cycle's record.
// (As a launch per operation a cycle of l = 4 took 108 launches; 16^4 with 20-bit
// spinors, m = 0.05 to 1e-12: 39 -> 14.0 ms.)
// A cycle whose |r_0|^2 asks for a reliable update, or that breaks down, lowers
// the guard of the cycles behind it; the host reads each cycle's record from
// pinned memory, with the next cycle already enqueued.
//
// A whole-lattice field is two single-parity fields back to back: the even
// sites, then the odd sites, each in the usual packed layout of Vh sites.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <chrono>
#include <cmath>
#include <cstring>
#include <mutex>

#include "hisq_dslash_kernels.h"

namespace hisq {

using dsl::SpinRaw;
using dsl::spin_decode;
using dsl::spin_load;

namespace {

constexpr int BL_BLOCK = 256;

constexpr int BL_MAXL = HISQ_MAX_BICGSTAB_L;

constexpr int BL_WAVES = BL_BLOCK / 64;

struct VecList {
    char *p[BL_MAXL + 1];
};

// device scalars of one solve (complex values as re, im).  A kernel reads no
// field that its own first block writes, but for stop (see Guard).
struct BlCtl {
    int stop;     // guard of a cycle's launches, which run up to this one: STOP_NEVER while the method goes on, the
                  // launch that broke down, -1 once its cycle is recorded, -2 when a reliable update is due
    int broke;    // 1: a BiCG or minimal-residual denominator vanished, 2: non-finite residual
    int cycles;   // completed
    unsigned long long seq;   // records published
    double rho_c[2], alpha_c[2];                            // entering the cycle
    double rho[BL_MAXL][2], alpha[BL_MAXL][2];              // of the cycle's steps
    double tau[BL_MAXL + 1][BL_MAXL + 1][2];
    double sigma[BL_MAXL + 1];
    double gp[BL_MAXL + 1][2];
    double rs2, rmax2, delta2, tol2;
    double red[2 * BL_MAXL + 2];   // sums of block partials too many for every consumer block to add up
};
// what the host reads after a cycle or a true residual
struct BlRecord {
    unsigned long long seq;
    int stop, broke, cycles;
    double rs2;       // |r_0|^2 (a cycle) or |b - M x|^2 (a true residual)
    double lead;      // |r_0|^2 over the value that asks for a reliable update
};
constexpr int BL_RING = 8;
struct BlHost {
    BlRecord ring[BL_RING];
    unsigned long long launched;
};

__device__ __forceinline__ size_t bl_tid() { return (size_t)blockIdx.x * blockDim.x + threadIdx.x; }
__device__ __forceinline__ size_t bl_stride() { return (size_t)gridDim.x * blockDim.x; }
__device__ __forceinline__ bool bl_first() { return blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0; }

__device__ __forceinline__ void bl_mul(const double *a, const double *b, double *o) {
    const double re = a[0] * b[0] - a[1] * b[1], im = a[0] * b[1] + a[1] * b[0];
    o[0] = re;
    o[1] = im;
}
// a / b with Smith's scaling (no overflow of |b|^2)
__device__ __forceinline__ void bl_div(const double *a, const double *b, double *o) {
    double re, im;
    if (fabs(b[0]) >= fabs(b[1])) {
        const double r = b[1] / b[0], d = b[0] + b[1] * r;
        re = (a[0] + a[1] * r) / d;
        im = (a[1] - a[0] * r) / d;
    } else {
        const double r = b[0] / b[1], d = b[0] * r + b[1];
        re = (a[0] * r + a[1]) / d;
        im = (a[1] * r - a[0]) / d;
    }
    o[0] = re;
    o[1] = im;
}
__device__ __forceinline__ bool bl_zero(const double *a) { return a[0] == 0.0 && a[1] == 0.0; }
__device__ __forceinline__ bool bl_finite(const double *a) { return __builtin_isfinite(a[0]) && __builtin_isfinite(a[1]); }

// v += c x, c complex
template <class R> __device__ __forceinline__ void bl_axpy(CVec<R> &v, const double *c, const CVec<R> &x) {
    const R cr = (R)c[0], ci = (R)c[1];
#pragma unroll
    for (int q = 0; q < 3; q++) {
        v.re[q] = fma(cr, x.re[q], fma(-ci, x.im[q], v.re[q]));
        v.im[q] = fma(cr, x.im[q], fma(ci, x.re[q], v.im[q]));
    }
}
template <class R> __device__ __forceinline__ void bl_xaxpy(CVec<double> &x, const double *c, const CVec<R> &v) {
#pragma unroll
    for (int q = 0; q < 3; q++) {
        x.re[q] += c[0] * (double)v.re[q] - c[1] * (double)v.im[q];
        x.im[q] += c[0] * (double)v.im[q] + c[1] * (double)v.re[q];
    }
}
// acc += conj(v) w (re, im)
template <class R> __device__ __forceinline__ void bl_cdot(double *acc, const CVec<R> &v, const CVec<R> &w) {
#pragma unroll
    for (int q = 0; q < 3; q++) {
        acc[0] += (double)v.re[q] * w.re[q] + (double)v.im[q] * w.im[q];
        acc[1] += (double)v.re[q] * w.im[q] - (double)v.im[q] * w.re[q];
    }
}
template <class R> __device__ __forceinline__ double bl_norm(const CVec<R> &w) {
    double a = 0.0;
#pragma unroll
    for (int q = 0; q < 3; q++) a += (double)w.re[q] * w.re[q] + (double)w.im[q] * w.im[q];
    return a;
}

// sums of block partials too many for every block of the consumer (one block, fixed order)
template <int NV> __global__ void k_bl_sum(const double *partial, int n, double *out, Guard gd) {
    __shared__ double lds[16 * NV];
    if (!gd.pass()) return;
    double v[NV];
    all_sums<NV>(partial, n, v, lds);
    if (threadIdx.x == 0) {
#pragma unroll
        for (int k = 0; k < NV; k++) out[k] = v[k];
    }
}

// Step j, first half: rho1 = <r~, r_j> (in: Re, Im first of each partial's nv),
// beta = alpha rho1 / rho0, u_i = r_i - beta u_i; block row i <= j.
template <int SF, class R>
__global__ void __launch_bounds__(BL_BLOCK) k_bl_dir(VecList u, VecList r, BlCtl *c, Sums in, int nv, int j, size_t vh,
                                                     size_t fb, Guard gd) {
    __shared__ double lds[3 * BL_WAVES];
    if (!gd.pass()) return;
    // the first site's words are on their way while the partials are added up
    char *ui = u.p[blockIdx.y];
    const char *ri = r.p[blockIdx.y];
    size_t i = bl_tid();
    SpinRaw<SF> y0, x0;
    auto fetch = [&](size_t k) {
        const size_t h = k >= vh ? 1 : 0, s = k - h * vh;
        y0 = spin_load<SF>(ui + h * fb, vh, s);
        x0 = spin_load<SF>(ri + h * fb, vh, s);
    };
    if (i < 2 * vh) fetch(i);
    double v[3];
    if (nv == 3) {
        all_sums<3>(in.p, in.n, v, lds);
    } else {
        double w[2];
        all_sums<2>(in.p, in.n, w, lds);
        v[0] = w[0];
        v[1] = w[1];
    }
    const double rho1[2] = {v[0], v[1]};
    const double *rho0 = j ? c->rho[j - 1] : c->rho_c, *alpha = j ? c->alpha[j - 1] : c->alpha_c;
    const bool bad = bl_zero(rho0) || !bl_finite(rho1);
    if (bl_first()) {
        c->rho[j][0] = rho1[0];
        c->rho[j][1] = rho1[1];
        if (bad) {
            c->broke = 1;
            c->stop = gd.j;
        }
    }
    if (bad) return;
    double t[2], beta[2];
    bl_mul(alpha, rho1, t);
    bl_div(t, rho0, beta);
    const R br = (R)-beta[0], bi = (R)-beta[1];
    for (; i < 2 * vh; i += bl_stride()) {
        const size_t h = i >= vh ? 1 : 0, s = i - h * vh;
        const CVec<R> y = spin_decode<R>(y0), x = spin_decode<R>(x0);
        if (i + bl_stride() < 2 * vh) fetch(i + bl_stride());
        CVec<R> o;
#pragma unroll
        for (int q = 0; q < 3; q++) {
            o.re[q] = br * y.re[q] - bi * y.im[q] + x.re[q];
            o.im[q] = br * y.im[q] + bi * y.re[q] + x.im[q];
        }
        (void)SpinorIO<SF, R>::store(ui + h * fb, vh, s, o);
    }
}

// Step j, second half: gamma = <r~, u_{j+1}>, alpha = rho / gamma,
// r_i -= alpha u_{i+1} (block row i <= j) and x += alpha u_0 (row j + 1).
template <int SF, class R>
__global__ void __launch_bounds__(BL_BLOCK) k_bl_res(VecList u, VecList r, char *x64, BlCtl *c, Sums in, int j,
                                                     size_t vh, size_t fb, size_t fb64, Guard gd) {
    __shared__ double lds[2 * BL_WAVES];
    if (!gd.pass()) return;
    const int k = blockIdx.y;
    size_t i = bl_tid();
    SpinRaw<SF> r0, u0;   // row j + 1: u_0 alone
    SpinRaw<SF_F64> x0;
    auto fetch = [&](size_t t) {
        const size_t h = t >= vh ? 1 : 0, s = t - h * vh;
        if (k <= j) {
            r0 = spin_load<SF>(r.p[k] + h * fb, vh, s);
            u0 = spin_load<SF>(u.p[k + 1] + h * fb, vh, s);
        } else {
            u0 = spin_load<SF>(u.p[0] + h * fb, vh, s);
            x0 = spin_load<SF_F64>(x64 + h * fb64, vh, s);
        }
    };
    if (i < 2 * vh) fetch(i);
    double gam[2], alpha[2];
    all_sums<2>(in.p, in.n, gam, lds);
    const bool bad = bl_zero(gam) || !bl_finite(gam);
    if (!bad) bl_div(c->rho[j], gam, alpha);
    if (bl_first()) {
        if (bad) {
            c->broke = 1;
            c->stop = gd.j;
        } else {
            c->alpha[j][0] = alpha[0];
            c->alpha[j][1] = alpha[1];
        }
    }
    if (bad) return;
    const double an[2] = {-alpha[0], -alpha[1]};
    for (; i < 2 * vh; i += bl_stride()) {
        const size_t h = i >= vh ? 1 : 0, s = i - h * vh, nx = i + bl_stride();
        const CVec<R> uv = spin_decode<R>(u0);
        if (k <= j) {
            CVec<R> o = spin_decode<R>(r0);
            if (nx < 2 * vh) fetch(nx);
            bl_axpy<R>(o, an, uv);
            (void)SpinorIO<SF, R>::store(r.p[k] + h * fb, vh, s, o);
        } else {
            CVec<double> x = spin_decode<double>(x0);
            if (nx < 2 * vh) fetch(nx);
            bl_xaxpy<R>(x, alpha, uv);
            SpinorIO<SF_F64, double>::store(x64 + h * fb64, vh, s, x);
        }
    }
}

// the scalars of a finished row i: sigma_i = |r_i|^2, gamma'_i = <r_i, r_0> / sigma_i, tau_ij =
// <r_i, r_j> / sigma_i; v: <r_0, r_i>, |r_i|^2, <r_i, r_{i+1}>, ...  Returns false when sigma_i
// vanishes, and launch `here` is then the last of the cycle.
__device__ __forceinline__ bool bl_row(BlCtl *c, const double *v, int i, int l, int here) {
    const double s2 = v[2];
    const bool bad = !(s2 > 0.0) || !__builtin_isfinite(s2);
    if (bl_first()) {
        c->sigma[i] = s2;
        if (bad) {
            c->broke = 1;
            c->stop = here;
        } else {
            c->gp[i][0] = v[0] / s2;
            c->gp[i][1] = -v[1] / s2;
            for (int j = i + 1; j <= l; j++) {
                c->tau[i][j][0] = v[3 + 2 * (j - i - 1)] / s2;
                c->tau[i][j][1] = v[4 + 2 * (j - i - 1)] / s2;
            }
        }
    }
    return !bad;
}

// Row i of the modified Gram-Schmidt: r_j -= tau_{i-1,j} r_{i-1} for j = i..l
// (i > 1; tau from the partials `in` of row i-1), then the dot products of row i
// on the vectors in registers.  m = l - i + 1 vectors, at most M (the registers).
// partial[block * (2 m + 1) + k]: <r_0, r_i>, |r_i|^2, <r_i, r_{i+1}>, ...
template <int SF, class R, int M>
__global__ void __launch_bounds__(BL_BLOCK) k_bl_mgs(VecList r, BlCtl *c, Sums in, int i, int l, size_t vh, size_t fb,
                                                     double *partial, Guard gd) {
    constexpr int NV = 2 * M + 1, NP = 2 * (M + 1) + 1;
    __shared__ double lds[NP * BL_WAVES], tl[M][2];
    if (!gd.pass()) return;
    const int m = l - i + 1;
    size_t t = bl_tid();
    SpinRaw<SF> w0, wp, w[M];
    auto fetch = [&](size_t k) {
        const size_t h = k >= vh ? 1 : 0, s = k - h * vh;
        w0 = spin_load<SF>(r.p[0] + h * fb, vh, s);
        if (i > 1) wp = spin_load<SF>(r.p[i - 1] + h * fb, vh, s);
#pragma unroll
        for (int q = 0; q < M; q++) w[q] = spin_load<SF>(r.p[min(i + q, l)] + h * fb, vh, s);
    };
    if (t < 2 * vh) fetch(t);
    if (i > 1) {
        // the previous row's m + 1 vectors left 2 m + 3 sums
        if (in.n == 1) {
            if (threadIdx.x < NP) lds[threadIdx.x] = threadIdx.x < 2 * m + 3 ? in.p[threadIdx.x] : 0.0;
        } else {
            // wave w sums the values k = w, w + BL_WAVES, ...
            for (int k = threadIdx.x >> 6; k < 2 * m + 3; k += BL_WAVES) {
                double t = 0.0;
                for (int b = threadIdx.x & 63; b < in.n; b += 64) t += in.p[(size_t)b * (2 * m + 3) + k];
                t = wave_sum(t);
                if ((threadIdx.x & 63) == 0) lds[k] = t;
            }
        }
        __syncthreads();
        const bool ok = bl_row(c, lds, i - 1, l, gd.j);
        if (!ok) return;
        if (threadIdx.x < M) {
            const int k = threadIdx.x;
            tl[k][0] = k < m ? -lds[3 + 2 * k] / lds[2] : 0.0;
            tl[k][1] = k < m ? -lds[4 + 2 * k] / lds[2] : 0.0;
        }
        __syncthreads();
    }
    double acc[NV];
#pragma unroll
    for (int k = 0; k < NV; k++) acc[k] = 0.0;
    for (; t < 2 * vh; t += bl_stride()) {
        const size_t h = t >= vh ? 1 : 0, s = t - h * vh;
        CVec<R> v[M], prev;
        const CVec<R> r0 = spin_decode<R>(w0);
        if (i > 1) prev = spin_decode<R>(wp);
#pragma unroll
        for (int k = 0; k < M; k++) v[k] = spin_decode<R>(w[k]);
        if (t + bl_stride() < 2 * vh) fetch(t + bl_stride());
        if (i > 1) {
#pragma unroll
            for (int k = 0; k < M; k++) {
                if (k >= m) break;
                bl_axpy<R>(v[k], tl[k], prev);
                v[k] = SpinorIO<SF, R>::store(r.p[i + k] + h * fb, vh, s, v[k]);
            }
        }
        bl_cdot<R>(acc, r0, v[0]);
        acc[2] += bl_norm<R>(v[0]);
#pragma unroll
        for (int k = 1; k < M; k++) {
            if (k >= m) break;
            bl_cdot<R>(acc + 1 + 2 * k, v[0], v[k]);
        }
    }
    __syncthreads();
    block_sum<NV>(acc, lds);
    if (threadIdx.x == 0) {
#pragma unroll
        for (int k = 0; k < NV; k++)
            if (k < 2 * m + 1) partial[(size_t)blockIdx.x * (2 * m + 1) + k] = acc[k];
    }
}

// The closing updates: gamma_l, gamma_j by back substitution, gamma''_j, then
// (block row 0) u_0 -= sum gamma_j u_j and (row 1) x += gamma_1 r_0 + sum_{j<l}
// gamma''_j r_j, r_0 -= sum gamma'_j r_j with <r~, r_0> and |r_0|^2 of the new one.
template <int SF, class R>
__global__ void __launch_bounds__(BL_BLOCK) k_bl_close(VecList u, VecList r, const char *rt, char *x64, BlCtl *c,
                                                       Sums in, int l, size_t vh, size_t fb, size_t fb64,
                                                       double *partial, Guard gd) {
    __shared__ double lds[3 * BL_WAVES], gm[BL_MAXL + 1][2], cx[BL_MAXL][2], cu[BL_MAXL][2], cr[BL_MAXL][2];
    if (!gd.pass()) return;
    double v[3];
    all_sums<3>(in.p, in.n, v, lds);   // <r_0, r_l>, |r_l|^2
    if (!bl_row(c, v, l, l, gd.j)) return;
    if (threadIdx.x == 0) {
        gm[l][0] = v[0] / v[2];
        gm[l][1] = -v[1] / v[2];
        cr[l - 1][0] = -gm[l][0];
        cr[l - 1][1] = -gm[l][1];
        for (int jj = l - 1; jj >= 1; jj--) {
            double sr = c->gp[jj][0], si = c->gp[jj][1];
            cr[jj - 1][0] = -sr;
            cr[jj - 1][1] = -si;
            for (int ii = jj + 1; ii <= l; ii++) {
                double t[2];
                bl_mul(c->tau[jj][ii], gm[ii], t);
                sr -= t[0];
                si -= t[1];
            }
            gm[jj][0] = sr;
            gm[jj][1] = si;
        }
        cx[0][0] = gm[1][0];
        cx[0][1] = gm[1][1];
        for (int jj = 1; jj < l; jj++) {
            double sr = gm[jj + 1][0], si = gm[jj + 1][1];
            for (int ii = jj + 1; ii < l; ii++) {
                double t[2];
                bl_mul(c->tau[jj][ii], gm[ii + 1], t);
                sr += t[0];
                si += t[1];
            }
            cx[jj][0] = sr;
            cx[jj][1] = si;
        }
        for (int jj = 1; jj <= l; jj++) {
            cu[jj - 1][0] = -gm[jj][0];
            cu[jj - 1][1] = -gm[jj][1];
        }
        if (bl_first()) {   // the next cycle's rho_0 = -omega rho, omega = gamma_l, and its alpha
            double t[2];
            bl_mul(gm[l], c->rho[l - 1], t);
            c->rho_c[0] = -t[0];
            c->rho_c[1] = -t[1];
            c->alpha_c[0] = c->alpha[l - 1][0];
            c->alpha_c[1] = c->alpha[l - 1][1];
        }
    }
    __syncthreads();
    double acc[3] = {0.0, 0.0, 0.0};
    for (size_t i = bl_tid(); i < 2 * vh; i += bl_stride()) {
        const size_t h = i >= vh ? 1 : 0, s = i - h * vh;
        if (blockIdx.y == 0) {
            CVec<R> o = SpinorIO<SF, R>::load(u.p[0] + h * fb, vh, s);
#pragma unroll 4
            for (int k = 1; k <= l; k++) bl_axpy<R>(o, cu[k - 1], SpinorIO<SF, R>::load(u.p[k] + h * fb, vh, s));
            (void)SpinorIO<SF, R>::store(u.p[0] + h * fb, vh, s, o);
            continue;
        }
        CVec<R> o = SpinorIO<SF, R>::load(r.p[0] + h * fb, vh, s);
        const CVec<R> w = SpinorIO<SF, R>::load(rt + h * fb, vh, s);
        CVec<double> x = SpinorIO<SF_F64, double>::load(x64 + h * fb64, vh, s);
        bl_xaxpy<R>(x, cx[0], o);
#pragma unroll 4
        for (int k = 1; k <= l; k++) {
            const CVec<R> y = SpinorIO<SF, R>::load(r.p[k] + h * fb, vh, s);
            if (k < l) bl_xaxpy<R>(x, cx[k], y);
            bl_axpy<R>(o, cr[k - 1], y);
        }
        SpinorIO<SF_F64, double>::store(x64 + h * fb64, vh, s, x);
        const CVec<R> st = SpinorIO<SF, R>::store(r.p[0] + h * fb, vh, s, o);
        bl_cdot<R>(acc, w, st);
        acc[2] += bl_norm<R>(st);
    }
    if (blockIdx.y == 0) return;
    block_sum<3>(acc, lds);
    if (threadIdx.x == 0) {
#pragma unroll
        for (int k = 0; k < 3; k++) partial[3 * (size_t)blockIdx.x + k] = acc[k];
    }
}

// r_0 = pack(r64) (and the shadow residual, at the start), with <r~, r_0> and
// |r_0|^2 as the closing updates leave them
template <int SF, class R>
__global__ void __launch_bounds__(BL_BLOCK) k_bl_restart(char *r0, char *rt, int start, const char *r64, size_t vh,
                                                         size_t fb, size_t fb64, double *partial) {
    __shared__ double lds[3 * BL_WAVES];
    double acc[3] = {0.0, 0.0, 0.0};
    for (size_t i = bl_tid(); i < 2 * vh; i += bl_stride()) {
        const size_t h = i >= vh ? 1 : 0, s = i - h * vh;
        const CVec<double> t = SpinorIO<SF_F64, double>::load(r64 + h * fb64, vh, s);
        const CVec<double> o = SpinorIO<SF, double>::store(r0 + h * fb, vh, s, t);
        CVec<double> w = o;
        if (start)
            (void)SpinorIO<SF, double>::store(rt + h * fb, vh, s, t);
        else
            w = SpinorIO<SF, double>::load(rt + h * fb, vh, s);
        bl_cdot<double>(acc, w, o);
        acc[2] += bl_norm<double>(o);
    }
    block_sum<3>(acc, lds);
    if (threadIdx.x == 0) {
#pragma unroll
        for (int k = 0; k < 3; k++) partial[3 * (size_t)blockIdx.x + k] = acc[k];
    }
}

// The record of a cycle (op 0; in: the closing updates' partials), of a true
// residual (op 1; in: |b - M x|^2 partials) or of |b|^2 (op 2: the target is
// tol^2 |b|^2 from then on), and what it decides: a cycle that asks for a
// reliable update closes the cycles behind it, a true residual opens them again.
__global__ void k_bl_record(BlCtl *c, Sums in, int op, BlHost *host) {
    __shared__ double lds[16 * 3];
    const bool ran = op != 0 || c->stop == STOP_NEVER;
    double v[3] = {0.0, 0.0, 0.0};
    if (ran) {
        if (op == 0) {
            all_sums<3>(in.p, in.n, v, lds);
        } else {
            double w[1];
            all_sums<1>(in.p, in.n, w, lds);
            v[2] = w[0];
        }
    }
    if (threadIdx.x) return;
    double lead = 0.0;
    if (ran && op == 0) {
        c->cycles++;
        const double rs2 = v[2], rmax2 = fmax(c->rmax2, rs2);
        c->rs2 = rs2;
        c->rmax2 = rmax2;
        const double t = fmax(c->delta2 * rmax2, c->tol2);
        lead = t > 0.0 ? rs2 / t : 0.0;
        if (!__builtin_isfinite(rs2)) {
            c->broke = 2;
            c->stop = -1;
        } else if (rs2 < c->delta2 * rmax2 || rs2 <= c->tol2) {
            c->stop = -2;
        }
    } else if (op == 1) {
        c->rmax2 = v[2];
        if (!__builtin_isfinite(v[2])) {
            c->broke = 2;
            c->stop = -1;
        }
        if (!c->broke) c->stop = STOP_NEVER;
    } else if (op == 2) {
        c->tol2 *= v[2];   // tol^2 |b|^2
    } else if (c->stop >= 0) {
        c->stop = -1;      // broken down in this cycle: those behind it do nothing
    }
    const unsigned long long seq = c->seq + 1;
    c->seq = seq;
    BlRecord *o = &host->ring[seq % BL_RING];
    o->stop = c->stop;
    o->broke = c->broke;
    o->cycles = c->cycles;
    o->rs2 = v[2];
    o->lead = lead;
    __hip_atomic_store(&o->seq, seq, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}

// canonical lexicographic [V][3] <-> (even field, odd field) in F64 layout
__global__ void k_bl_split(char *dst, const double *src, Geom g, size_t fb64) {
    const size_t V = 2 * (size_t)g.vh;
    for (size_t i = bl_tid(); i < V; i += bl_stride()) {
        size_t r = i;
        const int x = (int)(r % g.X); r /= g.X;
        const int y = (int)(r % g.Y); r /= g.Y;
        const int z = (int)(r % g.Z);
        const int t = (int)(r / g.Z);
        const int par = (x + y + z + t) & 1;
        CVec<double> v;
#pragma unroll
        for (int q = 0; q < 3; q++) {
            v.re[q] = src[6 * i + 2 * q];
            v.im[q] = src[6 * i + 2 * q + 1];
        }
        SpinorIO<SF_F64, double>::store(dst + par * fb64, g.vh, i >> 1, v);
    }
}

__global__ void k_bl_merge(double *dst, const char *src, Geom g, size_t fb64) {
    const size_t V = 2 * (size_t)g.vh;
    for (size_t i = bl_tid(); i < V; i += bl_stride()) {
        size_t r = i;
        const int x = (int)(r % g.X); r /= g.X;
        const int y = (int)(r % g.Y); r /= g.Y;
        const int z = (int)(r % g.Z);
        const int t = (int)(r / g.Z);
        const int par = (x + y + z + t) & 1;
        const CVec<double> v = SpinorIO<SF_F64, double>::load(src + par * fb64, g.vh, i >> 1);
#pragma unroll
        for (int q = 0; q < 3; q++) {
            dst[6 * i + 2 * q] = v.re[q];
            dst[6 * i + 2 * q + 1] = v.im[q];
        }
    }
}

#define HISQ_BL_DISPATCH(sf, compute, CALL)                                                          \
    do {                                                                                             \
        switch ((sf) * 2 + ((compute) == 64)) {                                                      \
        case SF_F64 * 2 + 1: { constexpr int SFc = SF_F64; typedef double Rc; CALL; } break;         \
        case SF_F32 * 2 + 0: { constexpr int SFc = SF_F32; typedef float Rc; CALL; } break;          \
        case SF_HALF16 * 2 + 0: { constexpr int SFc = SF_HALF16; typedef float Rc; CALL; } break;    \
        case SF_INT20 * 2 + 0: { constexpr int SFc = SF_INT20; typedef float Rc; CALL; } break;      \
        case SF_INT30 * 2 + 1: { constexpr int SFc = SF_INT30; typedef double Rc; CALL; } break;     \
        case SF_INT30 * 2 + 0: { constexpr int SFc = SF_INT30; typedef float Rc; CALL; } break;      \
        case SF_INT24 * 2 + 0: { constexpr int SFc = SF_INT24; typedef float Rc; CALL; } break;      \
        default: return set_error(HISQ_EINVAL, "bicgstab: unsupported sloppy triplet");             \
        }                                                                                            \
    } while (0)

struct Bl {
    Geom g;
    size_t vh, fb, fb64;          // bytes of one parity field: sloppy, FP64
    hisq_fmt f;
    const hisq_gauge *g64, *gs;
    double mass;
    hipStream_t st;
    int l;
    int nbl;                      // grid of the vector kernels
    double *dpart;                // partials of the operator (both parities, two each)
    double *vpart[3];             // partials of the vector kernels: closing updates, Gram-Schmidt rows in turn
    VecList r, u;
    char *rt;
    DslashPlan plan_s{}, plan_64{};
    int nb_s = 0, nb64 = 0;
    long matvecs = 0, f64apps = 0;
    double alg = 0.0;
    BlCtl *ctl = nullptr;         // device scalars
    const int *stopp = nullptr;   // &ctl->stop
    int at = 0;                   // of the cycle's next guarded launch
    BlHost *host = nullptr;

    Guard guard() { return Guard{stopp, at++, 0}; }

    // block partials for the next kernel: as they are when few, else added up in a launch
    template <int NV> hisq_status sums(const double *partial, int n, Sums *out) {
        *out = Sums{partial, n};
        if (n * NV <= SUMS_DIRECT) return HISQ_OK;
        hipLaunchKernelGGL((k_bl_sum<NV>), dim3(1), dim3(1024), 0, st, partial, n, ctl->red, guard());
        HISQ_TRY_HIP(hipGetLastError());
        *out = Sums{ctl->red, 1};
        return HISQ_OK;
    }
    // for the Gram-Schmidt rows, whose blocks add up nv values with a wave each: up to 512
    // blocks' tuples directly (a launch of its own took 10 us at 16^4)
    hisq_status sums_n(const double *partial, int nv, Sums *out) {
        *out = Sums{partial, nbl};
        if (nbl <= 512 && nv > 3) return HISQ_OK;
        switch (nv) {
        case 3: return sums<3>(partial, nbl, out);
        case 5: return sums<5>(partial, nbl, out);
        case 7: return sums<7>(partial, nbl, out);
        case 9: return sums<9>(partial, nbl, out);
        case 11: return sums<11>(partial, nbl, out);
        case 13: return sums<13>(partial, nbl, out);
        case 15: return sums<15>(partial, nbl, out);
        case 17: return sums<17>(partial, nbl, out);
        default: return set_error(HISQ_EINVAL, "bicgstab: l out of range");
        }
    }

    DslashArgs dargs(const hisq_gauge *gg, int sf) const {
        DslashArgs a;
        memset(&a, 0, sizeof(a));
        a.b = 1.0;
        a.g = g;
        a.red = RED_NONE;
        a.nrhs = 1;
        a.field_stride = spinor_field_bytes(vh, sf);
        gauge_args(a, gg);
        return a;
    }

    // out = M in = 2m in + D in (sloppy) on both parities, one launch: per output parity
    // p, out_p = D in_q + 2m in_p (skipped after a breakdown in the cycle); dot: the
    // partials of <r~, out>
    hisq_status matvec(char *out, const char *in, bool dot) {
        DslashArgs a = dargs(gs, f.spinor);
        a.both = 1;
        a.half = fb;
        a.out = out;
        a.in = in;
        a.x = in;
        a.a = 2.0 * mass;
        a.guard = guard();
        if (dot) {
            a.red = RED_CDOT;
            a.z = rt;
            a.partial = dpart;
        }
        HISQ_TRY_HIP(launch_dslash(a, f, plan_s, st, nullptr));
        alg += 2.0 * vh * (dslash_link_bytes(gs) + (dot ? 4.0 : 3.0) * spinor_site_bytes(f.spinor));
        return HISQ_OK;
    }

    template <int M> hisq_status mgs_row(int i, const Sums &in, double *out) {
        HISQ_BL_DISPATCH(f.spinor, f.compute,
                         hipLaunchKernelGGL((k_bl_mgs<SFc, Rc, M>), dim3(nbl), dim3(BL_BLOCK), 0, st, r, ctl, in, i, l,
                                            vh, fb, out, guard()));
        HISQ_TRY_HIP(hipGetLastError());
        return HISQ_OK;
    }

    // one cycle: l BiCG steps, the minimal-residual step by modified Gram-Schmidt, the record
    hisq_status enq_cycle(char *x64) {
        const double bs = spinor_site_bytes(f.spinor);
        Sums in;
        at = 0;
        for (int j = 0; j < l; j++) {
            const int nv = j ? 2 : 3;
            if (j)
                HISQ_TRY(sums<2>(dpart, 2 * nb_s, &in));
            else
                HISQ_TRY(sums<3>(vpart[0], nbl, &in));
            HISQ_BL_DISPATCH(f.spinor, f.compute,
                             hipLaunchKernelGGL((k_bl_dir<SFc, Rc>), dim3(nbl, j + 1), dim3(BL_BLOCK), 0, st, u, r, ctl,
                                                in, nv, j, vh, fb, guard()));
            HISQ_TRY_HIP(hipGetLastError());
            HISQ_TRY(matvec(u.p[j + 1], u.p[j], true));
            HISQ_TRY(sums<2>(dpart, 2 * nb_s, &in));
            HISQ_BL_DISPATCH(f.spinor, f.compute,
                             hipLaunchKernelGGL((k_bl_res<SFc, Rc>), dim3(nbl, j + 2), dim3(BL_BLOCK), 0, st, u, r, x64,
                                                ctl, in, j, vh, fb, fb64, guard()));
            HISQ_TRY_HIP(hipGetLastError());
            HISQ_TRY(matvec(r.p[j + 1], r.p[j], j + 1 < l));
            alg += 2.0 * vh * ((j + 1) * 6.0 * bs + bs + 96.0);
        }
        in = Sums{nullptr, 0};
        for (int i = 1; i <= l; i++) {
            const int m = l - i + 1;
            double *out = vpart[1 + (i & 1)];
            if (m == 1)
                HISQ_TRY(mgs_row<1>(i, in, out));
            else if (m == 2)
                HISQ_TRY(mgs_row<2>(i, in, out));
            else if (m == 3)
                HISQ_TRY(mgs_row<3>(i, in, out));
            else if (m == 4)
                HISQ_TRY(mgs_row<4>(i, in, out));
            else
                HISQ_TRY(mgs_row<BL_MAXL>(i, in, out));
            HISQ_TRY(sums_n(out, 2 * m + 1, &in));
            alg += 2.0 * vh * bs * (i > 1 ? 2.0 + 2.0 * m : 1.0 + m);
        }
        HISQ_BL_DISPATCH(f.spinor, f.compute,
                         hipLaunchKernelGGL((k_bl_close<SFc, Rc>), dim3(nbl, 2), dim3(BL_BLOCK), 0, st, u, r, rt, x64,
                                            ctl, in, l, vh, fb, fb64, vpart[0], guard()));
        HISQ_TRY_HIP(hipGetLastError());
        alg += 2.0 * vh * (bs * (2.0 * l + 5.0) + 96.0);
        HISQ_TRY(record(Sums{vpart[0], nbl}, 0));
        return HISQ_OK;
    }

    hisq_status record(const Sums &in, int op) {
        hipLaunchKernelGGL(k_bl_record, dim3(1), dim3(1024), 0, st, ctl, in, op, host);
        HISQ_TRY_HIP(hipGetLastError());
        return HISQ_OK;
    }
    hisq_status wait(unsigned long long seq, BlRecord *out) {
        return wait_record(&host->ring[seq % BL_RING], seq, st, out);
    }

    // r64 = b64 - M x64 with the FP64 operator (both parities in one launch); *r2 = |r64|^2
    hisq_status residual64(char *r64, const char *x64, const char *b64, double *r2) {
        const hisq_fmt f64 = {HISQ_GAUGE_F64, HISQ_SPINOR_F64, 64};
        DslashArgs a = dargs(g64, SF_F64);
        a.both = 1;
        a.half = fb64;
        a.out = r64;
        a.in = x64;
        a.x = x64;
        a.y = b64;
        a.b = -1.0;
        a.a = -2.0 * mass;
        a.c = 1.0;
        a.red = RED_NORM;
        a.partial = dpart;
        HISQ_TRY_HIP(launch_dslash(a, f64, plan_64, st, nullptr));
        f64apps++;
        alg += 2.0 * vh * (dslash_link_bytes(g64) + 4.0 * 48);
        HISQ_TRY(record(Sums{dpart, 2 * nb64}, 1));
        BlRecord rec;
        HISQ_TRY(wait(++host->launched, &rec));
        *r2 = rec.rs2;
        return HISQ_OK;
    }

    hisq_status restart(const char *r64, bool start) {
        HISQ_BL_DISPATCH(f.spinor, f.compute,
                         hipLaunchKernelGGL((k_bl_restart<SFc, Rc>), dim3(nbl), dim3(BL_BLOCK), 0, st, r.p[0], rt,
                                            start ? 1 : 0, r64, vh, fb, fb64, vpart[0]));
        HISQ_TRY_HIP(hipGetLastError());
        alg += 2.0 * vh * (48.0 + 2.0 * spinor_site_bytes(f.spinor));
        return HISQ_OK;
    }
};

inline size_t al256(size_t v) { return (v + 255) & ~(size_t)255; }

// library-owned stream per device (default priority), ordered after the caller's
// stream with an event; a cycle is captured from it (the caller's stream may be
// the null stream, which cannot be captured)
struct BlDev {
    hipStream_t stream = nullptr;
    hipEvent_t ev = nullptr;
    BlHost *host = nullptr;   // pinned: the records the device leaves
    std::mutex mu;
};
BlDev g_bldev[64];

struct BlLayout {
    size_t fb, fb64, dpart, vpart, part_doubles, total;
    size_t off_part, off_ctl, off_x64, off_b64, off_r64, off_vec;
    int nvec;
};

BlLayout bl_layout(const Geom &g, int l, const hisq_fmt &f) {
    BlLayout L;
    L.fb = al256(spinor_field_bytes(g.vh, f.spinor));
    L.fb64 = al256(spinor_field_bytes(g.vh, SF_F64));
    const size_t nbl = (size_t)blas_blocks(2 * (size_t)g.vh);
    // the operator's partials: two per block of the largest one-system launch, both parities
    L.dpart = 4 * (size_t)std::max(dslash_blocks(g.vh, 64), 8 * g.T * slab_tiles(g, 1, 64));
    L.vpart = nbl * (2 * BL_MAXL + 1);
    L.part_doubles = L.dpart + 3 * L.vpart;
    L.nvec = 2 * (l + 1) + 1;   // r_0..r_l, u_0..u_l, shadow
    size_t off = 0;
    L.off_part = off;
    off += al256(L.part_doubles * sizeof(double));
    L.off_ctl = off;
    off += al256(sizeof(BlCtl));
    L.off_x64 = off;
    off += 2 * L.fb64;
    L.off_b64 = off;
    off += 2 * L.fb64;
    L.off_r64 = off;
    off += 2 * L.fb64;
    L.off_vec = off;
    off += (size_t)L.nvec * 2 * L.fb;
    L.total = off;
    return L;
}

}  // namespace

}  // namespace hisq

using namespace hisq;

extern "C" size_t hisq_bicgstab_workspace_bytes(const int dims[4], int l, hisq_fmt sloppy) {
    if (!dims || !dims_ok(dims) || !triplet_ok(sloppy) || l < 1 || l > HISQ_MAX_BICGSTAB_L) return 0;
    return bl_layout(make_geom(dims), l, sloppy).total;
}

extern "C" hisq_status hisq_bicgstab_solve(double *x, const double *b, const hisq_gauge *g64, const hisq_gauge *gs,
                                           double mass, double tol, int l, hisq_fmt sloppy,
                                           const hisq_solver_params *p, void *ws, size_t ws_bytes,
                                           hisq_solver_stats *stats, void *stream) {
    auto t0 = std::chrono::steady_clock::now();
    hisq_solver_stats tmp;
    hisq_solver_stats *sto = stats ? stats : &tmp;
    memset(sto, 0, sizeof(*sto));
    sto->status = HISQ_EINVAL;
    if (!x || !b || !g64 || !gs || !ws) return set_error(HISQ_EINVAL, "hisq_bicgstab_solve: null argument");
    if (l < 1 || l > HISQ_MAX_BICGSTAB_L) return set_error(HISQ_EINVAL, "l must be in [1,%d]", HISQ_MAX_BICGSTAB_L);
    if (!(tol > 0.0) || !(mass > 0.0)) return set_error(HISQ_EINVAL, "tol and mass must be > 0");
    if (!triplet_ok(sloppy)) return set_error(HISQ_EINVAL, "unsupported sloppy triplet");
    if (!aligned16(x) || !aligned16(b) || !aligned16(ws)) return set_error(HISQ_EALIGN, "unaligned pointer");
    const int *dims = g64->dims;
    if (!dims_ok(dims)) return set_error(HISQ_EINVAL, "bad lattice dims");
    if (g64->fmt != HISQ_GAUGE_F64 || !g64->fat || !g64->lng) return set_error(HISQ_EINVAL, "g64 must hold FP64 links");
    if (gs->fmt != sloppy.gauge || !gs->fat || !gs->lng) return set_error(HISQ_EINVAL, "gs does not match the sloppy triplet");
    if (!recon_ok(sloppy, gs->long_recon, false) ||
        !recon_ok(hisq_fmt{HISQ_GAUGE_F64, HISQ_SPINOR_F64, 64}, g64->long_recon, false))
        return set_error(HISQ_EINVAL, "eight-parameter long links need FP64 arithmetic on F64 or FIX32 links");
    for (int k = 0; k < 4; k++)
        if (gs->dims[k] != dims[k]) return set_error(HISQ_EINVAL, "gauge dims differ");
    hisq_solver_params q;
    hisq_solver_params_default(&q);
    if (p) q = *p;
    if (q.maxiter <= 0) q.maxiter = 100000;
    const Geom g = make_geom(dims);
    const BlLayout L = bl_layout(g, l, sloppy);
    if (ws_bytes < L.total) return set_error(HISQ_EWORKSPACE, "workspace %zu bytes, need %zu", ws_bytes, L.total);

    char *w = (char *)ws;
    Bl B;
    B.g = g;
    B.vh = g.vh;
    B.fb = L.fb;
    B.fb64 = L.fb64;
    B.f = sloppy;
    B.g64 = g64;
    B.gs = gs;
    B.mass = mass;
    int dev = 0;
    HISQ_TRY_HIP(hipGetDevice(&dev));
    if (dev < 0 || dev >= 64) return set_error(HISQ_EINVAL, "device index %d out of range", dev);
    BlDev &dv = g_bldev[dev];
    std::unique_lock<std::mutex> lk(dv.mu);
    if (!dv.stream) {
        HISQ_TRY_HIP(hipStreamCreateWithFlags(&dv.stream, hipStreamNonBlocking));
        HISQ_TRY_HIP(hipEventCreateWithFlags(&dv.ev, hipEventDisableTiming));
    }
    if (!dv.host) {
        HISQ_TRY_HIP(hipHostMalloc((void **)&dv.host, sizeof(BlHost), hipHostMallocCoherent));
        memset(dv.host, 0, sizeof(BlHost));
    }
    HISQ_TRY_HIP(hipEventRecord(dv.ev, (hipStream_t)stream));
    HISQ_TRY_HIP(hipStreamWaitEvent(dv.stream, dv.ev, 0));
    B.st = dv.stream;
    B.host = dv.host;
    B.l = l;
    B.nbl = blas_blocks(2 * (size_t)g.vh);
    B.dpart = (double *)(w + L.off_part);
    for (int k = 0; k < 3; k++) B.vpart[k] = B.dpart + L.dpart + k * L.vpart;
    B.ctl = (BlCtl *)(w + L.off_ctl);
    B.stopp = &B.ctl->stop;
    char *x64 = w + L.off_x64, *b64 = w + L.off_b64, *r64 = w + L.off_r64;
    memset(&B.r, 0, sizeof(B.r));
    memset(&B.u, 0, sizeof(B.u));
    for (int i = 0; i <= l; i++) {
        B.r.p[i] = w + L.off_vec + (size_t)i * 2 * L.fb;
        B.u.p[i] = w + L.off_vec + (size_t)(l + 1 + i) * 2 * L.fb;
    }
    B.rt = w + L.off_vec + (size_t)(2 * l + 2) * 2 * L.fb;

    // launch shapes (autotuned on first use)
    {
        DslashArgs ps = B.dargs(gs, sloppy.spinor);
        ps.out = B.r.p[1];
        ps.in = B.r.p[0] + L.fb;
        B.plan_s = dslash_plan(sloppy, g, 1, &ps, B.st);
        dslash_keep_links(sloppy, g, ps.long_recon, B.plan_s);
        B.nb_s = dslash_tile_blocks(g, B.plan_s.tile[0]);
        const hisq_fmt f64 = {HISQ_GAUGE_F64, HISQ_SPINOR_F64, 64};
        DslashArgs p64 = B.dargs(g64, SF_F64);
        p64.out = r64;
        p64.in = x64 + L.fb64;
        B.plan_64 = dslash_plan(f64, g, 1, &p64, B.st);
        B.nb64 = dslash_tile_blocks(g, B.plan_64.tile[0]);
    }

    hipLaunchKernelGGL(k_bl_split, dim3(B.nbl), dim3(BL_BLOCK), 0, B.st, x64, x, g, L.fb64);
    hipLaunchKernelGGL(k_bl_split, dim3(B.nbl), dim3(BL_BLOCK), 0, B.st, b64, b, g, L.fb64);
    HISQ_TRY_HIP(hipGetLastError());
    {   // rho0 = 1, alpha = 0, omega = 1 (entering a cycle: -omega rho0); tol2 is multiplied by |b|^2 in its record
        BlCtl c0;
        memset(&c0, 0, sizeof(c0));
        c0.stop = STOP_NEVER;
        c0.rho_c[0] = -1.0;
        c0.delta2 = q.delta > 0 ? q.delta * q.delta : 0.0;
        c0.tol2 = tol * tol;
        c0.seq = B.host->launched;
        HISQ_TRY_HIP(hipMemcpyAsync(B.ctl, &c0, sizeof(c0), hipMemcpyHostToDevice, B.st));
        HISQ_TRY_HIP(hipStreamSynchronize(B.st));
    }
    double b2 = 0.0;
    {   // both halves' block partials, then one fixed-order sum
        int nbe = 0, nbo = 0;
        HISQ_TRY_HIP(launch_norm2_f64(b64, g.vh, B.vpart[0], &nbe, B.st));
        HISQ_TRY_HIP(launch_norm2_f64(b64 + L.fb64, g.vh, B.vpart[0] + nbe, &nbo, B.st));
        HISQ_TRY(B.record(Sums{B.vpart[0], nbe + nbo}, 2));
        BlRecord rec;
        HISQ_TRY(B.wait(++B.host->launched, &rec));
        b2 = rec.rs2;
    }
    double r2 = 0.0;
    HISQ_TRY(B.residual64(r64, x64, b64, &r2));
    hisq_status status = HISQ_OK;
    long rus = 0;
    const double tol2 = tol * tol * b2;
    if (b2 == 0.0) {   // x = 0
        HISQ_TRY_HIP(hipMemsetAsync(x, 0, 2 * (size_t)g.vh * 6 * sizeof(double), B.st));
        HISQ_TRY_HIP(hipStreamSynchronize(B.st));
        sto->status = HISQ_OK;
        return HISQ_OK;
    }
    if (!std::isfinite(b2) || !std::isfinite(r2)) {
        status = set_error(HISQ_EBREAKDOWN, "bicgstab: non-finite initial residual");
    } else if (r2 > tol2) {
        HISQ_TRY(B.restart(r64, true));
        HISQ_TRY_HIP(hipMemsetAsync(B.u.p[0], 0, 2 * L.fb, B.st));
        hipGraphExec_t exec = nullptr;
        struct ExecFree {
            hipGraphExec_t *e;
            hipStream_t st;
            ~ExecFree() {
                (void)hipStreamSynchronize(st);   // a cycle behind the last one may still be returning from its guards
                if (*e) (void)hipGraphExecDestroy(*e);
            }
        } exec_free{&exec, B.st};
        double cyc_alg = 0.0;
        int inflight = 0, cycles = 0;
        Pace pace;
        while (status == HISQ_OK) {
            // the next cycle is enqueued before the running one is read, unless
            // that one is about to ask for a reliable update
            while (inflight < 2 && (inflight == 0 || pace.left > (double)inflight) &&
                   B.matvecs + 2L * l * inflight < q.maxiter) {
                const double a0 = B.alg;
                if (q.use_graph) {
                    if (!exec) {
                        hipGraph_t gr = nullptr;
                        HISQ_TRY_HIP(hipStreamBeginCapture(B.st, hipStreamCaptureModeThreadLocal));
                        hisq_status cs = B.enq_cycle(x64);
                        hipError_t e = hipStreamEndCapture(B.st, &gr);
                        if (cs != HISQ_OK) {
                            if (gr) (void)hipGraphDestroy(gr);
                            return cs;
                        }
                        HISQ_TRY_HIP(e);
                        e = hipGraphInstantiate(&exec, gr, nullptr, nullptr, 0);
                        (void)hipGraphDestroy(gr);
                        HISQ_TRY_HIP(e);
                        cyc_alg = B.alg - a0;
                    }
                    HISQ_TRY_HIP(hipGraphLaunch(exec, B.st));
                } else {
                    HISQ_TRY(B.enq_cycle(x64));
                    cyc_alg = B.alg - a0;
                }
                B.alg = a0;
                B.host->launched++;
                inflight++;
            }
            if (inflight == 0) {
                status = set_error(HISQ_ENOCONV, "bicgstab: no convergence in %ld operator applications", B.matvecs);
                break;
            }
            BlRecord rec;
            HISQ_TRY(B.wait(B.host->launched - (unsigned long long)inflight + 1, &rec));
            inflight--;
            cycles = rec.cycles;
            B.matvecs += 2 * l;   // of a cycle that broke down too
            B.alg += cyc_alg;
            if (rec.broke == 2) {
                status = set_error(HISQ_EBREAKDOWN, "bicgstab: non-finite residual");
                break;
            }
            if (rec.broke) {
                status = set_error(HISQ_EBREAKDOWN, "bicgstab: breakdown after %ld operator applications", B.matvecs);
                break;
            }
            Status s;
            s.lead = rec.lead;
            s.k = cycles;
            pace.update(s);
            if (rec.stop == STOP_NEVER) continue;
            // ---- reliable update ----
            inflight = 0;   // the cycle behind, if any, does nothing; its record is skipped
            pace.reset();
            HISQ_TRY(B.residual64(r64, x64, b64, &r2));
            rus++;
            if (!std::isfinite(r2)) {
                status = set_error(HISQ_EBREAKDOWN, "bicgstab: non-finite true residual");
                break;
            }
            if (r2 <= tol2) break;
            HISQ_TRY(B.restart(r64, false));
        }
    }
    if (status == HISQ_ENOCONV || status == HISQ_EBREAKDOWN) {
        double rf = 0.0;   // report the true residual of the iterate handed back
        if (B.residual64(r64, x64, b64, &rf) == HISQ_OK) r2 = rf;
    }
    hipLaunchKernelGGL(k_bl_merge, dim3(B.nbl), dim3(BL_BLOCK), 0, B.st, x, x64, g, L.fb64);
    hipError_t e = hipGetLastError();
    if (e == hipSuccess) e = hipStreamSynchronize(B.st);
    if (e != hipSuccess && status == HISQ_OK) status = set_error(HISQ_EHIP, "bicgstab: %s", hipGetErrorString(e));
    sto->status = status;
    sto->iters = (int)B.matvecs;
    sto->reliable_updates = (int)rus;
    sto->dslash_sloppy = (int)(2 * B.matvecs);
    sto->dslash_f64 = (int)(2 * B.f64apps);
    sto->true_resid = std::sqrt(r2 / b2);
    sto->alg_bytes = B.alg;
    sto->seconds = std::chrono::duration<double>(std::chrono::steady_clock::now() - t0).count();
    return status;
}
