// Conjugate-gradient vector kernels for the quadratic reconstruction
// (E^H E + lambda T^H T) x = b of Sec. IV-B: T = I (CG-SENSE) or T = the
// first differences along each image axis (QPLS), zero beyond the image
// edge; residual norm ||r|| / ||b|| of Sec. IV-A.  A launch serves a batch
// of independent images: one grid row per image, each with its own partial
// sums and scalars.
//
// Inner products are reduced deterministically: a fixed grid for a given
// length, one FP64 partial per block in a fixed order, and every kernel that
// uses a scalar sums the partials in a fixed order, so no host round trip is
// needed between iterations and a solve gives the same bits whatever else runs
// on the GPU.  An iteration takes three of these kernels; with the coil sum of
// E^H E p and the scalars in kernels of their own it took six, each bound by
// its launch and one round trip to memory (256^2, 8 coils: 20 -> 13 us of
// kernels an iteration, ten iterations 1054 -> 990 us).
#include <algorithm>

#include "kbn_internal.h"

namespace {

constexpr int TPB = 256;

// Sum over the workgroup in a fixed order: lanes of a wave by halving
// distances, then the waves in order.
__device__ inline double block_sum(double v, double *sh) {
    for (int off = 32; off > 0; off >>= 1) v += __shfl_down(v, off, 64);
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = v;
    __syncthreads();
    double s = sh[0];
#pragma unroll
    for (int w = 1; w < TPB / 64; ++w) s += sh[w];
    return s;
}

// Sum of an image's block partials, the same in every workgroup: the kernels
// that use a scalar sum the partials themselves (8 KB from L2) instead of
// waiting for a kernel that does.
__device__ inline double parts_sum(const double *__restrict__ part, int nparts, double *sh) {
    double acc = 0.0;
    for (int i = threadIdx.x; i < nparts; i += TPB) acc += part[i];
    return block_sum(acc, sh);
}

// x = 0, p = r, partial |r|^2
__global__ __launch_bounds__(TPB) void k_cg_init(float2 *__restrict__ x, const float2 *__restrict__ r,
                                                 float2 *__restrict__ p, int64_t n,
                                                 double *__restrict__ part) {
    __shared__ double sh[TPB / 64];
    const int64_t im = blockIdx.y;  // image of this block
    x += im * n;
    r += im * n;
    p += im * n;
    part += im * KBN_CG_PARTS;
    double acc = 0.0;
    for (int64_t i = (int64_t)blockIdx.x * TPB + threadIdx.x; i < n; i += (int64_t)gridDim.x * TPB) {
        const float2 v = r[i];
        x[i] = make_float2(0.f, 0.f);
        p[i] = v;
        acc += (double)v.x * v.x + (double)v.y * v.y;
    }
    const double s = block_sum(acc, sh);
    if (threadIdx.x == 0) part[blockIdx.x] = s;
}

// q = sum_c src[c] + lambda T^H T p, partial Re <p, q>.  src holds the C coil
// images of each image's E^H E p (C = 1: its sum, which may be q itself),
// added in coil order.  T = I, or (FD) the first differences along each axis:
// the path-graph Laplacian per axis, the sum over in-image neighbours of p_i -
// p_nb on an image [n0][n1][n2], row-major.
template <bool FD>
__global__ __launch_bounds__(TPB) void k_cg_q(float2 *q, const float2 *src, int C, const float2 *__restrict__ p,
                                              float lam, int n0, int n1, int n2, int64_t n,
                                              double *__restrict__ part) {
    __shared__ double sh[TPB / 64];
    const int64_t im = blockIdx.y;  // image of this block
    q += im * n;
    src += im * C * n;
    p += im * n;
    part += im * KBN_CG_PARTS;
    const int64_t s0 = (int64_t)n1 * n2;
    double acc = 0.0;
    for (int64_t i = (int64_t)blockIdx.x * TPB + threadIdx.x; i < n; i += (int64_t)gridDim.x * TPB) {
        const float2 c = p[i];
        float2 qv = src[i];
        for (int k = 1; k < C; ++k) {
            const float2 v = src[k * n + i];
            qv.x += v.x;
            qv.y += v.y;
        }
        float lx = c.x, ly = c.y;
        if (FD) {
            const int i2 = (int)(i % n2);
            const int64_t t = i / n2;
            const int i1 = (int)(t % n1);
            const int i0 = (int)(t / n1);
            lx = ly = 0.f;
            if (i0 > 0) { const float2 v = p[i - s0]; lx += c.x - v.x; ly += c.y - v.y; }
            if (i0 < n0 - 1) { const float2 v = p[i + s0]; lx += c.x - v.x; ly += c.y - v.y; }
            if (i1 > 0) { const float2 v = p[i - n2]; lx += c.x - v.x; ly += c.y - v.y; }
            if (i1 < n1 - 1) { const float2 v = p[i + n2]; lx += c.x - v.x; ly += c.y - v.y; }
            if (i2 > 0) { const float2 v = p[i - 1]; lx += c.x - v.x; ly += c.y - v.y; }
            if (i2 < n2 - 1) { const float2 v = p[i + 1]; lx += c.x - v.x; ly += c.y - v.y; }
        }
        qv.x += lam * lx;
        qv.y += lam * ly;
        q[i] = qv;
        acc += (double)c.x * qv.x + (double)c.y * qv.y;
    }
    const double s = block_sum(acc, sh);
    if (threadIdx.x == 0) part[blockIdx.x] = s;
}

// alpha = rr / <p, q> from the partials of k_cg_q (0 unless both are > 0),
// x += alpha p, r -= alpha q, partial |r|^2 (in the second half of the partials,
// the first being read).  Workgroup 0 keeps <p, q>, alpha and the previous rr.
__global__ __launch_bounds__(TPB) void k_cg_xr(float2 *__restrict__ x, float2 *__restrict__ r,
                                               const float2 *__restrict__ p,
                                               const float2 *__restrict__ q, double *scal, int64_t n,
                                               double *part) {
    __shared__ double sh[TPB / 64], sh2[TPB / 64];
    const int64_t im = blockIdx.y;  // image of this block
    x += im * n;
    r += im * n;
    p += im * n;
    q += im * n;
    scal += im * KBN_CG_NSCAL;
    part += im * KBN_CG_PARTS;
    const double rr = scal[KBN_CG_RR];
    const double pq = parts_sum(part, gridDim.x, sh);
    const double alpha = (pq > 0.0 && rr > 0.0) ? rr / pq : 0.0;
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        scal[KBN_CG_PQ] = pq;
        scal[KBN_CG_ALPHA] = alpha;
        scal[KBN_CG_RRPREV] = rr;
    }
    const float a = (float)alpha;
    double acc = 0.0;
    for (int64_t i = (int64_t)blockIdx.x * TPB + threadIdx.x; i < n; i += (int64_t)gridDim.x * TPB) {
        const float2 pv = p[i], qv = q[i];
        float2 xv = x[i], rv = r[i];
        xv.x += a * pv.x;
        xv.y += a * pv.y;
        rv.x -= a * qv.x;
        rv.y -= a * qv.y;
        x[i] = xv;
        r[i] = rv;
        acc += (double)rv.x * rv.x + (double)rv.y * rv.y;
    }
    const double s = block_sum(acc, sh2);
    if (threadIdx.x == 0) part[KBN_CG_MAXPARTS + blockIdx.x] = s;
}

// new rr from the partials of k_cg_xr, beta = rr / previous rr (0 unless that
// is > 0), p = r + beta p.  Workgroup 0 keeps rr, beta, ||r|| / ||b|| and the
// iteration count; no workgroup reads what it writes.
__global__ __launch_bounds__(TPB) void k_cg_p(float2 *__restrict__ p, const float2 *__restrict__ r, double *scal,
                                              int64_t n, const double *__restrict__ part) {
    __shared__ double sh[TPB / 64];
    const int64_t im = blockIdx.y;  // image of this block
    p += im * n;
    r += im * n;
    scal += im * KBN_CG_NSCAL;
    part += im * KBN_CG_PARTS + KBN_CG_MAXPARTS;
    const double prev = scal[KBN_CG_RRPREV];
    const double rr = parts_sum(part, gridDim.x, sh);
    const double beta = prev > 0.0 ? rr / prev : 0.0;
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        const double bb = scal[KBN_CG_BB];
        scal[KBN_CG_BETA] = beta;
        scal[KBN_CG_RR] = rr;
        scal[KBN_CG_REL] = bb > 0.0 ? sqrt(rr / bb) : 0.0;
        scal[KBN_CG_ITERS] += 1.0;
    }
    const float b = (float)beta;
    for (int64_t i = (int64_t)blockIdx.x * TPB + threadIdx.x; i < n; i += (int64_t)gridDim.x * TPB) {
        const float2 rv = r[i];
        float2 pv = p[i];
        pv.x = rv.x + b * pv.x;
        pv.y = rv.y + b * pv.y;
        p[i] = pv;
    }
}

// Start: rr = bb = |b|^2 from the partials of k_cg_init, rel = 1 (0 when b = 0).
__global__ __launch_bounds__(TPB) void k_cg_start(const double *__restrict__ part, int nparts,
                                                  double *__restrict__ scal) {
    __shared__ double sh[TPB / 64];
    const int64_t im = blockIdx.x;  // one block per image
    scal += im * KBN_CG_NSCAL;
    const double s = parts_sum(part + im * KBN_CG_PARTS, nparts, sh);
    if (threadIdx.x != 0) return;
    scal[KBN_CG_RR] = s;
    scal[KBN_CG_BB] = s;
    scal[KBN_CG_REL] = s > 0.0 ? 1.0 : 0.0;
    scal[KBN_CG_ITERS] = 0.0;
    scal[KBN_CG_ALPHA] = 0.0;
    scal[KBN_CG_BETA] = 0.0;
    scal[KBN_CG_PQ] = 0.0;
    scal[KBN_CG_RRPREV] = 0.0;
}

}  // namespace

int kbn_cg_nparts(int64_t n) {
    const int64_t b = (n + TPB - 1) / TPB;
    return (int)std::max<int64_t>(1, std::min<int64_t>(b, KBN_CG_MAXPARTS));
}

hipError_t kbn_launch_cg(int kind, int nimg, int64_t n, float2 *x, float2 *r, float2 *p, float2 *q, const float2 *src,
                         int C, float lam, KbnCgImage img, double *scal, double *part, hipStream_t s) {
    // one grid row per image; partials [nimg][KBN_CG_PARTS], scalars [nimg][KBN_CG_NSCAL]
    if (nimg < 1 || nimg > 65535) return hipErrorInvalidValue;
    const int g = kbn_cg_nparts(n);
    const dim3 grid(g, nimg);
    switch (kind) {
    case KBN_CGK_INIT:
        k_cg_init<<<grid, dim3(TPB), 0, s>>>(x, r, p, n, part);
        k_cg_start<<<dim3(nimg), dim3(TPB), 0, s>>>(part, g, scal);
        break;
    case KBN_CGK_Q:
        if (img.reg == KBN_REG_FINITE_DIFF) {
            if ((int64_t)img.n0 * img.n1 * img.n2 != n) return hipErrorInvalidValue;
            k_cg_q<true><<<grid, dim3(TPB), 0, s>>>(q, src, C, p, lam, img.n0, img.n1, img.n2, n, part);
        } else {
            k_cg_q<false><<<grid, dim3(TPB), 0, s>>>(q, src, C, p, lam, img.n0, img.n1, img.n2, n, part);
        }
        break;
    case KBN_CGK_XR:
        k_cg_xr<<<grid, dim3(TPB), 0, s>>>(x, r, p, q, scal, n, part);
        break;
    case KBN_CGK_P:
        k_cg_p<<<grid, dim3(TPB), 0, s>>>(p, r, scal, n, part);
        break;
    default:
        return hipErrorInvalidValue;
    }
    return hipGetLastError();
}
