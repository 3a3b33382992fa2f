// Kernels of the J-symmetric QMR-from-BCG iteration with J = T (arXiv 2103.00438, Section
// "Solution strategies", QMR paragraph, and the J-symmetry DA = A^T D of Eq. (a-matrix-d)).
//
// Because M^T T = T M for M = L T + z I, the BCG shadow sequence is T r_k and every inner product is
// the bilinear form x^T T y (no conjugation). Per step the only dense product is T r_k (a block
// product over all active systems); T p_k follows from the recurrence T p_k = T r_k + beta T p_{k-1},
// so M p_k = L (T p_k) + z p_k costs a sparse product only. The QMR iterate comes from the BCG one by
// quasi-minimal residual smoothing: 1/tau_k^2 = 1/tau_{k-1}^2 + 1/||r_k||^2, eta_k = tau_k^2/||r_k||^2,
// xq += eta_k (x_k - xq), s += eta_k (r_k - s).
//
// Vector slots of the per-system basis Q: 0 r, 1 p, 2 T p, 3 q = M p, 4 x (BCG), 5 xq (QMR), 6 s.
#include "device_util.h"
#include "krylov.h"

namespace wfq {

namespace {

__device__ inline double* slot(const Basis& V, int s, int j) {
    return V.base + (int64_t)s * V.sys_stride + (int64_t)j * V.vec_stride;
}

__device__ inline double block_sum4(double v, double* sh) {
    v = wave_sum(v);
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    __syncthreads();
    if (lane == 0) sh[wave] = v;
    __syncthreads();
    return sh[0] + sh[1] + sh[2] + sh[3];
}

// The sum of a system's nb block partials, formed by every work-group that needs it (staged in LDS, added in order):
// a launch of one thread per system for it took 2.7 to 3.7 us between kernels of 3 to 4 (4 100 atoms, 14 systems).
__device__ inline double2 ordered_sum(const double2* __restrict__ p, int nb, double2* sh) {
    double a = 0.0, b = 0.0;
    for (int b0 = 0; b0 < nb; b0 += 256) {
        __syncthreads();
        if ((int)threadIdx.x < nb - b0) sh[threadIdx.x] = p[b0 + threadIdx.x];
        __syncthreads();
        const int cnt = min(256, nb - b0);
#pragma unroll 8
        for (int q = 0; q < cnt; ++q) {
            a += sh[q].x;
            b += sh[q].y;
        }
    }
    return make_double2(a, b);
}

// partial rho = sum_i r_i (T r)_i, with T r in the packed block Y (rows 2k, 2k + 1)
template <typename YE>
__global__ void __launch_bounds__(256) rho_kernel(const YE* __restrict__ Y, int64_t ld, const int* __restrict__ sys,
                                                  Basis Q, int64_t n, double2* __restrict__ partial, int nblk) {
    __shared__ double sh[4];
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const int k = blockIdx.y;
    const int s = sys[k];
    double a = 0.0, b = 0.0;
    if (i < n) {
        const double* r = slot(Q, s, 0);
        const double rr = r[i], ri = r[i + Q.npad];
        const double tr = widen(Y[(int64_t)(2 * k) * ld + i]), ti = widen(Y[(int64_t)(2 * k + 1) * ld + i]);
        a = rr * tr - ri * ti;
        b = rr * ti + ri * tr;
    }
    a = block_sum4(a, sh);
    b = block_sum4(b, sh);
    if (threadIdx.x == 0) partial[(int64_t)s * nblk + blockIdx.x] = make_double2(a, b);
}

// rho_new = the sum of its partials; beta = rho_new / rho_old (0 on the first step); p = r + beta p; T p = T r + beta T p
template <typename YE>
__global__ void __launch_bounds__(256) dirs_kernel(const YE* __restrict__ Y, int64_t ld, const int* __restrict__ sys,
                                                   Basis Q, int64_t n, const double2* __restrict__ partial, int nblk,
                                                   double2* __restrict__ rho_new,
                                                   const double2* __restrict__ rho_old, const int* __restrict__ first,
                                                   double* __restrict__ tpb) {
    __shared__ double2 stage[256];
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const int k = blockIdx.y;
    const int s = sys[k];
    const double2 a = ordered_sum(partial + (int64_t)s * nblk, nblk, stage);
    if (i == 0) rho_new[s] = a;
    if (i >= n) return;
    double br = 0.0, bi = 0.0;
    if (!first[s]) {
        const double2 c = rho_old[s];
        const double dd = c.x * c.x + c.y * c.y;
        br = (a.x * c.x + a.y * c.y) / dd;
        bi = (a.y * c.x - a.x * c.y) / dd;
    }
    const double* r = slot(Q, s, 0);
    double* p = slot(Q, s, 1);
    double* tp = slot(Q, s, 2);
    const int64_t o = Q.npad;
    const double pr = p[i], pi = p[i + o];
    p[i] = r[i] + br * pr - bi * pi;
    p[i + o] = r[i + o] + br * pi + bi * pr;
    const double tr = widen(Y[(int64_t)(2 * k) * ld + i]), ti = widen(Y[(int64_t)(2 * k + 1) * ld + i]);
    const double qr = tp[i], qi = tp[i + o];
    const double nr = tr + br * qr - bi * qi, ni = ti + br * qi + bi * qr;
    tp[i] = nr;
    tp[i + o] = ni;
    reinterpret_cast<double2*>(tpb)[(int64_t)s * ld + i] = make_double2(nr, ni);   // interleaved for the SpMM
}

// partial sums over 256-row blocks of sigma = (T p)^T q, ||T p||^2 and ||q||^2
__global__ void __launch_bounds__(256) q_sums_kernel(int64_t n, const int* __restrict__ sys, Basis Q,
                                                     double2* __restrict__ part_sig, double2* __restrict__ part_nrm,
                                                     int nblk) {
    __shared__ double sh[4];
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const int s = sys[blockIdx.y];
    double sr = 0.0, si = 0.0, nt = 0.0, nq = 0.0;
    if (i < n) {
        const int64_t o = Q.npad;
        const double* tp = slot(Q, s, 2);
        const double* q = slot(Q, s, 3);
        const double qr = q[i], qi = q[i + o], tr = tp[i], ti = tp[i + o];
        sr = tr * qr - ti * qi;
        si = tr * qi + ti * qr;
        nt = tr * tr + ti * ti;
        nq = qr * qr + qi * qi;
    }
    sr = block_sum4(sr, sh);
    si = block_sum4(si, sh);
    nt = block_sum4(nt, sh);
    nq = block_sum4(nq, sh);
    if (threadIdx.x == 0) {
        part_sig[(int64_t)s * nblk + blockIdx.x] = make_double2(sr, si);
        part_nrm[(int64_t)s * nblk + blockIdx.x] = make_double2(nt, nq);
    }
}

// sigma = the sum of its partials, with the breakdown test (Lanczos breakdown: no look-ahead); x += alpha p,
// r -= alpha q with alpha = rho / sigma, and the partial sums of |r|^2
__global__ void __launch_bounds__(256) xr_kernel(const int* __restrict__ sys, Basis Q, int64_t n,
                                                 const double2* __restrict__ part_sig, const double2* __restrict__ part_nrm,
                                                 const double2* __restrict__ rho, int* __restrict__ flags, double thr,
                                                 double* __restrict__ norm2, int nblk) {
    __shared__ double sh[4];
    __shared__ double2 stage[256];
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const int s = sys[blockIdx.y];
    const double2 a = rho[s], c = ordered_sum(part_sig + (int64_t)s * nblk, nblk, stage);
    if (blockIdx.x == 0) {
        const double2 nrm = ordered_sum(part_nrm + (int64_t)s * nblk, nblk, stage);
        int f = 0;
        const double sabs = hypot(c.x, c.y), rabs = hypot(a.x, a.y);
        if (!(sabs > thr * sqrt(nrm.x * nrm.y)) || !(rabs > 0.0)) f |= 8;
        if (!(sabs == sabs) || !(rabs == rabs)) f |= 4;
        if (threadIdx.x == 0) flags[s] = f;
    }
    // contracted by hand, so that the rounding does not depend on where the compiler takes sigma from
    const double dd = fma(c.x, c.x, c.y * c.y);
    const double alr = fma(c.x, a.x, a.y * c.y) / dd, ali = fma(a.y, c.x, -(a.x * c.y)) / dd;
    double nn = 0.0;
    if (i < n) {
        const int64_t o = Q.npad;
        double* r = slot(Q, s, 0);
        const double* p = slot(Q, s, 1);
        const double* q = slot(Q, s, 3);
        double* x = slot(Q, s, 4);
        const double pr = p[i], pi = p[i + o], qr = q[i], qi = q[i + o];
        x[i] += fma(alr, pr, -(ali * pi));
        x[i + o] += fma(alr, pi, ali * pr);
        const double rr = r[i] - fma(alr, qr, -(ali * qi)), ri = r[i + o] - fma(ali, qr, alr * qi);
        r[i] = rr;
        r[i + o] = ri;
        nn = fma(rr, rr, ri * ri);
    }
    nn = block_sum4(nn, sh);
    if (threadIdx.x == 0) norm2[(int64_t)s * nblk + blockIdx.x] = nn;
}

// smoothing weights from the new BCG residual norm (the sum of its partials): 1 / tau'^2 = 1 / tau^2 + 1 / |r|^2, eta =
// tau'^2 / |r|^2; xq += eta (x - xq); s += eta (r - s); partial ||s||^2. tau^2 goes from one array to another, since every
// work-group of a system reads the old one; the first-step flag is cleared.
__global__ void __launch_bounds__(256) smooth_kernel(const int* __restrict__ sys, Basis Q, int64_t n,
                                                     const double* __restrict__ rn_part, const double* __restrict__ tau2,
                                                     double* __restrict__ tau2_new, int* __restrict__ first,
                                                     double* __restrict__ norm2, int nblk) {
    __shared__ double sh[4];
    __shared__ double stage[256];
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const int s = sys[blockIdx.y];
    double nr = 0.0;
    for (int b0 = 0; b0 < nblk; b0 += 256) {
        __syncthreads();
        if ((int)threadIdx.x < nblk - b0) stage[threadIdx.x] = rn_part[(int64_t)s * nblk + b0 + threadIdx.x];
        __syncthreads();
        const int cnt = min(256, nblk - b0);
#pragma unroll 8
        for (int q = 0; q < cnt; ++q) nr += stage[q];
    }
    const double t2 = tau2[s];
    const double t2n = nr > 0.0 ? 1.0 / (1.0 / t2 + 1.0 / nr) : 0.0;
    const double e = nr > 0.0 ? t2n / nr : 1.0;
    if (i == 0) {
        tau2_new[s] = t2n;
        first[s] = 0;
    }
    double nn = 0.0;
    if (i < n) {
        const int64_t o = Q.npad;
        const double* x = slot(Q, s, 4);
        double* xq = slot(Q, s, 5);
        const double* r = slot(Q, s, 0);
        double* sv = slot(Q, s, 6);
        xq[i] += e * (x[i] - xq[i]);
        xq[i + o] += e * (x[i + o] - xq[i + o]);
        const double a = sv[i] + e * (r[i] - sv[i]), b = sv[i + o] + e * (r[i + o] - sv[i + o]);
        sv[i] = a;
        sv[i + o] = b;
        nn = a * a + b * b;
    }
    nn = block_sum4(nn, sh);
    if (threadIdx.x == 0) norm2[(int64_t)s * nblk + blockIdx.x] = nn;
}

// restart: x = xq; p = 0, T p = 0; s = r (r holds the FP64 residual of xq)
__global__ void __launch_bounds__(256) restart_kernel(const int* __restrict__ sys, Basis Q, int64_t npad) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const int s = sys[blockIdx.y];
    for (int h = 0; h < 2; ++h) {
        const int64_t j = i + h * npad;
        slot(Q, s, 4)[j] = slot(Q, s, 5)[j];
        slot(Q, s, 1)[j] = 0.0;
        slot(Q, s, 2)[j] = 0.0;
        slot(Q, s, 6)[j] = slot(Q, s, 0)[j];
    }
}
}  // namespace

void qmr_rho(bool y_is_f64, const void* Y, int64_t ld, const int* sys, int nsys, const Basis& Q, int64_t n,
             double2* partial, int nblk, hipStream_t st) {
    if (nsys <= 0) return;
    dim3 grd((unsigned)nblk, (unsigned)nsys);
    if (y_is_f64)
        hipLaunchKernelGGL(rho_kernel<double>, grd, dim3(256), 0, st, static_cast<const double*>(Y), ld, sys, Q, n,
                           partial, nblk);
    else
        hipLaunchKernelGGL(rho_kernel<float>, grd, dim3(256), 0, st, static_cast<const float*>(Y), ld, sys, Q, n,
                           partial, nblk);
    WFQ_CHECK_LAUNCH();
}

void qmr_dirs(bool y_is_f64, const void* Y, int64_t ld, const int* sys, int nsys, const Basis& Q, int64_t n,
              const double2* partial, int nblk, double2* rho_new, const double2* rho_old, const int* first, double* tpb, hipStream_t st) {
    if (nsys <= 0) return;
    dim3 grd((unsigned)((n + 255) / 256), (unsigned)nsys);
    if (y_is_f64)
        hipLaunchKernelGGL(dirs_kernel<double>, grd, dim3(256), 0, st, static_cast<const double*>(Y), ld, sys, Q, n,
                           partial, nblk, rho_new, rho_old, first, tpb);
    else
        hipLaunchKernelGGL(dirs_kernel<float>, grd, dim3(256), 0, st, static_cast<const float*>(Y), ld, sys, Q, n,
                           partial, nblk, rho_new, rho_old, first, tpb);
    WFQ_CHECK_LAUNCH();
}

void qmr_q(const Structure& S, const int* sys, int nsys, const Basis& Q, const double2* z, const double* tpb,
           double2* part_sig, double2* part_nrm, int nblk, hipStream_t st) {
    if (nsys <= 0) return;
    // q (slot 3) = L (T p) + z p (slot 1), gathering T p from the compact interleaved block that
    // qmr_dirs wrote (one pair of doubles per atom and system)
    spmm_shift_interleaved(S, tpb, S.npad, sys, nsys, z, Q, 1, 3, st);
    dim3 grd((unsigned)nblk, (unsigned)nsys);
    hipLaunchKernelGGL(q_sums_kernel, grd, dim3(256), 0, st, S.n, sys, Q, part_sig, part_nrm, nblk);
    WFQ_CHECK_LAUNCH();
}

void qmr_xr(const int* sys, int nsys, const Basis& Q, int64_t n, const double2* part_sig, const double2* part_nrm,
            const double2* rho, int* flags, double thr, double* norm2, int nblk, hipStream_t st) {
    if (nsys <= 0) return;
    dim3 grd((unsigned)nblk, (unsigned)nsys);
    hipLaunchKernelGGL(xr_kernel, grd, dim3(256), 0, st, sys, Q, n, part_sig, part_nrm, rho, flags, thr, norm2, nblk);
    WFQ_CHECK_LAUNCH();
}

void qmr_smooth(const int* sys, int nsys, const Basis& Q, int64_t n, const double* rn_part, const double* tau2,
                double* tau2_new, int* first, double* norm2, int nblk, hipStream_t st) {
    if (nsys <= 0) return;
    dim3 grd((unsigned)nblk, (unsigned)nsys);
    hipLaunchKernelGGL(smooth_kernel, grd, dim3(256), 0, st, sys, Q, n, rn_part, tau2, tau2_new, first, norm2, nblk);
    WFQ_CHECK_LAUNCH();
}

void qmr_restart(const int* sys, int nsys, const Basis& Q, hipStream_t st) {
    if (nsys <= 0) return;
    dim3 grd((unsigned)(Q.npad / 256), (unsigned)nsys);
    hipLaunchKernelGGL(restart_kernel, grd, dim3(256), 0, st, sys, Q, Q.npad);
    WFQ_CHECK_LAUNCH();
}

}  // namespace wfq
