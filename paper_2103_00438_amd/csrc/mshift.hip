// Multi-shift GMRES: one Krylov basis for every frequency of a field direction.
//
// The scaled system (L T + z I) q = b_k has a real, frequency-independent matrix L T; the frequency
// only enters as the uniform complex diagonal shift z (arXiv 2103.00438, the remark after Eq.
// wfq-a-matrix), and b_k = E0 L r_k does not depend on it. Krylov spaces are invariant under such
// shifts (the conclusions point to this property for spectra): with the Arnoldi relation
// A V_k = V_{k+1} Hbar_k of A = L T started from b_k,
//     (A + z I) V_k = V_{k+1} (Hbar_k + z Ibar_k),   Ibar_k = [I_k; 0],
// so the GMRES iterate of every shifted system is x = V_k y_z with y_z the least-squares solution of
// (Hbar_k + z Ibar_k) y ~ ||b_k|| e_1. A and b_k are real, hence V and Hbar are real: one real
// Arnoldi process per direction (one T product on a real vector per step, shared by all
// frequencies) and one small complex Givens recurrence per (frequency, direction) system.
//
// Layouts: basis of direction d, slot j at V + (d * mdim1 + j) * npad (FP64, padding rows zero); the
// kept products T u_j (FP64 solves) in the same layout; Hessenberg column j of direction d at
// H + (d * m + j) * (m + 1) (entries 0..j+1), and the triangular factor S of U = Q S likewise.
// Per-system arrays are system-minor (entry e of system s at e * S + s, S = systems of the batch):
// rotations cs/sn (m entries), g (m + 1), R packed by columns (column j from entry j (j + 1) / 2).
// The phase's own orthogonalisation is the one-reduction form below (ms_dcgs_*); ms_dot and ms_update
// serve the starting norms and the relaxed phase's product-error probe.
#include <algorithm>
#include <type_traits>

#include "device_util.h"
#include "krylov.h"

namespace wfq {

namespace {

// (the fused products are named: left to the compiler, they change with the code around a call)
__device__ inline double2 cmul(double2 a, double2 b) {
    return make_double2(fma(a.x, b.x, -(a.y * b.y)), fma(a.x, b.y, a.y * b.x));
}
__device__ inline double2 cconj(double2 a) { return make_double2(a.x, -a.y); }
__device__ inline double2 cadd(double2 a, double2 b) { return make_double2(a.x + b.x, a.y + b.y); }
__device__ inline double2 csub(double2 a, double2 b) { return make_double2(a.x - b.x, a.y - b.y); }
__device__ inline double2 cscale(double c, double2 a) { return make_double2(c * a.x, c * a.y); }
__device__ inline double cabs(double2 a) { return hypot(a.x, a.y); }
__device__ inline double2 cdiv(double2 a, double2 b) {
    const double d = b.x * b.x + b.y * b.y;
    return make_double2((a.x * b.x + a.y * b.y) / d, (a.y * b.x - a.x * b.y) / d);
}

// divide by, and multiply with, an entry of a real or a complex triangle
__device__ inline double2 tri_div(double2 a, double b) { return cscale(1.0 / b, a); }
__device__ inline double2 tri_div(double2 a, double2 b) { return cdiv(a, b); }
__device__ inline double2 tri_mul(double a, double2 b) { return cscale(a, b); }
__device__ inline double2 tri_mul(double2 a, double2 b) { return cmul(a, b); }

__device__ inline double* slot(double* V, int64_t npad, int mdim1, int d, int j) {
    return V + ((int64_t)d * mdim1 + j) * npad;
}

// 1 / |p| from the block sums of p^2 that the update sweep left in norm[0 .. nblk - 1] (fixed order; 0 when p = 0),
// computed by a whole wave; nrm receives |p|
__device__ inline double inv_norm(const double* __restrict__ norm, int64_t nblk, double& nrm) {
    double s0 = 0.0, s1 = 0.0;
    for (int64_t q = threadIdx.x & 63; q < nblk; q += 128) {
        s0 += norm[q];
        s1 += q + 64 < nblk ? norm[q + 64] : 0.0;
    }
    nrm = sqrt(wave_sum(s0) + wave_sum(s1));
    return nrm > 0.0 ? 1.0 / nrm : 0.0;
}

// X[c][i] = cast(v) with v = V(d_c, j)[i] / |V(d_c, j)|, which is also written back (normalises the
// new basis vector on its way into the product). The norm comes from its block sums, which every wave adds
// for itself (nu and inv_h keep it for the step's other kernels), or, without them, 1 / norm is inv_h[d].
template <typename E>
__global__ void __launch_bounds__(256) ms_pack_kernel(double* __restrict__ V, int64_t npad, int mdim1, int j,
                                                      DirList dirs, const double* __restrict__ norm,
                                                      double* __restrict__ nu, double* __restrict__ inv_h,
                                                      E* __restrict__ X, int64_t ld) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const int c = blockIdx.y;
    const int d = dirs[c];
    double* v = slot(V, npad, mdim1, d, j);
    const double x = v[i];
    double sc, nrm;
    if (norm) {
        sc = inv_norm(norm + (int64_t)d * (npad / 64), npad / 64, nrm);
        if (i == 0) {
            nu[d] = nrm;
            inv_h[d] = sc;
        }
    } else {
        sc = inv_h[d];
    }
    const double a = x * sc;
    v[i] = a;
    X[(int64_t)c * ld + i] = cast_from_double<E>(a);
}

// The product of a small stored FP64 T with the newest basis vectors, taken straight from the basis:
// Y[c][i] = sum_k T[i][k] v_c[k], v_c = V(d_c, j) / |V(d_c, j)|. One launch in place of the pack, the product and the
// norm's reduction, whose latencies bound a step of a few thousand atoms (600 atoms, 3 directions: 4.7 + 5.6 + 2.3 us,
// now 5.1). A wave owns kMsRowsT rows of T and sums as tx_skinny_kernel does; every work-group adds the norms'
// block sums for itself while its first rows of T are on their way. The basis vectors are normalised in registers
// and stay as they are in memory until ms_spmm.
constexpr int kMsRowsT = 2;
template <int NC>
__global__ void __launch_bounds__(256) ms_skinny_kernel(const double* __restrict__ T, int64_t npad,
                                                        const double* __restrict__ V, int mdim1, int j,
                                                        DirList dirs, const double* __restrict__ norm,
                                                        double* __restrict__ nu, double* __restrict__ inv_h,
                                                        double* __restrict__ Y) {
    constexpr int R = kMsRowsT;
    __shared__ double inv[4];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int64_t row0 = ((int64_t)blockIdx.x * 4 + wave) * R;
    if (wave < NC) {   // wave c: the norm of column c
        const int d = dirs[wave];
        double sc, nrm;
        if (norm) {
            sc = inv_norm(norm + (int64_t)d * (npad / 64), npad / 64, nrm);
            if (blockIdx.x == 0 && lane == 0) {
                nu[d] = nrm;
                inv_h[d] = sc;
            }
        } else {
            sc = inv_h[d];
        }
        if (lane == 0) inv[wave] = sc;
    }
    const double* u[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c) u[c] = V + ((int64_t)dirs[c] * mdim1 + j) * npad;
    __syncthreads();
    double sc[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c) sc[c] = inv[c];
    double acc[R][NC];
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
        for (int c = 0; c < NC; ++c) acc[r][c] = 0.0;
#pragma unroll 4
    for (int64_t k = 2 * lane; k < npad; k += 128) {
        double2 x[NC], t[R];
#pragma unroll
        for (int r = 0; r < R; ++r) t[r] = *reinterpret_cast<const double2*>(T + (row0 + r) * npad + k);
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            x[c] = *reinterpret_cast<const double2*>(u[c] + k);
            x[c] = make_double2(x[c].x * sc[c], x[c].y * sc[c]);
        }
#pragma unroll
        for (int r = 0; r < R; ++r)
#pragma unroll
            for (int c = 0; c < NC; ++c) acc[r][c] = fma(t[r].y, x[c].y, fma(t[r].x, x[c].x, acc[r][c]));
    }
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            const double s = wave_sum(acc[r][c]);
            if (lane == 0) Y[(int64_t)c * npad + row0 + r] = s;
        }
}

// V(d_c, jdst) = L Y[c] for the NC columns c0 .. c0 + NC - 1 (real ELL rows, each entry read once
// for all columns; padding rows get 0), with TV(d_c, jdst - 1) = Y[c] kept and, with scale, V(d_c, jdst - 1) *=
// scale[d_c] (a basis vector that entered its product unnormalised).
template <typename YE, int NC>
__global__ void __launch_bounds__(256) ms_spmm_kernel(int64_t n, int64_t npad, int w, const int32_t* __restrict__ ecol,
                                                      const double* __restrict__ eval, const YE* __restrict__ Y,
                                                      int64_t ld, DirList dirs, double* __restrict__ V,
                                                      int mdim1, int jdst, int c0, double* __restrict__ TV,
                                                      const double* __restrict__ Yi, const double* __restrict__ scale) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    double acc[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c) acc[c] = 0.0;
    const YE* y = Y + (int64_t)c0 * ld;
    if (i < n) {
        if (Yi) {
            // the interleaved copy: all columns of neighbour j in one aligned 32-byte load
#pragma unroll 4
            for (int e = 0; e < w; ++e) {
                const double v = eval[(int64_t)e * npad + i];
                const int64_t j = ecol[(int64_t)e * npad + i];
                const doublex4 yj = *reinterpret_cast<const doublex4*>(Yi + 4 * j);
                const double yv[4] = {yj.x, yj.y, yj.z, yj.w};
#pragma unroll
                for (int c = 0; c < NC; ++c) acc[c] += v * yv[c];
            }
        } else {
#pragma unroll 4
            for (int e = 0; e < w; ++e) {
                const double v = eval[(int64_t)e * npad + i];
                const int64_t j = ecol[(int64_t)e * npad + i];
#pragma unroll
                for (int c = 0; c < NC; ++c) acc[c] += v * widen(y[c * ld + j]);
            }
        }
    }
#pragma unroll
    for (int c = 0; c < NC; ++c) {
        const int d = dirs[c0 + c];
        slot(V, npad, mdim1, d, jdst)[i] = acc[c];
        if (TV) slot(TV, npad, mdim1, d, jdst - 1)[i] = i < n ? widen(y[c * ld + i]) : 0.0;
        if (scale) slot(V, npad, mdim1, d, jdst - 1)[i] *= scale[d];
    }
}

// The same for structures of a few thousand rows, where the time is the latency of a row's chain and not the
// entries' traffic: 16 rows per work-group, their entries staged in LDS by all its threads at once (chunks of kMsEnt), so that a
// lane waits for gathers alone, and one column per lane group of 16 (600 atoms, 3 columns: 7.7 us, now 4.7).
constexpr int kMsEnt = 128;
template <typename YE, int NC>
__global__ void __launch_bounds__(64) ms_spmm_small_kernel(int64_t n, int64_t npad, int w, const int32_t* __restrict__ ecol,
                                                           const double* __restrict__ eval, const YE* __restrict__ Y,
                                                           int64_t ld, DirList dirs, double* __restrict__ V, int mdim1,
                                                           int jdst, double* __restrict__ TV,
                                                           const double* __restrict__ scale) {
    __shared__ double lval[kMsEnt * 16];
    __shared__ int32_t lcol[kMsEnt * 16];
    const int r = threadIdx.x & 15, c = threadIdx.x >> 4;
    const int64_t i0 = (int64_t)blockIdx.x * 16, i = i0 + r;
    const YE* y = Y + (int64_t)min(c, NC - 1) * ld;
    double acc = 0.0;
    for (int e0 = 0; e0 < w; e0 += kMsEnt) {
        const int en = min(kMsEnt, w - e0);
        __syncthreads();
#pragma unroll 8
        for (int q = threadIdx.x; q < en * 16; q += 64) {
            const int64_t at = (int64_t)(e0 + (q >> 4)) * npad + i0 + (q & 15);
            lcol[q] = ecol[at];
            lval[q] = eval[at];
        }
        __syncthreads();
#pragma unroll 16
        for (int e = 0; e < en; ++e) acc += lval[e * 16 + r] * widen(y[lcol[e * 16 + r]]);
    }
    if (c >= NC) return;
    const int d = dirs[c];
    const bool in = i < n;
    slot(V, npad, mdim1, d, jdst)[i] = in ? acc : 0.0;
    if (TV) slot(TV, npad, mdim1, d, jdst - 1)[i] = in ? widen(y[i]) : 0.0;
    if (scale) slot(V, npad, mdim1, d, jdst - 1)[i] *= scale[d];
}

// partial[d][i][wc] = sum over wave chunk wc (512 rows) of V(d, i) * V(d, jw) for i < nvec; with
// self_norm also partial[d][nvec][wc] = sum of V(d, jw)^2. One wave per (chunk, vector): the
// launch has thousands of waves even for one direction, and each sum has a fixed order.
__global__ void __launch_bounds__(256) ms_dot_kernel(const double* __restrict__ V, int64_t n, int64_t npad, int mdim1,
                                                     int nvec, int jw, DirList dirs,
                                                     double* __restrict__ partial, int pslots, int64_t nwc,
                                                     int self_norm) {
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int64_t wc = blockIdx.x;
    const int i = blockIdx.y * 4 + wave;
    if (i >= nvec + self_norm) return;
    const int d = dirs[blockIdx.z];
    const double* w = V + ((int64_t)d * mdim1 + jw) * npad;
    const double* v = i < nvec ? V + ((int64_t)d * mdim1 + i) * npad : w;
    const int64_t row0 = wc * kWaveRows + lane;
    double s = 0.0;
#pragma unroll
    for (int r = 0; r < 8; ++r) {
        const int64_t row = row0 + 64 * r;
        if (row < n) s += v[row] * w[row];
    }
    s = wave_sum(s);
    if (lane == 0) partial[((int64_t)d * pslots + i) * nwc + wc] = s;
}

// h[d][i] = sum_wc partial[d][i][wc], i < count: one wave per (value, direction); lane l adds the
// chunks l, l + 64, ... and the lanes are combined by a fixed butterfly (same order every call)
__global__ void __launch_bounds__(256) ms_reduce_kernel(DirList dirs, const double* __restrict__ partial,
                                                        int pslots, int64_t nwc, int count, double* __restrict__ h) {
    const int d = dirs[blockIdx.y];
    const int i = blockIdx.x * 4 + (threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    if (i >= count) return;   // uniform over the wave
    const double* p = partial + ((int64_t)d * pslots + i) * nwc;
    double s = 0.0;
    for (int64_t q = lane; q < nwc; q += 64) s += p[q];
    s = wave_sum(s);
    if (lane == 0) h[(int64_t)d * pslots + i] = s;
}

// V(d, jw) -= sum_{i < nvec} h[d][i] V(d, i); with norm != NULL also norm[d][blk] = the sum of
// V(d, jw)^2 over the 64 rows of block blk. A block owns 64 rows; its 4 waves take every 4th basis
// vector and their partial sums are combined in LDS in a fixed order.
constexpr int kMsRows = 64;
__global__ void __launch_bounds__(256) ms_update_kernel(double* __restrict__ V, int64_t n, int64_t npad, int mdim1,
                                                        int nvec, int jw, DirList dirs,
                                                        const double* __restrict__ h, int pslots,
                                                        double* __restrict__ norm) {
    __shared__ double part[4][kMsRows];
    const int r = threadIdx.x & 63, q = threadIdx.x >> 6;
    const int64_t row = (int64_t)blockIdx.x * kMsRows + r;
    const int d = dirs[blockIdx.y];
    const double* hd = h + (int64_t)d * pslots;
    double acc = 0.0;
    if (row < n) {
#pragma unroll 4
        for (int i = q; i < nvec; i += 4) acc += hd[i] * V[((int64_t)d * mdim1 + i) * npad + row];
    }
    part[q][r] = acc;
    __syncthreads();
    if (q == 0) {
        double* w = V + ((int64_t)d * mdim1 + jw) * npad;
        double x = 0.0;
        if (row < n) {
            x = w[row] - ((part[0][r] + part[1][r]) + (part[2][r] + part[3][r]));
            w[row] = x;
        }
        if (norm) {
            const double s2 = wave_sum_sq(x);
            if (r == 0) norm[(int64_t)d * (npad / kMsRows) + blockIdx.x] = s2;
        }
    }
}

// ---- Arnoldi with one reduction per step on the real basis of each direction: classical
// Gram-Schmidt with delayed reorthogonalisation (DCGS2, Swirydowicz, Langou, Ananthan, Yang and
// Thomas 2020), the real counterpart of the batched GMRES's. At step k, q_0 .. q_{k-1} are final,
// slot k holds u (the previous step's once-projected vector p, normalised by the pack) and slot
// k + 1 holds z = A u. One sweep gives a = Q^T u, alpha = u^T u, b = Q^T z and beta = u^T z
// (dots[d][e]: e = t < k: a_t; e = k: alpha; e = k + 1 + t: b_t; e = 2 k + 1: beta); then with
// rho = sqrt(alpha - |a|^2) and nu = |p|:
//   q_k = (u - Q a) / rho;  H(0:k-1, k-1) = hp + nu a,  H(k, k-1) = nu rho   (column k-1 complete)
//   gamma = q_k^T z = (beta - a^T b) / rho;  p' = (z - Q b - gamma q_k) / rho
//   hp'(0:k-1) = (b - (Hbar a)(0:k-1)) / rho,  hp'(k) = (gamma - H(k, k-1) a_{k-1}) / rho
// since A q_k = (z - Q_{k+1} Hbar a) / rho by A Q_k = Q_{k+1} Hbar. The basis is read twice per step
// instead of four times; column k-1 is complete (and its Givens step taken) at step k, and a last
// step without product completes column m-1. As u_k = rho q_k + Q a, the vectors that entered the
// products relate to the final basis by U = Q S with S upper triangular (S(t, k) = a_t,
// S(k, k) = rho), kept column by column in the layout of H when the products T u_k are kept.

// partial[d][e][wc] for the entries e above over wave chunk wc (512 rows). One wave per (chunk, group
// of kGroup basis vectors t <= k, direction): u and z of the chunk stay in registers while the
// wave computes v_t . u and v_t . z for its vectors (t = k: alpha and beta). 16 vectors per wave where that fills
// the chip, 4 where a wave's chain of vectors is the time (ms_dcgs_dot).
template <int kGroup>
__global__ void __launch_bounds__(256) ms_dcgs_dot_kernel(const double* __restrict__ V, int64_t n, int64_t npad,
                                                          int mdim1, int k, int with_z, DirList dirs,
                                                          double* __restrict__ partial, int ps, int64_t nwc) {
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int64_t wc = (int64_t)blockIdx.x * 4 + wave;
    if (wc >= nwc) return;   // uniform over the wave
    const int t0 = blockIdx.y * kGroup, t1 = min(t0 + kGroup, k + 1);
    const int d = dirs[blockIdx.z];
    const double* u = V + ((int64_t)d * mdim1 + k) * npad;
    const double* zv = u + npad;   // slot k + 1 (read only with z)
    const int64_t row0 = wc * kWaveRows + lane;
    double xu[8], xz[8];
#pragma unroll
    for (int r = 0; r < 8; ++r) {
        const int64_t row = row0 + 64 * r;
        xu[r] = row < n ? u[row] : 0.0;
        xz[r] = (with_z && row < n) ? zv[row] : 0.0;
    }
    double* P = partial + (int64_t)d * ps * nwc + wc;
#pragma unroll 2
    for (int t = t0; t < t1; ++t) {
        const double* v = V + ((int64_t)d * mdim1 + t) * npad;
        double sa = 0.0, sb = 0.0;
#pragma unroll
        for (int r = 0; r < 8; ++r) {
            const int64_t row = row0 + 64 * r;
            const double x = row < n ? v[row] : 0.0;
            sa += x * xu[r];
            sb += x * xz[r];
        }
        sa = wave_sum(sa);
        sb = wave_sum(sb);
        if (lane == 0) {
            P[(int64_t)t * nwc] = sa;
            if (with_z) P[(int64_t)(k + 1 + t) * nwc] = sb;
        }
    }
}

// sum over the work-group of one value per thread, in a fixed order (waves' sums in order)
__device__ inline double block_sum256(double x, double* red) {
    x = wave_sum(x);
    __syncthreads();
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = x;
    __syncthreads();
    return (red[0] + red[1]) + (red[2] + red[3]);
}

// One work-group per direction: column k-1 of H (k >= 1), column k of S (with z, S != NULL), and with
// z gamma and 1 / rho. With z the step's product has left nu[d] = |p|; without (the last step, k >= 1) u is the
// unnormalised p, whose dots are scaled by 1 / |p| from its block sums.
__global__ void __launch_bounds__(256) ms_dcgs_coeff_kernel(DirList dirs, int k, int with_z, int m,
                                                            const double* __restrict__ dots, int ps,
                                                            double* __restrict__ hp, double* __restrict__ H,
                                                            double* __restrict__ Sm, const double* __restrict__ nu,
                                                            const double* __restrict__ norm, int64_t nblk,
                                                            double* __restrict__ gam, double* __restrict__ inv_rho) {
    __shared__ double red[4];
    const int d = dirs[blockIdx.x];
    const int tid = threadIdx.x;
    const double* dt = dots + (int64_t)d * ps;
    double* hpd = hp + (int64_t)d * (m + 1);
    double nud = 0.0, sc = 1.0;
    if (with_z)
        nud = nu[d];
    else
        sc = inv_norm(norm + (int64_t)d * nblk, nblk, nud);
    double asq = 0.0;
    for (int i = tid; i < k; i += 256) {
        const double ai = sc * dt[i];
        asq += ai * ai;
    }
    asq = block_sum256(asq, red);
    const double r2 = dt[k] * sc * sc - asq;
    const double rho = r2 > 0.0 ? sqrt(r2) : 0.0;
    if (k >= 1) {
        double* col = H + ((int64_t)d * m + (k - 1)) * (m + 1);
        for (int i = tid; i < k; i += 256) col[i] = hpd[i] + nud * sc * dt[i];
        if (tid == 0) col[k] = nud * rho;
    }
    if (!with_z) return;
    if (Sm) {
        double* sk = Sm + ((int64_t)d * m + k) * (m + 1);
        for (int i = tid; i < k; i += 256) sk[i] = dt[i];
        if (tid == 0) sk[k] = rho;
    }
    double ab = 0.0;
    for (int i = tid; i < k; i += 256) ab += dt[i] * dt[k + 1 + i];
    ab = block_sum256(ab, red);
    const double ir = rho > 0.0 ? 1.0 / rho : 0.0;
    if (tid == 0) {
        gam[d] = (dt[2 * k + 1] - ab) * ir;
        inv_rho[d] = ir;
    }
}

// The next column's first-pass coefficients, hp(i) = (b_i - (Hbar a)_i) / rho for i < k and
// hp(k) = (gamma - H(k, k-1) a_{k-1}) / rho, after column k-1 of H is complete. One work-group of
// 16 waves per (64 rows, direction): lane = row, wave w adds the columns c = w, w + 16, ... (Hbar is
// upper Hessenberg: c >= i - 1 only), and the 16 partial sums are added in order.
__global__ void __launch_bounds__(1024) ms_dcgs_hp_kernel(DirList dirs, int k, int m,
                                                          const double* __restrict__ dots, int ps,
                                                          const double* __restrict__ H, const double* __restrict__ gam,
                                                          const double* __restrict__ inv_rho, double* __restrict__ hp) {
    __shared__ double red[16][64];
    const int d = dirs[blockIdx.y];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int i = blockIdx.x * 64 + lane;
    const double* dt = dots + (int64_t)d * ps;
    const double* Hd = H + (int64_t)d * m * (m + 1);
    const int c0 = max(0, (int)blockIdx.x * 64 - 1);
    double acc = 0.0;
    if (i < k) {
#pragma unroll 4
        for (int c = c0 + wave; c < k; c += 16)
            if (c >= i - 1) acc += Hd[(int64_t)c * (m + 1) + i] * dt[c];
    }
    red[wave][lane] = acc;
    __syncthreads();
    if (wave == 0 && i <= k) {
        const double ir = inv_rho[d];
        double* hpd = hp + (int64_t)d * (m + 1);
        if (i < k) {
            double s = 0.0;
#pragma unroll
            for (int w = 0; w < 16; ++w) s += red[w][lane];
            hpd[i] = (dt[k + 1 + i] - s) * ir;
        } else {
            const double last = k >= 1 ? Hd[(int64_t)(k - 1) * (m + 1) + k] * dt[k - 1] : 0.0;
            hpd[k] = (gam[d] - last) * ir;
        }
    }
}

// The three kernels between the two sweeps (reduction of the dots, ms_dcgs_coeff, ms_dcgs_hp) as one, for a
// few hundred basis vectors of up to some tens of chunks: one work-group of 16 waves per direction. The dots
// are reduced into LDS (and global memory, for the update sweep), the norms and scalar products in one pass, and
// H a row block by row block as in ms_dcgs_hp_kernel, with column k-1 taken from LDS.
constexpr int kStepMax = 384;   // largest k; above, the three kernels' parallelism over H pays
__global__ void __launch_bounds__(1024) ms_dcgs_step_kernel(DirList dirs, int k, int with_z, int m,
                                                            const double* __restrict__ partial, int ps, int64_t nwc,
                                                            const double* __restrict__ nu,
                                                            const double* __restrict__ norm, int64_t nblk,
                                                            double* __restrict__ dots, double* __restrict__ hp,
                                                            double* __restrict__ H, double* __restrict__ Sm,
                                                            double* __restrict__ gam, double* __restrict__ inv_rho) {
    __shared__ double sd[2 * kStepMax + 2], hcol[kStepMax + 1], red[16][64], part[2][4];
    const int d = dirs[blockIdx.x];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    double* hpd = hp + (int64_t)d * (m + 1);
    double* Hd = H + (int64_t)d * m * (m + 1);
    double* dt = dots + (int64_t)d * ps;
    // column k-1's first-pass coefficients, loaded ahead of the reductions
    double hold = 0.0;
    if (tid < k) hold = hpd[tid];
    double nud = 0.0, sc = 1.0;
    if (with_z)
        nud = nu[d];
    else
        sc = inv_norm(norm + (int64_t)d * nblk, nblk, nud);
    {
        // the order of ms_reduce_kernel (a butterfly over up to 64 chunks), with 4 or 16 lanes per dot
        const int count = with_z ? 2 * k + 2 : k + 1;
        const int L = nwc <= 4 ? 4 : 16;
        const int sub = tid % L;
        for (int e = tid / L; e < count; e += 1024 / L) {
            const double* p = partial + ((int64_t)d * ps + e) * nwc;
            auto at = [&](int q) { return q < nwc ? p[q] : 0.0; };
            double s = L == 4 ? at(sub) : (at(sub) + at(sub + 32)) + (at(sub + 16) + at(sub + 48));
            for (int off = L / 2; off >= 1; off >>= 1) s += __shfl_xor(s, off, 64);
            if (sub == 0) {
                sd[e] = s;
                dt[e] = s;
            }
        }
    }
    __syncthreads();
    if (wave < 4) {   // the sums of ms_dcgs_coeff_kernel's 256 threads
        double asq = 0.0, ab = 0.0;
        for (int i = tid; i < k; i += 256) {
            const double ai = sc * sd[i];
            asq += ai * ai;
            if (with_z) ab += sd[i] * sd[k + 1 + i];
        }
        asq = wave_sum(asq);
        ab = wave_sum(ab);
        if (lane == 0) {
            part[0][wave] = asq;
            part[1][wave] = ab;
        }
    }
    __syncthreads();
    const double asq = (part[0][0] + part[0][1]) + (part[0][2] + part[0][3]);
    const double ab = (part[1][0] + part[1][1]) + (part[1][2] + part[1][3]);
    const double r2 = sd[k] * sc * sc - asq;
    const double rho = r2 > 0.0 ? sqrt(r2) : 0.0;
    if (k >= 1) {
        double* col = Hd + (int64_t)(k - 1) * (m + 1);
        if (tid < k) col[tid] = hcol[tid] = hold + nud * sc * sd[tid];
        if (tid == 0) col[k] = hcol[k] = nud * rho;
    }
    if (!with_z) return;
    if (Sm) {
        double* sk = Sm + ((int64_t)d * m + k) * (m + 1);
        if (tid < k) sk[tid] = sd[tid];
        if (tid == 0) sk[k] = rho;
    }
    const double ir = rho > 0.0 ? 1.0 / rho : 0.0;
    const double gm = (sd[2 * k + 1] - ab) * ir;
    if (tid == 0) {
        gam[d] = gm;
        inv_rho[d] = ir;
    }
    __syncthreads();   // hcol
    for (int rb = 0; rb <= k / 64; ++rb) {
        const int i = rb * 64 + lane, c0 = max(0, rb * 64 - 1);
        double acc = 0.0;
        if (i < k) {
#pragma unroll 4
            for (int c = c0 + wave; c < k - 1; c += 16)
                if (c >= i - 1) acc += Hd[(int64_t)c * (m + 1) + i] * sd[c];
            if (((k - 1 - c0) & 15) == wave) acc += hcol[i] * sd[k - 1];   // that wave's last column
        }
        red[wave][lane] = acc;
        __syncthreads();
        if (wave == 0 && i <= k) {
            if (i < k) {
                double s = 0.0;
#pragma unroll
                for (int w = 0; w < 16; ++w) s += red[w][lane];
                hpd[i] = (sd[k + 1 + i] - s) * ir;
            } else {
                hpd[k] = (gm - (k >= 1 ? hcol[k] * sd[k - 1] : 0.0)) * ir;
            }
        }
        __syncthreads();
    }
}

// q_k = (u - Q a) / rho into slot k and p' = (z - Q b - gamma q_k) / rho into slot k + 1, with the
// sums of p'^2 over 64-row blocks in norm[d][blk]. A work-group owns 256 rows (4 per lane); its 4
// waves take every 4th basis vector (both sums from one read) and are combined in LDS in a fixed
// order. Rows past n (below npad) are read but neither written nor counted in the norm.
__global__ void __launch_bounds__(256) ms_dcgs_update_kernel(double* __restrict__ V, int64_t n, int64_t npad,
                                                             int mdim1, int k, DirList dirs,
                                                             const double* __restrict__ dots, int ps,
                                                             const double* __restrict__ gam,
                                                             const double* __restrict__ inv_rho,
                                                             double* __restrict__ norm) {
    __shared__ double pa[4][256], pb[4][256];
    const int lane = threadIdx.x & 63, q = threadIdx.x >> 6;
    const int64_t base = (int64_t)blockIdx.x * 256;   // npad is a multiple of 256
    const int d = dirs[blockIdx.y];
    const double* dt = dots + (int64_t)d * ps;
    double sa[4] = {0.0, 0.0, 0.0, 0.0}, sb[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll 2
    for (int i = q; i < k; i += 4) {
        const double* v = V + ((int64_t)d * mdim1 + i) * npad + base + lane;
        const double ai = dt[i], bi = dt[k + 1 + i];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const double x = v[64 * r];
            sa[r] += ai * x;
            sb[r] += bi * x;
        }
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        pa[q][lane + 64 * r] = sa[r];
        pb[q][lane + 64 * r] = sb[r];
    }
    __syncthreads();
    const int t = threadIdx.x;
    const int64_t row = base + t;
    double* u = V + ((int64_t)d * mdim1 + k) * npad;
    double* zv = u + npad;
    double x = 0.0;
    if (row < n) {
        const double ir = inv_rho[d], g = gam[d];
        const double qk = (u[row] - ((pa[0][t] + pa[1][t]) + (pa[2][t] + pa[3][t]))) * ir;
        x = (zv[row] - ((pb[0][t] + pb[1][t]) + (pb[2][t] + pb[3][t])) - g * qk) * ir;
        u[row] = qk;
        zv[row] = x;
    }
    const double s2 = wave_sum_sq(x);
    if (lane == 0) norm[(int64_t)d * (npad / kMsRows) + (base / kMsRows) + q] = s2;
}

// Back substitution of one system by one work-group: y (K entries, in LDS) <- U^-1 y, U upper triangular with
// entry (i, c) from at(c, i). Column by column it would wait for memory and two barriers K times; here panels of
// kPanel columns are solved: the first wave solves the panel's triangle from registers, and the rows above take
// all of the panel's columns at once, loaded before the triangle is solved.
constexpr int kPanel = 16;
template <typename E, typename At>
__device__ inline void back_substitute(double2* ys, int K, At&& at) {
    const int tid = threadIdx.x;
    __syncthreads();
    for (int c1 = K; c1 > 0; c1 -= kPanel) {
        const int c0 = max(0, c1 - kPanel), p = c1 - c0;
        // this thread's first row above the panel: its entries, in flight while the triangle is solved
        E own[kPanel];
#pragma unroll
        for (int q = 0; q < kPanel; ++q) own[q] = at(min(c0 + q, c1 - 1), min(tid, c0));
        if (tid < 64) {
            // lane r holds y and the entries of row c0 + r; column q's solution is broadcast from lane q
            E tri[kPanel];
#pragma unroll
            for (int q = 0; q < kPanel; ++q) tri[q] = at(min(c0 + q, c1 - 1), c0 + min(tid, min(q, p - 1)));
            double2 v = tid < p ? ys[c0 + tid] : make_double2(0.0, 0.0);
#pragma unroll
            for (int q = kPanel - 1; q >= 0; --q) {
                if (q >= p) continue;
                const double2 w = tri_div(v, tri[q]);
                const double2 x = make_double2(__shfl(w.x, q, 64), __shfl(w.y, q, 64));
                if (tid == q) v = x;
                if (tid < q) v = csub(v, tri_mul(tri[q], x));
            }
            if (tid < p) ys[c0 + tid] = v;
        }
        __syncthreads();
        for (int r = tid; r < c0; r += 256) {
            double2 v = ys[r];
            if (r == tid) {
#pragma unroll
                for (int q = kPanel - 1; q >= 0; --q)
                    if (q < p) v = csub(v, tri_mul(own[q], ys[c0 + q]));
            } else {
#pragma unroll 8
                for (int q = p - 1; q >= 0; --q) v = csub(v, tri_mul(at(c0 + q, r), ys[c0 + q]));
            }
            ys[r] = v;
        }
        __syncthreads();
    }
}

// y[s] <- S^-1 y[s] over the first k[s] entries (S of the system's direction), one work-group per system
__global__ void __launch_bounds__(256) ms_sinv_kernel(const int* __restrict__ sys, const int* __restrict__ ksteps,
                                                      int m, const double* __restrict__ Sm,
                                                      const int* __restrict__ sdir, double2* __restrict__ y) {
    extern __shared__ double2 ys[];
    const int s = sys[blockIdx.x];
    const int K = ksteps[s];
    const double* Sd = Sm + (int64_t)sdir[s] * m * (m + 1);
    for (int i = threadIdx.x; i < K; i += blockDim.x) ys[i] = y[(int64_t)s * m + i];
    back_substitute<double>(ys, K, [&](int c, int i) { return Sd[(int64_t)c * (m + 1) + i]; });
    for (int i = threadIdx.x; i < K; i += blockDim.x) y[(int64_t)s * m + i] = ys[i];
}

// One Givens step of system s on column j of Hbar + z Ibar (direction sdir[s], shift z[s]): the
// rotations of the earlier steps are applied, a new rotation zeroes the subdiagonal, the rotated
// column is stored as column j of R, and |g_{j+1}| is the residual norm of the shifted system.
// One wave per system. Applying rotation i maps the running entry affinely,
// cur' = -conj(s_i) cur + c_i y_{i+1}, and emits c_i cur + s_i y_{i+1}: each lane composes the maps
// of a contiguous chunk of the rotations, an inclusive scan across the lanes gives every chunk its
// incoming entry, and the lanes then replay their chunks to emit the rotated entries (about
// 2 j / 64 + 6 dependent steps instead of j).
struct GivensArgs {
    const int* sys;
    int nsys, j, m;
    const int* sdir;
    const double2* z;
    const double* H;
    double* cs;
    double2 *sn, *g, *R;
    int64_t S;
    double* est;
    const double* tol_abs;
    int *flags, *run, *ksteps;
};
__device__ inline void givens_wave(int k, int lane, const int* __restrict__ sys, int nsys, int j, int m,
                                                       const int* __restrict__ sdir, const double2* __restrict__ z,
                                                       const double* __restrict__ H, double* __restrict__ cs,
                                                       double2* __restrict__ sn, double2* __restrict__ g,
                                                       double2* __restrict__ R, int64_t S, double* __restrict__ est,
                                                       const double* __restrict__ tol_abs, int* __restrict__ flags,
                                                       int* __restrict__ run, int* __restrict__ ksteps) {
    const int s = sys[k];
    // everything that hangs on s alone is loaded at once: the step is a chain of memory latencies
    const int go = run[s], sd = sdir[s];
    const double2 zs = z[s], gj = g[(int64_t)j * S + s];
    const double tol = tol_abs[s];
    if (!go) return;   // stopped earlier in this chunk of steps (uniform over the wave)
    const double* hc = H + ((int64_t)sd * m + j) * (m + 1);
    double2* col = R + ((int64_t)j * (j + 1) / 2) * S + s;   // entry i of the column at col[i * S]
    auto yv = [&](int i) {   // entry i + 1 of column j of Hbar + z Ibar
        return make_double2(hc[i + 1] + (i + 1 == j ? zs.x : 0.0), i + 1 == j ? zs.y : 0.0);
    };
    const int L = (j + 63) / 64;
    const int i0 = min(j, lane * L), i1 = min(j, i0 + L);
    // the chunk's map: cur_out = A cur_in + B
    double2 A = make_double2(1.0, 0.0), B = make_double2(0.0, 0.0);
    for (int i = i0; i < i1; ++i) {
        const double2 a = cscale(-1.0, cconj(sn[(int64_t)i * S + s]));
        A = cmul(a, A);
        B = cadd(cmul(a, B), cscale(cs[(int64_t)i * S + s], yv(i)));
    }
    // inclusive scan of the maps over the lanes (lane l: the maps of chunks 0 .. l, applied in order)
    for (int off = 1; off < 64; off <<= 1) {
        const double2 Ap = make_double2(__shfl_up(A.x, off, 64), __shfl_up(A.y, off, 64));
        const double2 Bp = make_double2(__shfl_up(B.x, off, 64), __shfl_up(B.y, off, 64));
        if (lane >= off) {
            B = cadd(cmul(A, Bp), B);
            A = cmul(A, Ap);
        }
    }
    const double2 cur0 = make_double2(hc[0] + (j == 0 ? zs.x : 0.0), j == 0 ? zs.y : 0.0);
    double2 Ae = make_double2(__shfl_up(A.x, 1, 64), __shfl_up(A.y, 1, 64));
    double2 Be = make_double2(__shfl_up(B.x, 1, 64), __shfl_up(B.y, 1, 64));
    if (lane == 0) {
        Ae = make_double2(1.0, 0.0);
        Be = make_double2(0.0, 0.0);
    }
    double2 cur = cadd(cmul(Ae, cur0), Be);
    for (int i = i0; i < i1; ++i) {
        const double2 y = yv(i);
        const double ci = cs[(int64_t)i * S + s];
        const double2 si = sn[(int64_t)i * S + s];
        col[(int64_t)i * S] = cadd(cscale(ci, cur), cmul(si, y));
        cur = cadd(cscale(-1.0, cmul(cconj(si), cur)), cscale(ci, y));
    }
    // entry j after every earlier rotation: the whole composition applied to the first entry
    const double2 At = make_double2(__shfl(A.x, 63, 64), __shfl(A.y, 63, 64));
    const double2 Bt = make_double2(__shfl(B.x, 63, 64), __shfl(B.y, 63, 64));
    if (lane != 0) return;
    const double hn = hc[j + 1];
    const double2 x = cadd(cmul(At, cur0), Bt);
    // rotation [c s; -conj(s) c] with c real zeroing hn below col[j]
    const double ax = cabs(x);
    double c;
    double2 sv;
    if (hn == 0.0) {
        c = 1.0;
        sv = make_double2(0.0, 0.0);
    } else if (ax == 0.0) {
        c = 0.0;
        sv = make_double2(1.0, 0.0);
    } else {
        const double nu = hypot(ax, hn);
        c = ax / nu;
        sv = make_double2(x.x / ax * hn / nu, x.y / ax * hn / nu);
    }
    cs[(int64_t)j * S + s] = c;
    sn[(int64_t)j * S + s] = sv;
    const double2 cj = cadd(cscale(c, x), cscale(hn, sv));
    col[(int64_t)j * S] = cj;
    const double2 gn = cscale(-1.0, cmul(cconj(sv), gj));
    g[(int64_t)(j + 1) * S + s] = gn;
    g[(int64_t)j * S + s] = cscale(c, gj);
    const double e = cabs(gn);
    est[s] = e;
    int f = 0;
    if (e <= tol) f |= 1;
    if (hn <= 1e-14 * cabs(cj)) f |= 2;   // the Krylov space is invariant: the iterate is exact
    if (!(e == e) || !(hn == hn)) f |= 4;
    flags[s] = f;
    ksteps[s] = j + 1;
    if (f) run[s] = 0;
}

__global__ void __launch_bounds__(64) ms_givens_kernel(GivensArgs a) {
    givens_wave(blockIdx.x, threadIdx.x, a.sys, a.nsys, a.j, a.m, a.sdir, a.z, a.H, a.cs, a.sn, a.g, a.R, a.S, a.est,
                a.tol_abs, a.flags, a.run, a.ksteps);
}

// The update sweep of step k and the Givens step on column k-1, which do not depend on each other, in one launch
// for structures of some thousand atoms, where each alone is a few microseconds of latency on a part of the chip.
// The first nupd work-groups update 64 rows of one direction each (the sums of ms_dcgs_update_kernel, one row per
// lane); the others take the Givens steps of gper systems each.
__global__ void __launch_bounds__(256) ms_update_givens_kernel(double* __restrict__ V, int64_t n, int64_t npad, int mdim1,
                                                               int k, DirList dirs,
                                                               const double* __restrict__ dots, int ps,
                                                               const double* __restrict__ gam,
                                                               const double* __restrict__ inv_rho,
                                                               double* __restrict__ norm, int nupd, int gper, GivensArgs a) {
    __shared__ double pa[4][64], pb[4][64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if ((int)blockIdx.x >= nupd) {
        const int q = ((int)blockIdx.x - nupd) * gper + wave;
        if (wave < gper && q < a.nsys)
            givens_wave(q, lane, a.sys, a.nsys, a.j, a.m, a.sdir, a.z, a.H, a.cs, a.sn, a.g, a.R, a.S, a.est, a.tol_abs,
                        a.flags, a.run, a.ksteps);
        return;
    }
    const int nrb = (int)(npad / kMsRows);
    const int64_t rb = blockIdx.x % nrb;
    const int d = dirs[blockIdx.x / nrb];
    const int64_t row = rb * kMsRows + lane;
    const double* dt = dots + (int64_t)d * ps;
    const double* v = V + (int64_t)d * mdim1 * npad + row;
    double* u = V + ((int64_t)d * mdim1 + k) * npad;
    double* zv = u + npad;
    const double ur = u[row], zr = zv[row], ir = inv_rho[d], g = gam[d];   // ahead of the sums (wave 0 uses them)
    double sa = 0.0, sb = 0.0;
#pragma unroll 8
    for (int i = wave; i < k; i += 4) {
        const double x = v[(int64_t)i * npad];
        const double ai = dt[i], bi = dt[k + 1 + i];
        sa += ai * x;
        sb += bi * x;
    }
    pa[wave][lane] = sa;
    pb[wave][lane] = sb;
    __syncthreads();
    if (wave != 0) return;
    const int t = lane;
    double x = 0.0;
    if (row < n) {
        const double qk = (ur - ((pa[0][t] + pa[1][t]) + (pa[2][t] + pa[3][t]))) * ir;
        x = (zr - ((pb[0][t] + pb[1][t]) + (pb[2][t] + pb[3][t])) - g * qk) * ir;
        u[row] = qk;
        zv[row] = x;
    }
    const double s2 = wave_sum_sq(x);
    if (lane == 0) norm[(int64_t)d * nrb + rb] = s2;
}

// y = R^-1 g over the first k[s] columns, one work-group per system; packed R: entry i of column c at
// ((c (c + 1) / 2) + i) S + s
__global__ void __launch_bounds__(256) ms_solve_kernel(const int* __restrict__ sys, const int* __restrict__ ksteps,
                                                       int m, const double2* __restrict__ R, int64_t S,
                                                       const double2* __restrict__ g, double2* __restrict__ y) {
    extern __shared__ double2 ys[];
    const int s = sys[blockIdx.x];
    const int K = ksteps[s];
    for (int i = threadIdx.x; i < K; i += blockDim.x) ys[i] = g[(int64_t)i * S + s];
    back_substitute<double2>(ys, K, [&](int c, int i) { return R[((int64_t)c * (c + 1) / 2 + i) * S + s]; });
    for (int i = threadIdx.x; i < K; i += blockDim.x) y[(int64_t)s * m + i] = ys[i];
}

// x(s) = sum_{i < k[s]} y[s][i] V(d, i) for groups of up to 8 systems of one direction (the basis
// is read once per group); rows >= n and systems with k = 0 get 0. Real part at out + col sys_stride,
// imaginary part im_off further, with col = pos[s] (skipped when negative) or s when pos is NULL.
// Each thread owns kRows rows, 256 apart; the coefficients of 64 steps at a time are staged in LDS, so the loop over the
// steps waits for the basis alone (600 atoms, 600 systems: 118 us, now 40).
template <int kRows>
__global__ void __launch_bounds__(256) ms_xupdate_kernel(const double* __restrict__ V, int64_t n, int64_t npad,
                                                         int mdim1, const int* __restrict__ grp_sys,
                                                         const int* __restrict__ grp_dir, const int* __restrict__ ksteps,
                                                         const double2* __restrict__ y, int m,
                                                         double* __restrict__ out, int64_t sys_stride, int64_t im_off,
                                                         const int* __restrict__ pos) {
    constexpr int kStage = 64;
    __shared__ double2 sy[kStage][kMsGroup];
    const int64_t i0 = (int64_t)blockIdx.x * 256 * kRows + threadIdx.x;
    const int gi = blockIdx.y;
    const int d = grp_dir[gi];
    int kk[kMsGroup], kmax = 0, kmin = m;   // steps of each system, the most, and the fewest
#pragma unroll
    for (int t = 0; t < kMsGroup; ++t) {
        const int s = grp_sys[gi * kMsGroup + t];
        kk[t] = s >= 0 ? ksteps[s] : 0;
        kmax = max(kmax, kk[t]);
        kmin = min(kmin, kk[t]);
    }
    double ar[kRows][kMsGroup], ai[kRows][kMsGroup];
#pragma unroll
    for (int r = 0; r < kRows; ++r)
#pragma unroll
        for (int t = 0; t < kMsGroup; ++t) ar[r][t] = ai[r][t] = 0.0;
    const double* v = V + (int64_t)d * mdim1 * npad;
    for (int c0 = 0; c0 < kmax; c0 += kStage) {
        __syncthreads();
        for (int q = threadIdx.x; q < kStage * kMsGroup; q += 256) {
            const int t = q / kStage, c = c0 + q % kStage, s = grp_sys[gi * kMsGroup + t];
            if (s >= 0 && c < ksteps[s]) sy[q % kStage][t] = y[(int64_t)s * m + c];
        }
        __syncthreads();
        auto steps = [&](int from, int to, auto all) {   // all: every system takes these steps
#pragma unroll 4
            for (int c = from; c < to; ++c) {
                double x[kRows];
#pragma unroll
                for (int r = 0; r < kRows; ++r) {
                    const int64_t i = i0 + 256 * r;
                    x[r] = i < npad ? v[(int64_t)c * npad + i] : 0.0;
                }
#pragma unroll
                for (int t = 0; t < kMsGroup; ++t)
                    if (all.value || c < kk[t]) {
                        const double2 yc = sy[c - c0][t];
#pragma unroll
                        for (int r = 0; r < kRows; ++r) {
                            ar[r][t] = fma(yc.x, x[r], ar[r][t]);
                            ai[r][t] = fma(yc.y, x[r], ai[r][t]);
                        }
                    }
            }
        };
        const int to = min(c0 + kStage, kmax), full = min(to, max(c0, kmin));
        steps(c0, full, std::true_type{});
        steps(full, to, std::false_type{});
    }
#pragma unroll
    for (int t = 0; t < kMsGroup; ++t) {
        const int s = grp_sys[gi * kMsGroup + t];
        const int col = s < 0 ? -1 : pos ? pos[s] : s;
        if (col < 0) continue;
        double* xr = out + (int64_t)col * sys_stride;
#pragma unroll
        for (int r = 0; r < kRows; ++r) {
            const int64_t i = i0 + 256 * r;
            if (i >= npad) continue;
            xr[i] = i < n ? ar[r][t] : 0.0;
            xr[i + im_off] = i < n ? ai[r][t] : 0.0;
        }
    }
}

}  // namespace

void ms_pack(int prec, double* V, int64_t npad, int mdim1, int j, const DirList& dirs, int ndir, const double* norm,
             double* nu, double* inv_h, void* X, int64_t ld, hipStream_t st) {
    if (ndir <= 0) return;
    dim3 grd((unsigned)(npad / 256), (unsigned)ndir);
    auto go = [&](auto tag) {
        using E = decltype(tag);
        hipLaunchKernelGGL(ms_pack_kernel<E>, grd, dim3(256), 0, st, V, npad, mdim1, j, dirs, norm, nu, inv_h,
                           static_cast<E*>(X), ld);
    };
    if (prec == WFQ_PREC_FP64) go(double{});
    else if (prec == WFQ_PREC_FP32) go(float{});
    else go(uint16_t{});
    WFQ_CHECK_LAUNCH();
}

void ms_skinny(const Structure& S, const double* V, int mdim1, int j, const DirList& dirs, int ndir, const double* norm,
               double* nu, double* inv_h, double* Y, hipStream_t st) {
    if (ndir <= 0) return;
    if (ndir > 4 || !S.T64) throw Error{WFQ_EINVAL, "ms_skinny: up to 4 columns of a stored FP64 T"};
    auto go = [&](auto ncv) {
        constexpr int NC = decltype(ncv)::value;
        hipLaunchKernelGGL(ms_skinny_kernel<NC>, dim3((unsigned)(S.npad / (4 * kMsRowsT))), dim3(256), 0, st, S.T64, S.npad, V,
                           mdim1, j, dirs, norm, nu, inv_h, Y);
    };
    if (ndir == 1) go(std::integral_constant<int, 1>{});
    else if (ndir == 2) go(std::integral_constant<int, 2>{});
    else if (ndir == 3) go(std::integral_constant<int, 3>{});
    else go(std::integral_constant<int, 4>{});
    WFQ_CHECK_LAUNCH();
}

void ms_spmm(const Structure& S, bool y_is_f64, const void* Y, int64_t ld, const DirList& dirs, int ndir, double* V,
             int mdim1, int jdst, double* TV, hipStream_t st, const double* Yi, const double* scale) {
    if (ndir <= 0) return;
    if (Yi && (!y_is_f64 || ndir > 4)) throw Error{WFQ_EINVAL, "ms_spmm: the interleaved copy holds up to 4 FP64 columns"};
    const dim3 grd((unsigned)(S.npad / 256));
    if (ms_merged(S.npad) && ndir <= 4 && !Yi) {
        auto small = [&](auto tag, auto ncv) {
            using YE = decltype(tag);
            constexpr int NC = decltype(ncv)::value;
            hipLaunchKernelGGL((ms_spmm_small_kernel<YE, NC>), dim3((unsigned)(S.npad / 16)), dim3(64), 0, st, S.n, S.npad,
                               S.ell_w, S.ell_col, S.ell_val, static_cast<const YE*>(Y), ld, dirs, V, mdim1, jdst, TV, scale);
        };
        auto by = [&](auto tag) {
            if (ndir == 1) small(tag, std::integral_constant<int, 1>{});
            else if (ndir == 2) small(tag, std::integral_constant<int, 2>{});
            else if (ndir == 3) small(tag, std::integral_constant<int, 3>{});
            else small(tag, std::integral_constant<int, 4>{});
        };
        if (y_is_f64) by(double{});
        else by(float{});
        WFQ_CHECK_LAUNCH();
        return;
    }
    // columns in chunks of at most 4 (3 for the usual three field directions in one pass)
    for (int c0 = 0; c0 < ndir; c0 += 4) {
        const int nc = std::min(4, ndir - c0);
        auto go = [&](auto tag, auto ncv) {
            using YE = decltype(tag);
            constexpr int NC = decltype(ncv)::value;
            hipLaunchKernelGGL((ms_spmm_kernel<YE, NC>), grd, dim3(256), 0, st, S.n, S.npad, S.ell_w, S.ell_col,
                               S.ell_val, static_cast<const YE*>(Y), ld, dirs, V, mdim1, jdst, c0, TV, Yi, scale);
        };
        auto by_nc = [&](auto tag) {
            if (nc == 1) go(tag, std::integral_constant<int, 1>{});
            else if (nc == 2) go(tag, std::integral_constant<int, 2>{});
            else if (nc == 3) go(tag, std::integral_constant<int, 3>{});
            else go(tag, std::integral_constant<int, 4>{});
        };
        if (y_is_f64)
            by_nc(double{});
        else
            by_nc(float{});
        WFQ_CHECK_LAUNCH();
    }
}

void ms_dot(const double* V, int64_t n, int64_t npad, int mdim1, int nvec, int jw, const DirList& dirs, int ndir,
            double* partial, int pslots, bool self_norm, hipStream_t st) {
    const int ntot = nvec + (self_norm ? 1 : 0);
    if (ndir <= 0 || ntot <= 0) return;
    const int64_t nwc = wave_chunks(n);
    dim3 grd((unsigned)nwc, (unsigned)((ntot + 3) / 4), (unsigned)ndir);
    hipLaunchKernelGGL(ms_dot_kernel, grd, dim3(256), 0, st, V, n, npad, mdim1, nvec, jw, dirs, partial, pslots, nwc,
                       (int)self_norm);
    WFQ_CHECK_LAUNCH();
}

void ms_reduce(const DirList& dirs, int ndir, const double* partial, int pslots, int64_t n, int count, double* h,
               hipStream_t st) {
    if (ndir <= 0 || count <= 0) return;
    hipLaunchKernelGGL(ms_reduce_kernel, dim3((unsigned)((count + 3) / 4), (unsigned)ndir), dim3(256), 0, st, dirs,
                       partial, pslots, wave_chunks(n), count, h);
    WFQ_CHECK_LAUNCH();
}

void ms_update(double* V, int64_t n, int64_t npad, int mdim1, int nvec, int jw, const DirList& dirs, int ndir,
               const double* h, int pslots, double* norm, hipStream_t st) {
    if (ndir <= 0) return;
    dim3 grd((unsigned)(npad / kMsRows), (unsigned)ndir);
    hipLaunchKernelGGL(ms_update_kernel, grd, dim3(256), 0, st, V, n, npad, mdim1, nvec, jw, dirs, h, pslots, norm);
    WFQ_CHECK_LAUNCH();
}

void ms_givens(const int* sys, int nsys, int j, int m, const int* sdir, const double2* z, const double* H, double* cs,
               double2* sn, double2* g, double2* R, int64_t S, double* est, const double* tol_abs, int* flags,
               int* run, int* ksteps, hipStream_t st) {
    if (nsys <= 0) return;
    hipLaunchKernelGGL(ms_givens_kernel, dim3((unsigned)nsys), dim3(64), 0, st,
                       GivensArgs{sys, nsys, j, m, sdir, z, H, cs, sn, g, R, S, est, tol_abs, flags, run, ksteps});
    WFQ_CHECK_LAUNCH();
}

bool ms_merged(int64_t npad) { return npad <= 8192; }

void ms_update_givens(double* V, int64_t n, int64_t npad, int mdim1, int k, bool with_z, const DirList& dirs, int ndir,
                      const double* dots, int ps, const double* gam, const double* irho, double* norm, const int* sys,
                      int nsys, int m, const int* sdir, const double2* z, const double* H, double* cs, double2* sn,
                      double2* g, double2* R, int64_t S, double* est, const double* tol_abs, int* flags, int* run,
                      int* ksteps, hipStream_t st) {
    const int nupd = with_z ? (int)(npad / kMsRows) * ndir : 0, ngiv = k >= 1 ? nsys : 0;
    if (nupd + ngiv == 0) return;
    // Givens steps spread over the chip: one to a work-group (its other waves end at once) up to 1 024 systems
    // (600 systems in work-groups of 16 waves: 5.8 us; 4 to a work-group 6.4, 16 to a work-group 10.2)
    const int gper = std::min(4, 1 + ngiv / 1024);
    hipLaunchKernelGGL(ms_update_givens_kernel, dim3((unsigned)(nupd + (ngiv + gper - 1) / gper)), dim3(256), 0, st, V, n,
                       npad, mdim1, k, dirs, dots, ps, gam, irho, norm, nupd, gper,
                       GivensArgs{sys, ngiv, k - 1, m, sdir, z, H, cs, sn, g, R, S, est, tol_abs, flags, run, ksteps});
    WFQ_CHECK_LAUNCH();
}

void ms_dcgs_dot(const double* V, int64_t n, int64_t npad, int mdim1, int k, bool with_z, const DirList& dirs, int ndir,
                 double* partial, int ps, hipStream_t st) {
    if (ndir <= 0) return;
    if (2 * k + 2 > ps) throw Error{WFQ_EINVAL, "ms_dcgs_dot: too few partial slots"};
    const int64_t nwc = wave_chunks(n);
    // four vectors per wave while 16 would leave fewer than 2 048 waves (two per SIMD)
    const bool few = nwc * (k / 16 + 1) * ndir < 2048;
    const int group = few ? 4 : 16;
    dim3 grd((unsigned)((nwc + 3) / 4), (unsigned)(k / group + 1), (unsigned)ndir);
    hipLaunchKernelGGL(few ? ms_dcgs_dot_kernel<4> : ms_dcgs_dot_kernel<16>, grd, dim3(256), 0, st, V, n, npad, mdim1, k,
                       with_z ? 1 : 0, dirs, partial, ps, nwc);
    WFQ_CHECK_LAUNCH();
}

void ms_dcgs_step(const DirList& dirs, int ndir, int k, bool with_z, int m, const double* partial, int ps, int64_t n,
                  int64_t npad, const double* nu, const double* norm, double* dots, double* hp, double* H, double* Sm,
                  double* gam, double* inv_rho, hipStream_t st) {
    if (ndir <= 0) return;
    const int64_t nwc = wave_chunks(n), nblk = npad / kMsRows;
    if (k <= kStepMax && nwc <= 64) {
        hipLaunchKernelGGL(ms_dcgs_step_kernel, dim3((unsigned)ndir), dim3(1024), 0, st, dirs, k, with_z ? 1 : 0, m, partial,
                           ps, nwc, nu, norm, nblk, dots, hp, H, Sm, gam, inv_rho);
        WFQ_CHECK_LAUNCH();
        return;
    }
    ms_reduce(dirs, ndir, partial, ps, n, with_z ? 2 * k + 2 : k + 1, dots, st);
    hipLaunchKernelGGL(ms_dcgs_coeff_kernel, dim3((unsigned)ndir), dim3(256), 0, st, dirs, k, with_z ? 1 : 0, m, dots,
                       ps, hp, H, Sm, nu, norm, nblk, gam, inv_rho);
    WFQ_CHECK_LAUNCH();
    if (!with_z) return;
    hipLaunchKernelGGL(ms_dcgs_hp_kernel, dim3((unsigned)(k / 64 + 1), (unsigned)ndir), dim3(1024), 0, st, dirs, k, m,
                       dots, ps, H, gam, inv_rho, hp);
    WFQ_CHECK_LAUNCH();
}

void ms_dcgs_update(double* V, int64_t n, int64_t npad, int mdim1, int k, const DirList& dirs, int ndir,
                    const double* dots, int ps, const double* gam, const double* inv_rho, double* norm, hipStream_t st) {
    if (ndir <= 0) return;
    dim3 grd((unsigned)(npad / 256), (unsigned)ndir);
    hipLaunchKernelGGL(ms_dcgs_update_kernel, grd, dim3(256), 0, st, V, n, npad, mdim1, k, dirs, dots, ps, gam, inv_rho,
                       norm);
    WFQ_CHECK_LAUNCH();
}

void ms_sinv(const int* sys, int nsys, const int* ksteps, int m, const double* Sm, const int* sdir, double2* y,
             hipStream_t st) {
    if (nsys <= 0) return;
    hipLaunchKernelGGL(ms_sinv_kernel, dim3((unsigned)nsys), dim3(256), (size_t)m * sizeof(double2), st, sys, ksteps,
                       m, Sm, sdir, y);
    WFQ_CHECK_LAUNCH();
}

void ms_solve(const int* sys, int nsys, const int* ksteps, int m, const double2* R, int64_t S, const double2* g,
              double2* y, hipStream_t st) {
    if (nsys <= 0) return;
    hipLaunchKernelGGL(ms_solve_kernel, dim3((unsigned)nsys), dim3(256), (size_t)m * sizeof(double2), st, sys, ksteps,
                       m, R, S, g, y);
    WFQ_CHECK_LAUNCH();
}

namespace {
void launch_xupdate(const double* V, int64_t n, int64_t npad, int mdim1, const int* grp_sys, const int* grp_dir, int ngrp,
                    const int* ksteps, const double2* y, int m, double* out, int64_t sys_stride, int64_t im_off,
                    const int* pos, hipStream_t st) {
    // four rows per thread (each coefficient read from LDS serves four products of the FP64 units, which bound it) from
    // 2 048 waves on, two per SIMD
    const int rows = npad / 256 * ngrp >= 2048 ? 4 : 1;
    hipLaunchKernelGGL(rows == 4 ? ms_xupdate_kernel<4> : ms_xupdate_kernel<1>,
                       dim3((unsigned)((npad + 256 * rows - 1) / (256 * rows)), (unsigned)ngrp), dim3(256), 0, st, V, n, npad, mdim1,
                       grp_sys, grp_dir, ksteps, y, m, out, sys_stride, im_off, pos);
    WFQ_CHECK_LAUNCH();
}
}  // namespace

void ms_xupdate(const double* V, int64_t n, int64_t npad, int mdim1, const int* grp_sys, const int* grp_dir, int ngrp,
                const int* ksteps, const double2* y, int m, const Basis& X, hipStream_t st) {
    if (ngrp <= 0) return;
    launch_xupdate(V, n, npad, mdim1, grp_sys, grp_dir, ngrp, ksteps, y, m, X.base, X.sys_stride, X.npad, nullptr, st);
}

void ms_txupdate(const double* TV, int64_t n, int64_t npad, int mdim1, const int* grp_sys, const int* grp_dir,
                 int ngrp, const int* ksteps, const double2* y, int m, const int* pos, double* Y, int64_t ld,
                 hipStream_t st) {
    if (ngrp <= 0) return;
    if (ld < npad) throw Error{WFQ_EINVAL, "ms_txupdate: leading dimension below the padded length"};
    launch_xupdate(TV, n, npad, mdim1, grp_sys, grp_dir, ngrp, ksteps, y, m, Y, 2 * ld, ld, pos, st);
}

}  // namespace wfq
