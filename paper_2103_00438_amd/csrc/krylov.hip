// Krylov-side kernels: the packing of vectors into a product's block, the sparse half of the operator (L Y + z V),
// the triangular solve of the least-squares problem (the Arnoldi sweeps and the column step are in dcgs.hip), the solution
// update, the FP64 refinement residual and the observables (arXiv 2103.00438, Section
// "Solution strategies": GMRES paragraph and restarted GMRES(k); Eq. (long-cross) for the dipole).
//
// All of these are bandwidth-bound vector sweeps. Reductions are deterministic: each wave sums a
// fixed 512-row chunk with a fixed butterfly, and per-chunk partials are added in chunk order.
#include "device_util.h"
#include "krylov.h"

namespace wfq {

namespace {

__device__ inline double* vre(const Basis& V, int s, int j) { return V.base + (int64_t)s * V.sys_stride + (int64_t)j * V.vec_stride; }

__device__ inline double2 cmul(double2 a, double2 b) { return make_double2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x); }

// block of 256 threads -> one value, fixed order
__device__ inline double block_sum(double v, double* sh) {
    v = wave_sum(v);
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    __syncthreads();
    if (lane == 0) sh[wave] = v;
    __syncthreads();
    double t = sh[0] + sh[1] + sh[2] + sh[3];
    return t;
}

template <typename E>
__global__ void __launch_bounds__(256) pack_kernel(Basis V, const int* __restrict__ sys, int j,
                                                   const double* __restrict__ scale, int write_back, E* __restrict__ X,
                                                   int64_t ld, const int* __restrict__ run, NormSums norm) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const int k = blockIdx.y;
    const int s = sys[k];
    if (run && !run[s]) {   // a system that stopped inside this chunk of steps: zero columns
        X[(int64_t)(2 * k) * ld + i] = cast_from_double<E>(0.0);
        X[(int64_t)(2 * k + 1) * ld + i] = cast_from_double<E>(0.0);
        return;
    }
    double* re = vre(V, s, j);
    double* im = re + V.npad;
    const double re_i = re[i], im_i = im[i];
    double sc = scale ? scale[s] : 1.0;
    if (norm.norm2) {   // few chunks: every thread adds them, in order
        double sum = 0.0;
        for (int64_t w = 0; w < norm.nwc; ++w) sum += norm.norm2[(int64_t)s * norm.nwc + w];
        const double nu = sqrt(sum);
        sc = nu > 0.0 ? 1.0 / nu : 0.0;
        if (i == 0) {
            norm.nu[s] = nu;
            norm.inv_h[s] = sc;
        }
    }
    const double a = re_i * sc, b = im_i * sc;
    if (write_back) {
        re[i] = a;
        im[i] = b;
    }
    X[(int64_t)(2 * k) * ld + i] = cast_from_double<E>(a);
    X[(int64_t)(2 * k + 1) * ld + i] = cast_from_double<E>(b);
}

// the block of the operator entry points, straight from a caller's vectors (rows from 2 nsys on are zeroed)
template <typename E>
__global__ void __launch_bounds__(256) load_kernel(int64_t n, int64_t ld, const int32_t* __restrict__ perm, int nsys,
                                                   const double* __restrict__ x_re, const double* __restrict__ x_im,
                                                   E* __restrict__ X) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const int64_t k = blockIdx.y;
    double a = 0.0, b = 0.0;
    if (k < nsys && i < n) {
        const int64_t o = k * n + perm[i];
        a = x_re[o];
        b = x_im[o];
    }
    X[(2 * k) * ld + i] = cast_from_double<E>(a);
    X[(2 * k + 1) * ld + i] = cast_from_double<E>(b);
}

// ---- L Y + z V. Row blocks are laid out so that the work-groups of one XCD (ids congruent mod 8) own one contiguous
// run of rows: they gather overlapping neighbour windows of Y at about the same time, and that XCD's L2 serves them.
template <typename YE> struct Pair2;
template <> struct Pair2<float> { using type = float2; };
template <> struct Pair2<double> { using type = double2; };

// Yr[i][k] = (Y[2k][i], Y[2k+1][i]), ldk pairs per row: every system's value of one atom side by side, so
// that the SpMM below fetches whole lines. 32 rows x 8 systems per work-group, a wave 8 x 8 of them.
template <typename YE>
__global__ void __launch_bounds__(256) row_pairs_kernel(const YE* __restrict__ Y, int64_t ld, int nsys, int64_t ldk,
                                                        typename Pair2<YE>::type* __restrict__ Yr) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int64_t i = (int64_t)blockIdx.x * 32 + wave * 8 + (lane >> 3);   // grid: ld / 32 blocks
    const int64_t k = (int64_t)blockIdx.y * 8 + (lane & 7);
    if (k >= nsys) return;
    typename Pair2<YE>::type v;
    v.x = Y[(2 * k) * ld + i];
    v.y = Y[(2 * k + 1) * ld + i];
    Yr[i * ldk + k] = v;
}

// Where a row's sum goes: slot jdst of the systems' bases, or a caller's vectors in its own atom order. kParts: a row's
// entries may be summed in parts (the solves keep one sum per row, whose order their results hang on).
struct ToBasis {
    static constexpr bool kParts = false;
    const int* sys;
    const double2* z;
    Basis Vs, V;
    int jsrc, jdst;
    __device__ void operator()(int k, int64_t i, double ar, double ai) const {
        const int s = sys[k];
        const double* sr = vre(Vs, s, jsrc);
        const double vr = sr[i], vi = sr[i + Vs.npad];
        const double2 zz = z[s];
        double* dr = vre(V, s, jdst);
        dr[i] = ar + zz.x * vr - zz.y * vi;
        dr[i + V.npad] = ai + zz.x * vi + zz.y * vr;
    }
};
struct ToUser {
    static constexpr bool kParts = true;
    const double *z_re, *z_im, *x_re, *x_im;
    double *y_re, *y_im;
    const int32_t* perm;
    int64_t n;
    __device__ void operator()(int k, int64_t i, double ar, double ai) const {
        const int64_t o = k * n + perm[i];
        const double vr = x_re[o], vi = x_im[o], zr = z_re[k], zi = z_im[k];
        y_re[o] = ar + zr * vr - zi * vi;
        y_im[o] = ai + zr * vi + zi * vr;
    }
};

// L Y + z V with the lanes of a wave on 8 rows x 8: L groups of SPL adjacent systems times 8 / L parts of the rows'
// entries. From row pairs (PAIRS), what a row group gathers from one neighbour is one 128-byte line (8 FP64 or
// 16 FP32 systems), which the load path, the bound of this product, moves in an eighth of the line visits of one
// lane per row and system: 6 603 atoms with 321 neighbours, 37 systems in FP64 181 -> 67 us (and 5 to put the pairs
// together), 20 000 atoms with 37, 192 systems in FP32 197 -> 104 (14), 64 systems 78 -> 42 (7). The row block and the number of
// work-groups make no difference there. For few systems the parts of the entries share the latency of the row's
// chain and are added by lane shuffles in a fixed order (612 atoms, one system: 6.3 -> 5.1 us). The ELL rows of the
// work-group's R rows are staged in LDS (STAGED; neighbour lists too long for that are read where they are used).
template <typename YE, int L, int Q, int SPL, int R, bool PAIRS, bool STAGED, typename Out>
__global__ void __launch_bounds__(256) spmm_sys_kernel(int64_t n, int64_t npad, int w,
                                                       const int32_t* __restrict__ ecol,
                                                       const double* __restrict__ eval, const YE* __restrict__ Y,
                                                       int64_t ld, int nsys, int per_group, Out out) {
    extern __shared__ char smem[];
    constexpr int RW = 64 / (L * Q) < R ? 64 / (L * Q) : R;   // rows per wave
    double* lval = reinterpret_cast<double*>(smem);
    int32_t* lcol = reinterpret_cast<int32_t*>(smem + (size_t)w * R * sizeof(double));
    const int per_xcd = (int)(gridDim.x >> 3);
    const int64_t rb = (int64_t)(blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);   // one run of rows per XCD
    const int64_t r0 = rb * R;
    if (r0 >= n) return;   // whole work-group: grid padded to a multiple of 8 row blocks
    if constexpr (STAGED) {
        for (int q = threadIdx.x; q < w * R; q += 256) {
            const int e = q / R, r = q % R;
            const int64_t i = r0 + r;   // < npad: npad is a multiple of R
            lcol[q] = ecol[(int64_t)e * npad + i];
            lval[q] = eval[(int64_t)e * npad + i];
        }
        __syncthreads();
    }
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    constexpr int nrg = R / RW < 4 ? R / RW : 4;   // row groups; the waves beyond them take other systems
    static_assert(nrg * RW == R, "a work-group's waves cover its rows");
    // in pairs the systems of a row lie side by side, in planes without parts the rows of a system
    constexpr bool kByRows = !PAIRS && Q == 1;
    static_assert(!kByRows || RW * L == 64, "planes: every lane has a row and a system");
    const int lr = kByRows ? lane % RW : lane / (L * Q), g = kByRows ? lane / RW : lane % L, part = lane % (L * Q) / L;
    if (lr >= RW) return;   // fewer rows than lanes (long neighbour lists, few systems)
    const int r = wave % nrg * RW + lr;
    const int64_t i = r0 + r;
    const int k_end = min(nsys, (int)(blockIdx.y + 1) * per_group);
    for (int kb = (int)blockIdx.y * per_group + wave / nrg * L * SPL; kb < k_end; kb += 4 / nrg * L * SPL) {
        if (kByRows && kb + SPL * g >= k_end) break;
        int k[SPL];   // lanes past the end repeat the last system and store nothing
        double ar[SPL], ai[SPL];
        const int kl = kb + SPL * g < k_end ? kb + SPL * g : kb;
#pragma unroll
        for (int t = 0; t < SPL; ++t) {
            k[t] = min(kb + SPL * g + t, k_end - 1);
            ar[t] = ai[t] = 0.0;
        }
#pragma unroll 8
        for (int e = part; e < w; e += Q) {
            const int64_t c = STAGED ? lcol[e * R + r] : ecol[(int64_t)e * npad + i];
            const double v = STAGED ? lval[e * R + r] : eval[(int64_t)e * npad + i];
#pragma unroll
            for (int t = 0; t < SPL; ++t) {
                if constexpr (PAIRS) {
                    const YE* y = Y + 2 * (c * ld + kl) + 2 * t;
                    ar[t] += v * widen(y[0]);
                    ai[t] += v * widen(y[1]);
                } else {
                    ar[t] += v * widen(Y[(int64_t)(2 * k[t]) * ld + c]);
                    ai[t] += v * widen(Y[(int64_t)(2 * k[t] + 1) * ld + c]);
                }
            }
        }
#pragma unroll
        for (int t = 0; t < SPL; ++t) {
#pragma unroll
            for (int o = L; o < L * Q; o <<= 1) {
                ar[t] += __shfl_xor(ar[t], o, 64);
                ai[t] += __shfl_xor(ai[t], o, 64);
            }
            if (part == 0 && kb + SPL * g + t < k_end && i < n) out(k[t], i, ar[t], ai[t]);
        }
    }
}

template <typename YE, int L, int Q, int SPL, int R, bool PAIRS, bool STAGED, typename Out>
void launch_spmm_tile(const Structure& S, const YE* Y, int64_t ld, int nsys, const Out& out, hipStream_t st) {
    const int64_t nb8 = (S.npad / R + 7) / 8 * 8;
    constexpr int RW = 64 / (L * Q) < R ? 64 / (L * Q) : R;
    const int lanes = 4 / (R / RW) * L * SPL;   // systems per pass of a work-group
    const int64_t want = (2048 + nb8 - 1) / nb8;
    // planes of few rows: a wave's systems to a work-group while there are no more than two work-groups a CU (321-atom
    // sphere, 24 systems, FP32 operator: 44 -> 31 us)
    const int64_t spread = !PAIRS && Q == 1 ? std::min<int64_t>(512 / nb8, (nsys + L * SPL - 1) / (L * SPL)) : 1;
    const int gy = (int)std::max<int64_t>({1, spread, std::min<int64_t>(want, (nsys + lanes - 1) / lanes)});
    const int per_group = ((nsys + gy - 1) / gy + L * SPL - 1) / (L * SPL) * (L * SPL);
    const dim3 grd((unsigned)nb8, (unsigned)((nsys + per_group - 1) / per_group));
    hipLaunchKernelGGL((spmm_sys_kernel<YE, L, Q, SPL, R, PAIRS, STAGED, Out>), grd, dim3(256), STAGED ? (size_t)S.ell_w * 12 * R : 0,
                       st, S.n, S.npad, S.ell_w, S.ell_col, S.ell_val, Y, ld, nsys, per_group, out);
    WFQ_CHECK_LAUNCH();
}
// Rows of a work-group: the most whose ELL rows leave four work-groups to a CU's LDS, up to 32 (a row group per wave)
template <typename YE, int L, int Q, int SPL, bool PAIRS, typename Out>
void launch_spmm_sys(const Structure& S, const YE* Y, int64_t ld, int nsys, const Out& out, hipStream_t st) {
    const size_t per_row = (size_t)S.ell_w * 12;
    if (per_row * 32 <= 40960) launch_spmm_tile<YE, L, Q, SPL, 32, PAIRS, true>(S, Y, ld, nsys, out, st);
    else if (per_row * 16 <= 40960) launch_spmm_tile<YE, L, Q, SPL, 16, PAIRS, true>(S, Y, ld, nsys, out, st);
    else if (per_row * 8 <= 40960) launch_spmm_tile<YE, L, Q, SPL, 8, PAIRS, true>(S, Y, ld, nsys, out, st);
    else launch_spmm_tile<YE, L, Q, SPL, 8, PAIRS, false>(S, Y, ld, nsys, out, st);
}
// Planes, a row's entries in one sum: up to 64 rows, one system per wave (neighbouring rows' neighbours share lines). Where
// long lists leave fewer rows than lanes, the others take further systems: spheres with 321 neighbours in FP64, us with
// the lanes idle / taken, 5 979 atoms 4 systems 68 / 29, 40 systems 583 / 135; 1 505 atoms 40 systems 161 / 51; lists too
// long for LDS, 5 979 atoms, 40 systems 4 092 / 1 224.
template <typename YE, typename Out>
void launch_spmm_planes(const Structure& S, const YE* Y, int64_t ld, int nsys, const Out& out, hipStream_t st) {
    const size_t per_row = (size_t)S.ell_w * 12;
    if (per_row * 64 <= 40960) launch_spmm_tile<YE, 1, 1, 1, 64, false, true>(S, Y, ld, nsys, out, st);
    else if (per_row * 32 <= 40960) launch_spmm_tile<YE, 2, 1, 1, 32, false, true>(S, Y, ld, nsys, out, st);
    else if (per_row * 16 <= 40960) launch_spmm_tile<YE, 4, 1, 1, 16, false, true>(S, Y, ld, nsys, out, st);
    else if (per_row * 8 <= 40960) launch_spmm_tile<YE, 8, 1, 1, 8, false, true>(S, Y, ld, nsys, out, st);
    else launch_spmm_tile<YE, 8, 1, 1, 8, false, false>(S, Y, ld, nsys, out, st);
}

// Yr != NULL (room for round_up(nsys, 8) pairs per row): from four systems on the product's planes are first turned
// into row pairs there. FP64 gains from four systems on at every size (3 043-atom sphere, 4 systems: 52 -> 45 us for the
// whole operator, 12: 92 -> 56; 600-atom tube, 12: 28 -> 26). FP32 planes are half as long, and the extra
// launch only pays from about 4 M gathered pairs (4 000-atom tube, 12 systems, 2.4 M: 30 -> 33 us; sphere, 6
// systems, 4.0 M: equal; 12 systems: 62 -> 50; 16 000-atom tube, 12 systems, 9.6 M: 222 -> 214). In the solves two
// systems are enough where lists are too long for 64 rows, in whose planes lanes would idle (10 005-atom sphere, FP64, 2
// systems: 57 -> 37 us).
template <typename YE, typename Out>
void spmm_sys(const Structure& S, const YE* Y, int64_t ld, void* Yr, int nsys, const Out& out, hipStream_t st) {
    constexpr bool f64 = std::is_same<YE, double>::value;
    const bool idle = !Out::kParts && nsys >= 2 && (size_t)S.ell_w * 12 * 64 > 40960;   // planes would leave lanes idle
    if (Yr && (nsys >= 4 || idle) && (f64 || S.npad * S.ell_w * nsys >= (int64_t)4 << 20)) {
        const int64_t ldk = (nsys + 7) / 8 * 8;
        hipLaunchKernelGGL(row_pairs_kernel<YE>, dim3((unsigned)(S.npad / 32), (unsigned)(ldk / 8)), dim3(256), 0, st, Y, ld,
                           nsys, ldk, static_cast<typename Pair2<YE>::type*>(Yr));
        WFQ_CHECK_LAUNCH();
        const YE* P = static_cast<const YE*>(Yr);
        if (nsys <= 4) launch_spmm_sys<YE, 4, Out::kParts ? 2 : 1, 1, true>(S, P, ldk, nsys, out, st);
        else if (f64 || nsys <= 8) launch_spmm_sys<YE, 8, 1, 1, true>(S, P, ldk, nsys, out, st);
        else launch_spmm_sys<YE, 8, 1, 2, true>(S, P, ldk, nsys, out, st);
    } else if (!Out::kParts || nsys > 4) {
        launch_spmm_planes(S, Y, ld, nsys, out, st);
    } else if (nsys == 1) {
        launch_spmm_sys<YE, 1, 8, 1, false>(S, Y, ld, nsys, out, st);
    } else if (nsys == 2) {
        launch_spmm_sys<YE, 2, 4, 1, false>(S, Y, ld, nsys, out, st);
    } else {
        launch_spmm_sys<YE, 4, 2, 1, false>(S, Y, ld, nsys, out, st);
    }
}

// L Y + z V from per-system interleaved columns (Yp[s][i] = (re, im)), the layout in which QMR's direction update
// leaves T p. A work-group owns R consecutive rows for one group of systems, their ELL rows staged once in LDS
// ([entry][row], so lanes read consecutive words); each wave works on 64 / R systems at a time, one lane per (row,
// system).
template <int R>
__global__ void __launch_bounds__(256) spmm_rows_kernel(int64_t n, int64_t npad, int w,
                                                        const int32_t* __restrict__ ecol,
                                                        const double* __restrict__ eval, const double2* __restrict__ Yp,
                                                        int64_t ld, const int* __restrict__ sys, int nsys, int per_group,
                                                        ToBasis out) {
    extern __shared__ char smem[];
    double* lval = reinterpret_cast<double*>(smem);
    int32_t* lcol = reinterpret_cast<int32_t*>(smem + (size_t)w * R * sizeof(double));
    constexpr int G = 64 / R;
    const int per_xcd = (int)(gridDim.x >> 3);
    const int64_t rb = (int64_t)(blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
    const int64_t r0 = rb * R;
    if (r0 >= n) return;   // whole work-group: grid padded to a multiple of 8 row blocks
    for (int q = threadIdx.x; q < w * R; q += 256) {
        const int e = q / R, r = q % R;
        const int64_t i = r0 + r;   // < npad: npad is a multiple of R
        lcol[q] = ecol[(int64_t)e * npad + i];
        lval[q] = eval[(int64_t)e * npad + i];
    }
    __syncthreads();
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int r = lane % R, g = lane / R;
    const int64_t i = r0 + r;
    if (i >= n) return;
    const int k_end = min(nsys, (int)(blockIdx.y + 1) * per_group);
    for (int k = (int)blockIdx.y * per_group + wave * G + g; k < k_end; k += 4 * G) {
        double ar = 0.0, ai = 0.0;
        const double2* yp = Yp + (int64_t)sys[k] * ld;
#pragma unroll 4
        for (int e = 0; e < w; ++e) {
            const int c = lcol[e * R + r];
            const double v = lval[e * R + r];
            const double2 y = yp[c];
            ar += v * y.x;
            ai += v * y.y;
        }
        out(k, i, ar, ai);
    }
}

template <int R>
void launch_spmm_rows(const Structure& S, const double2* Yp, int64_t ld, int nsys, const ToBasis& out, hipStream_t st) {
    constexpr int G = 64 / R;
    const int64_t nb = S.npad / R;
    const int64_t nb8 = (nb + 7) / 8 * 8;
    // enough work-groups to fill the chip (about 8 per CU), but at least one system per wave
    const int64_t want = (2048 + nb8 - 1) / nb8;
    const int gy = (int)std::max<int64_t>(1, std::min<int64_t>(want, (nsys + 4 * G - 1) / (4 * G)));
    const int per_group = (nsys + gy - 1) / gy;
    const size_t lds = (size_t)S.ell_w * R * 12;
    hipLaunchKernelGGL(spmm_rows_kernel<R>, dim3((unsigned)nb8, (unsigned)gy), dim3(256), lds, st, S.n, S.npad, S.ell_w,
                       S.ell_col, S.ell_val, Yp, ld, out.sys, nsys, per_group, out);
}

// One wave per system: column-oriented back substitution on R y = g (k <= mdim - 1 steps).
__global__ void __launch_bounds__(64) tri_solve_kernel(const int* __restrict__ sys, const int* __restrict__ ksteps,
                                                       int mdim, const double2* __restrict__ R,
                                                       const double2* __restrict__ g, double2* __restrict__ y) {
    const int s = sys[blockIdx.x];
    const int lane = threadIdx.x;
    const int kk = ksteps[s];
    const double2* Rs = R + (int64_t)s * mdim * mdim;
    const double2* gs = g + (int64_t)s * (mdim + 1);
    double2* ys = y + (int64_t)s * mdim;
    // each lane keeps the right-hand side entries l = lane, lane + 64, ...
    double2 rhs[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int l = lane + 64 * q;
        rhs[q] = l < kk ? gs[l] : make_double2(0.0, 0.0);
    }
    for (int i = kk - 1; i >= 0; --i) {
        const int owner = i & 63, slot = i >> 6;
        double2 ri = make_double2(0.0, 0.0);
#pragma unroll
        for (int q = 0; q < 4; ++q)
            if (q == slot) ri = rhs[q];
        ri.x = __shfl(ri.x, owner, 64);
        ri.y = __shfl(ri.y, owner, 64);
        const double2 d = Rs[(int64_t)i * mdim + i];
        const double dd = d.x * d.x + d.y * d.y;
        const double2 yi = make_double2((ri.x * d.x + ri.y * d.y) / dd, (ri.y * d.x - ri.x * d.y) / dd);
        if (lane == 0) ys[i] = yi;
        // rhs_l -= R_li y_i for l < i (column i of R)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int l = lane + 64 * q;
            if (l < i) {
                const double2 t = cmul(Rs[(int64_t)i * mdim + l], yi);
                rhs[q].x -= t.x;
                rhs[q].y -= t.y;
            }
        }
    }
}

__global__ void __launch_bounds__(256) x_update_kernel(Basis V, Basis X, int64_t n, const int* __restrict__ sys,
                                                       const int* __restrict__ ksteps, const double2* __restrict__ y,
                                                       int mdim) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= n) return;
    const int s = sys[blockIdx.y];
    const int kk = ksteps[s];
    double ar = 0.0, ai = 0.0;
    for (int l = 0; l < kk; ++l) {
        const double2 yy = y[(int64_t)s * mdim + l];
        const double* vr = vre(V, s, l);
        const double a = vr[i], b = vr[i + V.npad];
        ar += yy.x * a - yy.y * b;
        ai += yy.x * b + yy.y * a;
    }
    double* xr = vre(X, s, 0);
    xr[i] += ar;
    xr[i + X.npad] += ai;
}

// V(s, 0) = b_dir(s) - (L Y_s + z_s x_s), system s = sys[k] with its product in columns 2k and 2k + 1 of
// Y; norm2[s][blk] = the block's sum of |r_i|^2 and qtq[s][blk] (if not NULL) that of
// Re(conj(x_i) (T x)_i). The grid's x index is the system and its y index the row block, so the
// work-groups of one row block run together and read its rows of L through the L2 cache once.
__global__ void __launch_bounds__(256) residual_kernel(int64_t n, int64_t npad, int w,
                                                       const int32_t* __restrict__ ecol,
                                                       const double* __restrict__ eval,
                                                       const double* __restrict__ Y, int64_t ld,
                                                       const int* __restrict__ sys, const double2* __restrict__ z,
                                                       Basis X, const double* __restrict__ b, const int* __restrict__ dir,
                                                       Basis V, double* __restrict__ norm2, int nblk,
                                                       double* __restrict__ qtq) {
    __shared__ double sh[4];
    const int64_t i = (int64_t)blockIdx.y * 256 + threadIdx.x;
    const int k = blockIdx.x;
    const int s = sys[k];
    double nn = 0.0, et = 0.0;
    if (i < n) {
        double ar = 0.0, ai = 0.0;
        for (int p = 0; p < w; ++p) {
            const int c = ecol[(int64_t)p * npad + i];
            const double v = eval[(int64_t)p * npad + i];
            ar += v * Y[(int64_t)(2 * k) * ld + c];
            ai += v * Y[(int64_t)(2 * k + 1) * ld + c];
        }
        const double* xr = vre(X, s, 0);
        const double xre = xr[i], xim = xr[i + X.npad];
        const double2 zz = z[s];
        const double rr = b[(int64_t)dir[s] * V.npad + i] - (ar + zz.x * xre - zz.y * xim);
        const double ri = -(ai + zz.x * xim + zz.y * xre);
        double* vr = vre(V, s, 0);
        vr[i] = rr;
        vr[i + V.npad] = ri;
        nn = rr * rr + ri * ri;
        // Re(conj(x_i) (T x)_i); T is real and symmetric, so the sum over i is x^H T x
        et = xre * Y[(int64_t)(2 * k) * ld + i] + xim * Y[(int64_t)(2 * k + 1) * ld + i];
    }
    nn = block_sum(nn, sh);
    if (threadIdx.x == 0) norm2[(int64_t)s * nblk + blockIdx.y] = nn;
    if (qtq) {
        et = block_sum(et, sh);   // block_sum synchronises before it reuses sh
        if (threadIdx.x == 0) qtq[(int64_t)s * nblk + blockIdx.y] = et;
    }
}

__global__ void __launch_bounds__(256) copy_rhs_kernel(int64_t n, const int* __restrict__ sys,
                                                       const double* __restrict__ b, const int* __restrict__ dir, Basis V,
                                                       double* __restrict__ norm2, int nblk) {
    __shared__ double sh[4];
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const int s = sys[blockIdx.y];
    double nn = 0.0;
    if (i < n) {
        const double v = b[(int64_t)dir[s] * V.npad + i];
        double* vr = vre(V, s, 0);
        vr[i] = v;
        vr[i + V.npad] = 0.0;
        nn = v * v;
    }
    nn = block_sum(nn, sh);
    if (threadIdx.x == 0) norm2[(int64_t)s * nblk + blockIdx.x] = nn;
}

__global__ void sumsq_kernel(const int* __restrict__ sys, int nsys, const double* __restrict__ norm2, int nb,
                             double* __restrict__ out) {
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= nsys) return;
    const int s = sys[k];
    double acc = 0.0;
    for (int b = 0; b < nb; ++b) acc += norm2[(int64_t)s * nb + b];
    out[s] = sqrt(acc);
}

__global__ void __launch_bounds__(256) observables_kernel(int64_t n, int64_t npad, const double* __restrict__ pos,
                                                          const int* __restrict__ sys, Basis X, double E0,
                                                          double2* __restrict__ alpha) {
    __shared__ double sh[4];
    const int s = sys[blockIdx.x];
    const double* xr = vre(X, s, 0);
    const double* xi = xr + X.npad;
    double acc[6] = {0, 0, 0, 0, 0, 0};
    for (int64_t i = threadIdx.x; i < n; i += 256) {
        const double a = xr[i], b = xi[i];
#pragma unroll
        for (int l = 0; l < 3; ++l) {
            const double r = pos[l * npad + i];
            acc[2 * l] += r * a;
            acc[2 * l + 1] += r * b;
        }
    }
#pragma unroll
    for (int q = 0; q < 6; ++q) acc[q] = block_sum(acc[q], sh);
    if (threadIdx.x == 0)
        for (int l = 0; l < 3; ++l) alpha[(int64_t)s * 3 + l] = make_double2(acc[2 * l] / E0, acc[2 * l + 1] / E0);
}

__global__ void __launch_bounds__(256) scatter_kernel(int64_t n, const int32_t* __restrict__ perm,
                                                      const int* __restrict__ sys, Basis X, double* __restrict__ qr,
                                                      double* __restrict__ qi) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= n) return;
    const int s = sys[blockIdx.y];
    const double* xr = vre(X, s, 0);
    const int64_t o = (int64_t)s * n + perm[i];
    if (qr) qr[o] = xr[i];
    if (qi) qi[o] = xr[i + X.npad];
}

// x(sys[k]) = x(src_a[k]) + t[k] (x(src_b[k]) - x(src_a[k])), complex t (the targets are distinct from
// every source)
__global__ void __launch_bounds__(256) interp_kernel(int64_t n, const int* __restrict__ sys,
                                                     const int* __restrict__ src_a, const int* __restrict__ src_b,
                                                     const double2* __restrict__ t, Basis X) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= n) return;
    const int k = blockIdx.y;
    const double* ar = vre(X, src_a[k], 0);
    const double* br = vre(X, src_b[k], 0);
    double* xr = vre(X, sys[k], 0);
    const double2 tk = t[k];
    const double dr = br[i] - ar[i], di = br[i + X.npad] - ar[i + X.npad];
    xr[i] = ar[i] + (tk.x * dr - tk.y * di);
    xr[i + X.npad] = ar[i + X.npad] + (tk.x * di + tk.y * dr);
}

}  // namespace

void interp_start(const int* sys, int nsys, const int* src_a, const int* src_b, const double2* t, const Basis& x,
                  int64_t n, hipStream_t st) {
    if (nsys <= 0) return;
    dim3 grd((unsigned)((n + 255) / 256), (unsigned)nsys);
    hipLaunchKernelGGL(interp_kernel, grd, dim3(256), 0, st, n, sys, src_a, src_b, t, x);
    WFQ_CHECK_LAUNCH();
}

void pack_columns(int prec, const Basis& V, const int* sys, int nsys, int j, const double* scale, bool write_back,
                  void* X, int64_t ld, hipStream_t st, const int* run, const NormSums& norm) {
    if (nsys <= 0) return;
    dim3 grd((unsigned)(V.npad / 256), (unsigned)nsys);
    if (prec == WFQ_PREC_FP64)
        hipLaunchKernelGGL(pack_kernel<double>, grd, dim3(256), 0, st, V, sys, j, scale, (int)write_back,
                           static_cast<double*>(X), ld, run, norm);
    else if (prec == WFQ_PREC_FP32)
        hipLaunchKernelGGL(pack_kernel<float>, grd, dim3(256), 0, st, V, sys, j, scale, (int)write_back,
                           static_cast<float*>(X), ld, run, norm);
    else
        hipLaunchKernelGGL(pack_kernel<uint16_t>, grd, dim3(256), 0, st, V, sys, j, scale, (int)write_back,
                           static_cast<uint16_t*>(X), ld, run, norm);
    WFQ_CHECK_LAUNCH();
}

void load_columns(const Structure& S, int prec, const double* x_re, const double* x_im, int nsys, int64_t rows, void* X,
                  hipStream_t st) {
    const dim3 grd((unsigned)(S.npad / 256), (unsigned)(rows / 2));
    auto go = [&](auto tag) {
        using E = decltype(tag);
        hipLaunchKernelGGL(load_kernel<E>, grd, dim3(256), 0, st, S.n, S.npad, S.dperm, nsys, x_re, x_im,
                           static_cast<E*>(X));
    };
    if (prec == WFQ_PREC_FP64) go(double{});
    else if (prec == WFQ_PREC_FP32) go(float{});
    else go(uint16_t{});
    WFQ_CHECK_LAUNCH();
}

void spmm_shift(const Structure& S, bool y_is_f64, const void* Y, int64_t ld, void* Yr, const int* sys, int nsys,
                const double2* z, const Basis& V, int jsrc, int jdst, hipStream_t st, const Basis* shift_src) {
    if (nsys <= 0) return;
    const ToBasis out{sys, z, shift_src ? *shift_src : V, V, jsrc, jdst};
    if (y_is_f64) spmm_sys(S, static_cast<const double*>(Y), ld, Yr, nsys, out, st);
    else spmm_sys(S, static_cast<const float*>(Y), ld, Yr, nsys, out, st);
}

void spmm_user(const Structure& S, bool y_is_f64, const void* Y, int64_t ld, void* Yr, int nsys, const double* z_re,
               const double* z_im, const double* x_re, const double* x_im, double* y_re, double* y_im, hipStream_t st) {
    if (nsys <= 0) return;
    const ToUser out{z_re, z_im, x_re, x_im, y_re, y_im, S.dperm, S.n};
    if (y_is_f64) spmm_sys(S, static_cast<const double*>(Y), ld, Yr, nsys, out, st);
    else spmm_sys(S, static_cast<const float*>(Y), ld, Yr, nsys, out, st);
}

void spmm_shift_interleaved(const Structure& S, const double* Yp, int64_t ld, const int* sys, int nsys,
                            const double2* z, const Basis& V, int jsrc, int jdst, hipStream_t st) {
    if (nsys <= 0) return;
    // the largest row block whose ELL rows fit in 40 KB of LDS (4 work-groups per CU)
    const size_t per_row = (size_t)S.ell_w * 12;
    const int R = per_row * 64 <= 40960 ? 64 : per_row * 32 <= 40960 ? 32 : per_row * 16 <= 40960 ? 16
                  : per_row * 8 <= 40960 ? 8 : 0;
    if (R == 0) throw Error{WFQ_EINVAL, "neighbour lists too long for the sparse product"};
    const ToBasis out{sys, z, V, V, jsrc, jdst};
    const double2* Y = reinterpret_cast<const double2*>(Yp);
    if (R == 64) launch_spmm_rows<64>(S, Y, ld, nsys, out, st);
    else if (R == 32) launch_spmm_rows<32>(S, Y, ld, nsys, out, st);
    else if (R == 16) launch_spmm_rows<16>(S, Y, ld, nsys, out, st);
    else launch_spmm_rows<8>(S, Y, ld, nsys, out, st);
    WFQ_CHECK_LAUNCH();
}

void tri_solve(const int* sys, int nsys, const int* ksteps, int mdim, const double2* R, const double2* g,
               double2* y, hipStream_t st) {
    if (nsys <= 0) return;
    if (mdim > 257) throw Error{WFQ_EINVAL, "restart length above 256 is not supported"};
    hipLaunchKernelGGL(tri_solve_kernel, dim3(nsys), dim3(64), 0, st, sys, ksteps, mdim, R, g, y);
    WFQ_CHECK_LAUNCH();
}

void x_update(const Basis& V, const Basis& x, int64_t n, const int* sys, int nsys, const int* ksteps,
              const double2* y, int mdim, hipStream_t st) {
    if (nsys <= 0) return;
    dim3 grd((unsigned)((n + 255) / 256), (unsigned)nsys);
    hipLaunchKernelGGL(x_update_kernel, grd, dim3(256), 0, st, V, x, n, sys, ksteps, y, mdim);
    WFQ_CHECK_LAUNCH();
}

void residual(const Structure& S, const double* Y, int64_t ld, const int* sys, int nsys, const double2* z,
              const Basis& x, const double* b, const int* dir, const Basis& V, double* norm2, int nblk,
              double* qtq, hipStream_t st) {
    if (nsys <= 0) return;
    if (nblk > 65535) throw Error{WFQ_EINVAL, "residual: more row blocks than the grid's y dimension holds"};
    dim3 grd((unsigned)nsys, (unsigned)nblk);
    hipLaunchKernelGGL(residual_kernel, grd, dim3(256), 0, st, S.n, S.npad, S.ell_w, S.ell_col, S.ell_val, Y, ld, sys,
                       z, x, b, dir, V, norm2, nblk, qtq);
    WFQ_CHECK_LAUNCH();
}

void sumsq(const int* sys, int nsys, const double* norm2, int nb, double* out, hipStream_t st) {
    if (nsys <= 0) return;
    hipLaunchKernelGGL(sumsq_kernel, dim3((nsys + 63) / 64), dim3(64), 0, st, sys, nsys, norm2, nb, out);
    WFQ_CHECK_LAUNCH();
}

void copy_rhs(const Structure& S, const int* sys, int nsys, const double* b, const int* dir, const Basis& V,
              double* norm2, int nblk, hipStream_t st) {
    if (nsys <= 0) return;
    dim3 grd((unsigned)nblk, (unsigned)nsys);
    hipLaunchKernelGGL(copy_rhs_kernel, grd, dim3(256), 0, st, S.n, sys, b, dir, V, norm2, nblk);
    WFQ_CHECK_LAUNCH();
}

void observables(const Structure& S, const int* sys, int nsys, const Basis& x, double E0, double2* alpha,
                 hipStream_t st) {
    if (nsys <= 0) return;
    hipLaunchKernelGGL(observables_kernel, dim3(nsys), dim3(256), 0, st, S.n, S.npad, S.pos, sys, x, E0, alpha);
    WFQ_CHECK_LAUNCH();
}

void scatter_q(const Structure& S, const int32_t* perm, const int* sys, int nsys, const Basis& x, double* q_re,
               double* q_im, hipStream_t st) {
    if (nsys <= 0 || (!q_re && !q_im)) return;
    dim3 grd((unsigned)((S.n + 255) / 256), (unsigned)nsys);
    hipLaunchKernelGGL(scatter_kernel, grd, dim3(256), 0, st, S.n, perm, sys, x, q_re, q_im);
    WFQ_CHECK_LAUNCH();
}

}  // namespace wfq
