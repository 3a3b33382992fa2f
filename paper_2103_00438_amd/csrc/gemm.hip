// Block products Y = T X with the stored damped Coulomb matrix (the dense half of the operator
// A = (Kbar - P) D of Eq. (a-matrix-product); arXiv 2103.00438). T is symmetric, so each output
// column is a row-times-row product: Y[c][i] = sum_k T[i][k] X[c][k]. Both operands are contiguous
// along k, which is the layout the matrix cores want.
//
// Wide blocks (many Krylov columns) run on MFMA: FP64 v_mfma_f64_16x16x4, FP32 v_mfma_f32_16x16x4,
// BF16 v_mfma_f32_16x16x32 (FP32 accumulation). A work-group (4 or 8 waves) owns a BM x BN output
// tile, stages 64-, 128- or 256-byte k-slices of its X rows and T rows in LDS (double buffered,
// rows padded by 16 bytes so that each group of 8 lanes reading 16 bytes covers all 32 banks) and
// each wave computes a (16 WM) x (16 WN) sub-tile. Each lane feeds the matrix core 16 bytes of k per operand; the k
// order inside a slice is a permutation that is the same for both operands, so the sum is exact.
// Narrow blocks (<= 8 columns, e.g. one frequency at a time) stream T once with vector loads.
#include <cmath>
#include <cstring>
#include <iterator>

#include "common.h"
#include "device_util.h"

namespace wfq {

namespace {

template <int P>
struct Prec;
template <>
struct Prec<WFQ_PREC_FP64> {
    using elem = double;
    using out = double;
    using acc = doublex4;
    using sacc = double;
};
template <>
struct Prec<WFQ_PREC_FP32> {
    using elem = float;
    using out = float;
    using acc = floatx4;
    using sacc = float;
};
template <>
struct Prec<WFQ_PREC_BF16> {
    using elem = uint16_t;
    using out = float;
    using acc = floatx4;
    using sacc = float;
};

__device__ inline void mma(doublex4& c, const u32x4& a, const u32x4& b) {
    double a0 = __hiloint2double(a.y, a.x), a1 = __hiloint2double(a.w, a.z);
    double b0 = __hiloint2double(b.y, b.x), b1 = __hiloint2double(b.w, b.z);
    c = __builtin_amdgcn_mfma_f64_16x16x4f64(a0, b0, c, 0, 0, 0);
    c = __builtin_amdgcn_mfma_f64_16x16x4f64(a1, b1, c, 0, 0, 0);
}

template <int P>
__device__ inline void mma(floatx4& c, const u32x4& a, const u32x4& b);

template <>
__device__ inline void mma<WFQ_PREC_FP32>(floatx4& c, const u32x4& a, const u32x4& b) {
    c = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(a.x), __uint_as_float(b.x), c, 0, 0, 0);
    c = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(a.y), __uint_as_float(b.y), c, 0, 0, 0);
    c = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(a.z), __uint_as_float(b.z), c, 0, 0, 0);
    c = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(a.w), __uint_as_float(b.w), c, 0, 0, 0);
}

template <>
__device__ inline void mma<WFQ_PREC_BF16>(floatx4& c, const u32x4& a, const u32x4& b) {
    bf16x8 av = __builtin_bit_cast(bf16x8, a);
    bf16x8 bv = __builtin_bit_cast(bf16x8, b);
    c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av, bv, c, 0, 0, 0);
}

// Element-outer issue order: for each k element, one MFMA into every accumulator in turn, so
// consecutive MFMAs never depend on each other.
template <int P, int WM, int WN, typename A>
__device__ inline void mma_block_interleaved(A (&acc)[WM][WN], const u32x4 (&af)[WM], const u32x4 (&bf)[WN]) {
    if constexpr (P == WFQ_PREC_FP32) {
        float a[WM][4], b[WN][4];
#pragma unroll
        for (int x = 0; x < WM; ++x) {
            a[x][0] = __uint_as_float(af[x].x); a[x][1] = __uint_as_float(af[x].y);
            a[x][2] = __uint_as_float(af[x].z); a[x][3] = __uint_as_float(af[x].w);
        }
#pragma unroll
        for (int y = 0; y < WN; ++y) {
            b[y][0] = __uint_as_float(bf[y].x); b[y][1] = __uint_as_float(bf[y].y);
            b[y][2] = __uint_as_float(bf[y].z); b[y][3] = __uint_as_float(bf[y].w);
        }
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
            for (int x = 0; x < WM; ++x)
#pragma unroll
                for (int y = 0; y < WN; ++y)
                    acc[x][y] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[x][e], b[y][e], acc[x][y], 0, 0, 0);
    } else if constexpr (P == WFQ_PREC_FP64) {
        double a[WM][2], b[WN][2];
#pragma unroll
        for (int x = 0; x < WM; ++x) {
            a[x][0] = __hiloint2double(af[x].y, af[x].x);
            a[x][1] = __hiloint2double(af[x].w, af[x].z);
        }
#pragma unroll
        for (int y = 0; y < WN; ++y) {
            b[y][0] = __hiloint2double(bf[y].y, bf[y].x);
            b[y][1] = __hiloint2double(bf[y].w, bf[y].z);
        }
#pragma unroll
        for (int e = 0; e < 2; ++e)
#pragma unroll
            for (int x = 0; x < WM; ++x)
#pragma unroll
                for (int y = 0; y < WN; ++y)
                    acc[x][y] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[x][e], b[y][e], acc[x][y], 0, 0, 0);
    } else {
#pragma unroll
        for (int x = 0; x < WM; ++x)
#pragma unroll
            for (int y = 0; y < WN; ++y) mma<P>(acc[x][y], af[x], bf[y]);
    }
}

template <int P, typename A>
__device__ inline void mma_any(A& c, const u32x4& a, const u32x4& b) {
    if constexpr (P == WFQ_PREC_FP64)
        mma(c, a, b);
    else
        mma<P>(c, a, b);
}

constexpr int kRowStride = 144;  // bytes per staged row (128 data + 16 pad)

// Map a linear work-group id to a (m-tile, n-tile) pair so that the work-groups dispatched to one
// XCD (ids congruent mod 8) get a contiguous run of tiles, m fastest: the m-tiles that share one
// slab of T rows then run on the same XCD and reuse it from that XCD's L2.
__device__ inline int xcd_logical(int b, int total) {
    int xcd = b & 7, slot = b >> 3;
    int q = total >> 3, r = total & 7;
    return xcd < r ? xcd * (q + 1) + slot : r * (q + 1) + (xcd - r) * q + slot;
}

// KB = bytes of k staged per row and stage (64, 128 or 256); rows are padded by 16 bytes in LDS.
//
// Split k: with split > 1 the k range is cut into `split` equal parts and each (m-tile, part,
// n-tile) is one work-group, m fastest, so the m-tiles that share one slab of T and one k part
// stay adjacent (same XCD, same time) and T is still read once. Part 0 writes Y, part p > 0 writes
// its partial tile to ws + (p - 1) * mrows * ld in the layout of Y; split_reduce_kernel then adds
// the parts to Y in part order (a fixed summation order, so results are reproducible).
template <int P, int WM, int WN, int WAVES_M, int WAVES_N, int KB, int OCC, int ILV>
__global__ void __launch_bounds__(64 * WAVES_M * WAVES_N, OCC)
    tx_mfma_kernel(const typename Prec<P>::elem* __restrict__ X, const typename Prec<P>::elem* __restrict__ T,
                   typename Prec<P>::out* __restrict__ Y, int64_t ld, int ncol, int mt_count, int nt_count, int split,
                   int unit, typename Prec<P>::out* __restrict__ ws) {
    using elem = typename Prec<P>::elem;
    using acc_t = typename Prec<P>::acc;
    constexpr int NT = 64 * WAVES_M * WAVES_N;
    constexpr int BM = 16 * WM * WAVES_M;
    constexpr int BN = 16 * WN * WAVES_N;
    constexpr int ROWS = BM + BN;
    constexpr int CH = KB / 16;          // 16-byte chunks per staged row
    constexpr int RS = KB + 16;          // padded LDS row stride
    constexpr int TOTAL = ROWS * CH;     // 16-byte chunks per stage
    constexpr int PER_T = (TOTAL + NT - 1) / NT;
    // chunk u of this thread exists (only the last one can be missing)
#define WFQ_CHUNK_OK(u) (TOTAL % NT == 0 || (u) < PER_T - 1 || r0 + (u) * RSTEP < ROWS)
    __shared__ __attribute__((aligned(16))) char lds[2 * ROWS * RS];

    const int logical = xcd_logical(blockIdx.x, mt_count * nt_count * split);
    const int mt = logical % mt_count;
    const int part = (logical / mt_count) % split;
    const int nt = logical / (mt_count * split);
    const int64_t m0 = (int64_t)mt * BM, n0 = (int64_t)nt * BN;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = wave % WAVES_M, wn = wave / WAVES_M;

    // chunk u of this thread: row r0 + u * RSTEP (X rows first, then T rows), byte column cc * 16
    static_assert(NT % CH == 0, "whole rows per pass");
    constexpr int RSTEP = NT / CH;
    const int r0 = tid / CH, cc = tid % CH;
    const int64_t ldb = ld * (int64_t)sizeof(elem);
    const char* xb = reinterpret_cast<const char*>(X) + m0 * ldb + cc * 16;
    const char* tb = reinterpret_cast<const char*>(T) + n0 * ldb + cc * 16;
    const int dst0 = r0 * RS + cc * 16;
    // A missing last chunk re-reads the last row, and X rows past the last column (the tile can
    // be wider than the rows the caller holds) re-read the last column: loads stay unconditional
    // and in bounds; what they feed lands only in Y rows >= ncol, which are not stored.
    const int xlast = ncol - 1 - (int)m0;
    auto src_of = [&](int u) {
        const int row = min(r0 + u * RSTEP, ROWS - 1);
        return row < BM ? xb + min(row, xlast) * ldb : tb + (row - BM) * ldb;
    };

    acc_t acc[WM][WN];
#pragma unroll
    for (int a = 0; a < WM; ++a)
#pragma unroll
        for (int b = 0; b < WN; ++b) acc[a][b] = acc_t{0, 0, 0, 0};

    const int nu = (int)(ld * (int64_t)sizeof(elem) / KB) / unit;   // parts begin at multiples of `unit` stages
    const int kb = (int)((int64_t)nu * part / split) * unit, ke = (int)((int64_t)nu * (part + 1) / split) * unit;
    u32x4 reg[PER_T];
#pragma unroll
    for (int u = 0; u < PER_T; ++u)
        reg[u] = *reinterpret_cast<const u32x4*>(src_of(u) + (int64_t)kb * KB);
#pragma unroll
    for (int u = 0; u < PER_T; ++u)
        if (WFQ_CHUNK_OK(u)) *reinterpret_cast<u32x4*>(lds + dst0 + u * RSTEP * RS) = reg[u];
    __syncthreads();

    const int frag_row = lane & 15, frag_chunk = lane >> 4;
    for (int kt = kb; kt < ke; ++kt) {
        // prefetch the next k-step (the last step re-reads its own: loads stay unconditional, so
        // the staging registers live in VGPRs across the MFMA block instead of going to scratch)
        {
            const int64_t off = (int64_t)min(kt + 1, ke - 1) * KB;
#pragma unroll
            for (int u = 0; u < PER_T; ++u)
                reg[u] = *reinterpret_cast<const u32x4*>(src_of(u) + off);
        }
        // keep the loads ahead of the MFMA block: issued late, their latency is not hidden
        __builtin_amdgcn_sched_barrier(0);
        const char* L = lds + ((kt - kb) & 1) * ROWS * RS;
#pragma unroll
        for (int cg = 0; cg < CH / 4; ++cg) {
            u32x4 af[WM], bf[WN];
            const int coff = (cg * 4 + frag_chunk) * 16;
#pragma unroll
            for (int a = 0; a < WM; ++a)
                af[a] = *reinterpret_cast<const u32x4*>(L + (wm * 16 * WM + a * 16 + frag_row) * RS + coff);
#pragma unroll
            for (int b = 0; b < WN; ++b)
                bf[b] = *reinterpret_cast<const u32x4*>(L + (BM + wn * 16 * WN + b * 16 + frag_row) * RS + coff);
            if constexpr (ILV) {
                mma_block_interleaved<P, WM, WN>(acc, af, bf);
            } else {
#pragma unroll
                for (int a = 0; a < WM; ++a)
#pragma unroll
                    for (int b = 0; b < WN; ++b) mma_any<P>(acc[a][b], af[a], bf[b]);
            }
        }
        // the other buffer was last read in step kt - 1, which every wave left at its barrier;
        // the stores wait for the loads, so they stay behind the MFMA block
        __builtin_amdgcn_sched_barrier(0);
        {
            char* S = lds + ((kt + 1 - kb) & 1) * ROWS * RS;
#pragma unroll
            for (int u = 0; u < PER_T; ++u)
                if (WFQ_CHUNK_OK(u)) *reinterpret_cast<u32x4*>(S + dst0 + u * RSTEP * RS) = reg[u];
        }
        __syncthreads();
    }

    // Accumulator layout of one 16 x 16 block: column j = lane % 16 in every case; the row of
    // element r is 4 (lane / 16) + r for the FP32 and BF16 instructions and lane / 16 + 4 r for
    // the FP64 one.
    typename Prec<P>::out* out = part == 0 ? Y : ws + (int64_t)(part - 1) * mt_count * BM * ld;
#pragma unroll
    for (int a = 0; a < WM; ++a)
#pragma unroll
        for (int b = 0; b < WN; ++b)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int row = P == WFQ_PREC_FP64 ? (lane >> 4) + 4 * r : 4 * (lane >> 4) + r;
                int64_t c = m0 + wm * 16 * WM + a * 16 + row;
                int64_t i = n0 + wn * 16 * WN + b * 16 + (lane & 15);
                if (c < ncol) out[c * ld + i] = acc[a][b][r];
            }
}

#undef WFQ_CHUNK_OK

// ---- FP64 products of a few to a hundred columns: both operands straight into the fragment layout
//
// FP64 matrix instructions take 64 clocks for 512 B per operand, so a wave that holds 16 CF columns x 16 RF rows
// needs no LDS to feed them. T is symmetric, so Y[c][i] = sum_k T[k][i] X[c][k] walks down T's rows: the 16 lanes of a
// fragment's row index read adjacent elements (32 or 64 bytes of every line per load; along a row of T, each lane
// would be a line visit of its own, and those bound the kernel). A lane's 16 bytes are two neighbouring
// columns of T and feed two fragments; X is laid out the same way beforehand (xt_kernel: [k][columns]).
// What this spares against the LDS tiles of tx_mfma_kernel is column padding (128 columns' work for 74; the granule is 16
// here) and barriers. The four waves of a work-group take every fourth 16 k of the same tile, their sums are
// added in LDS in order at the end, and the loads of a wave's next 16 k are in flight during the products of this
// one (two register buffers). Split k and the order of the tiles as in tx_mfma_kernel.
// Bound: the FP64 matrix cores and, below some 48 columns, T's 8 bytes per element. Against the fastest LDS tile, us:
// 20 000 atoms 588 / 753 at 16 columns, 717 / 1 017 at 48, 1 111 / 1 770 at 80 (59 TFLOP/s), 1 676 / 1 787 at 128,
// 4 507 / 5 208 at 384; 6 603 atoms 72 / 75, 101 / 126, 150 / 202, 191 / 239, 514 / 607; 2 000 atoms 11 / 19, 16 / 20, 23 / 30, 28 / 32,
// 57 / 75 (X's turning and the adding of parts included). Along T's rows instead (each lane its own line): 1 300 at
// 20 000 atoms and 80 columns.
__global__ void __launch_bounds__(256) xt_kernel(const double* __restrict__ X, int64_t ld, int ncol, int64_t ldc,
                                                 double* __restrict__ Xt) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int64_t k = (int64_t)blockIdx.x * 32 + wave * 8 + (lane & 7);   // grid: ld / 32 blocks
    const int c = blockIdx.y * 8 + (lane >> 3);
    __shared__ double tile[4][8][9];
    tile[wave][lane >> 3][lane & 7] = c < ncol ? X[(int64_t)c * ld + k] : 0.0;   // 8 columns x 8 k, each wave its own
    __syncthreads();
    Xt[((int64_t)blockIdx.x * 32 + wave * 8 + (lane >> 3)) * ldc + blockIdx.y * 8 + (lane & 7)] =
        tile[wave][lane & 7][lane >> 3];
}

template <int CF, int RF>
__global__ void __launch_bounds__(256, 2) tx_frag_kernel(const double* __restrict__ Xt, int64_t ldc,
                                                         const double* __restrict__ T, double* __restrict__ Y, int64_t ld,
                                                         int ncol, int mt_count, int nt_count, int split,
                                                         double* __restrict__ ws) {
    static_assert(RF % 2 == 0, "rows of T come in pairs of fragments");
    constexpr int BM = 16 * CF, BN = 16 * RF, CP = CF / 2;
    __shared__ double sum[2][4][16 * BN];
    const int logical = xcd_logical(blockIdx.x, mt_count * nt_count * split);
    const int mt = logical % mt_count;
    const int part = (logical / mt_count) % split;
    const int nt = logical / (mt_count * split);
    const int m0 = mt * BM;
    const int64_t n0 = (int64_t)nt * BN;
    const int lane = threadIdx.x & 63, col = lane & 15, kg = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);   // (scalar: the addresses' base stays scalar)
    const int units = (int)(ld / 64);   // 64 k: 16 per wave
    const int ub = (int)((int64_t)units * part / split), ue = (int)((int64_t)units * (part + 1) / split);
    const double* tb = T + (int64_t)16 * wave * ld + n0;
    const double* xb = Xt + (int64_t)16 * wave * ldc + m0;
    const uint32_t to = (uint32_t)(kg * ld + 2 * col), xo = (uint32_t)(kg * ldc + 2 * col),
                   xo1 = (uint32_t)(kg * ldc + 16 * (CF - 1) + col);
    struct Frag {
        double2 t[4][RF / 2], x[4][CP > 0 ? CP : 1];
        double x1[4];
    };
    auto load = [&](Frag& f, int u) {
#pragma unroll
        for (int s = 0; s < 4; ++s) {   // 4 k each
            const double* tu = tb + ((int64_t)64 * u + 4 * s) * ld;
            const double* xu = xb + ((int64_t)64 * u + 4 * s) * ldc;
#pragma unroll
            for (int r = 0; r < RF / 2; ++r) f.t[s][r] = *reinterpret_cast<const double2*>(tu + 32 * r + to);
#pragma unroll
            for (int c = 0; c < CP; ++c) f.x[s][c] = *reinterpret_cast<const double2*>(xu + 32 * c + xo);
            if constexpr (CF % 2 == 1) f.x1[s] = xu[xo1];
        }
    };
    doublex4 acc[CF][RF];
#pragma unroll
    for (int c = 0; c < CF; ++c)
#pragma unroll
        for (int r = 0; r < RF; ++r) acc[c][r] = doublex4{0, 0, 0, 0};
    auto mul = [&](const Frag& f) {
#pragma unroll
        for (int s = 0; s < 4; ++s)
#pragma unroll
            for (int c = 0; c < CF; ++c)
#pragma unroll
                for (int r = 0; r < RF; ++r) {
                    const double a = c / 2 < CP ? (c % 2 ? f.x[s][c / 2].y : f.x[s][c / 2].x) : f.x1[s];
                    const double b = r % 2 ? f.t[s][r / 2].y : f.t[s][r / 2].x;
                    acc[c][r] = __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, acc[c][r], 0, 0, 0);
                }
    };
    Frag f0, f1;
    load(f0, ub);
    int u = ub;
    for (; u + 1 < ue; u += 2) {
        load(f1, u + 1);
        __builtin_amdgcn_sched_barrier(0);
        mul(f0);
        __builtin_amdgcn_sched_barrier(0);
        load(f0, min(u + 2, ue - 1));   // the last step re-reads its own: loads stay unconditional
        __builtin_amdgcn_sched_barrier(0);
        mul(f1);
        __builtin_amdgcn_sched_barrier(0);
    }
    if (u < ue) mul(f0);
    double* out = part == 0 ? Y : ws + (int64_t)(part - 1) * mt_count * BM * ld;
#pragma unroll
    for (int c = 0; c < CF; ++c) {
        // element e of a block: fragment row (X) lane / 16 + 4 e, fragment column (T) lane % 16. Column c of the tile
        // is 32 (c / 2) + 2 row + c % 2 where X came in pairs, rows of T likewise
        double(*buf)[16 * BN] = sum[c & 1];
#pragma unroll
        for (int r = 0; r < RF; ++r)
#pragma unroll
            for (int e = 0; e < 4; ++e) buf[wave][(kg + 4 * e) * BN + 32 * (r / 2) + 2 * col + r % 2] = acc[c][r][e];
        __syncthreads();
#pragma unroll
        for (int q = 0; q < RF; ++q) {
            const int at = q * 256 + threadIdx.x, fr = at / BN;
            const int j = m0 + (c / 2 < CP ? 32 * (c / 2) + 2 * fr + c % 2 : 16 * c + fr);
            if (j < ncol) out[(int64_t)j * ld + n0 + at % BN] = (buf[0][at] + buf[1][at]) + (buf[2][at] + buf[3][at]);
        }
    }
}

// ---- FP32 products through the FP16 matrix cores: each FP32 operand is split into two FP16 parts
//
// v_mfma_f32_16x16x4_f32 does 256 multiply-adds per CU and clock, the FP16 form sixteen times as many
// from half the bits per operand. An FP32 value scaled into FP16's range is h + l + e with h its FP16
// rounding, l the FP16 rounding of x - h and |e| <= 2^-23 |x|, and x y = h h' + h l' + l h' + O(2^-22) x y:
// three FP16 products with FP32 accumulation stand for the FP32 one. The scales are powers of two
// (exact): one for T from its largest element, and one per column of X from that column's largest
// entry, taken out again in the epilogue. The sum over k rounds 3 k / 32 times in FP32 instead of k
// times, so the error against 64 bits falls (figures at any_variant).
//
// Layout: T goes straight from global memory into the matrix cores' fragment layout (a wave owns 16 WN
// rows of T and all 16 WM columns of its work-group, so no other wave needs its rows). T is symmetric and is
// walked down its rows: the 16 lanes of a fragment's row index read 16 WN adjacent elements of each of a lane's
// 8 k (along a row of T every lane would visit a line of its own: 430 us instead of 379 for 20 000 atoms and 128 columns).
// The split is done in registers, and the loads of the next stage are in flight during the matrix products of this one. X is split beforehand (split_x_kernel) into
// groups of 8 h and 8 l halves and staged through LDS for the four waves, double buffered, rows padded
// by 16 bytes (distinct banks for 8 lanes reading 16 bytes).
// Bound: the matrix cores and their operand reads with several hundred columns (20 000 atoms, 384 columns:
// 929 us = 1 020 TFLOP/s of FP16 products, 338 of the FP32 product's; 2 410 us and 130 TFLOP/s with the FP32
// instruction, whose peak is 157), below about 100 columns the HBM reads of T (32 columns: 293 us, 5.6 TB/s).

// One work-group per column of X: its largest magnitude gives the scale (the scaled entries stay below
// 2^15), then every group of 8 entries is written as 8 h and 8 l halves (32 bytes, like the FP32 entries).
__global__ void __launch_bounds__(1024) split_x_kernel(const float* __restrict__ X, int64_t ld, char* __restrict__ Xs,
                                                       ColInfo* __restrict__ info) {
    __shared__ unsigned red[16], redf[16];
    const int64_t c = blockIdx.x;
    const float* x = X + c * ld;
    unsigned m = 0, f = 0;   // largest magnitude (bits); bit 0: +inf, 1: -inf, 2: NaN
    for (int64_t i = (int64_t)threadIdx.x * 4; i < ld; i += 4096) {
        const u32x4 v = *reinterpret_cast<const u32x4*>(x + i);
        const unsigned w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const unsigned a = w[e] & 0x7fffffffu;
            m = max(m, a);
            if (a >= 0x7f800000u) f |= a > 0x7f800000u ? 4u : (w[e] >> 31) ? 2u : 1u;
        }
    }
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) {
        m = max(m, (unsigned)__shfl_xor((int)m, off, 64));
        f |= (unsigned)__shfl_xor((int)f, off, 64);
    }
    if ((threadIdx.x & 63) == 0) {
        red[threadIdx.x >> 6] = m;
        redf[threadIdx.x >> 6] = f;
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < 16; ++q) {
        m = max(m, red[q]);
        f |= redf[q];
    }
    int ex = 0;
    if (m > 0 && f == 0) {
        (void)frexpf(__uint_as_float(m), &ex);   // m = fraction in [1/2, 1) times 2^ex
        ex = 15 - ex;
    }
    if (threadIdx.x == 0) info[c] = ColInfo{ex, f == 0 ? 0 : f == 1 ? 1 : f == 2 ? 2 : 3};
    char* o = Xs + c * ld * 4;
    for (int64_t i = (int64_t)threadIdx.x * 8; i < ld; i += 8192) {
        float v[8];
        *reinterpret_cast<floatx4*>(v) = *reinterpret_cast<const floatx4*>(x + i);
        *reinterpret_cast<floatx4*>(v + 4) = *reinterpret_cast<const floatx4*>(x + i + 4);
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = ldexpf(v[e], ex);
        const halfx8 h = split_hi(v);
        *reinterpret_cast<halfx8*>(o + i * 4) = h;
        *reinterpret_cast<halfx8*>(o + i * 4 + 16) = split_lo(v, h);
    }
}

// BM = 16 WM columns, BN = 64 WN rows of T, KS values of k per stage. Split k and the tile order as in
// tx_mfma_kernel.
template <int WM, int WN, int KS, int OCC>
__global__ void __launch_bounds__(256, OCC)
    tx_split_kernel(const char* __restrict__ Xs, const ColInfo* __restrict__ info, const float* __restrict__ T,
                    float* __restrict__ Y, int64_t ld, int ncol, int mt_count, int nt_count, int split,
                    float* __restrict__ ws, float tscale, int texp) {
    constexpr int BM = 16 * WM, BN = 64 * WN;
    constexpr int SUB = KS / 32;         // 32-wide matrix steps per stage
    constexpr int RS = KS * 4 + 16;      // padded LDS row
    constexpr int CH = KS / 4;           // 16-byte chunks per row and stage
    constexpr int PER_T = BM * CH / 256;
    static_assert(BM * CH % 256 == 0 && 256 % CH == 0, "whole rows per pass");
    __shared__ __attribute__((aligned(16))) char lds[2 * BM * RS];

    const int logical = xcd_logical(blockIdx.x, mt_count * nt_count * split);
    const int mt = logical % mt_count;
    const int part = (logical / mt_count) % split;
    const int nt = logical / (mt_count * split);
    const int64_t m0 = (int64_t)mt * BM, n0 = (int64_t)nt * BN;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int fr = lane & 15, fk = lane >> 4;

    // X staging: chunk u of this thread is row r0 + u * RSTEP (columns past the last one re-read it: what
    // they feed is not stored)
    constexpr int RSTEP = 256 / CH;
    const int r0 = tid / CH, cc = tid % CH;
    const int xlast = ncol - 1 - (int)m0;
    const char* xp[PER_T];
#pragma unroll
    for (int u = 0; u < PER_T; ++u) xp[u] = Xs + (m0 + min(r0 + u * RSTEP, xlast)) * ld * 4 + cc * 16;
    const int dst0 = r0 * RS + cc * 16;
    // this lane's 8 values of k of WN neighbouring columns of T, one for each of the wave's fragments
    typedef float tvec __attribute__((ext_vector_type(WN)));
    const uint32_t to = (uint32_t)(8 * fk * ld + n0 + wave * 16 * WN + WN * fr);

    floatx4 acc[WM][WN];
#pragma unroll
    for (int a = 0; a < WM; ++a)
#pragma unroll
        for (int b = 0; b < WN; ++b) acc[a][b] = floatx4{0, 0, 0, 0};

    const int nk = (int)(ld / KS);
    const int kb = (int)((int64_t)nk * part / split), ke = (int)((int64_t)nk * (part + 1) / split);
    u32x4 xr[PER_T];
    tvec raw[SUB][8];
    auto load_t = [&](int kt, int s) {
#pragma unroll
        for (int e = 0; e < 8; ++e)
            raw[s][e] = *reinterpret_cast<const tvec*>(T + (int64_t)(kt * KS + s * 32 + e) * ld + to);
    };
#pragma unroll
    for (int u = 0; u < PER_T; ++u) xr[u] = *reinterpret_cast<const u32x4*>(xp[u] + (int64_t)kb * KS * 4);
#pragma unroll
    for (int s = 0; s < SUB; ++s) load_t(kb, s);
#pragma unroll
    for (int u = 0; u < PER_T; ++u) *reinterpret_cast<u32x4*>(lds + dst0 + u * RSTEP * RS) = xr[u];
    __syncthreads();

    for (int kt = kb; kt < ke; ++kt) {
        const int kn = min(kt + 1, ke - 1);   // the last stage re-reads its own: loads stay unconditional
#pragma unroll
        for (int u = 0; u < PER_T; ++u) xr[u] = *reinterpret_cast<const u32x4*>(xp[u] + (int64_t)kn * KS * 4);
        const char* L = lds + ((kt - kb) & 1) * BM * RS;
#pragma unroll
        for (int s = 0; s < SUB; ++s) {
            halfx8 th[WN], tl[WN];
#pragma unroll
            for (int b = 0; b < WN; ++b) {
                float v[8];
#pragma unroll
                for (int e = 0; e < 8; ++e) v[e] = raw[s][e][b] * tscale;
                th[b] = split_hi(v);
                tl[b] = split_lo(v, th[b]);
            }
            load_t(kn, s);
            // keep the loads ahead of the matrix products: issued late, their latency is not hidden
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int a = 0; a < WM; ++a) {
                const char* lp = L + (a * 16 + fr) * RS + s * 128 + fk * 32;
                const halfx8 xh = *reinterpret_cast<const halfx8*>(lp);
                const halfx8 xl = *reinterpret_cast<const halfx8*>(lp + 16);
#pragma unroll
                for (int b = 0; b < WN; ++b) acc[a][b] = __builtin_amdgcn_mfma_f32_16x16x32_f16(xl, th[b], acc[a][b], 0, 0, 0);
#pragma unroll
                for (int b = 0; b < WN; ++b) acc[a][b] = __builtin_amdgcn_mfma_f32_16x16x32_f16(xh, tl[b], acc[a][b], 0, 0, 0);
#pragma unroll
                for (int b = 0; b < WN; ++b) acc[a][b] = __builtin_amdgcn_mfma_f32_16x16x32_f16(xh, th[b], acc[a][b], 0, 0, 0);
            }
        }
        // the other buffer was last read in stage kt - 1, which every wave left at its barrier
        char* S = lds + ((kt + 1 - kb) & 1) * BM * RS;
#pragma unroll
        for (int u = 0; u < PER_T; ++u) *reinterpret_cast<u32x4*>(S + dst0 + u * RSTEP * RS) = xr[u];
        __syncthreads();
    }

    float* out = part == 0 ? Y : ws + (int64_t)(part - 1) * mt_count * BM * ld;
#pragma unroll
    for (int a = 0; a < WM; ++a)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int64_t c = m0 + a * 16 + 4 * fk + r;
            if (c >= ncol) continue;
            const ColInfo ci = info[c];
            tvec y;
#pragma unroll
            for (int b = 0; b < WN; ++b) {
                y[b] = ldexpf(acc[a][b][r], -(ci.exp + texp));
                // every element of T is positive, so a column with an infinite entry gives that infinity
                if (ci.cls) y[b] = ci.cls == 1 ? __builtin_inff() : ci.cls == 2 ? -__builtin_inff() : __builtin_nanf("");
            }
            *reinterpret_cast<tvec*>(out + c * ld + n0 + wave * 16 * WN + WN * fr) = y;
        }
}

// Y[q] += ws_1[q] + ws_2[q] + ... for the first `count` elements, parts added in order.
template <typename O>
__global__ void __launch_bounds__(256) split_reduce_kernel(O* __restrict__ Y, const O* __restrict__ ws,
                                                            int64_t count, int64_t stride, int parts) {
    const int64_t q = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (q >= count) return;
    O v = Y[q];
    for (int p = 0; p < parts; ++p) v += ws[p * stride + q];
    Y[q] = v;
}

// ---- narrow blocks: each wave streams R rows of T once and keeps up to NC columns of X in registers.

__device__ inline void unpack(const u32x4& v, float (&f)[4]) {
    f[0] = __uint_as_float(v.x); f[1] = __uint_as_float(v.y); f[2] = __uint_as_float(v.z); f[3] = __uint_as_float(v.w);
}
__device__ inline void unpack(const u32x4& v, double (&f)[2]) {
    f[0] = __hiloint2double(v.y, v.x); f[1] = __hiloint2double(v.w, v.z);
}
__device__ inline void unpack(const u32x4& v, float (&f)[8]) {
    uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        f[2 * q] = __uint_as_float(w[q] << 16);
        f[2 * q + 1] = __uint_as_float(w[q] & 0xffff0000u);
    }
}

template <int P>
struct SkinnyVec;
template <>
struct SkinnyVec<WFQ_PREC_FP64> { static constexpr int E = 2; };
template <>
struct SkinnyVec<WFQ_PREC_FP32> { static constexpr int E = 4; };
template <>
struct SkinnyVec<WFQ_PREC_BF16> { static constexpr int E = 8; };

// A wave computes R rows for all NC columns, U steps of its lanes' k loaded at once (the loads' latency bounds a small T),
// W waves a work-group. Each lane adds up every 64th 16-byte piece of a row, then the lanes are added.
template <int P, int NC, int R, int U, int W>
__global__ void __launch_bounds__(64 * W) tx_skinny_kernel(const typename Prec<P>::elem* __restrict__ X,
                                                           const typename Prec<P>::elem* __restrict__ T,
                                                           typename Prec<P>::out* __restrict__ Y, int64_t ld, int ncol) {
    using S = typename Prec<P>::sacc;
    constexpr int E = SkinnyVec<P>::E;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int64_t row0 = ((int64_t)blockIdx.x * W + wave) * R;
    S acc[R][NC];
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
        for (int c = 0; c < NC; ++c) acc[r][c] = 0;
    u32x4 x[U][NC], t[U][R];
    const auto load = [&](int u, int64_t k) {
#pragma unroll
        for (int r = 0; r < R; ++r) t[u][r] = *reinterpret_cast<const u32x4*>(T + (row0 + r) * ld + k);
#pragma unroll
        for (int c = 0; c < NC; ++c) x[u][c] = *reinterpret_cast<const u32x4*>(X + c * ld + k);
    };
    const auto add = [&](int u) {
        S xv[NC][E];
#pragma unroll
        for (int c = 0; c < NC; ++c) unpack(x[u][c], xv[c]);
#pragma unroll
        for (int r = 0; r < R; ++r) {
            S tv[E];
            unpack(t[u][r], tv);
#pragma unroll
            for (int c = 0; c < NC; ++c)
#pragma unroll
                for (int e = 0; e < E; ++e) acc[r][c] += tv[e] * xv[c][e];
        }
    };
    int64_t k = (int64_t)lane * E;
    for (; k + (U - 1) * 64 * E < ld; k += U * 64 * E) {
#pragma unroll
        for (int u = 0; u < U; ++u) load(u, k + u * 64 * E);
#pragma unroll
        for (int u = 0; u < U; ++u) add(u);
    }
    for (; k < ld; k += 64 * E) {
        load(0, k);
        add(0);
    }
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            S v = acc[r][c];
#pragma unroll
            for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off, 64);
            acc[r][c] = v;
        }
    if (lane == 0) {
#pragma unroll
        for (int c = 0; c < NC; ++c)
            if (c < ncol)
#pragma unroll
                for (int r = 0; r < R; ++r) Y[c * ld + row0 + r] = acc[r][c];
    }
}

// ---- variant registry: every kernel shape that can compute a block product, per precision.

struct KParts {
    int split, stage_bytes;
};
struct Variant {
    const char* name;
    int bm, bn;        // output tile (m = columns of Y, n = atoms); bm = 0 for the narrow kernel
    int max_ncol;      // largest ncol the variant accepts (narrow kernels hold columns in registers)
    // NULL: T recomputed, the stored copy not read (otf_narrow_f64). With parts (LDS-tile shapes only) k is divided as given
    void (*launch)(const Structure& s, const void* X, const void* T, void* Y, int64_t ld, int ncol, hipStream_t st,
                   const KParts* parts);
    KParts (*parts)(const Structure& s, int64_t ld, int ncol);   // how the shape divides k; NULL but for LDS tiles
};

// Number of k parts for a grid of `tiles` work-groups over nk k-steps when `slots` work-groups fit
// on the chip at once: the time is taken as proportional to (rounds of work-groups) x (k-steps per
// part), plus two k-steps per extra part for writing and adding the partial tiles. A split must
// win by 3 % and keep parts >= 8 k-steps and the partial tiles within the work-space cap.
int choose_split(int64_t tiles, int nk, int64_t slots, uint64_t part_bytes, uint64_t cap) {
    auto cost = [&](int sp) { return (double)((tiles * sp + slots - 1) / slots) * ((nk + sp - 1) / sp) + 2.0 * (sp - 1); };
    int best = 1;
    double best_cost = cost(1);
    for (int sp = 2; sp <= 8; ++sp) {
        if (nk / sp < 8 || (uint64_t)(sp - 1) * part_bytes > cap) break;
        const double c = cost(sp);
        if (c < 0.97 * best_cost) {
            best = sp;
            best_cost = c;
        }
    }
    return best;
}


// How a shape divides k: into `split` parts that begin at multiples of stage_bytes of a row
template <int P, int WM, int WN, int WAVES_M, int WAVES_N, int KB, int OCC, int ILV>
KParts mfma_parts(const Structure& s, int64_t ld, int ncol) {
    constexpr int BM = 16 * WM * WAVES_M, BN = 16 * WN * WAVES_N;
    constexpr int NT = 64 * WAVES_M * WAVES_N;
    static const int per_cu = [&] {
        int nb = 0;
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(
                &nb, reinterpret_cast<const void*>(tx_mfma_kernel<P, WM, WN, WAVES_M, WAVES_N, KB, OCC, ILV>), NT, 0) !=
                hipSuccess || nb < 1)
            nb = 1;
        return nb;
    }();
    const int mtc = (ncol + BM - 1) / BM, ntc = (int)(ld / BN);
    const int nk = (int)(ld * (int64_t)sizeof(typename Prec<P>::elem) / KB);
    const uint64_t part_bytes = (uint64_t)mtc * BM * ld * sizeof(typename Prec<P>::out);
    const uint64_t cap = s.split_fixed ? s.split_fixed_bytes : kSplitWsCap;
    return {choose_split((int64_t)mtc * ntc, nk, (int64_t)per_cu * device_cus(s.device), part_bytes, cap), KB};
}

template <int P, int WM, int WN, int WAVES_M, int WAVES_N, int KB, int OCC, int ILV = 0>
void launch_mfma(const Structure& s, const void* X, const void* T, void* Y, int64_t ld, int ncol, hipStream_t st,
                 const KParts* as = nullptr) {
    constexpr int BM = 16 * WM * WAVES_M, BN = 16 * WN * WAVES_N;
    using elem = typename Prec<P>::elem;
    using out = typename Prec<P>::out;
    const KParts kp = as ? *as : mfma_parts<P, WM, WN, WAVES_M, WAVES_N, KB, OCC, ILV>(s, ld, ncol);
    if (kp.stage_bytes % KB != 0) throw Error{WFQ_EINVAL, "block product: parts that are no whole stages"};
    const int mtc = (ncol + BM - 1) / BM, ntc = (int)(ld / BN), split = kp.split;
    const uint64_t part_bytes = (uint64_t)mtc * BM * ld * sizeof(out);
    out* ws = split > 1 ? static_cast<out*>(split_workspace(s, (split - 1) * part_bytes)) : nullptr;
    hipLaunchKernelGGL((tx_mfma_kernel<P, WM, WN, WAVES_M, WAVES_N, KB, OCC, ILV>), dim3(mtc * ntc * split),
                       dim3(64 * WAVES_M * WAVES_N), 0, st, static_cast<const elem*>(X), static_cast<const elem*>(T),
                       static_cast<out*>(Y), ld, ncol, mtc, ntc, split, kp.stage_bytes / KB, ws);
    if (split > 1) {
        const int64_t count = (int64_t)ncol * ld;
        hipLaunchKernelGGL(split_reduce_kernel<out>, dim3((unsigned)((count + 255) / 256)), dim3(256), 0, st,
                           static_cast<out*>(Y), ws, count, (int64_t)mtc * BM * ld, split - 1);
    }
}

// columns of X per pass of the fragment-layout product: the count of 16-column fragments (1 to 5 a pass) that
// pads least; of equal ones the wider, but 3 for 6, 11 and 12 fragments (6 603 to 20 000 atoms, 96 and 192 columns: no slower)
int frag_columns(int ncol) {
    const int f = (ncol + 15) / 16;
    if (f <= 5) return f;
    int best = 3;
    for (int c = 4; c <= 5; ++c)
        if ((f + c - 1) / c * c < (f + best - 1) / best * best) best = c;
    return best;
}
uint64_t frag_x_bytes(int64_t ld, int64_t ldc) { return (uint64_t)ld * ldc * sizeof(double); }
bool frag_fits(const Structure& s, int ncol) {
    const int bm = 16 * frag_columns(ncol);
    return frag_x_bytes(s.npad, (int64_t)(ncol + bm - 1) / bm * bm) <= (s.split_fixed ? s.split_fixed_bytes : kSplitWsCap);
}

template <int CF, int RF>
void launch_frag(const Structure& s, const void* X, const void* T, void* Y, int64_t ld, int ncol, hipStream_t st, const KParts*) {
    constexpr int BM = 16 * CF, BN = 16 * RF;
    const int mtc = (ncol + BM - 1) / BM, ntc = (int)(ld / BN), units = (int)(ld / 64);
    const int64_t ldc = (int64_t)mtc * BM;
    const uint64_t head = frag_x_bytes(ld, ldc), part_bytes = (uint64_t)ldc * ld * sizeof(double);
    const uint64_t cap = s.split_fixed ? s.split_fixed_bytes : kSplitWsCap;
    if (head > cap) {   // no room for the turned X
        launch_mfma<WFQ_PREC_FP64, 4, 4, 2, 4, 128, 1, 1>(s, X, T, Y, ld, ncol, st);
        return;
    }
    // k parts: the work-groups of the fullest CU times a part's time (64 k of a tile: the CU's 128 FP64 operations a
    // clock, or its share of the memory's rate), and for each further part its tile written and added
    const int64_t cus = device_cus(s.device);
    const double unit_us = 64.0 * BN * std::max(BM * 2 / (128 * 2400.0), 8 / (5.0e6 / (double)cus));
    auto cost = [&](int sp) {
        return (double)(((int64_t)mtc * ntc * sp + cus - 1) / cus) * ((units + sp - 1) / sp) * unit_us +
               (sp > 1 ? 3.0 + (sp - 1) * 2.0 * (double)part_bytes / 5.0e6 : 0.0);
    };
    int split = 1;
    for (int sp = 2; sp <= 16 && units / sp >= 4 && head + (uint64_t)(sp - 1) * part_bytes <= cap; ++sp)
        if (cost(sp) < 0.98 * cost(split)) split = sp;
    char* w = static_cast<char*>(split_workspace(s, head + (split - 1) * part_bytes));
    double *Xt = reinterpret_cast<double*>(w), *ws = reinterpret_cast<double*>(w + head);
    hipLaunchKernelGGL(xt_kernel, dim3((unsigned)(ld / 32), (unsigned)(ldc / 8)), dim3(256), 0, st,
                       static_cast<const double*>(X), ld, ncol, ldc, Xt);
    hipLaunchKernelGGL((tx_frag_kernel<CF, RF>), dim3(mtc * ntc * split), dim3(256), 0, st, Xt, ldc,
                       static_cast<const double*>(T), static_cast<double*>(Y), ld, ncol, mtc, ntc, split, ws);
    if (split > 1) {
        const int64_t count = (int64_t)ncol * ld;
        hipLaunchKernelGGL(split_reduce_kernel<double>, dim3((unsigned)((count + 255) / 256)), dim3(256), 0, st,
                           static_cast<double*>(Y), ws, count, (int64_t)mtc * BM * ld, split - 1);
    }
}

template <int WM, int WN, int KS, int OCC>
void launch_split(const Structure& s, const void* X, const void* T, void* Y, int64_t ld, int ncol, hipStream_t st, const KParts*) {
    constexpr int BM = 16 * WM, BN = 64 * WN;
    auto kern = tx_split_kernel<WM, WN, KS, OCC>;
    static const int per_cu = [&] {
        int nb = 0;
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, reinterpret_cast<const void*>(kern), 256, 0) != hipSuccess ||
            nb < 1)
            nb = 1;
        return nb;
    }();
    const uint64_t head = split_x_bytes(ld, ncol), info_bytes = round_up((int64_t)ncol * sizeof(ColInfo), 256);
    if (!split_scale_ok(s) || !split_fits(s, ld, ncol)) {
        // no room for the split X (or a T outside the split's range): the FP32 matrix instruction
        launch_mfma<WFQ_PREC_FP32, 4, 4, 2, 4, 64, 2>(s, X, T, Y, ld, ncol, st);
        return;
    }
    const int mtc = (ncol + BM - 1) / BM, ntc = (int)(ld / BN);
    const uint64_t part_bytes = (uint64_t)mtc * BM * ld * sizeof(float);
    const int split = choose_split((int64_t)mtc * ntc, (int)(ld / KS), (int64_t)per_cu * device_cus(s.device), part_bytes,
                                   (s.split_fixed ? s.split_fixed_bytes : kSplitWsCap) - head);
    char* ws = static_cast<char*>(split_workspace(s, head + (split - 1) * part_bytes));
    ColInfo* info = reinterpret_cast<ColInfo*>(ws);
    float* parts = reinterpret_cast<float*>(ws + head);
    const int texp = split_t_exp(s);
    split_x(static_cast<const float*>(X), ld, ncol, ws, st);
    hipLaunchKernelGGL(kern, dim3(mtc * ntc * split), dim3(256), 0, st, ws + info_bytes, info,
                       static_cast<const float*>(T), static_cast<float*>(Y), ld, ncol, mtc, ntc, split, parts,
                       (float)std::ldexp(1.0, texp), texp);
    if (split > 1)
        add_parts_f32(static_cast<float*>(Y), parts, (int64_t)ncol * ld, (int64_t)mtc * BM * ld, split - 1, st);
}

template <int P, int NC, int R, int U = 1, int W = 4>
void launch_skinny_rows(const Structure&, const void* X, const void* T, void* Y, int64_t ld, int ncol, hipStream_t st,
                        const KParts*) {
    using elem = typename Prec<P>::elem;
    using out = typename Prec<P>::out;
    hipLaunchKernelGGL((tx_skinny_kernel<P, NC, R, U, W>), dim3((unsigned)(ld / (W * R))), dim3(64 * W), 0, st,
                       static_cast<const elem*>(X), static_cast<const elem*>(T), static_cast<out*>(Y), ld, ncol);
}

// Rows per wave by size: few rows a wave where T has few of them, 4 where the waves fill the chip anyway and X, read again
// by every wave, bounds instead. One wave a work-group, so that the CUs get equal shares. us, 4 rows in work-groups of 4
// waves (what all sizes had) / 2 rows and two loads ahead / 4 rows, one wave a work-group: FP64, 2 columns 600 atoms 5.3 /
// 3.3 / 3.8, 2 000 12.3 / 8.0 / -, 4 000 31.4 / 21.1 / 26.0, 5 000 41.7 / 30.4 / 34.0, 7 000 92 / 92 / 86, 20 000 650 / 665 /
// 635; 4 columns 600 7.5 / 4.1 / -, 4 000 40.5 / 26.6 / 39.9, 7 000 131 / 129 / 127; 8 columns 1 500 16.1 / 13.9 / 10.2, 4 000
// 41.0 / - / 35.5, 10 000 247 / 329 / 220 and with one row at 250 atoms 3.5 against 5.5, 600 6.3 and 7.1. FP32, 8 columns
// 2 000 20.0 / 6.7 / -, 7 000 69 / 40 / 68, 10 000 155 / 127 / 158, 20 000 366 / 468 / 350; 4 columns 4 000 18.4 / 12.2 / 13.7,
// 7 000 30.5 / 31.9 / 30.7; 8 rows in work-groups of 4 waves ("r8", tuned handles only) took 206 at 15 800, 229 at 16 480 and 298
// at 20 000 atoms against 182, 207 and 294 of 4 rows. A row's sums are the same in all of them.
template <int P, int NC>
void launch_skinny(const Structure& s, const void* X, const void* T, void* Y, int64_t ld, int ncol, hipStream_t st,
                   const KParts* parts) {
    constexpr bool wide64 = P == WFQ_PREC_FP64 && NC == 8;
    if (wide64 ? ld < 1024 : ld < (NC == 8 ? 12288 : 6144))
        launch_skinny_rows<P, NC, wide64 ? 1 : 2, wide64 ? 4 : 2, 1>(s, X, T, Y, ld, ncol, st, parts);
    else
        launch_skinny_rows<P, NC, 4, 1, 1>(s, X, T, Y, ld, ncol, st, parts);
}

template <int P, int WM, int WN, int WAVES_M, int WAVES_N, int KB, int OCC, int ILV = 0>
Variant tile(const char* name) {
    return {name, 16 * WM * WAVES_M, 16 * WN * WAVES_N, 1 << 30, launch_mfma<P, WM, WN, WAVES_M, WAVES_N, KB, OCC, ILV>,
            mfma_parts<P, WM, WN, WAVES_M, WAVES_N, KB, OCC, ILV>};
}

template <int P>
const std::vector<Variant>& variants() {
    constexpr int OCC2 = P == WFQ_PREC_FP64 ? 1 : 2;
    static const std::vector<Variant> v = {
        {"skinny2", 0, 4, 2, launch_skinny<P, 2>, nullptr},
        {"skinny4", 0, 4, 4, launch_skinny<P, 4>, nullptr},
        {"skinny8", 0, 4, 8, launch_skinny<P, 8>, nullptr},
        {"skinny2r8", 0, 8, 2, launch_skinny_rows<P, 2, 8>, nullptr},
        {"skinny4r8", 0, 8, 4, launch_skinny_rows<P, 4, 8>, nullptr},
        tile<P, 2, 2, 1, 4, 128, 2>("m32n128"),
        tile<P, 4, 2, 1, 4, 128, 2>("m64n128"),
        tile<P, 4, 4, 2, 2, 128, OCC2>("m128n128"),
        tile<P, 4, 2, 2, 2, 128, 2>("m128n64"),
        tile<P, 4, 4, 1, 4, 128, 1>("m64n256"),
        tile<P, 4, 4, 2, 4, 128, 1>("m128n256w8"),
        tile<P, 4, 4, 4, 2, 128, 1>("m256n128w8"),
        tile<P, 4, 4, 2, 2, 256, 1>("m128n128k256"),
        tile<P, 4, 2, 1, 4, 256, 1>("m64n128k256"),
        tile<P, 4, 4, 2, 4, 128, 1, 1>("m128n256w8i"),
        tile<P, 4, 4, 4, 2, 128, 1, 1>("m256n128w8i"),
        tile<P, 4, 2, 1, 4, 128, 2, 1>("m64n128i"),
        tile<P, 4, 2, 2, 2, 128, 2, 1>("m128n64i"),
        tile<P, 4, 2, 1, 4, 256, 1, 1>("m64n128k256i"),
    };
    return v;
}

// Wider column tiles for FP32 and BF16 (their accumulators are half the size of FP64 ones), so
// that column counts between the powers of two are not padded up to the next multiple of 128.
template <int P>
const std::vector<Variant>& variants_all() {
    static const std::vector<Variant> v = [] {
        std::vector<Variant> r = variants<P>();
        if constexpr (P == WFQ_PREC_FP64) {
            r.push_back({"otfn2", 0, 4, 2, nullptr, nullptr});
            r.push_back({"otfn4", 0, 4, 4, nullptr, nullptr});
            r.push_back({"otfn8", 0, 4, 8, nullptr, nullptr});
            // fragment-layout products (f<columns>n<rows of T>)
            r.push_back({"f16n64", 16, 64, 1 << 30, launch_frag<1, 4>, nullptr});
            r.push_back({"f32n64", 32, 64, 1 << 30, launch_frag<2, 4>, nullptr});
            r.push_back({"f48n32", 48, 32, 1 << 30, launch_frag<3, 2>, nullptr});
            r.push_back({"f48n64", 48, 64, 1 << 30, launch_frag<3, 4>, nullptr});
            r.push_back({"f64n32", 64, 32, 1 << 30, launch_frag<4, 2>, nullptr});
            r.push_back({"f80n32", 80, 32, 1 << 30, launch_frag<5, 2>, nullptr});
        }
        if constexpr (P != WFQ_PREC_FP64) {
            r.push_back(tile<P, 3, 4, 2, 4, 128, 1>("m96n256w8"));
            r.push_back(tile<P, 5, 4, 2, 4, 128, 1>("m160n256w8"));
            r.push_back(tile<P, 6, 4, 2, 4, 128, 1>("m192n256w8"));
            r.push_back(tile<P, 3, 4, 4, 2, 128, 1>("m192n128w8"));
            r.push_back(tile<P, 7, 4, 2, 4, 128, 1>("m224n256w8"));
            r.push_back(tile<P, 7, 2, 2, 4, 128, 1>("m224n128w8"));
            // 64-byte k stages: half the LDS, so two work-groups share a CU and one's matrix-core
            // work covers the other's barrier
            r.push_back(tile<P, 4, 4, 2, 4, 64, 2>("m128n256w8k64"));
        }
        if constexpr (P == WFQ_PREC_FP32) {
            // FP16-split products (s<columns>n<rows of T>k<k per stage>)
            r.push_back({"s32n256k32", 32, 256, 1 << 30, launch_split<2, 4, 32, 2>, nullptr});
            r.push_back({"s64n256k32", 64, 256, 1 << 30, launch_split<4, 4, 32, 2>, nullptr});
            r.push_back({"s96n256k32", 96, 256, 1 << 30, launch_split<6, 4, 32, 2>, nullptr});
            r.push_back({"s128n256k32", 128, 256, 1 << 30, launch_split<8, 4, 32, 2>, nullptr});
            r.push_back({"s64n128k64", 64, 128, 1 << 30, launch_split<4, 2, 64, 2>, nullptr});
            r.push_back({"s96n128k64", 96, 128, 1 << 30, launch_split<6, 2, 64, 2>, nullptr});
            r.push_back({"s128n128k64", 128, 128, 1 << 30, launch_split<8, 2, 64, 2>, nullptr});
            r.push_back({"s192n128k32", 192, 128, 1 << 30, launch_split<12, 2, 32, 2>, nullptr});
        }
        return r;
    }();
    return v;
}

const std::vector<Variant>& variants_of(int prec) {
    return prec == WFQ_PREC_FP64 ? variants_all<WFQ_PREC_FP64>()
           : prec == WFQ_PREC_FP32 ? variants_all<WFQ_PREC_FP32>() : variants_all<WFQ_PREC_BF16>();
}

int find_variant(int prec, const char* name) {
    const auto& v = variants_of(prec);
    for (size_t k = 0; k < v.size(); ++k)
        if (std::strcmp(v[k].name, name) == 0) return (int)k;
    return -1;
}

struct Pick { int upto; const char* name; };
int pick_name(int prec, const Pick* t, int ncol) {
    while (ncol > t->upto) ++t;
    const int k = find_variant(prec, t->name);
    return k >= 0 ? k : find_variant(prec, "m128n256w8");   // present for every precision
}

// Built-in choice of the kept order when no tuning result covers ncol: the fastest shapes measured on MI355X for
// a 20 000-atom T, per precision and column count.
int default_variant(int prec, int ncol) {
    static const Pick f64[] = {{2, "skinny2"}, {4, "skinny4"}, {8, "skinny8"}, {32, "m32n128"}, {64, "m64n128i"},
                               {96, "m128n256w8i"}, {128, "m128n256w8"}, {192, "m64n128i"}, {256, "m128n256w8i"},
                               {320, "m64n128"}, {1 << 30, "m128n256w8i"}};
    static const Pick f32[] = {{2, "skinny2"}, {4, "skinny4"}, {32, "m32n128"}, {64, "m64n128k256i"},
                               {96, "m96n256w8"}, {128, "m128n256w8k64"}, {160, "m160n256w8"}, {192, "m96n256w8"},
                               {224, "m224n128w8"}, {256, "m128n256w8k64"}, {288, "m96n256w8"}, {320, "m160n256w8"},
                               {1 << 30, "m128n256w8k64"}};
    // BF16 T is 2 bytes per element: even one column streams it faster through the matrix cores
    static const Pick b16[] = {{64, "m64n128i"}, {128, "m128n128"}, {192, "m192n256w8"}, {256, "m256n128w8i"},
                               {320, "m160n256w8"}, {1 << 30, "m192n256w8"}};
    return pick_name(prec, prec == WFQ_PREC_FP64 ? f64 : prec == WFQ_PREC_FP32 ? f32 : b16, ncol);
}

// FP32 products through the FP16 matrix cores: applications of the operator only, no solves
bool is_split(const char* name) { return name[0] == 's' && name[1] >= '0' && name[1] <= '9'; }

// Built-in choice in any order for FP32 and BF16, by padded size too: the fastest shapes measured at 700, 1 000, 1 400,
// 2 000, 2 800, 4 000, 5 200, 6 600, 8 000, 10 000 and 20 000 atoms. A small T has few tiles of many rows, so
// narrower and shorter ones fill the chip; us against the kept order's shape: FP32 2 000 atoms 15 / 26 at 64 columns,
// 2 800 atoms 11 / 17 at 4, BF16 2 000 atoms 9 / 13 at 128, 11 / 15 at 192.
// The FP16-split FP32 shapes (s...) where they are faster and no less accurate than the FP32 matrix instruction, us of the
// two: N 20 000 280 / 362 at 8 columns, 310 / 556 at 64, 379 / 846 at 128, 929 / 2 427 at 384; N 10 000 117 / 117, 135 / 214, 262 / 600;
// N 5 200 33 / 38, 39 / 46, 49 / 80, 92 / 160; N 4 000 42 / 48 at 128; N 2 800 31 / 37 at 128. Error against 64 bits, random
// vectors: N 612 2.7e-7 / 2.6e-7, N 2 600 2.7e-7 / 3.7e-7, N 20 000 6.5e-7 to 9.5e-7 / 1.0e-6 to 1.5e-6 (the more k parts, the
// smaller).
int any_variant(const Structure& s, int prec, int ncol) {
    constexpr int rest = 1 << 30;
    struct Range { int64_t below; Pick t[9]; };
    static const Range f32[] = {
        {1280, {{2, "skinny2"}, {4, "skinny4"}, {8, "skinny8"}, {256, "m32n128"}, {rest, "m64n128i"}}},
        {1536, {{2, "skinny2"}, {4, "skinny4"}, {160, "m32n128"}, {288, "m64n128i"}, {rest, "s64n128k64"}}},
        {1792, {{2, "skinny2"}, {4, "skinny4"}, {160, "m32n128"}, {rest, "s64n128k64"}}},
        {3072, {{2, "skinny2"}, {4, "skinny4"}, {96, "m32n128"}, {rest, "s64n128k64"}}},
        {4608, {{2, "skinny2"}, {4, "skinny4"}, {32, "m32n128"}, {64, "m64n128i"}, {rest, "s64n128k64"}}},
        {6144, {{2, "skinny2"}, {4, "skinny4"}, {256, "s64n128k64"}, {rest, "s96n256k32"}}},
        {9216, {{2, "skinny2"}, {4, "skinny4"}, {32, "m32n128"}, {64, "s64n128k64"}, {96, "s96n128k64"}, {128, "s64n256k32"},
                {192, "s96n256k32"}, {rest, "s128n256k32"}}},
        {16384, {{2, "skinny2"}, {4, "skinny4"}, {32, "m32n128"}, {64, "s64n256k32"}, {96, "s96n128k64"}, {128, "s128n128k64"},
                 {192, "s192n128k32"}, {rest, "s128n256k32"}}},
        {INT64_MAX, {{2, "skinny2"}, {4, "skinny4"}, {96, "s96n256k32"}, {128, "s128n256k32"}, {192, "s192n128k32"},
                     {256, "s128n256k32"}, {288, "s96n256k32"}, {rest, "s128n256k32"}}}};
    static const Range b16[] = {
        {1536, {{2, "skinny2"}, {4, "skinny4"}, {192, "m32n128"}, {rest, "m64n128i"}}},
        {3072, {{2, "skinny2"}, {128, "m32n128"}, {rest, "m64n128i"}}},
        {6144, {{96, "m32n128"}, {256, "m64n128i"}, {rest, "m192n128w8"}}},
        {9216, {{64, "m32n128"}, {128, "m64n128i"}, {160, "m160n256w8"}, {192, "m192n128w8"}, {256, "m128n256w8i"},
                {320, "m160n256w8"}, {rest, "m192n256w8"}}},
        {16384, {{64, "m64n128i"}, {128, "m128n128"}, {160, "m160n256w8"}, {192, "m192n128w8"}, {256, "m128n256w8i"},
                 {320, "m160n256w8"}, {rest, "m192n256w8"}}},
        {INT64_MAX, {{64, "m64n128i"}, {128, "m128n128"}, {192, "m192n256w8"}, {256, "m256n128w8i"}, {320, "m160n256w8"},
                     {rest, "m192n256w8"}}}};
    const Range* r = prec == WFQ_PREC_FP32 ? f32 : b16;
    while (s.npad >= r->below) ++r;
    const int k = pick_name(prec, r->t, ncol);
    // no room for the split X, or a T outside the split's range: the FP32 instruction's shape
    if (is_split(variants_of(prec)[k].name) && (!split_scale_ok(s) || !split_fits(s, s.npad, ncol)))
        return default_variant(prec, ncol);
    return k;
}

// padded size from which untuned narrow FP64 products are recomputed rather than streamed: in the symmetric form
// (5 000 atoms, 1 to 4 columns: 22 / 26 / 31 / 33 us recomputed, 31 / 31 / 35 / 35 streamed; 4 000: 21 / 24 / 29 / 31 and
// 27 / 27 / 27 / 28), and one-sided, in the kept order (20 000 atoms, 3 columns: 252 us recomputed, 475 streamed)
constexpr int64_t kSymNarrowFrom = 4608, kOtfNarrowFrom = 16384;
// Matrix-free FP64 products of up to this many columns go through the narrow kernel, 4 at a time; the wide one's time
// hardly depends on its columns. From 3 072 rows on 64, by measurement: narrow / wide, us, 4 096 atoms 502 / 875 at 64, 988 /
// 882 at 128; 16 384 atoms 1 126 / 3 027 at 32, 2 230 / 3 021 at 64, 4 444 / 4 499 at 128. Below, the wide kernel
// takes about 20 us and 0.25 us a row; a narrow pass 23 us up to 1 024 rows and 27.5 above, and 0.048 us an entry of the
// longest near-field list (some 40 on graphene, 458 on a metal sphere). Operator, narrow / wide, us: tubes of 200 atoms, 12
// columns 76 / 81, 16 columns 98 / 81; 880, 40 columns 231 / 279, 56 columns 319 / 279; spheres of 381 atoms, 12 columns
// 134 / 152, 16 columns 171 / 152; 935, 24 columns 281 / 307, 64 columns 713 / 321; 1 985, 40 columns 527 / 588, 64 columns 828 / 607.
int otf_narrow_columns(const Structure& s) {
    if (s.npad >= 3072) return 64;
    const double wide = 20.0 + 0.25 * s.npad, pass = (s.npad <= 1024 ? 23.0 : 27.5) + 0.048 * s.near_w;
    return std::min(64, 4 * (int)(wide / pass));
}
bool otf_takes_narrow(const Structure& s, int prec, int ncol, Order order) {
    return prec == WFQ_PREC_FP64 && ncol <= otf_narrow_columns(s) && otf_narrow_fits(s, ncol, order);
}

// The tuned entry with the smallest ncol >= this one (or the largest tuned one), used only when
// it was tuned for a comparable width (within a factor of two); -1 without one
int tuned_variant(const Structure& s, int prec, int ncol, Order order) {
    const auto& tuned = s.tuned[prec][(int)order];
    auto it = tuned.lower_bound(ncol);
    if (it == tuned.end() && !tuned.empty()) it = std::prev(tuned.end());
    if (it != tuned.end() && it->first <= 2 * ncol && ncol <= 2 * it->first) {
        const Variant& v = variants_of(prec)[it->second];
        if (ncol <= v.max_ncol && (v.launch || otf_narrow_fits(s, ncol, order))) return it->second;
    }
    return -1;
}

int pick_variant(const Structure& s, int prec, int ncol, Order order) {
    const int tuned = tuned_variant(s, prec, ncol, order);
    if (tuned >= 0) return tuned;
    if (prec == WFQ_PREC_FP64 && order == Order::any && ncol > 4) {
        // in any order: two narrow recomputed products for 5 to 8 columns of a large structure (20 000 atoms, 8
        // columns: 380 us, streamed through the matrix cores 576; 10 000: 144 and 161; 8 000: 138 and 94), and the fragment-layout shapes (figures at
        // tx_frag_kernel) but for 5 to 8 columns of the smallest, whose one launch is quicker than two, and for up to 32
        // columns beyond 16 384 rows, where T's bytes bound both and the tile is nearer to the memory's rate (operator,
        // fragment layout / tile: 16 480 atoms, 24 columns 495 / 450, 17 200 535 / 474, 19 280 633 / 576; 16 320: 387 / 432)
        if (ncol <= 8 && s.npad >= 10240 && otf_narrow_sym(s, 4, order)) return find_variant(prec, "otfn8");
        if ((ncol > 8 || s.npad >= 1536) && (ncol > 32 || s.npad <= 16384) && frag_fits(s, ncol)) {
            static const char* const name[] = {"f16n64", "f32n64", "f48n32", "f64n32", "f80n32"};
            const int cf = frag_columns(ncol);
            return find_variant(prec, cf == 3 && s.npad >= 16384 ? "f48n64" : name[cf - 1]);
        }
    }
    // narrow FP64 products of large structures: recomputing the elements on the vector ALUs
    // (about 16 FP64 operations per pair) beats streaming 8 bytes per pair of the stored copy
    if (prec == WFQ_PREC_FP64 && ncol <= 4 && s.npad >= kSymNarrowFrom && otf_narrow_fits(s, ncol, order) &&
        (s.npad >= kOtfNarrowFrom || otf_narrow_sym(s, ncol, order)))
        return find_variant(prec, ncol <= 2 ? "otfn2" : "otfn4");
    return order == Order::any && prec != WFQ_PREC_FP64 ? any_variant(s, prec, ncol) : default_variant(prec, ncol);
}

void run_variant(const Structure& s, int prec, int var, const void* X, void* Y, int ncol, hipStream_t st,
                 Order order = Order::any, const KParts* parts = nullptr) {
    const void* T = prec == WFQ_PREC_FP64 ? (const void*)s.T64 : prec == WFQ_PREC_FP32 ? (const void*)s.T32
                                                                                       : (const void*)s.T16;
    if (T == nullptr) throw Error{WFQ_EINVAL, "the stored copy of T for this precision was not built"};
    const Variant& v = variants_of(prec)[var];
    if (ncol > v.max_ncol) throw Error{WFQ_EINVAL, "kernel variant cannot take that many columns"};
    if (v.launch) {
        v.launch(s, X, T, Y, s.npad, ncol, st, parts);
    } else {
        for (int c0 = 0; c0 < ncol; c0 += 4)
            otf_narrow_f64(s, static_cast<const double*>(X) + (int64_t)c0 * s.npad,
                           static_cast<double*>(Y) + (int64_t)c0 * s.npad, s.npad, std::min(4, ncol - c0),
                           device_cus(s.device), st, order);
    }
    WFQ_CHECK_LAUNCH();
}

// The product of the shape that pick_variant names. In the kept order the default shapes are those of a 20 000-atom T;
// on a small T their tiles are few, and a smaller tile gives the same sums (k is walked in the same order inside a
// stage of any size) when it divides k as they do. A tuned shape runs as it was measured. FP64, 989 atoms: 60 us
// in the old shape and 14 in the new at 80 columns, 21 and 14 at 48.
// In any order the smaller FP32 tiles divide k into no fewer parts than those shapes, and up to 64 columns into two more than
// they would themselves, or as those shapes do where that is more than a work-group a CU: an FP32 sum's error grows with its length. Error after L and us of the operator, their own parts /
// these (that of the kept order's shape): 1 289-atom sphere, 256 columns 2.14e-6 / 1.88e-6 (1.88e-6), 37 / 36; 1 721, 40
// columns 2.64e-6 / 2.10e-6 (2.37e-6), 25.4 / 23.3; 2 315, 48 columns 2.58e-6 / 2.33e-6 (2.33e-6).
void run_picked(const Structure& s, int prec, int ncol, Order order, const void* X, void* Y, hipStream_t st) {
    const int var = pick_variant(s, prec, ncol, order);
    const Variant& v = variants_of(prec)[var];
    int other = -1;
    if (order == Order::kept && v.parts && tuned_variant(s, prec, ncol, order) < 0) {
        if (prec == WFQ_PREC_FP64 && ncol > 32) {
            if (ncol <= (s.npad < 3072 ? 192 : s.npad < 10240 ? 112 : 0)) other = find_variant(prec, "m32n128");
            else if (s.npad < 3072) other = find_variant(prec, "m64n128i");
        } else if (prec == WFQ_PREC_FP32 && s.npad < 3072 && ncol > 32 && ncol <= 224) {
            other = find_variant(prec, ncol <= 96 || s.npad < 1536 ? "m32n128" : "m64n128i");
        }
    }
    if (other >= 0 && other != var) {
        const KParts kp = v.parts(s, s.npad, ncol);
        if (kp.stage_bytes % 128 == 0) {   // both shapes' stages are 128 bytes
            run_variant(s, prec, other, X, Y, ncol, st, order, &kp);
            return;
        }
    }
    if (order == Order::any && prec == WFQ_PREC_FP32 && v.parts && tuned_variant(s, prec, ncol, order) < 0) {
        const Variant& d = variants_of(prec)[default_variant(prec, ncol)];
        KParts kp = v.parts(s, s.npad, ncol);
        const int own = kp.split, stages = (int)(s.npad * (int64_t)sizeof(float) / kp.stage_bytes);
        const KParts dp = d.parts ? d.parts(s, s.npad, ncol) : kp;
        kp.split = std::max(own, dp.split);
        if (ncol <= 64 && s.npad < 3072) {
            const int64_t tiles = (ncol + v.bm - 1) / v.bm * (s.npad / v.bn);
            if (tiles * (kp.split + 2) <= device_cus(s.device)) kp.split += 2;
            else if (dp.stage_bytes % 128 == 0) kp = dp;
        }
        const uint64_t part_bytes = (uint64_t)round_up(ncol, v.bm) * s.npad * sizeof(float);
        if ((kp.split != own || kp.stage_bytes != 128) && kp.split <= stages / 2 &&
            (kp.split - 1) * part_bytes <= (s.split_fixed ? s.split_fixed_bytes : kSplitWsCap)) {
            run_variant(s, prec, var, X, Y, ncol, st, order, &kp);
            return;
        }
    }
    run_variant(s, prec, var, X, Y, ncol, st, order);
}

template <typename E>
__global__ void convert_kernel(const double* __restrict__ src, E* __restrict__ dst, int64_t count) {
    int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i < count) dst[i] = cast_from_double<E>(src[i]);
}

}  // namespace

bool split_scale_ok(const Structure& s) { return s.eta_max > 0x1p-60 && s.eta_max < 0x1p60; }

int split_t_exp(const Structure& s) {
    int ex = 0;
    (void)std::frexp(s.eta_max, &ex);
    return 15 - ex;
}

uint64_t split_x_bytes(int64_t ld, int ncol) {
    return round_up((int64_t)ncol * sizeof(ColInfo), 256) + (uint64_t)ncol * ld * 4;
}

bool split_fits(const Structure& s, int64_t ld, int ncol) {
    return split_x_bytes(ld, ncol) <= (s.split_fixed ? s.split_fixed_bytes : kSplitWsCap);
}

void split_x(const float* X, int64_t ld, int ncol, char* ws, hipStream_t st) {
    const int64_t info_bytes = round_up((int64_t)ncol * sizeof(ColInfo), 256);
    hipLaunchKernelGGL(split_x_kernel, dim3((unsigned)ncol), dim3(1024), 0, st, X, ld, ws + info_bytes,
                       reinterpret_cast<ColInfo*>(ws));
    WFQ_CHECK_LAUNCH();
}

void add_parts_f32(float* Y, const float* ws, int64_t count, int64_t stride, int parts, hipStream_t st) {
    hipLaunchKernelGGL(split_reduce_kernel<float>, dim3((unsigned)((count + 255) / 256)), dim3(256), 0, st, Y, ws, count,
                       stride, parts);
    WFQ_CHECK_LAUNCH();
}

int device_cus(int device) {
    int cus = 0;
    WFQ_HIP(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, device));
    return cus > 0 ? cus : 1;
}

void* split_workspace(const Structure& s, uint64_t bytes) {
    if (s.split_fixed) {
        // a caller-provided region (the allocation-free entry point): never allocate
        if (bytes > s.split_fixed_bytes) throw Error{WFQ_ENOMEM, "split-k partial tiles exceed the fixed work space"};
        return s.split_fixed;
    }
    if (bytes > s.split_ws_bytes) {
        if (s.split_ws) {
            WFQ_HIP(hipFree(s.split_ws));
            s.split_ws = nullptr;
            s.split_ws_bytes = 0;
        }
        ++s.epoch;
        hipError_t e = hipMalloc(&s.split_ws, bytes);
        if (e != hipSuccess) throw Error{WFQ_ENOMEM, std::string("hipMalloc failed: ") + hipGetErrorString(e)};
        s.split_ws_bytes = bytes;
    }
    return s.split_ws;
}

void convert_from_f64(int prec, const double* src, void* dst, int64_t count, hipStream_t st) {
    if (count <= 0) return;
    dim3 grd((unsigned)((count + 255) / 256));
    if (prec == WFQ_PREC_FP64)
        WFQ_HIP(hipMemcpyAsync(dst, src, count * 8, hipMemcpyDeviceToDevice, st));
    else if (prec == WFQ_PREC_FP32)
        hipLaunchKernelGGL(convert_kernel<float>, grd, dim3(256), 0, st, src, static_cast<float*>(dst), count);
    else
        hipLaunchKernelGGL(convert_kernel<uint16_t>, grd, dim3(256), 0, st, src, static_cast<uint16_t*>(dst), count);
    WFQ_CHECK_LAUNCH();
}

void tx_f64(const Structure& s, const double* X, double* Y, int ncol, hipStream_t st, Order order) {
    if (ncol > 0) run_picked(s, WFQ_PREC_FP64, ncol, order, X, Y, st);
}
void tx_f32(const Structure& s, const float* X, float* Y, int ncol, hipStream_t st, Order order) {
    if (ncol > 0) run_picked(s, WFQ_PREC_FP32, ncol, order, X, Y, st);
}
void tx_bf16(const Structure& s, const uint16_t* X, float* Y, int ncol, hipStream_t st, Order order) {
    if (ncol > 0) run_picked(s, WFQ_PREC_BF16, ncol, order, X, Y, st);
}

void tx_any(const Structure& s, int prec, const void* X, void* Y, int ncol, hipStream_t st, Order order) {
    if (s.t_mode == WFQ_TMODE_OTF) {
        if (prec == WFQ_PREC_FP32)
            otf_tx_f32(s, static_cast<const float*>(X), static_cast<float*>(Y), ncol, st);
        else if (otf_takes_narrow(s, prec, ncol, order))
            for (int c0 = 0; c0 < ncol; c0 += 4)
                otf_narrow_f64(s, static_cast<const double*>(X) + (int64_t)c0 * s.npad,
                               static_cast<double*>(Y) + (int64_t)c0 * s.npad, s.npad, std::min(4, ncol - c0),
                               device_cus(s.device), st, order);
        else if (prec == WFQ_PREC_FP64)
            otf_tx_f64(s, static_cast<const double*>(X), static_cast<double*>(Y), ncol, st);
        else
            throw Error{WFQ_EINVAL, "matrix-free T runs in FP32 or FP64"};
        return;
    }
    if (prec == WFQ_PREC_FP64)
        tx_f64(s, static_cast<const double*>(X), static_cast<double*>(Y), ncol, st, order);
    else if (prec == WFQ_PREC_FP32)
        tx_f32(s, static_cast<const float*>(X), static_cast<float*>(Y), ncol, st, order);
    else
        tx_bf16(s, static_cast<const uint16_t*>(X), static_cast<float*>(Y), ncol, st, order);
}

void tx_variant_run(const Structure& s, int prec, int var, const void* X, void* Y, int ncol, hipStream_t st) {
    if (ncol > 0) run_variant(s, prec, var, X, Y, ncol, st);
}

bool tx_is_otf_narrow(const Structure& s, int prec, int ncol, Order order) {
    if (prec != WFQ_PREC_FP64) return false;
    if (s.t_mode == WFQ_TMODE_OTF) return otf_takes_narrow(s, prec, ncol, order);
    if (ncol > 4) return false;
    return std::strncmp(variants_of(prec)[pick_variant(s, prec, ncol, order)].name, "otfn", 4) == 0;
}

bool tx_is_skinny(const Structure& s, int prec, int ncol, Order order) {
    if (s.t_mode == WFQ_TMODE_OTF) return false;
    return std::strncmp(variants_of(prec)[pick_variant(s, prec, ncol, order)].name, "skinny", 6) == 0;
}

int tx_variant_count(int precision) { return (int)variants_of(precision).size(); }
const char* tx_variant_name(int precision, int k) { return variants_of(precision)[k].name; }
int tx_variant_max_ncol(int precision, int k) { return variants_of(precision)[k].max_ncol; }

// Time every variant that accepts ncol (reps launches each, after one warm-up launch) on random
// device data and keep the fastest for this ncol in s.tuned, for the solves (kept order, no FP16-split shape) and for any
// order. ms[k] = average time of variant k (negative when the variant does not apply); the recomputed shapes
// run another kernel in each order and are timed in both, ms[k] being the kept order's.
void tune_tx(Structure& s, int prec, int ncol, int reps, double* ms, hipStream_t st) {
    const int64_t rows = round_up(ncol, kColPad);
    const int es = prec == WFQ_PREC_FP64 ? 8 : prec == WFQ_PREC_FP32 ? 4 : 2;
    const int os = prec == WFQ_PREC_FP64 ? 8 : 4;
    void *X = nullptr, *Y = nullptr;
    double* X64 = nullptr;
    WFQ_HIP(hipMalloc(&X, rows * s.npad * es));
    WFQ_HIP(hipMalloc(&Y, rows * s.npad * os));
    WFQ_HIP(hipMalloc(&X64, rows * s.npad * 8));
    {
        std::vector<double> h(rows * s.npad, 0.0);
        uint64_t state = 0x9E3779B97F4A7C15ull * (uint64_t)(ncol + 1);
        for (int64_t c = 0; c < ncol; ++c)
            for (int64_t i = 0; i < s.n; ++i) {
                state = state * 6364136223846793005ull + 1442695040888963407ull;
                h[c * s.npad + i] = (double)(state >> 11) * (1.0 / 9007199254740992.0) - 0.5;
            }
        h2d_sync(s, X64, h.data(), h.size() * 8, st);
        WFQ_HIP(hipStreamSynchronize(st));
    }
    convert_from_f64(prec, X64, X, rows * s.npad, st);
    hipEvent_t a, b;
    WFQ_HIP(hipEventCreate(&a));
    WFQ_HIP(hipEventCreate(&b));
    const auto& vs = variants_of(prec);
    auto time_of = [&](size_t k, Order order) {
        run_variant(s, prec, (int)k, X, Y, ncol, st, order);
        WFQ_HIP(hipEventRecord(a, st));
        for (int r = 0; r < reps; ++r) run_variant(s, prec, (int)k, X, Y, ncol, st, order);
        WFQ_HIP(hipEventRecord(b, st));
        WFQ_HIP(hipEventSynchronize(b));
        float t = 0.f;
        WFQ_HIP(hipEventElapsedTime(&t, a, b));
        return (double)t / reps;
    };
    double best[2] = {1e300, 1e300};
    int best_k[2] = {-1, -1};
    auto keep = [&](Order order, size_t k, double t) {
        if (t >= best[(int)order]) return;
        best[(int)order] = t;
        best_k[(int)order] = (int)k;
    };
    for (size_t k = 0; k < vs.size(); ++k) {
        ms[k] = -1.0;
        if (ncol > vs[k].max_ncol) continue;
        ms[k] = time_of(k, Order::kept);
        keep(Order::any, k, vs[k].launch ? ms[k] : time_of(k, Order::any));
        if (!is_split(vs[k].name)) keep(Order::kept, k, ms[k]);
    }
    (void)hipEventDestroy(a);
    (void)hipEventDestroy(b);
    (void)hipFree(X);
    (void)hipFree(Y);
    (void)hipFree(X64);
    for (int o = 0; o < 2; ++o)
        if (best_k[o] >= 0) s.tuned[prec][o][ncol] = best_k[o];
    ++s.epoch;
}

}  // namespace wfq
