// tboa_quantize_layer: Algorithm 1 (lines 2-13) for one projection weight, all arithmetic in fp64.
//
// Heads are independent and run side by side: the N rows of the current step of every head form one
// "block" of n_heads*N rows (block row R = h*nbr + r  <->  layer row h*d_h + i0 + r).  Per step:
//   grid search   (Alg. 1 line 9)  candidates -> approximate costs of all of them on the matrix cores (integer codes against
//                                  digits of H_in, or pairs of errors against half terms) -> exact fp64 costs of the near-minimal ones -> argmin
//                                  (narrow layers and group-wise grids: every candidate exactly, one kernel or one fp64 GEMM)
//   in-channel sweep (Algorithm 3) groups of 512 columns (sweep.hip); the columns right of a group get one rank-512 GEMM update per term
//   compensation  (Prop. 3.1/3.2)  T = [U_out^T]_{i1:,B} [U_out^T]_{B,B}^-1 per head, then W~[i1:] -= T E as a
//                                  batched GEMM, E = (W_B - Q_B) - ((W_B R) U_in^T) U_in
// and after the last step the coordinate descent of Algorithm 2 on precomputed Gram matrices (d_h x d_h per head; per
// pair of groups when the grids are group-wise), then the outputs and the loss.
#include "internal.h"
#include <hip/hip_fp16.h>
#include <algorithm>
#include <string.h>
#include <stdlib.h>
#include <math.h>

namespace {

__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}

__device__ __forceinline__ double quant_code(double w, double s, double z, double maxq) {
    return fmin(fmax(rint(w / s) + z, 0.0), maxq);
}

// ------------------------------------------------------------------------------------------------ rows
__global__ void gather_rows_kernel(const double* __restrict__ src, double* __restrict__ dst, double* __restrict__ work, BlockMap m, int n) {
    const int R = blockIdx.y;
    const double* s = src + layer_row(m, R) * n;
    const long long o = (long long)R * n;
    for (int c = blockIdx.x * blockDim.x + threadIdx.x; c < n; c += gridDim.x * blockDim.x) { const double v = s[c]; dst[o + c] = v; work[o + c] = v; }
}

// ------------------------------------------------------------------------------------------------ grid search
// one wavefront per row: range of the row, then the candidate list (s_k, z_k)
__global__ __launch_bounds__(256) void grid_candidates_kernel(const double* __restrict__ Wk, long long ldw, int c0, int ncols,
                                                              int rows, int ncand, int grid_points, double maxq,
                                                              double* __restrict__ cand_s, double* __restrict__ cand_z) {
    const int lane = threadIdx.x & 63, row = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (row >= rows) return;
    const double* w = Wk + (long long)row * ldw + c0;
    double lo = 0.0, hi = 0.0;
    for (int c = lane; c < ncols; c += 64) { const double v = w[c]; lo = fmin(lo, v); hi = fmax(hi, v); }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) { lo = fmin(lo, __shfl_xor(lo, o, 64)); hi = fmax(hi, __shfl_xor(hi, o, 64)); }
    if (lo == hi) { lo = -1.0; hi = 1.0; }
    for (int k = lane; k < ncand; k += 64) {
        const double p = 1.0 - (double)k / (double)grid_points;
        const double s = (p * hi - p * lo) / maxq;
        const double z = rint(-(p * lo) / s);
        cand_s[(long long)row * ncand + k] = s;
        cand_z[(long long)row * ncand + k] = z;
    }
}

// Delta[(row, k), c] = s_k (clamp(round(w_c / s_k) + z_k) - z_k) - w_c
__global__ __launch_bounds__(256) void grid_delta_kernel(const double* __restrict__ Wk, long long ldw, int c0, int ncols, int ncand,
                                                         double maxq, const double* __restrict__ cand_s,
                                                         const double* __restrict__ cand_z, double* __restrict__ Delta) {
    const int row = blockIdx.y;
    const int c = blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= ncols) return;
    const double w = Wk[(long long)row * ldw + c0 + c];
    const double* cs = cand_s + (long long)row * ncand;
    const double* cz = cand_z + (long long)row * ncand;
    double* out = Delta + (long long)row * ncand * ncols + c;
    for (int k = 0; k < ncand; ++k) {
        const double s = cs[k], z = cz[k];
        const double q = quant_code(w, s, z, maxq);
        out[(long long)k * ncols] = s * (q - z) - w;
    }
}

// out[i] = sum_c A[i, c] B[i, c], one wavefront per row
__global__ __launch_bounds__(256) void rowdot_kernel(const double* __restrict__ A, long long lda, const double* __restrict__ B,
                                                     long long ldb, long long rows, int ncols, double* __restrict__ out) {
    const int lane = threadIdx.x & 63;
    const long long row = (long long)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (row >= rows) return;
    const double* a = A + row * lda; const double* b = B + row * ldb;
    double s = 0.0;
    for (int c = lane; c < ncols; c += 64) s += a[c] * b[c];
    s = wave_sum(s);
    if (lane == 0) out[row] = s;
}

// lowest (value, index) over the wavefront; an index of INT_MAX loses to every other one
__device__ __forceinline__ void wave_argmin(double& v, int& k) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        const double v2 = __shfl_xor(v, o, 64); const int k2 = __shfl_xor(k, o, 64);
        if (k2 != 0x7fffffff && (k == 0x7fffffff || v2 < v || (v2 == v && k2 < k))) { v = v2; k = k2; }
    }
}

// lowest k among the minima of cost[row, :] -> (s, z) of that candidate; one wavefront per row (one thread per row took 16 us for
// 80 dependent loads).  A NaN at k = 0 stays the minimum, as it does in a loop over k that replaces what is larger.
__global__ __launch_bounds__(256) void grid_argmin_kernel(const double* __restrict__ cost, const double* __restrict__ cand_s,
                                   const double* __restrict__ cand_z, int rows, int ncand, BlockMap m, int r_off,
                                   double* __restrict__ s_out, double* __restrict__ z_out, int ng, int gi) {
    const int lane = threadIdx.x & 63, row = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (row >= rows) return;
    const double* c = cost + (long long)row * ncand;
    double bc = 0.0; int best = 0x7fffffff;
    for (int k = lane; k < ncand; k += 64) { const double v = c[k]; if (v == v && (best == 0x7fffffff || v < bc)) { bc = v; best = k; } }
    wave_argmin(bc, best);
    if (lane != 0) return;
    if (best == 0x7fffffff || !(c[0] == c[0])) best = 0;
    const long long lr = layer_row(m, r_off + row);
    s_out[lr * ng + gi] = cand_s[(long long)row * ncand + best];
    z_out[lr * ng + gi] = cand_z[(long long)row * ncand + best];
}

// clamp(round(w / s) + z) - z of one weight.  The quotient is that of fp64: fl32(w) fl32(1 / s) is within 2^-22 (relative) of it, so wherever it is further than
// 2^-20 |t| from a half-integer both round to the same integer; only the others take the fp64 division.
__device__ __forceinline__ float grid_code(float wf, float inv, float z, float maxq, const double* w, bool exists, double s) {
    const float t = wf * inv;
    float r = rintf(t);
    const bool safe = inv != 0.f && fabsf(t - r) < 0.5f - (fabsf(t) * 9.5367431640625e-7f + 9.5367431640625e-7f);
    if (!safe && exists) r = (float)fmin(fmax(rint(*w / s), -1024.0), 1024.0);
    return fminf(fmaxf(r + z, 0.f), maxq) - z;
}

// The whole search over 32, 64 or 128 columns with exact costs (a grid per group of columns, narrow layers): candidates, their errors, the products with H_in and
// the minimum of a row in one workgroup, nothing of it in memory.  H_in's block stays in registers for all rows of a workgroup, in the lanes of the fp64 MFMA's right operand: wavefront
// w owns the tiles w and NT - 1 - w of 16 columns (NT = 4, 2: tile w), and of the symmetric block each column tile only takes the rows up to its own (doubled
// above it: delta H delta^T = delta T delta^T).  Sixteen candidates at a time: every thread forms delta for its column, LDS hands it to the wavefronts as left operand
// and, after the products, to be multiplied with them.  The MFMAs are 36 of 64 tiles, 24 us of those 82; forming delta and handing it over are the rest.
// Separate launches (candidates, delta, product, row sums, minimum) wrote and read delta and the products, 105 MB each for 1280 rows x 80 candidates x 128 columns:
// 144 us, now 82 us.
template <int NT>
__global__ __launch_bounds__(256) void grid_group_kernel(const double* __restrict__ Wk, long long ldw, int c0, const double* __restrict__ H, long long h_stride, int n, int rows_per_mat,
                                                         int rows_wg, int ncand, int grid_points, double maxq, BlockMap m, double* __restrict__ s_out, double* __restrict__ z_out,
                                                         int ng, int gi) {
    typedef double v4d __attribute__((ext_vector_type(4)));
    constexpr int NC = 16 * NT, P = NC + 4, PER = 256 / NC, MAXC = 256;      // (pitch: 16 rows fall into different banks)
    constexpr bool PAIR = NT == 8;
    __shared__ double D[2][16][P], cs[MAXC], cz[MAXC], part[4][MAXC], ws[NC];
    __shared__ float cr[MAXC];
    const int t = threadIdx.x, lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6), l16 = lane & 15, lk = lane >> 4;
    const int mat = blockIdx.y, r_lo = blockIdx.x * rows_wg, r_hi = min(rows_per_mat, r_lo + rows_wg), tiles = (ncand + 15) / 16;
    const int j2 = PAIR ? NT - 1 - wave : wave, j1 = wave;      // column tiles of this wavefront (j1: NT = 8)
    const double* Hm = H + mat * h_stride + (long long)c0 * n + c0;
    double b2[4 * NT], b1[PAIR ? 2 * NT : 1];
#pragma unroll
    for (int i = 0; i < 4 * NT; ++i) b2[i] = (j2 < NT && i / 4 <= j2) ? (i / 4 < j2 ? 2.0 : 1.0) * Hm[(long long)(4 * i + lk) * n + 16 * j2 + l16] : 0.0;
    if constexpr (PAIR) {
#pragma unroll
        for (int i = 0; i < 2 * NT; ++i) b1[i] = i / 4 <= j1 ? (i / 4 < j1 ? 2.0 : 1.0) * Hm[(long long)(4 * i + lk) * n + 16 * j1 + l16] : 0.0;
    }
    for (int r = r_lo; r < r_hi; ++r) {
        const int row = mat * rows_per_mat + r;
        const double* w = Wk + (long long)row * ldw + c0;
        double lo = 0.0, hi = 0.0;
        for (int c = lane; c < NC; c += 64) { const double v = w[c]; lo = fmin(lo, v); hi = fmax(hi, v); }
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) { lo = fmin(lo, __shfl_xor(lo, o, 64)); hi = fmax(hi, __shfl_xor(hi, o, 64)); }
        if (lo == hi) { lo = -1.0; hi = 1.0; }
        __syncthreads();      // the last row's costs have been read
        if (t < NC) ws[t] = w[t];
        for (int k = t; k < ncand; k += 256) {
            const double p = 1.0 - (double)k / (double)grid_points;
            const double s = (p * hi - p * lo) / maxq, i = 1.0 / s;
            cs[k] = s; cz[k] = rint(-(p * lo) / s);
            cr[k] = (i >= 1.17549435e-38 && i <= 3.4e38) ? (float)i : 0.f;
        }
        __syncthreads();
        const int c = t % NC;
        const double wv = ws[c];
        const float wf = (float)wv;
        for (int ct = 0; ct < tiles; ++ct) {
            double (&Db)[16][P] = D[ct & 1];
#pragma unroll
            for (int i = 0; i < 16 / PER; ++i) {
                const int q = i * PER + t / NC, k = min(16 * ct + q, ncand - 1);
                Db[q][c] = cs[k] * (double)grid_code(wf, cr[k], (float)cz[k], (float)maxq, &wv, true, cs[k]) - wv;
            }
            __syncthreads();      // (the other buffer is written after every wavefront has passed here, done with it)
            double cost[4] = {0.0, 0.0, 0.0, 0.0};
            if (j2 < NT) {
                v4d x2 = {0.0, 0.0, 0.0, 0.0}, x1 = x2;
#pragma unroll
                for (int kt = 0; kt < NT; ++kt) {
                    if (kt > j2) break;
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        const double a = Db[l16][16 * kt + 4 * u + lk];
                        x2 = __builtin_amdgcn_mfma_f64_16x16x4f64(a, b2[4 * kt + u], x2, 0, 0, 0);
                        if constexpr (PAIR) { if (kt < NT / 2 && kt <= j1) x1 = __builtin_amdgcn_mfma_f64_16x16x4f64(a, b1[(4 * kt + u) % (2 * NT)], x1, 0, 0, 0); }
                    }
                }
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    cost[v] = x2[v] * Db[lk + 4 * v][16 * j2 + l16];
                    if constexpr (PAIR) cost[v] += x1[v] * Db[lk + 4 * v][16 * j1 + l16];
                }
            }
#pragma unroll
            for (int v = 0; v < 4; ++v) {
#pragma unroll
                for (int o = 8; o > 0; o >>= 1) cost[v] += __shfl_xor(cost[v], o, 64);
                if (l16 == 0 && 16 * ct + lk + 4 * v < ncand) part[wave][16 * ct + lk + 4 * v] = cost[v];
            }
        }
        __syncthreads();
        if (wave == 0) {      // as grid_argmin_kernel
            double bc = 0.0; int best = 0x7fffffff;
            bool first = true;
            for (int k = lane; k < ncand; k += 64) {
                const double v = (part[0][k] + part[1][k]) + (part[2][k] + part[3][k]);
                if (k == 0) first = v == v;
                if (v == v && (best == 0x7fffffff || v < bc)) { bc = v; best = k; }
            }
            wave_argmin(bc, best);
            if (lane == 0) {
                if (best == 0x7fffffff || !first) best = 0;
                const long long lr = layer_row(m, row);
                s_out[lr * ng + gi] = cs[best]; z_out[lr * ng + gi] = cz[best];
            }
        }
    }
}

// ---- two-phase search: approximate costs of all candidates on the matrix cores, exact fp64 costs of the few
// candidates within GRID_TAU of the approximate minimum.
//
// With T the part of H below its diagonal, delta H delta^T = sum_c delta_c (2 (delta T^T)[c] + H_cc delta_c) (H is symmetric; the product then needs, for
// output column r, only the contraction indices c < r: its causal limit).  Two forms of the product:
//
// Integers (coarse grids, see grid_delta): delta_k = s_k qbar_k - w with qbar = code - zero, at most maxq in magnitude, so that
//     delta_k T^T = s_k G_k - G_w,   G_k = qbar_k T^T,  G_w = w T^T,
// and every row r of T is taken as integers times a step v_r, two or three digits to the base 256: the product runs on signed bytes at twice the rate of 16-bit
// operands, its sums are exact, and v_r is large enough that maxq sum |T'_r| stays below 2^31.  G_w comes from the 31-bit integer form of the weight rows, one product
// for every pair of digits, added in 64-bit integers.  So a cost is that of T' = v times the integers, the same T' for all candidates, and the one error is
// the rounding of T: expected relative error E = 2 sqrt(sum_r r v_r^2 / 12) / tr H, which the device forms per matrix.  Two digits where E <= 6e-7 and |H off the
// diagonal|_F is small enough for one half term (grid_one_term), three elsewhere (E 1e-9 - 8e-7, the latter on channels correlated by common factors).
// T itself is coarser than as halves, a fixed step per row where those have 11 or 22 bits of every entry: median relative error of an entry (2048 columns, 4096 tokens)
// 2.6e-6 with three digits against 2.2e-8 with two half terms, 6.5e-4 with two digits against 1.7e-4 with one.  The exact sums and the weights' 31 bits more than make up for it,
// because half terms lost more where G_k and G_w cancel in their fp32 sums.  Largest deviations of a cost, half terms -> digits, widths 320 - 8192:
//     independent channels   one term -> two digits 3e-6 -> 3e-7 - 1e-6,   two terms -> three digits 1e-7 - 5e-7 -> 5e-9 - 4e-8   (two digits there: 5e-7 - 1.3e-6)
//     outlier channels 5e-7 - 2.5e-6 -> 8e-9 - 6e-8,   common factors 1.3e-6 - 2.3e-5 -> 5e-7 - 5e-6,   a rank-4 map of the channels 7e-6 - 1.2e-4 -> 3e-6 - 4e-5
//     one direction with nearly all of the variance 9e-5 - 1.3e-3 -> 3e-5 - 5e-4 (equal on average at 4096 columns)
// 70B-shaped W_O (8192 x 8192, 80 candidates, three digits against two half terms): products 86 -> 63 ms.
//
// Pairs of delta (fine grids): delta itself as a (hi, lo) pair of halves against one or two half terms of T with half of H's diagonal, the channels
// equilibrated by powers of two: T'_rc = T_rc 2^(10 - e_r - e_c) with e_c half the exponent of H_cc, delta'_c = delta_c 2^(e_c - e_max), so that the entries of T' are at
// most 2^12 whatever the spread of the channels.  With one term what is left is the rounding of H, at most 2^-11 of an entry and the same for every
// candidate (the diagonal is exempt: its rounding is known and added back).  Its effect on a cost goes by rho = |H off the diagonal|_F / tr H: measured 2.9e-4 rho
// (root mean square over the near-minimal candidates) and up to 1.4e-3 rho below rho = 0.01, at every width and number of bits, and more of it above (up to 8e-3 rho
// at 0.4).  Three products of bf16 pairs were off by 1e-6 - 2e-6 with 3 and 4 bits, 0.6e-6 - 2.3e-6 with 8 (root mean square, widths 1024 - 8192, 16 - 131
// thousand tokens): one term is taken where it is off by no more than that, which is where channels are uncorrelated and the tokens many
// (grid_one_term), and two (22 bits) elsewhere: 1e-7 - 3e-7, on strongly correlated channels 1.5e-6 - 5.8e-6.  The device decides per matrix (grid_terms_kernel).
//
// As a guard, every exact re-evaluation is compared with its approximation, and a call whose largest deviation exceeds grid_guard GRID_TAU (a quarter of it by
// default) is repeated: with the longer form of T if a matrix had the shorter one, else with exact costs for every candidate (counted by tboa_counter).
constexpr int GRID_PAD = 256;        // extra elements per row of the operands (memory-channel spread)
constexpr int GRID_KS = 6;          // exact re-evaluations per row
// survivors: approximate cost <= (1 + tau) * approximate minimum.  The cheapest candidate is among them where no cost is off by more than g with (1 + g) / (1 - g) <= 1 + tau.
// A narrower margin, which covers the g = 5e-4 that the default guard lets pass, with integers where the expected error E of a cost is 10000 times below that:
// uncorrelated channels over many tokens, where the largest deviations seen are 8e-8, and fewer candidates need exact costs (70B-shaped W_O: the call 168.7 -> 163.6 ms).
// A caller's guard above the default keeps the whole margin.
constexpr double GRID_TAU = 2e-3, GRID_TAU_NARROW = 1.05e-3, GRID_NARROW_ERROR = 5e-8;
constexpr double GRID_TWO_DIGITS = 6e-7;      // expected relative error of a cost up to which two digits of T do, |H off the diagonal|_F permitting (grid_one_term)
// the left operand is delta as a pair of halves, else the integer codes: 3 levels of qbar over any width, 7 over 2048 columns.  The step of T grows with maxq times
// the width; beyond that the pairs are closer on correlated channels (4 bits, 8192 columns: 1.5e-6 - 5.8e-6 against 2e-5 expected of integers)
constexpr bool grid_delta(int bits, int n) { return bits > 3 || (bits == 3 && n > 2048); }
constexpr double grid_one_term(int bits) { return bits == 2 ? 0.005 : bits <= 4 ? 0.003 : 0.0; }      // one half term of T (or two digits) is enough for |H off the diagonal|_F up to this times tr H
constexpr int GRID_SPREAD = 14;     // channels whose variance is below 2^-28 of the largest share an exponent (no subnormal half values)

// columns of the operands: zeros beyond n (integers: whole output tiles, whose contraction then is whole turns of the LDS ring)
inline int grid_width(int n, bool delta) { return delta ? (n + 31) / 32 * 32 : (n + 255) / 256 * 256; }
inline long long grid_pitch(int np, bool delta) { return (delta ? np : np / 2) + GRID_PAD; }      // of an operand, in 16-bit elements
inline long long rows16(long long rows) { return (rows + 15) / 16 * 16; }

// What a matrix's equilibration leaves behind, [n_hin][np] each: up[c] = 2^(e_c - e_max) (0 beyond n), down[c] = 2^-e_c, dcorr[c] = H'_cc less
// twice what the half terms hold of T'_cc, off2[c] = sum of the squares of row c left of the diagonal; per matrix scale = 2^(2 e_max) and
// terms = number of half terms of T'.
struct GridScale { float* up; double* down; float* dcorr; double* off2; double* scale; int* terms; };
__global__ __launch_bounds__(256) void grid_scale_kernel(const double* __restrict__ H, int n, int np, GridScale g) {
    __shared__ int red[256];
    const double* Hm = H + (long long)blockIdx.x * n * n;
    const long long o = (long long)blockIdx.x * np;
    auto half_exponent = [&](int c) {
        const double v = Hm[(long long)c * n + c];
        return (v > 0.0 && v < 1.7976931348623157e308) ? (ilogb(v) >> 1) : -600;
    };
    int m = -600;
    for (int c = threadIdx.x; c < n; c += 256) m = max(m, half_exponent(c));
    red[threadIdx.x] = m;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) { if ((int)threadIdx.x < w) red[threadIdx.x] = max(red[threadIdx.x], red[threadIdx.x + w]); __syncthreads(); }
    const int emax = red[0];
    for (int c = threadIdx.x; c < np; c += 256) {
        if (c >= n) { g.up[o + c] = 0.f; g.down[o + c] = 0.0; continue; }
        const int e = max(half_exponent(c), emax - GRID_SPREAD);
        g.up[o + c] = ldexpf(1.f, e - emax); g.down[o + c] = ldexp(1.0, -e);
    }
    if (threadIdx.x == 0) g.scale[blockIdx.x] = ldexp(1.0, 2 * emax);
}

// T' as two half terms in the GEMM's 16 x 32 blocks, one [np, np + pad] matrix per H and term (all first terms, then all second ones); only
// what the causal limit reads (columns up to the end of the row's 256-tile) is written.  One workgroup per row, eight consecutive columns per thread.
__global__ __launch_bounds__(256) void grid_factor_kernel(const double* __restrict__ H, int n, int np, GridScale g, __half* __restrict__ out, long long term_stride) {
    __shared__ double red[4];
    const int r = blockIdx.x;
    const long long o = (long long)blockIdx.y * np, pitch = np + GRID_PAD;
    const double* h = H + (long long)blockIdx.y * n * n + (long long)r * n;
    _Float16* dst = (_Float16*)out + (long long)blockIdx.y * np * pitch;
    const double dr = 1024.0 * g.down[o + r];
    const int cend = min(np, (r / 256 + 1) * 256);
    double sq = 0.0;
    for (int c = 8 * threadIdx.x; c < cend; c += 2048) {
        union { _Float16 b[8]; uint4 u; } hi, lo;
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const int k = c + j;
            double t = 0.0;
            if (r < n && k <= r) {
                const double v = h[k];
                t = v * dr * g.down[o + k];
                if (k == r) t *= 0.5; else sq += v * v;
            }
            hi.b[j] = (_Float16)(float)t;
            lo.b[j] = (_Float16)(float)(t - (double)hi.b[j]);
        }
        const long long a = tboa_blocked_offset(r, c, pitch >> 5);
        *(uint4*)(dst + a) = hi.u; *(uint4*)(dst + term_stride + a) = lo.u;
    }
    sq = wave_sum(sq);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = sq;
    __syncthreads();
    if (threadIdx.x == 0) g.off2[o + r] = (red[0] + red[1]) + (red[2] + red[3]);
}

// number of half terms of each matrix (one up to |H off the diagonal|_F = one_term tr H; `at_least` 2: never one), and what they leave out of the diagonal
__global__ __launch_bounds__(256) void grid_terms_kernel(const double* __restrict__ H, int n, int np, GridScale g, int at_least, double one_term, int* __restrict__ gstat) {
    __shared__ double red[2][256];
    const double* Hm = H + (long long)blockIdx.x * n * n;
    const long long o = (long long)blockIdx.x * np;
    double tr = 0.0, off = 0.0;
    for (int c = threadIdx.x; c < n; c += 256) { tr += Hm[(long long)c * n + c]; off += g.off2[o + c]; }
    red[0][threadIdx.x] = tr; red[1][threadIdx.x] = off;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) { red[0][threadIdx.x] += red[0][threadIdx.x + w]; red[1][threadIdx.x] += red[1][threadIdx.x + w]; }
        __syncthreads();
    }
    const double lim = one_term * red[0][0];
    const int terms = (at_least < 2 && 2.0 * red[1][0] <= lim * lim) ? 1 : 2;
    if (threadIdx.x == 0) { g.terms[blockIdx.x] = terms; if (terms == 1) atomicOr(gstat, 1); }
    for (int c = threadIdx.x; c < np; c += 256) {
        double d = 0.0;
        if (c < n) {
            const double t = 0.5 * Hm[(long long)c * n + c] * (1024.0 * g.down[o + c]) * g.down[o + c];
            const _Float16 hi = (_Float16)(float)t, lo = (_Float16)(float)(t - (double)hi);
            d = 2.0 * (t - (double)hi - (terms > 1 ? (double)lo : 0.0)) / 1024.0;
        }
        g.dcorr[o + c] = (float)d;
    }
}

// Integer form of T.  Per row r and matrix, [n_hin][np]: v = step of the row, hd = H_rr (both 0 beyond n); v2, v3: the steps with two and three digits, e2: the row's part
// of E with two; off2: sum of the squares of row r left of the diagonal; terms: digits taken; tau: margin of the survivors.
struct GridInt { double *v, *hd, *v2, *v3, *e2, *off2, *tau; int* terms; };
constexpr double GRID_DIGITS2 = 32600.0, GRID_DIGITS3 = 8.3e6;      // largest magnitudes of two and three digits in [-128, 127]

__global__ __launch_bounds__(256) void grid_int_steps_kernel(const double* __restrict__ H, int n, int np, double maxq, GridInt g) {
    __shared__ double red[3][4];
    const int r = blockIdx.x, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const long long o = (long long)blockIdx.y * np;
    const double* h = H + (long long)blockIdx.y * n * n + (long long)r * n;
    double sum = 0.0, big = 0.0, sq = 0.0;
    if (r < n)
        for (int c = threadIdx.x; c < r; c += 256) { const double a = fabs(h[c]); sum += a; big = fmax(big, a); sq += a * a; }
    sum = wave_sum(sum); sq = wave_sum(sq);
#pragma unroll
    for (int w = 32; w > 0; w >>= 1) big = fmax(big, __shfl_xor(big, w, 64));
    if (lane == 0) { red[0][wave] = sum; red[1][wave] = big; red[2][wave] = sq; }
    __syncthreads();
    if (threadIdx.x != 0) return;
    sum = (red[0][0] + red[0][1]) + (red[0][2] + red[0][3]);
    big = fmax(fmax(red[1][0], red[1][1]), fmax(red[1][2], red[1][3]));
    // maxq sum |T'| <= maxq (sum / v + n / 2) < 2^31
    const double least = maxq * sum / (2147483000.0 - 0.5 * maxq * n), v2 = fmax(big / GRID_DIGITS2, least), v3 = fmax(big / GRID_DIGITS3, least);
    g.v2[o + r] = v2; g.v3[o + r] = sum == sum ? v3 : sum;      // (a sum that is undefined makes every cost undefined)
    g.e2[o + r] = (double)r * v2 * v2;
    g.off2[o + r] = (red[2][0] + red[2][1]) + (red[2][2] + red[2][3]);
    g.hd[o + r] = r < n ? h[r] : 0.0;
}

__global__ __launch_bounds__(256) void grid_int_terms_kernel(int n, int np, GridInt g, int longer, double shorter_off, int whole_margin, int* __restrict__ gstat) {
    __shared__ double red[4][256];
    const long long o = (long long)blockIdx.x * np;
    double tr = 0.0, e = 0.0, e3 = 0.0, off = 0.0;
    for (int c = threadIdx.x; c < n; c += 256) { tr += g.hd[o + c]; e += g.e2[o + c]; off += g.off2[o + c]; e3 += (double)c * g.v3[o + c] * g.v3[o + c]; }
    red[0][threadIdx.x] = tr; red[1][threadIdx.x] = e; red[2][threadIdx.x] = e3; red[3][threadIdx.x] = off;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w)
            for (int k = 0; k < 4; ++k) red[k][threadIdx.x] += red[k][threadIdx.x + w];
        __syncthreads();
    }
    auto within = [&](double ee, double lim) { lim *= red[0][0]; return ee / 3.0 <= lim * lim; };      // E = 2 sqrt(e / 12) / tr
    const double off_lim = shorter_off * red[0][0];
    const int terms = (!longer && within(red[1][0], GRID_TWO_DIGITS) && 2.0 * red[3][0] <= off_lim * off_lim) ? 2 : 3;
    if (threadIdx.x == 0) {
        g.terms[blockIdx.x] = terms;
        g.tau[blockIdx.x] = !whole_margin && within(red[terms == 2 ? 1 : 2][0], GRID_NARROW_ERROR) ? GRID_TAU_NARROW : GRID_TAU;
        if (terms == 2) atomicOr(gstat, 1);
    }
    for (int c = threadIdx.x; c < np; c += 256) g.v[o + c] = c < n ? (terms == 2 ? g.v2[o + c] : g.v3[o + c]) : 0.0;
}

// signed bytes d0, d1, d2 with t = d0 + 256 d1 + 65536 d2
__device__ __forceinline__ void digits(int t, signed char& d0, signed char& d1, signed char& d2) {
    d0 = (signed char)(t & 255); t = (t - d0) >> 8;
    d1 = (signed char)(t & 255); d2 = (signed char)((t - d1) >> 8);
}
__device__ __forceinline__ int clamped_int(double x, double lim) { return (int)fmin(fmax(rint(x), -lim), lim); }      // (an undefined value becomes -lim)

// the digits of T', the highest first, in the GEMM's blocks, one [np, pitch] matrix per H and digit (all highest digits, then ..); only what the causal limit reads
// is written.  One workgroup per row, sixteen consecutive columns per thread.
__global__ __launch_bounds__(256) void grid_int_factor_kernel(const double* __restrict__ H, int n, int np, long long pitch, GridInt g, signed char* __restrict__ out, long long term_bytes) {
    const int r = blockIdx.x;
    const long long o = (long long)blockIdx.y * np;
    const double* h = H + (long long)blockIdx.y * n * n + (long long)r * n;
    signed char* dst = out + 2LL * blockIdx.y * np * pitch;
    const double v = g.v[o + r], inv = v > 0.0 ? 1.0 / v : 0.0;
    const bool two = g.terms[blockIdx.y] == 2;
    const int cend = min(np, (r / 256 + 1) * 256);
    for (int c = 16 * threadIdx.x; c < cend; c += 4096) {
        union { signed char b[16]; uint4 u; } d[3];
#pragma unroll
        for (int j = 0; j < 16; ++j) {
            const int t = (r < n && c + j < r) ? clamped_int(h[c + j] * inv, two ? 32639.0 : 8355711.0) : 0;
            if (two) { digits(t, d[1].b[j], d[0].b[j], d[2].b[j]); d[2].b[j] = 0; }
            else digits(t, d[2].b[j], d[1].b[j], d[0].b[j]);
        }
        const long long a = 2 * tboa_blocked_offset(r, c / 2, pitch >> 5);
#pragma unroll
        for (int k = 0; k < 3; ++k) *(uint4*)(dst + k * term_bytes + a) = d[k].u;
    }
}

// Rows of a pass, in one array of matrices (the rows that share one H): matrix row of (weight row rl of the matrix, candidate k) is rl ncand + k.
struct GridRows { int per, ncand; long long mat_rows, pitch; int np; };
// integers: the four digits of the weight rows, digit i (the highest first) of row rl at i per + rl of [w_rows, pitch]; wu = step of a weight row
constexpr int GRID_WD = 4;
struct GridWeights { signed char* A; long long w_rows; double* wu; };

// per weight row (one wavefront): range, candidates (s_k, z_k) and 1 / s_k in fp32 (0 where that is no normal number), the row in fp32, and
// DELTA: wdown = 2^-t, 2^t bringing the row's largest magnitude into [2^13, 2^14); else the row's digits
template <bool DELTA>
__global__ __launch_bounds__(256) void grid_rows_kernel(const double* __restrict__ Wk, long long ldw, int n, int rows, int grid_points, double maxq,
                                                        GridRows m, GridWeights gw, double* __restrict__ cand_s, double* __restrict__ cand_z,
                                                        float* __restrict__ cand_r, float* __restrict__ Wf, float* __restrict__ wdown) {
    const int lane = threadIdx.x & 63, row = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (row >= rows) return;
    const double* w = Wk + (long long)row * ldw;
    double lo = 0.0, hi = 0.0;
    for (int c = lane; c < n; c += 64) { const double v = w[c]; lo = fmin(lo, v); hi = fmax(hi, v); }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) { lo = fmin(lo, __shfl_xor(lo, o, 64)); hi = fmax(hi, __shfl_xor(hi, o, 64)); }
    const double big = fmax(-lo, hi);
    const int e = (big > 0.0 && big < 1e300) ? ilogb(big) : 0;
    if (lo == hi) { lo = -1.0; hi = 1.0; }
    for (int k = lane; k < m.ncand; k += 64) {
        const double p = 1.0 - (double)k / (double)grid_points;
        const double s = (p * hi - p * lo) / maxq;
        cand_s[(long long)row * m.ncand + k] = s;
        cand_z[(long long)row * m.ncand + k] = rint(-(p * lo) / s);
        const double r = 1.0 / s;
        cand_r[(long long)row * m.ncand + k] = (r >= 1.17549435e-38 && r <= 3.4e38) ? (float)r : 0.f;
    }
    for (int c = lane; c < m.np; c += 64) Wf[(long long)row * m.np + c] = c < n ? (float)w[c] : 0.f;
    if constexpr (DELTA) {
        if (lane == 0) wdown[row] = ldexpf(1.f, e - 13);
    } else {
        const int mat = row / m.per, rl = row % m.per;
        signed char* A = gw.A + 2LL * mat * gw.w_rows * m.pitch;
        if (lane == 0) gw.wu[row] = ldexp(1.0, e - 29);
        for (int c = 16 * lane; c < m.np; c += 1024) {
            union { signed char b[16]; uint4 u; } d[GRID_WD];
#pragma unroll
            for (int j = 0; j < 16; ++j) {
                const int t = c + j < n ? clamped_int(ldexp(w[c + j], 29 - e), 1073741824.0) : 0;
                d[3].b[j] = (signed char)(t & 255);
                digits((t - d[3].b[j]) >> 8, d[2].b[j], d[1].b[j], d[0].b[j]);
            }
#pragma unroll
            for (int k = 0; k < GRID_WD; ++k) *(uint4*)(A + 2 * tboa_blocked_offset((long long)k * m.per + rl, c / 2, m.pitch >> 5)) = d[k].u;
        }
    }
}

// qbar of every (row, candidate) as bytes; a wavefront makes whole blocks of 16 rows x 64: lane = (row of the block lane / 4, sixteen columns of lane % 4)
__global__ __launch_bounds__(256) void grid_codes_kernel(const double* __restrict__ Wk, long long ldw, const float* __restrict__ Wf, int n, float maxq, GridRows m,
                                                         const double* __restrict__ cand_s, const double* __restrict__ cand_z, const float* __restrict__ cand_r,
                                                         signed char* __restrict__ Acat) {
    typedef float f4 __attribute__((ext_vector_type(4)));
    const int lane = threadIdx.x & 63, mat = blockIdx.z;
    const long long R = 16LL * (blockIdx.y * 4 + (threadIdx.x >> 6)) + (lane >> 2);
    if (R >= (long long)m.per * m.ncand) return;
    const int rl = (int)(R / m.ncand), k = (int)(R % m.ncand), row = mat * m.per + rl;
    const double s = cand_s[(long long)row * m.ncand + k];
    const float inv = cand_r[(long long)row * m.ncand + k], z = (float)cand_z[(long long)row * m.ncand + k];
    const float* wf = Wf + (long long)row * m.np; const double* w = Wk + (long long)row * ldw;
    signed char* A = Acat + 2LL * mat * m.mat_rows * m.pitch;
    const int nblk = m.np / 64, per = (nblk + gridDim.x - 1) / gridDim.x, b1 = min(nblk, ((int)blockIdx.x + 1) * per);
    for (int cb = blockIdx.x * per; cb < b1; ++cb) {
        const int c = 64 * cb + 16 * (lane & 3);
        union { signed char b[16]; uint4 u; } o;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const f4 wv = *(const f4*)(wf + c + 4 * q);
#pragma unroll
            for (int j = 0; j < 4; ++j) o.b[4 * q + j] = (signed char)(int)grid_code(wv[j], inv, z, maxq, w + c + 4 * q + j, c + 4 * q + j < n, s);
        }
        *(uint4*)(A + 2 * tboa_blocked_offset(R, c / 2, m.pitch >> 5)) = o.u;
    }
}

// delta up 2^t (2^t as for the weights) as a (hi, lo) pair of halves, the low parts lo_off elements further on, in blocks of 16 rows x 32.
// The finer the grid, the closer s qbar and w, whose products the integer form subtracts; deviations (largest, root mean square) on the Hessian of a 7B down
// projection (d_in 11008, rows of silu(gate) up over 131072 fake-quantized tokens): three products of bf16 pairs of delta and H 1.4e-4, 2.7e-5 and
// this form 2.9e-5, 5.8e-6 for any number of levels.
__global__ __launch_bounds__(256) void grid_delta_pair_kernel(const double* __restrict__ Wk, long long ldw, const float* __restrict__ Wf, int n, float maxq,
                                                         GridRows m, GridScale g, const double* __restrict__ cand_s, const double* __restrict__ cand_z,
                                                         const float* __restrict__ cand_r, const float* __restrict__ wdown, __half* __restrict__ Acat, long long lo_off) {
    const int lane = threadIdx.x & 63;
    const int mat = blockIdx.z;
    const long long R = 16LL * (blockIdx.y * 4 + (threadIdx.x >> 6)) + (lane >> 2);
    if (R >= (long long)m.per * m.ncand) return;
    const int rl = (int)(R / m.ncand), k = (int)(R % m.ncand), row = mat * m.per + rl;
    const double s = cand_s[(long long)row * m.ncand + k], up2 = 1.0 / (double)wdown[row];
    const float inv = cand_r[(long long)row * m.ncand + k], z = (float)cand_z[(long long)row * m.ncand + k];
    const float* wf = Wf + (long long)row * m.np; const float* up = g.up + (long long)mat * m.np; const double* w = Wk + (long long)row * ldw;
    _Float16* A = (_Float16*)Acat + (long long)mat * m.mat_rows * m.pitch;
    const int nblk = m.np / 32, per = (nblk + gridDim.x - 1) / gridDim.x, b1 = min(nblk, ((int)blockIdx.x + 1) * per);
    typedef float f4 __attribute__((ext_vector_type(4)));
    for (int cb = blockIdx.x * per; cb < b1; ++cb) {
        const int c = 32 * cb + 8 * (lane & 3);
        f4 wv[2] = {*(const f4*)(wf + c), *(const f4*)(wf + c + 4)}, uv[2] = {*(const f4*)(up + c), *(const f4*)(up + c + 4)};
        union { _Float16 b[8]; uint4 u; } o, l;
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const bool in = c + j < n;
            const double q = (double)grid_code(wv[j >> 2][j & 3], inv, z, maxq, w + c + j, in, s);
            const double d = (s * q - (in ? w[c + j] : 0.0)) * (double)uv[j >> 2][j & 3] * up2;
            o.b[j] = (_Float16)(float)d; l.b[j] = (_Float16)(float)(d - (double)o.b[j]);
        }
        const long long a = tboa_blocked_offset(R, c, m.pitch >> 5);
        *(uint4*)(A + a) = o.u;
        *(uint4*)(A + lo_off + a) = l.u;
    }
}

// cost[(row, k)] = 2^(2 e_max) sum_c delta'_c (2 G[c] 2^-10 + dcorr_c delta'_c), delta' the pair, G its product; one wavefront per (row, k)
__global__ __launch_bounds__(256) void grid_pair_cost_kernel(const float* __restrict__ G, const __half* __restrict__ Acat, int rows, GridRows m, GridScale g,
                                                        const float* __restrict__ wdown, double* __restrict__ out, long long lo_off) {
    typedef float f4 __attribute__((ext_vector_type(4)));
    typedef _Float16 h4 __attribute__((ext_vector_type(4)));
    const int lane = threadIdx.x & 63;
    const long long i = (long long)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (i >= (long long)rows * m.ncand) return;
    const int row = (int)(i / m.ncand), k = (int)(i % m.ncand), mat = row / m.per, rl = row % m.per;
    const long long kb = m.pitch >> 5, R = (long long)rl * m.ncand + k;
    const _Float16* A = (const _Float16*)Acat + (long long)mat * m.mat_rows * m.pitch;
    const float *g0 = G + ((long long)mat * m.mat_rows + R) * m.np, *dc = g.dcorr + (long long)mat * m.np;
    const double wd = wdown[row];
    double acc = 0.0;
    for (int c = 4 * lane; c < m.np; c += 256) {
        const f4 a = __builtin_nontemporal_load((const f4*)(g0 + c)), d = *(const f4*)(dc + c);
        const h4 q = *(const h4*)(A + tboa_blocked_offset(R, c, kb)), ql = *(const h4*)(A + lo_off + tboa_blocked_offset(R, c, kb));
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const double delta = wd * ((double)(float)q[j] + (double)(float)ql[j]);
            acc += delta * ((2.0 / 1024.0) * wd * (double)a[j] + (double)d[j] * delta);
        }
    }
    acc = wave_sum(acc);
    if (lane == 0) out[i] = g.scale[mat] * acc;
}

// Gw[row, c] = (w T'^T)[c] / v_c from the products of the digits, P[mat][digit of T][digit of w * per + row, c]
__global__ __launch_bounds__(256) void grid_weight_products_kernel(const int* __restrict__ P, GridRows m, GridWeights gw, GridInt g, double* __restrict__ Gw) {
    const int row = blockIdx.y, mat = row / m.per, rl = row % m.per, c = blockIdx.x * 256 + threadIdx.x;
    if (c >= m.np) return;
    const int terms = g.terms[mat];
    const int* p = P + 3LL * mat * gw.w_rows * m.np + (long long)rl * m.np + c;
    long long sum = 0;
#pragma unroll
    for (int i = 0; i < GRID_WD; ++i) {
        long long t = 0;
        for (int k = 0; k < terms; ++k) t = t * 256 + p[((long long)k * gw.w_rows + (long long)i * m.per) * m.np];
        sum = sum * 256 + t;
    }
    Gw[(long long)row * m.np + c] = gw.wu[row] * (double)sum;
}

// cost[(row, k)] = sum_c delta_c (2 v_c (s G[c] - Gw[c]) + H_cc delta_c), delta = s qbar - w.  One wavefront per row and GRID_KC candidates: bound by reading G, 4 bytes an
// entry, once; what belongs to the row and the columns is read once for them all (one candidate a wavefront read as much again from L2).
// least[row] = 2^-40 sum_c H_cc w_c^2: a candidate that costs less meets the weights up to the rounding of 24-bit numbers, which their 31 bits do not resolve well
// enough to tell costs apart (grid_count_kernel sends those of such a row to exact costs).
constexpr int GRID_KC = 8;
__global__ __launch_bounds__(256) void grid_cost_kernel(const int* __restrict__ G, const signed char* __restrict__ Acat, int rows, GridRows m, GridInt g,
                                                        const double* __restrict__ cand_s, const double* __restrict__ Wk, long long ldw, int n, const double* __restrict__ Gw,
                                                        double* __restrict__ out, double* __restrict__ least) {
    typedef int i4 __attribute__((ext_vector_type(4)));
    typedef double d4 __attribute__((ext_vector_type(4)));
    const int lane = threadIdx.x & 63, parts = (m.ncand + GRID_KC - 1) / GRID_KC;
    const long long i = (long long)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (i >= (long long)rows * parts) return;
    const int row = (int)(i / parts), k0 = (int)(i % parts) * GRID_KC, mat = row / m.per, rl = row % m.per;
    const long long kb = m.pitch >> 5, R0 = (long long)rl * m.ncand;
    const signed char* A = Acat + 2LL * mat * m.mat_rows * m.pitch;
    const int* Gm = G + ((long long)mat * m.mat_rows + R0) * m.np;
    double s[GRID_KC], acc[GRID_KC];
#pragma unroll
    for (int k = 0; k < GRID_KC; ++k) { s[k] = cand_s[(long long)row * m.ncand + min(k0 + k, m.ncand - 1)]; acc[k] = 0.0; }
    double norm = 0.0;
    for (int c = 4 * lane; c < m.np; c += 256) {
        double w[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) w[j] = c + j < n ? Wk[(long long)row * ldw + c + j] : 0.0;
        const d4 gw = *(const d4*)(Gw + (long long)row * m.np + c), v = *(const d4*)(g.v + (long long)mat * m.np + c), hd = *(const d4*)(g.hd + (long long)mat * m.np + c);
#pragma unroll
        for (int j = 0; j < 4; ++j) norm += hd[j] * w[j] * w[j];
#pragma unroll
        for (int k = 0; k < GRID_KC; ++k) {
            const int kk = min(k0 + k, m.ncand - 1);
            const i4 a = __builtin_nontemporal_load((const i4*)(Gm + (long long)kk * m.np + c));
            const int q = *(const int*)(A + 2 * tboa_blocked_offset(R0 + kk, (c / 16) * 8, kb) + (c & 15));
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const double delta = s[k] * (double)(signed char)(q >> (8 * j)) - w[j];
                acc[k] += delta * (2.0 * v[j] * (s[k] * (double)a[j] - gw[j]) + hd[j] * delta);
            }
        }
    }
#pragma unroll
    for (int k = 0; k < GRID_KC; ++k) {
        const double t = wave_sum(acc[k]);
        if (lane == 0 && k0 + k < m.ncand) out[(long long)row * m.ncand + k0 + k] = t;
    }
    norm = wave_sum(norm);
    if (lane == 0 && k0 == 0) least[row] = 9.094947017729282e-13 * norm;
}

// Device-side bookkeeping of the two-phase search, accumulated over every pass of a quantize_layer call and read once at
// its end: [0] set when a pass could not be trusted as it stands (non-finite approximate cost, more near-minimal
// candidates in a group of rows than the exact re-evaluation has room for), [1] near-minimal candidates evaluated exactly,
// [2] the largest |approximate - exact| / |exact| seen, as the bits of a non-negative float, [3] set when a matrix of the call has the shorter
// form of T (one half term, two digits), [4] rows of which some candidate costs less than approximate costs resolve.
enum { GS_TRIPPED = 0, GS_SURVIVORS = 1, GS_MAXDEV = 2, GS_SHORT = 3, GS_LOW = 4, GS_WORDS = 5 };

// per row (one wavefront): the candidates whose approximate cost makes them survivors (in increasing k, list[row][0 ..]), and the number that
// the exact pass evaluates.  A row with a single survivor needs none (that candidate wins), except every eighth row, whose
// exact cost is what the deviation guard of the pass measures.
// taus (integer form; null: GRID_TAU): the margin of each group of `per` rows.
// least (integer form; null: none): where the minimum lies below it (a row that one candidate meets, a constant row, a row of one weight) approximate costs
// do not tell which candidate it is: every candidate up to twice least[row] survives, all are evaluated, and the row stays out of the guard's relative
// deviation (its least changes sign for grid_argmin_sel_kernel).  Approximations of the survivors within half of least[row] leave nothing cheaper beyond twice least[row]; one
// that is further off (a cost below its own approximation's error) voids the pass.
__global__ __launch_bounds__(256) void grid_count_kernel(const double* __restrict__ cost, int rows, int ncand, const double* __restrict__ taus, int per,
                                                         double* __restrict__ least, int* __restrict__ list, int* __restrict__ cnt_out, int* __restrict__ gstat) {
    const int lane = threadIdx.x & 63, row = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (row >= rows) return;
    const double* c = cost + (long long)row * ncand; int* out = list + (long long)row * ncand;
    double m = INFINITY; int bad = 0;
    for (int k = lane; k < ncand; k += 64) { const double v = c[k]; m = fmin(m, v); bad |= !(v == v); }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) { m = fmin(m, __shfl_xor(m, o, 64)); bad |= __shfl_xor(bad, o, 64); }
    const double tau = taus ? taus[row / per] : GRID_TAU;
    const double lowest = least ? least[row] : 0.0;
    const bool low = least && m < lowest && 2.0 * lowest < INFINITY;
    const double lim = low ? fmax(m + tau * fabs(m), 2.0 * lowest) : m + tau * fabs(m);
    int cnt = 0;
    for (int k0 = 0; k0 < ncand; k0 += 64) {
        const int k = k0 + lane;
        const bool in = k < ncand && c[k] <= lim;
        const unsigned long long mask = __ballot(in);
        if (in) out[cnt + __popcll(mask & ((1ull << lane) - 1ull))] = k;
        cnt += __popcll(mask);
    }
    if (lane != 0) return;
    if (cnt == 0) out[0] = 0;
    if (bad || cnt == 0 || (least && m < lowest && !low)) { atomicOr(gstat + GS_TRIPPED, 1); cnt = 0; }
    if (low) { least[row] = -lowest; atomicAdd(gstat + GS_LOW, 1); }
    const int ev = (cnt > 1 || low || row % 8 == 0) ? cnt : 0;
    cnt_out[row] = ev;
    if (ev) atomicAdd(gstat + GS_SURVIVORS, ev);
}

// exclusive prefix sums of cnt over the rows of each group of `per` rows (one workgroup per group): off[row], total[group];
// a group with more survivors than `cap` slots trips the guard, and its total is cut to cap (rows beyond are not evaluated)
__global__ __launch_bounds__(256) void grid_scan_kernel(const int* __restrict__ cnt, int per, int cap, int* __restrict__ off,
                                                        int* __restrict__ total, int* __restrict__ gstat) {
    __shared__ int part[256];
    const int g = blockIdx.x, t = threadIdx.x;
    const int* c = cnt + (long long)g * per; int* o = off + (long long)g * per;
    const int chunk = (per + 255) / 256, lo = t * chunk, hi = min(per, lo + chunk);
    int s = 0;
    for (int i = lo; i < hi; ++i) s += c[i];
    part[t] = s;
    __syncthreads();
    if (t == 0) {
        int run = 0;
        for (int i = 0; i < 256; ++i) { const int v = part[i]; part[i] = run; run += v; }
        if (run > cap) { atomicOr(gstat + GS_TRIPPED, 1); run = cap; }
        total[g] = run;
    }
    __syncthreads();
    int run = part[t];
    for (int i = lo; i < hi; ++i) { o[i] = run; run += c[i]; }
}

// exact delta of the survivors, compacted per group of `per` rows: DeltaS[group][off[row] + j, c] for the j-th survivor of
// the row (increasing k); slots at or beyond cap do not exist
__global__ __launch_bounds__(256) void grid_delta_sel_kernel(const double* __restrict__ Wk, long long ldw, int n, int ncand, double maxq,
                                                             const double* __restrict__ cand_s, const double* __restrict__ cand_z,
                                                             const int* __restrict__ list, const int* __restrict__ cnt, const int* __restrict__ off,
                                                             int per, int cap, double* __restrict__ DeltaS) {
    const int row = blockIdx.y;
    const int c = blockIdx.x * blockDim.x + threadIdx.x;
    const int nc = cnt[row];
    if (c >= n || nc == 0) return;
    const double w = Wk[(long long)row * ldw + c];
    const int* l = list + (long long)row * ncand;
    double* out = DeltaS + ((long long)(row / per) * cap) * n + c;
    const int slot0 = off[row];
    for (int j = 0; j < nc && slot0 + j < cap; ++j) {
        const double s = cand_s[(long long)row * ncand + l[j]], z = cand_z[(long long)row * ncand + l[j]];
        out[(long long)(slot0 + j) * n] = s * (quant_code(w, s, z, maxq) - z) - w;
    }
}

// cost[i] = sum_c A[i, c] B[i, c] for the compacted rows: row i of group g (`slots` each) exists if i < total[g]
__global__ __launch_bounds__(256) void rowdot_limited_kernel(const double* __restrict__ A, const double* __restrict__ B, int n, int slots,
                                                             long long rows, const int* __restrict__ total, double* __restrict__ out) {
    const int lane = threadIdx.x & 63;
    const long long row = (long long)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (row >= rows) return;
    if ((int)(row % slots) >= total[row / slots]) return;
    const double* a = A + row * n; const double* b = B + row * n;
    double s = 0.0;
    for (int c = lane; c < n; c += 64) s += a[c] * b[c];
    s = wave_sum(s);
    if (lane == 0) out[row] = s;
}

// lowest exact cost among the survivors of a row (lowest k among equals); a row whose survivors were not evaluated takes its
// first one (it has a single one, or the pass is void anyway).  Every exact re-evaluation is compared with its approximation for
// the guard, in rows with least[row] < 0 by the distance and not in relation to the cost.  One wavefront per row, one survivor per lane.
__global__ __launch_bounds__(256) void grid_argmin_sel_kernel(const double* __restrict__ costS, const double* __restrict__ cost, const int* __restrict__ list,
                                       const int* __restrict__ cnt, const int* __restrict__ off, int per, int cap,
                                       const double* __restrict__ cand_s, const double* __restrict__ cand_z, int rows, int ncand,
                                       BlockMap m, int r_off, double* __restrict__ s_out, double* __restrict__ z_out, int ng, int gi,
                                       const double* __restrict__ least, int* __restrict__ gstat) {
    const int lane = threadIdx.x & 63, row = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (row >= rows) return;
    const double* cr = cost + (long long)row * ncand; const int* l = list + (long long)row * ncand;
    const double* ce = costS + (long long)(row / per) * cap;
    const int nc = cnt[row], slot0 = off[row];
    const double half = least && least[row] < 0.0 ? -0.5 * least[row] : 0.0;
    double bc = 0.0, dev = 0.0; int best = 0x7fffffff;
    for (int j = lane; j < nc && slot0 + j < cap; j += 64) {
        const int k = l[j];
        const double e = ce[slot0 + j], d = cr[k] == e ? 0.0 : fabs(cr[k] - e) / fabs(e);      // (equal: a row of zeros costs 0 both ways)
        if (best == 0x7fffffff || e < bc) { bc = e; best = k; }
        dev = fmax(dev, half > 0.0 ? (fabs(cr[k] - e) <= half ? 0.0 : 1.0) : (d == d) ? d : 1.0);
    }
    wave_argmin(bc, best);
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) dev = fmax(dev, __shfl_xor(dev, o, 64));
    if (lane != 0) return;
    if (nc > 0 && half == 0.0) atomicMax(gstat + GS_MAXDEV, __float_as_int((float)fmin(dev, 1.0)));
    if (half > 0.0 && dev > 0.0) atomicOr(gstat + GS_TRIPPED, 1);
    if (best == 0x7fffffff) best = l[0];
    const long long lr = layer_row(m, r_off + row);
    s_out[lr * ng + gi] = cand_s[(long long)row * ncand + best];
    z_out[lr * ng + gi] = cand_z[(long long)row * ncand + best];
}

__global__ void clear_words_kernel(int* p, int n) { if ((int)threadIdx.x < n) p[threadIdx.x] = 0; }

// ------------------------------------------------------------------------------------------------ Prop. 3.1 / 3.2
// E[R, c] = Wb[R, c] - Q[layer_row(R), c] (- S3[R, c])
__global__ void comp_error_kernel(const double* __restrict__ Wb, const double* __restrict__ Q, const double* __restrict__ S3,
                                  double* __restrict__ E, BlockMap m, int n) {
    const int R = blockIdx.y;
    const double* q = Q + layer_row(m, R) * n;
    for (int c = blockIdx.x * blockDim.x + threadIdx.x; c < n; c += gridDim.x * blockDim.x) {
        const long long i = (long long)R * n + c;
        double e = Wb[i] - q[c];
        if (S3) e -= S3[i];
        E[i] = e;
    }
}

// T[h, a, :] = Lo[a, B] Lo[B, B]^-1 for a = i1 .. dh-1, Lo = U_out[h]^T (lower): right-hand triangular solve, columns from the last to
// the first.  One wavefront per remaining row: lane k holds the right-hand side of the columns k, k + 64, .. in LDS, and a finished column
// is taken out of all the earlier ones at once (one thread per row, summing over the later columns, took 125 us for 48 columns; 10 us).
__global__ __launch_bounds__(256) void comp_T_kernel(const double* __restrict__ Uout, int dh, int i0, int i1, double* T, int TP, int lds) {
    extern __shared__ double rhs[];      // [4][nb]; without lds (blocks of thousands of rows) the right-hand side stands in T itself
    const int h = blockIdx.y, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int a = i1 + blockIdx.x * 4 + wave, nb = i1 - i0;
    if (a >= dh) return;
    const double* U = Uout + (long long)h * dh * dh + (long long)i0 * dh;      // row c: Lo[., i0 + c]
    double* t = T + ((long long)h * dh + a) * TP;
    double* x = lds ? rhs + (size_t)wave * nb : t;
    auto settle = [&]() { if (lds) __builtin_amdgcn_wave_barrier(); else __threadfence_block(); };
    for (int k = lane; k < nb; k += 64) x[k] = U[(long long)k * dh + a];
    settle();
    for (int c = nb - 1; c >= 0; --c) {
        const double tc = x[c] / U[(long long)c * dh + i0 + c];
        for (int k = lane; k < c; k += 64) x[k] = __builtin_fma(-tc, U[(long long)k * dh + i0 + c], x[k]);      // Lo[i0 + c, i0 + k]
        settle();
        if (lane == 0) t[c] = tc;
    }
}

// ------------------------------------------------------------------------------------------------ Algorithm 2
// Wbar = codes - z (per group)
__global__ void wbar_kernel(const uint8_t* __restrict__ codes, const double* __restrict__ z, int ng, int gsz, int n,
                            double* __restrict__ Wbar) {
    const int r = blockIdx.y;
    for (int c = blockIdx.x * blockDim.x + threadIdx.x; c < n; c += gridDim.x * blockDim.x)
        Wbar[(long long)r * n + c] = (double)codes[(long long)r * n + c] - z[(long long)r * ng + c / gsz];
}

// Per head: s_j += sum_k (F[j,k] - s_k C[j,k]) Ho[k,j] / (C[j,j] Ho[j,j]) in order j = 0..dh-1,
// F = Wbar (W (H_in - R))^T, C = Wbar H_in Wbar^T = (Cm + Cm^T) / 2   (Prop. 3.3 with Q = diag(s) Wbar; Cm from the half product, GemmF64::sym)
__global__ __launch_bounds__(256) void cd_head_kernel(const double* __restrict__ F, const double* __restrict__ Cm,
                                                      const double* __restrict__ Ho, int dh, int iters, double* __restrict__ s_all) {
    extern __shared__ double sh[];
    double* s = sh; double* red = sh + dh;
    const int h = blockIdx.x, t = threadIdx.x;
    const double* Fh = F + (long long)h * dh * dh; const double* Ch = Cm + (long long)h * dh * dh;
    const double* Hh = Ho + (long long)h * dh * dh;
    double* sg = s_all + (long long)h * dh;
    for (int i = t; i < dh; i += 256) s[i] = sg[i];
    __syncthreads();
    for (int it = 0; it < iters; ++it)
        for (int j = 0; j < dh; ++j) {
            double acc = 0.0;
            for (int k = t; k < dh; k += 256) acc += (Fh[(long long)j * dh + k] - s[k] * 0.5 * (Ch[(long long)j * dh + k] + Ch[(long long)k * dh + j])) * Hh[(long long)k * dh + j];
            acc = wave_sum(acc);
            if ((t & 63) == 0) red[t >> 6] = acc;
            __syncthreads();
            if (t == 0) {
                const double num = (red[0] + red[1]) + (red[2] + red[3]);
                const double den = Ch[(long long)j * dh + j] * Hh[(long long)j * dh + j];
                if (den > 0.0) s[j] = s[j] + num / den;
            }
            __syncthreads();
        }
    for (int i = t; i < dh; i += 256) sg[i] = s[i];
}

// Group-wise form of the same sweep: the coordinate is (row j, group g), visited in the order j = 0 .. dh-1,
// g = 0 .. ng-1, and Q = sum over (k, g') of s[k, g'] Wbar[k, G'] (rows masked to one group).  With
//   Cg[g][g'][j][k] = Wbar[j, G] H_in[G, G'] Wbar[k, G']^T      Fg[g][j][k] = Wbar[j, G] (W (H_in - R))[k, G]^T
// the step is  s[j, g] += sum_k Ho[k, j] (Fg[g][j][k] - sum_g' s[k, g'] Cg[g][g'][j][k]) / (Cg[g][g][j][j] Ho[j, j]).
// While the groups of row j are visited only the scales of row j itself change, so the numerators of all its groups are summed at once with the scales as they stand when the row
// begins, and a short recurrence over the groups then takes out what the steps before have changed: num[g] -= Ho[j, j] Cg[g][g'][j][j] (change of s[j, g']), g' < g.  The same goes for
// blocks of up to 16 rows: cd_group_sums_kernel sums the numerators of a block's rows over the whole chip with the scales as they stand when the block begins (it reads all of Cg, 8.4 GB
// for 40 heads of 128 rows and 40 groups), and in cd_group_chain_kernel, one workgroup per head, a row takes out what the rows of the block before it have changed, which needs 16
// columns of Cg at most.  (All sums in one kernel of a workgroup per head, at the rate of one CU each: 6.7 ms for these sizes; 1.8 + 1.5 this way.)
constexpr int CD_ROWS = 16;

// num0[h][j - j0][g] = sum_k Ho[k, j] (Fg[g][j][k] - sum_g' s[k, g'] Cg[g][g'][j][k]): a workgroup per (group, head) and share of the rows, a wavefront per row; the head's scales in LDS
__global__ __launch_bounds__(256) void cd_group_sums_kernel(const double* __restrict__ Fg, const double* __restrict__ Cg, const double* __restrict__ Ho, int dh, int ng, int j0, int nj,
                                                            int pitch, const double* __restrict__ s_all, double* __restrict__ num0) {
    extern __shared__ double s[];      // s[g pitch + k]
    const int g = blockIdx.x, h = blockIdx.y, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const long long rr = (long long)dh * dh;
    const double* Hh = Ho + (long long)h * rr;
    const double* sg = s_all + (long long)h * dh * ng;
    for (int i = threadIdx.x; i < dh * ng; i += 256) s[(i % ng) * pitch + i / ng] = sg[i];
    __syncthreads();
    for (int jj = blockIdx.z * 4 + wave; jj < nj; jj += 4 * gridDim.z) {
        const int j = j0 + jj;
        const double* F = Fg + (((long long)h * ng + g) * dh + j) * dh; const double* C = Cg + (((long long)h * ng + g) * ng * dh + j) * dh;
        double acc = 0.0;
        for (int k = lane; k < dh; k += 64) {
            double a = F[k];
            int g2 = 0;
            for (; g2 + 8 <= ng; g2 += 8) {
                double c[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) c[u] = C[(g2 + u) * rr + k];
#pragma unroll
                for (int u = 0; u < 8; ++u) a -= s[(g2 + u) * pitch + k] * c[u];
            }
            for (; g2 < ng; ++g2) a -= s[g2 * pitch + k] * C[g2 * rr + k];
            acc += a * Hh[(long long)k * dh + j];
        }
        acc = wave_sum(acc);
        if (lane == 0) num0[((long long)h * CD_ROWS + jj) * ng + g] = acc;
    }
}

// The rows j0 .. j0 + nj of a head one after the other.  LDS: ds[g nj + row of the block], the changes of the block's scales so far; where they fit beside it the numerators
// (lds & 1; else num_mem) and the diagonals Cg[g][g'][j][j] (lds & 2; else read from memory)
__global__ __launch_bounds__(1024) void cd_group_chain_kernel(const double* __restrict__ Cg, const double* __restrict__ Ho, int dh, int ng, int j0, int nj, int lds,
                                                              const double* __restrict__ num0, double* __restrict__ num_mem, double* __restrict__ s_all) {
    extern __shared__ double sh[];
    const int h = blockIdx.x, t = threadIdx.x, lane = t & 63, wave = t >> 6, kk = lane & 15;
    const bool cd_lds = lds & 2;
    double* ds = sh; double* num = lds & 1 ? ds + (size_t)nj * ng : num_mem + (long long)h * ng; double* cd = ds + (size_t)(nj + 1) * ng;
    const long long rr = (long long)dh * dh;
    const double* Ch = Cg + (long long)h * ng * ng * rr; const double* Hh = Ho + (long long)h * rr;
    double* sg = s_all + (long long)h * dh * ng;
    for (int jj = 0; jj < nj; ++jj) {
        const int j = j0 + jj;
        const double hkj = kk < jj ? Hh[(long long)(j0 + kk) * dh + j] : 0.0, hjj = Hh[(long long)j * dh + j];
        for (int g = wave; g < ng; g += 16) {
            // lanes: 16 rows of the block, 4 groups
            const double* C = Ch + ((long long)g * ng * dh + j) * dh + j0 + kk;
            const double start = num0[((long long)h * CD_ROWS + jj) * ng + g];
            double acc = 0.0;
            if (kk < jj || (cd_lds && kk == jj)) {
                int g2 = lane >> 4;
                for (; g2 + 28 < ng; g2 += 32) {
                    double c[8];
#pragma unroll
                    for (int u = 0; u < 8; ++u) c[u] = C[(g2 + 4 * u) * rr];
#pragma unroll
                    for (int u = 0; u < 8; ++u) {
                        if (kk < jj) acc += ds[(g2 + 4 * u) * nj + kk] * c[u];
                        else cd[g * ng + g2 + 4 * u] = c[u];
                    }
                }
                for (; g2 < ng; g2 += 4) {
                    const double c = C[g2 * rr];
                    if (kk < jj) acc += ds[g2 * nj + kk] * c;
                    else cd[g * ng + g2] = c;
                }
            }
            acc = wave_sum(acc * hkj);
            if (lane == 0) num[g] = start - acc;
        }
        __syncthreads();
        // the recurrence over the groups of row j.  A numerator per lane where they and the diagonals allow: every lane divides its own (a reciprocal, and the quotient's remainder
        // once more), the group whose turn it is passes its step on
        if (wave == 0 && cd_lds && ng <= 64) {
            const int own = min(lane, ng - 1);
            const double den = cd[own * ng + own] * hjj, inv = den > 0.0 ? 1.0 / den : 0.0;
            double x = lane < ng ? num[lane] : 0.0, mine = 0.0;
            for (int g = 0; g < ng; ++g) {
                const double c = hjj * cd[g * ng + own];      // (the diagonals of Cg[g][g'] and Cg[g'][g] are the same)
                const double q = x * inv, step = lane_value(den > 0.0 ? __builtin_fma(__builtin_fma(-q, den, x), inv, q) : 0.0, g);
                if (lane == g) mine = step;
                if (lane > g) x = __builtin_fma(-c, step, x);
            }
            if (lane < ng) { ds[lane * nj + jj] = mine; sg[(long long)j * ng + lane] += mine; }
        } else if (wave == 0) {
            for (int g = 0; g < ng; ++g) {
                const double den = (cd_lds ? cd[g * ng + g] : Ch[((long long)(g * ng + g) * dh + j) * dh + j]) * hjj;
                const double step = den > 0.0 ? num[g] / den : 0.0;
                for (int g2 = g + 1 + lane; g2 < ng; g2 += 64)
                    num[g2] -= hjj * (cd_lds ? cd[g2 * ng + g] : Ch[((long long)(g2 * ng + g) * dh + j) * dh + j]) * step;
                if (lane == 0) ds[g * nj + jj] = step;
                __builtin_amdgcn_wave_barrier();
            }
            for (int g = lane; g < ng; g += 64) sg[(long long)j * ng + g] += ds[g * nj + jj];
        }
        __syncthreads();
    }
}

// Cg[h][g'][g] = Cg[h][g][g']^T for g' < g, 64 x 64 pieces through LDS; grid.x runs over (pair, piece), grid.z over the heads.  Bound by memory: 40 heads, 40 groups,
// 128 x 128 each, 8.2 GB.
__global__ __launch_bounds__(256) void cd_group_mirror_kernel(double* __restrict__ Cg, int dh, int ng) {
    __shared__ double t[64][65];
    const int nt = (dh + 63) / 64, piece = blockIdx.x % (nt * nt), pair = blockIdx.x / (nt * nt);
    int g = (int)((sqrtf(8.f * (float)pair + 1.f) + 1.f) * 0.5f);      // pair = g (g - 1) / 2 + g'
    while ((long long)g * (g + 1) / 2 <= pair) ++g;
    while ((long long)g * (g - 1) / 2 > pair) --g;
    const int g2 = pair - g * (g - 1) / 2, r0 = (piece / nt) * 64, c0 = (piece % nt) * 64;
    const long long rr = (long long)dh * dh;
    double* C = Cg + (long long)blockIdx.z * ng * ng * rr;
    const double* src = C + ((long long)g * ng + g2) * rr; double* dst = C + ((long long)g2 * ng + g) * rr;
    for (int i = threadIdx.x; i < 64 * 64; i += 256) {
        const int r = i >> 6, c = i & 63;
        if (r0 + r < dh && c0 + c < dh) t[r][c] = src[(long long)(r0 + r) * dh + c0 + c];
    }
    __syncthreads();
    for (int i = threadIdx.x; i < 64 * 64; i += 256) {
        const int c = i >> 6, r = i & 63;
        if (r0 + r < dh && c0 + c < dh) dst[(long long)(c0 + c) * dh + r0 + r] = t[r][c];
    }
}

// out[row, seg] = sum over the columns c of segment seg of A[row, c] B[row, c]; one wavefront per (row, segment)
__global__ __launch_bounds__(256) void segdot_kernel(const double* __restrict__ A, const double* __restrict__ B, long long rows, int n, int gsz,
                                                     int ng, double* __restrict__ out, long long out_row_stride) {
    const int lane = threadIdx.x & 63;
    const long long w = (long long)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (w >= rows * ng) return;
    const long long row = w / ng; const int seg = (int)(w - row * ng);
    const double* a = A + row * n + (long long)seg * gsz; const double* b = B + row * n + (long long)seg * gsz;
    double s = 0.0;
    for (int c = lane; c < gsz; c += 64) s += a[c] * b[c];
    s = wave_sum(s);
    if (lane == 0) out[row * out_row_stride + seg] = s;
}

// identity H_out with groups: per row, s[g] += (Fd[g] - sum_g' s[g'] Cd[g][g']) / Cd[g][g] in the order g = 0 .. ng-1.
// Cd [rows, ng, ng], Fd [rows, ng].  One wavefront per row, its scales in LDS.
__global__ __launch_bounds__(256) void cd_group_diag_kernel(const double* __restrict__ Fd, const double* __restrict__ Cd, long long rows, int ng,
                                                            int iters, double* __restrict__ s_all) {
    extern __shared__ double sh[];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const long long row_raw = (long long)blockIdx.x * 4 + wv;
    const bool live = row_raw < rows;
    const long long row = live ? row_raw : rows - 1;
    double* s = sh + (size_t)wv * ng;
    for (int g = lane; g < ng; g += 64) s[g] = s_all[row * ng + g];
    __syncthreads();
    const double* C = Cd + row * ng * ng; const double* F = Fd + row * ng;
    for (int it = 0; it < iters; ++it)
        for (int g = 0; g < ng; ++g) {
            double acc = 0.0;
            for (int g2 = lane; g2 < ng; g2 += 64) acc += s[g2] * C[(long long)g * ng + g2];
            acc = wave_sum(acc);
            __syncthreads();
            if (lane == 0) { const double den = C[(long long)g * ng + g]; if (den > 0.0) s[g] = s[g] + (F[g] - acc) / den; }
            __syncthreads();
        }
    if (live) for (int g = lane; g < ng; g += 64) s_all[row * ng + g] = s[g];
}

// identity H_out: rows decouple, s_j += (F_jj - s_j C_jj) / C_jj
__global__ void cd_diag_kernel(const double* __restrict__ Fd, const double* __restrict__ Cd, int rows, int iters, double* __restrict__ s) {
    const int j = blockIdx.x * blockDim.x + threadIdx.x;
    if (j >= rows) return;
    double v = s[j];
    for (int it = 0; it < iters; ++it) if (Cd[j] > 0.0) v = v + (Fd[j] - v * Cd[j]) / Cd[j];
    s[j] = v;
}

// Q = s * Wbar, plus the fp32 outputs
__global__ void finalize_kernel(const double* __restrict__ Wbar, const double* __restrict__ s, const double* __restrict__ z,
                                int ng, int gsz, int n, double* __restrict__ Q, float* __restrict__ Wdeq,
                                float* __restrict__ scales, float* __restrict__ zeros) {
    const int r = blockIdx.y;
    for (int c = blockIdx.x * blockDim.x + threadIdx.x; c < n; c += gridDim.x * blockDim.x) {
        const double q = s[(long long)r * ng + c / gsz] * Wbar[(long long)r * n + c];
        Q[(long long)r * n + c] = q;
        Wdeq[(long long)r * n + c] = (float)q;
    }
    if (blockIdx.x == 0)
        for (int g = threadIdx.x; g < ng; g += blockDim.x) {
            scales[(long long)r * ng + g] = (float)s[(long long)r * ng + g];
            zeros[(long long)r * ng + g] = (float)z[(long long)r * ng + g];
        }
}

// identity H_out, one wavefront per row: C = Wbar H_in Wbar^T and F = Wbar (W (H_in - R))^T of the row alone, from the half products
// A = Wbar T, Gw = W T (T + T^T = 2 H_in) and WR = W R (or NULL)
__global__ __launch_bounds__(256) void cd_row_products_kernel(const double* __restrict__ A, const double* __restrict__ Wbar, const double* __restrict__ W,
                                                              const double* __restrict__ Gw, const double* __restrict__ WR, long long rows, int n,
                                                              double* __restrict__ Cd, double* __restrict__ Fd) {
    const int lane = threadIdx.x & 63;
    const long long row = (long long)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (row >= rows) return;
    const long long o = row * n;
    double c = 0.0, f = 0.0;
    for (int k = lane; k < n; k += 64) {
        const double a = A[o + k], wb = Wbar[o + k];
        c += a * wb;
        f += 0.5 * (a * W[o + k] + wb * Gw[o + k]) - (WR ? wb * WR[o + k] : 0.0);
    }
    c = wave_sum(c); f = wave_sum(f);
    if (lane == 0) { Cd[row] = c; Fd[row] = f; }
}

// (Q - W) T from products that the scale refinement already formed, for one scale per row (Q = diag(s) Wbar):
// DH = diag(s) (Wbar T) - W T.  Overwrites AH = Wbar T.
__global__ void dh_from_products_kernel(double* __restrict__ AH, const double* __restrict__ s, const double* __restrict__ Gw, int n) {
    const int r = blockIdx.y;
    const double sr = s[r];
    for (int c = blockIdx.x * blockDim.x + threadIdx.x; c < n; c += gridDim.x * blockDim.x) {
        const long long i = (long long)r * n + c;
        AH[i] = sr * AH[i] - Gw[i];
    }
}

// out[h] = scale * sum_{j,k} Ho[h][j,k] M[h][k,j]; sym: of the symmetric part of M (a half product)
__global__ __launch_bounds__(256) void head_trace_kernel(const double* __restrict__ Ho, const double* __restrict__ M, int dh,
                                                         double scale, int sym, double* __restrict__ out) {
    __shared__ double red[4];
    const int h = blockIdx.x, t = threadIdx.x;
    const double* Hh = Ho + (long long)h * dh * dh; const double* Mh = M + (long long)h * dh * dh;
    double acc = 0.0;
    for (int i = t; i < dh * dh; i += 256) { const int j = i / dh, k = i % dh; acc += Hh[i] * (sym ? 0.5 * (Mh[(long long)k * dh + j] + Mh[i]) : Mh[(long long)k * dh + j]); }
    acc = wave_sum(acc);
    if ((t & 63) == 0) red[t >> 6] = acc;
    __syncthreads();
    if (t == 0) out[h] = scale * ((red[0] + red[1]) + (red[2] + red[3]));
}

// out[h] = scale * sum over the rows of head h of v[row]
__global__ __launch_bounds__(256) void head_sum_kernel(const double* __restrict__ v, int dh, double scale, double* __restrict__ out) {
    __shared__ double red[4];
    const int h = blockIdx.x, t = threadIdx.x;
    double acc = 0.0;
    for (int i = t; i < dh; i += 256) acc += v[(long long)h * dh + i];
    acc = wave_sum(acc);
    if ((t & 63) == 0) red[t >> 6] = acc;
    __syncthreads();
    if (t == 0) out[h] = scale * ((red[0] + red[1]) + (red[2] + red[3]));
}

inline unsigned gx(long long n) { long long g = (n + 255) / 256; return (unsigned)(g < 1 ? 1 : (g > 64 ? 64 : g)); }

// ------------------------------------------------------------------------------------------------ host side
// products with d_in x d_in matrices: refinement and loss, exact grid costs, P, compensation, updates of the sweep
enum { RNS_REFINE = 1, RNS_EXACT = 2, RNS_P = 4, RNS_COMP = 8, RNS_SWEEP = 16 };

struct Layer {
    tboa_ctx* ctx; const tboa_layer_desc* d;
    int n, nh, dh, ng, gsz, nhin, ncand; double maxq;
    // workspace
    double *W64, *Wt, *Hi, *Hfac, *Uin, *Rd, *P, *Ho, *Hofac, *Uout, *ftmp, *fdinv;
    double *Q64, *s64, *z64;
    double *Wb, *Wk, *Epan, *Wsnap, *E, *S1, *S2, *T;
    double *cand_s, *cand_z, *Delta, *G, *cost, *DeltaS, *GS, *costS;
    __half* Hcat; int *sel, *list; int fast_grid, grid_terms;          // two-phase search: T' of every H_in, survivor bookkeeping
    GridScale gscale; float *cand_r, *Wf, *wdown;
    GridInt gint; GridWeights gwt; int* gwp; double *gwv, *gleast;      // integer form: T', digits of the weight rows, their products, w T'^T, costs that void a pass
    double *Wbar, *Abar, *Z, *WR, *Cm, *Fm, *dvec, *lossbuf;
    double *Cg, *Fg, *cdnum;    // group-wise refinement: Gram blocks per (group, group) pair
    int grid_chunk, fast_chunk;     // block rows (shared H_in) or heads (per-head H_in) per grid-search pass: exact, two-phase
    int lazy;           // the deviation term of the sweep goes through S = R U^T (see run_layer); nr, nv: its row arrays
    double *nr, *nv;
    int* gstat;         // device words of the two-phase search (GS_*), cleared at the start of a run
    long long nn;
    // Products with the d_in x d_in matrices on the integer matrix cores (gemm_rns.hip): the matrices as right operands, prepared once a call, and per stream of the call
    // (0: main, 1: aux) the left operand of a product, residues of its result and sums of squares
    int no_rns;                 // no room for residues: everything in fp64, the factorisation too
    int rns, rns_rows_max;      // rns: which products (RNS_*); rns_rows_max: rows of a product at a time
    RnsOperand hT, uR, uC, uS, pS, rC, left[2];      // H_in (its half T; group-wise: whole), rows of U, columns of U, columns of U and P for the sweep, columns of R
    unsigned char* rres[2]; CholRns frns; double *rsq, *rsq2, *rpart, *wsq; int *kexp, *hexp, *rexp, *pshift;      // kexp .. rexp: powers of two per channel (see run_layer)
};

RnsSource rows_of(const double* a, long long ld, int rows, int k) {
    RnsSource s{};
    s.a = a; s.ld = ld; s.kc = 1; s.rows = rows; s.k = k;
    return s;
}
RnsSource columns_of(const double* a, long long ld, int columns, int k) {
    RnsSource s = rows_of(a, ld, columns, k);
    s.kc = 0;
    return s;
}

// rows that are contracted over channels, with the powers of two that the right operand has the other way round
RnsSource left_of_channels(const double* a, long long ld, int rows, int k, const int* kexp) {
    RnsSource s = rows_of(a, ld, rows, k);
    s.kexp = kexp; s.ksign = -1;
    return s;
}

int rns_right_columns(Layer& L, const RnsSource& s, const RnsOperand& o) {
    TB_TRY(rns_norms(L.ctx, s, 1, L.rsq, 0, L.rpart));
    TB_TRY(rns_exps(L.ctx, L.n, 1, L.rsq, 0, RNS_BITS_B, o.e, 0));
    return rns_columns(L.ctx, s, 1, o, 0);
}

// Columns of U as right operand of the sweep's updates, with_P: and those of P beside them (its two terms), after U and P.  A column's updates come from the blocks of SWEEP_SP columns
// before its own: the entries within that block, the diagonal among them, are no part of its norm.  (With them, where the damping makes channels that are hardly in use as large as
// 1e-2 of the mean, their columns of U are little else than diagonal, and an update is rounded in units that it does not reach: 2^-38 - 2^-50 of sum |e u| instead of 2^-55.)
int rns_sweep_columns(Layer& L, bool with_P) {
    tboa_ctx* ctx = L.ctx;
    RnsSource u = columns_of(L.Uin, L.n, L.n, L.n), p = columns_of(L.P, L.n, L.n, L.n);
    u.before = p.before = SWEEP_SP;
    p.exp_shift = L.pshift; p.ksign = 1;
    TB_TRY(rns_norms(ctx, u, 1, L.rsq, 0, L.rpart));
    if (with_P) {
        RnsSource plain = p;
        plain.exp_shift = nullptr;
        TB_TRY(rns_norms(ctx, plain, 1, L.rsq2, 0, L.rpart));
        TB_TRY(rns_balance(ctx, L.n, L.rsq, L.rsq2, L.pshift));
    }
    TB_TRY(rns_exps(ctx, L.n, 1, L.rsq, 0, RNS_BITS_B, L.uS.e, 0));
    TB_TRY(rns_columns(ctx, u, 1, L.uS, 0));
    return with_P ? rns_columns(ctx, p, 1, L.pS, 0) : 0;
}

// C = A B, B a prepared right operand of n columns, at most rns_rows_max rows of A (contiguous) at a time
struct RnsProduct { const RnsOperand* B; double* C; int klo_m, klo_n, khi_n, upper; };
int rns_products(Layer& L, int which, const RnsSource& A, const RnsProduct& p) {
    tboa_ctx* ctx = L.ctx;
    for (int r0 = 0; r0 < A.rows; r0 += L.rns_rows_max) {
        RnsSource a = A;
        a.a += (long long)r0 * A.ld; a.rows = std::min(L.rns_rows_max, A.rows - r0);
        TB_TRY(rns_rows(ctx, a, nullptr, 1, RNS_BITS_A, L.left[which]));
        RnsGemm g{};
        g.A = &L.left[which]; g.B = p.B; g.M = a.rows; g.N = L.n; g.K = A.k; g.klo_m = p.klo_m; g.klo_n = p.klo_n; g.khi_n = p.khi_n; g.upper = p.upper; g.row0 = r0;
        g.alpha = 1.0; g.beta = 0.0; g.C = p.C + (long long)r0 * L.n; g.ldc = L.n; g.residues = L.rres[which]; g.m_limit = A.row_limit;
        TB_TRY(rns_gemm(ctx, g));
    }
    return 0;
}

// Algorithm 1 line 9 for the rows Wrows (block rows of every head, or whole heads for the fixed grid), columns [c0, c0 + ncols).
// Everything is enqueued; nothing is read back here.
int grid_search(Layer& L, const double* Wrows, long long ldw, int rows_per_head, BlockMap map, int c0, int ncols, int gi) {
    tboa_ctx* ctx = L.ctx;
    const int nh = L.nh, ncand = L.ncand;
    const bool ph = L.nhin > 1;
    const int total_rows = nh * rows_per_head;
    const int units = ph ? nh : total_rows;                 // chunk unit: a head or a row
    const int rows_per_unit = ph ? rows_per_head : 1;
    const bool fast = L.fast_grid && c0 == 0 && ncols == L.n;
    if (!fast && ncand <= 256 && (ncols == 32 || ncols == 64 || ncols == 128)) {
        const int mats = ph ? nh : 1, per = ph ? rows_per_head : total_rows, rows_wg = std::max(1, (total_rows + 511) / 512);      // two workgroups of 128 columns fit a CU
        const dim3 grid((unsigned)((per + rows_wg - 1) / rows_wg), (unsigned)mats);
        ProfRec rec{}; bool timed = false;
        if (ctx->prof_on) TB_TRY(prof_begin(ctx, TBOA_PROF_F64_GRID, (double)total_rows * ncand * ncols * (ncols + 16.0), rec, timed));
#define TB_GROUP(NT) hipLaunchKernelGGL(grid_group_kernel<NT>, grid, dim3(256), 0, ctx->stream, Wrows, ldw, c0, L.Hi, ph ? L.nn : 0LL, L.n, per, rows_wg, ncand, \
                                        L.d->grid_points, L.maxq, map, L.s64, L.z64, L.ng, gi)
        if (ncols == 128) TB_GROUP(8);
        else if (ncols == 64) TB_GROUP(4);
        else TB_GROUP(2);
#undef TB_GROUP
        TB_KERNEL_CHECK(ctx);
        return prof_end(ctx, rec, timed);
    }
    const int chunk = fast ? L.fast_chunk : L.grid_chunk;
    for (int u0 = 0; u0 < units; u0 += chunk) {
        const int nu = (units - u0 < chunk) ? units - u0 : chunk;
        const int r0 = u0 * rows_per_unit, rows = nu * rows_per_unit;
        const double* Wc = Wrows + (long long)r0 * ldw;
        if (fast) {
            const bool delta = grid_delta(L.d->bits, L.n);
            const int n = L.n, np = grid_width(n, delta);
            const int mats = ph ? nu : 1, per_mat = ph ? rows_per_head : rows;
            const long long pitch = grid_pitch(np, delta), mo = ph ? (long long)u0 * np : 0;
            const GridRows m{per_mat, ncand, rows16((long long)per_mat * ncand), pitch, np};
            GridWeights gw = L.gwt;
            gw.w_rows = rows16((long long)GRID_WD * per_mat);
            if (delta) hipLaunchKernelGGL(grid_rows_kernel<true>, dim3((rows + 3) / 4), dim3(256), 0, ctx->stream, Wc, ldw, n, rows, L.d->grid_points, L.maxq, m, gw,
                                          L.cand_s, L.cand_z, L.cand_r, L.Wf, L.wdown);
            else hipLaunchKernelGGL(grid_rows_kernel<false>, dim3((rows + 3) / 4), dim3(256), 0, ctx->stream, Wc, ldw, n, rows, L.d->grid_points, L.maxq, m, gw,
                                    L.cand_s, L.cand_z, L.cand_r, L.Wf, L.wdown);
            const unsigned rb = (unsigned)(((long long)m.per * ncand + 63) / 64);
            // (columns in up to 8 parts where there are few rows)
            const unsigned cparts = (long long)rb * mats >= 2048 ? 1u : (unsigned)std::min<long long>(8, 2048 / ((long long)rb * mats) + 1);
            GemmBf16 a{};
            a.M = (int)m.mat_rows; a.N = np; a.alpha = 1.f; a.lda = a.ldb = pitch; a.C = L.G; a.ldc = np;
            a.A = (const __hip_bfloat16*)L.Delta; a.B = (const __hip_bfloat16*)L.Hcat + (ph ? (long long)u0 * np * pitch : 0);
            a.batch = mats; a.strideA = m.mat_rows * pitch; a.strideB = (long long)np * pitch; a.strideC = m.mat_rows * np;
            a.c_dtype = TBOA_F32; a.accumulate = 0; a.tag = TBOA_PROF_GRID;
            const long long term = (long long)L.nhin * np * pitch;
            a.nterms = delta ? 2 : 3;
            for (int t = 0; t < a.nterms; ++t) { a.termA[t] = a.A; a.termB[t] = a.B + t * term; }
            a.flags = TBOA_GEMM_A_TILED | TBOA_GEMM_B_TILED | TBOA_GEMM_CAUSAL_K;     // T' is lower triangular
            const long long crow = (long long)rows * ncand;
            if (delta) {
                GridScale gs = L.gscale;      // of the first matrix of this pass
                gs.up += mo; gs.down += mo; gs.dcorr += mo; if (ph) { gs.scale += u0; gs.terms += u0; }
                __half* Acat = (__half*)L.Delta;
                const long long lo_off = (long long)mats * m.mat_rows * pitch;
                hipLaunchKernelGGL(grid_delta_pair_kernel, dim3(cparts, rb, mats), dim3(256), 0, ctx->stream, Wc, ldw, L.Wf, n, (float)L.maxq, m, gs,
                                   L.cand_s, L.cand_z, L.cand_r, L.wdown, Acat, lo_off);
                TB_KERNEL_CHECK(ctx);
                a.K = np; a.segs = gs.terms; a.flags |= TBOA_GEMM_F16;
                TB_TRY(gemm_bf16_nt(ctx, a));
                a.A += lo_off; a.segs = nullptr; a.nterms = 1; a.accumulate = 1;      // the low parts of delta against the first term of T'
                TB_TRY(gemm_bf16_nt(ctx, a));
                hipLaunchKernelGGL(grid_pair_cost_kernel, dim3((unsigned)((crow + 3) / 4)), dim3(256), 0, ctx->stream, (const float*)L.G, Acat, rows, m, gs, L.wdown, L.cost, lo_off);
            } else {
                GridInt gi2 = L.gint;
                gi2.v += mo; gi2.hd += mo; if (ph) gi2.terms += u0;
                signed char* Acat = (signed char*)L.Delta;
                hipLaunchKernelGGL(grid_codes_kernel, dim3(cparts, rb, mats), dim3(256), 0, ctx->stream, Wc, ldw, L.Wf, n, (float)L.maxq, m, L.cand_s, L.cand_z, L.cand_r, Acat);
                TB_KERNEL_CHECK(ctx);
                a.K = np / 2; a.segs = gi2.terms; a.flags |= TBOA_GEMM_I8;
                TB_TRY(gemm_bf16_nt(ctx, a));
                // the digits of the weight rows against every digit of T', one result each (a third digit that is not taken is zero)
                GemmBf16 w = a;
                w.M = (int)gw.w_rows; w.A = (const __hip_bfloat16*)gw.A; w.C = L.gwp; w.segs = nullptr; w.nterms = 1; w.tag = -1;
                w.batch = 3 * mats; w.batch_inner = 3; w.strideA = gw.w_rows * pitch; w.strideA2 = 0; w.strideB2 = term; w.strideC = 3 * gw.w_rows * np; w.strideC2 = gw.w_rows * np;
                TB_TRY(gemm_bf16_nt(ctx, w));
                hipLaunchKernelGGL(grid_weight_products_kernel, dim3((unsigned)((np + 255) / 256), rows), dim3(256), 0, ctx->stream, L.gwp, m, gw, gi2, L.gwv);
                const long long parts = (ncand + GRID_KC - 1) / GRID_KC;
                hipLaunchKernelGGL(grid_cost_kernel, dim3((unsigned)((rows * parts + 3) / 4)), dim3(256), 0, ctx->stream, (const int*)L.G, Acat, rows, m, gi2, L.cand_s,
                                   Wc, ldw, n, L.gwv, L.cost, L.gleast);
            }
            TB_KERNEL_CHECK(ctx);
            const int per = ph ? rows_per_head : rows, ngrp = rows / per;    // rows that share one H_in
            const int cap = per * GRID_KS;                                    // exact re-evaluations a group has room for
            int* cntv = L.sel; int* offv = cntv + rows; int* totv = offv + rows;
            hipLaunchKernelGGL(grid_count_kernel, dim3((rows + 3) / 4), dim3(256), 0, ctx->stream, L.cost, rows, ncand,
                               delta ? nullptr : L.gint.tau + (ph ? u0 : 0), per, delta ? nullptr : L.gleast, L.list, cntv, L.gstat);
            hipLaunchKernelGGL(grid_scan_kernel, dim3(ngrp), dim3(256), 0, ctx->stream, cntv, per, cap, offv, totv, L.gstat);
            hipLaunchKernelGGL(grid_delta_sel_kernel, dim3((n + 255) / 256, rows), dim3(256), 0, ctx->stream, Wc, ldw, n, ncand, L.maxq,
                               L.cand_s, L.cand_z, L.list, cntv, offv, per, cap, L.DeltaS);
            TB_KERNEL_CHECK(ctx);
            if (L.rns & RNS_EXACT) {
                RnsSource a = left_of_channels(L.DeltaS, n, cap, n, L.hexp);
                a.row_limit = totv;
                TB_TRY(rns_products(L, 0, a, {&L.hT, L.GS, 0, 0, 1, 0}));
            } else {
            GemmF64 g{};
            g.M = cap; g.N = n; g.K = n; g.alpha = 1.0; g.beta = 0.0; g.A = L.DeltaS; g.sam = n; g.sak = 1; g.sbk = n; g.sbn = 1;
            g.C = L.GS; g.ldc = n; g.batch = ngrp; g.strideA = (long long)g.M * n; g.strideC = g.strideA; g.m_limit = totv;
            g.B = L.Hi + (ph ? (long long)u0 * L.nn : 0); g.strideB = ph ? L.nn : 0;
            g.tag = TBOA_PROF_F64_GRID; g.sym = 1;      // delta H delta^T: half of H is enough
            TB_TRY(gemm_f64(ctx, g));
            }
            const long long srow = (long long)ngrp * cap;
            hipLaunchKernelGGL(rowdot_limited_kernel, dim3((unsigned)((srow + 3) / 4)), dim3(256), 0, ctx->stream, L.GS, L.DeltaS, n, cap,
                               srow, totv, L.costS);
            hipLaunchKernelGGL(grid_argmin_sel_kernel, dim3((rows + 3) / 4), dim3(256), 0, ctx->stream, L.costS, L.cost, L.list, cntv, offv, per, cap,
                               L.cand_s, L.cand_z, rows, ncand, map, r0, L.s64, L.z64, L.ng, gi, delta ? nullptr : L.gleast, L.gstat);
            TB_KERNEL_CHECK(ctx);
            ++ctx->counters[TBOA_CTR_GRID_PASSES];
            continue;
        }
        hipLaunchKernelGGL(grid_candidates_kernel, dim3((rows + 3) / 4), dim3(256), 0, ctx->stream, Wc, ldw, c0, ncols, rows,
                           ncand, L.d->grid_points, L.maxq, L.cand_s, L.cand_z);
        hipLaunchKernelGGL(grid_delta_kernel, dim3((ncols + 255) / 256, rows), dim3(256), 0, ctx->stream, Wc, ldw, c0, ncols, ncand,
                           L.maxq, L.cand_s, L.cand_z, L.Delta);
        TB_KERNEL_CHECK(ctx);
        GemmF64 g{};
        g.N = ncols; g.K = ncols; g.alpha = 1.0; g.beta = 0.0;
        g.A = L.Delta; g.sam = ncols; g.sak = 1;
        g.sbk = L.n; g.sbn = 1; g.C = L.G; g.ldc = ncols;
        g.tag = TBOA_PROF_F64_GRID; g.sym = 1;
        if (ph) {
            g.M = rows_per_head * ncand; g.batch = nu;
            g.B = L.Hi + (long long)u0 * L.nn + (long long)c0 * L.n + c0;
            g.strideA = (long long)g.M * ncols; g.strideB = L.nn; g.strideC = g.strideA;
        } else {
            g.M = rows * ncand; g.batch = 1;
            g.B = L.Hi + (long long)c0 * L.n + c0;
        }
        TB_TRY(gemm_f64(ctx, g));
        const long long crow = (long long)rows * ncand;
        hipLaunchKernelGGL(rowdot_kernel, dim3((unsigned)((crow + 3) / 4)), dim3(256), 0, ctx->stream, L.G, (long long)ncols, L.Delta,
                           (long long)ncols, crow, ncols, L.cost);
        hipLaunchKernelGGL(grid_argmin_kernel, dim3((rows + 3) / 4), dim3(256), 0, ctx->stream, L.cost, L.cand_s, L.cand_z, rows,
                           ncand, map, r0, L.s64, L.z64, L.ng, gi);
        TB_KERNEL_CHECK(ctx);
    }
    return 0;
}

// one GEMM over all block rows (shared H_in) or batched per head (per-head H_in): C = alpha A op(B) + beta C,
// A, C block arrays [nh*nbr, *]; B a d_in x d_in matrix (or one per head) addressed by (sbk, sbn) at offset boff.
int block_gemm(Layer& L, int nbr, int N, int K, double alpha, const double* A, long long lda, const double* B, long long boff,
               long long sbk, long long sbn, double beta, double* C, long long ldc, int tag, const GemmF64* flags = nullptr) {
    GemmF64 g{};
    if (flags) g = *flags;
    g.tag = tag;
    g.N = N; g.K = K; g.alpha = alpha; g.beta = beta;
    g.A = A; g.sam = lda; g.sak = 1; g.B = B + boff; g.sbk = sbk; g.sbn = sbn; g.C = C; g.ldc = ldc;
    if (L.nhin > 1) { g.M = nbr; g.batch = L.nh; g.strideA = (long long)nbr * lda; g.strideB = L.nn; g.strideC = (long long)nbr * ldc; }
    else { g.M = L.nh * nbr; g.batch = 1; }
    return gemm_f64(L.ctx, g);
}

// The two updates of a lazily corrected sweep (L.lazy) as one launch: Wk[:, col ..] -= Epan U and acc[:, col ..] -= Wsnap M, for the columns ecol .. of the
// panel arrays and the N columns at offset boff of U and of M (both d x d, or one per head).
int pair_gemm(Layer& L, int nbr, int N, int K, int ecol, long long boff, const double* M, int col, double* acc) {
    GemmF64 g{};
    g.N = N; g.K = K; g.alpha = -1.0; g.beta = 1.0; g.tag = TBOA_PROF_F64_SWEEP;
    g.A = L.Epan + ecol; g.sam = SWEEP_SP; g.sak = 1; g.B = L.Uin + boff; g.sbk = L.n; g.sbn = 1; g.C = L.Wk + col; g.ldc = L.n;
    g.batch_inner = 2; g.strideA2 = L.Wsnap - L.Epan; g.strideB2 = M - L.Uin; g.strideC2 = acc - L.Wk;
    if (L.nhin > 1) { g.M = nbr; g.batch = 2 * L.nh; g.strideA = (long long)nbr * SWEEP_SP; g.strideB = L.nn; g.strideC = (long long)nbr * L.n; }
    else { g.M = L.nh * nbr; g.batch = 2; }
    return gemm_f64(L.ctx, g);
}

// Wk[:, s1 ..] -= Epan U[s0 .. s1, s1 ..] + Wsnap P[s0 .. s1, s1 ..], both terms in one product of residues
int rns_sweep_update(Layer& L, int rows, int s0, int s1, bool with_P) {
    for (int r0 = 0; r0 < rows; r0 += L.rns_rows_max) {
        const int m = std::min(L.rns_rows_max, rows - r0);
        RnsSource e = rows_of(L.Epan + (long long)r0 * SWEEP_SP, SWEEP_SP, m, SWEEP_SP), w = rows_of(L.Wsnap + (long long)r0 * SWEEP_SP, SWEEP_SP, m, SWEEP_SP);
        w.exp_shift = L.pshift; w.ksign = -1;
        TB_TRY(rns_rows(L.ctx, e, with_P ? &w : nullptr, 1, RNS_BITS_A, L.left[0]));
        RnsGemm g{};
        g.A = &L.left[0]; g.B = &L.uS; g.B2 = with_P ? &L.pS : nullptr; g.b_row = s1; g.b_k = s0; g.M = m; g.N = L.n - s1; g.K = SWEEP_SP;
        g.alpha = -1.0; g.beta = 1.0; g.C = L.Wk + (long long)r0 * L.n + s1; g.ldc = L.n; g.residues = L.rres[0];
        TB_TRY(rns_gemm(L.ctx, g));
    }
    return 0;
}

// return values of run_layer: the approximate costs of the two-phase grid search could not be trusted somewhere in this
// run (see grid_search): the caller runs the layer again with exact costs for every candidate, or (the shorter form of H was not enough) with the longer one
constexpr int RUN_AGAIN_EXACT = 1, RUN_AGAIN_TWO_TERMS = 2;

int run_layer(Layer& L, const void* W, const float* H_in, const float* H_out, const float* R, uint8_t* codes, float* scales,
              float* zeros, float* W_deq, double* loss, double* loss_per_head) {
    tboa_ctx* ctx = L.ctx; const tboa_layer_desc* d = L.d;
    const int n = L.n, nh = L.nh, dh = L.dh, ng = L.ng, nhin = L.nhin;
    const long long nn = L.nn, wn = (long long)d->d_out * n;
    hipStream_t st = ctx->stream;

    hipLaunchKernelGGL(clear_words_kernel, dim3(1), dim3(64), 0, st, L.gstat, (int)GS_WORDS);
    TB_KERNEL_CHECK(ctx);

    TB_TRY(launch_cvt_to_f64(ctx, W, d->w_dtype, L.W64, wn));
    TB_HIP(ctx, hipMemcpyAsync(L.Wt, L.W64, wn * sizeof(double), hipMemcpyDeviceToDevice, st));
    // eq. 3 for H_in (and H_out).  The factorisation reads the upper triangle; the half products below read whatever triangle their tiles say, so
    // that an H_in that is symmetric up to rounding only must be made so first
    TB_TRY(launch_symmetric_f64_damp(ctx, n, nhin, H_in, d->damp, L.Hi));
    TB_TRY(launch_f32_to_f64_damp(ctx, n, nhin, H_in, d->damp, L.Hfac));
    if (L.fast_grid) {
        const bool delta = grid_delta(d->bits, n);
        const int np = grid_width(n, delta);
        const long long pitch = grid_pitch(np, delta), term = (long long)nhin * np * pitch;
        if (delta) {
            hipLaunchKernelGGL(grid_scale_kernel, dim3(nhin), dim3(256), 0, st, L.Hi, n, np, L.gscale);
            hipLaunchKernelGGL(grid_factor_kernel, dim3(np, nhin), dim3(256), 0, st, L.Hi, n, np, L.gscale, L.Hcat, term);
            hipLaunchKernelGGL(grid_terms_kernel, dim3(nhin), dim3(256), 0, st, L.Hi, n, np, L.gscale, L.grid_terms, grid_one_term(d->bits), L.gstat + GS_SHORT);
        } else {
            hipLaunchKernelGGL(grid_int_steps_kernel, dim3(np, nhin), dim3(256), 0, st, L.Hi, n, np, L.maxq, L.gint);
            hipLaunchKernelGGL(grid_int_terms_kernel, dim3(nhin), dim3(256), 0, st, n, np, L.gint, L.grid_terms >= 2, grid_one_term(d->bits), d->grid_guard > 0.25, L.gstat + GS_SHORT);
            hipLaunchKernelGGL(grid_int_factor_kernel, dim3(np, nhin), dim3(256), 0, st, L.Hi, n, np, pitch, L.gint, (signed char*)L.Hcat, 2 * term);
        }
        TB_KERNEL_CHECK(ctx);
    }
    if (L.rns) {
        // (R U^T and (W R) U^T: rows of R grow with a channel's size, U's entries fall)
        TB_TRY(rns_channel_sizes(ctx, n, L.Hi, L.kexp));
        // products of W (and what has its size: delta, codes less zeros, the rows of a step) with H_in and R: sizes of W's columns against those of H_in's and of R's rows
        if (L.hT.p || L.rC.p) TB_TRY(rns_norms(ctx, columns_of(L.W64, n, n, d->d_out), 1, L.wsq, 0, L.rpart));
        if (L.hT.p) {
            TB_TRY(rns_channel_exps(ctx, n, L.wsq, L.kexp, L.kexp, L.hexp));
            RnsSource h = rows_of(L.Hi, n, n, n);
            h.half = !d->group; h.kexp = L.hexp; h.ksign = 1;
            TB_TRY(rns_rows(ctx, h, nullptr, 1, RNS_BITS_B, L.hT));
        }
    }
    // U_in, P and U_out are first needed by the first in-channel sweep; the grid search before it needs only W and H_in.
    // The factorisations and the two P products (for one matrix: chains of small kernels that leave most of the GPU idle)
    // therefore run on the context's second stream, beside that grid search; setup_join() below is where they meet.
    // The breakdown status of the factorisations is read at the end of the call, with everything else that comes back.
    struct StreamSwap {      // everything enqueued while this lives goes to the second stream
        tboa_ctx* c; hipStream_t keep;
        explicit StreamSwap(tboa_ctx* c_) : c(c_), keep(c_->stream) { c->stream = c->aux; }
        ~StreamSwap() { c->stream = keep; }
    };
    bool joined = false;
    struct DrainAux {      // an error return before the join must not leave work running on the workspace
        tboa_ctx* c; const bool* joined;
        ~DrainAux() { if (!*joined) (void)hipStreamSynchronize(c->aux); }
    } drain{ctx, &joined};
    TB_HIP(ctx, hipEventRecord(ctx->ev_fork, st));
    {
    StreamSwap swap(ctx);
    TB_HIP(ctx, hipStreamWaitEvent(ctx->aux, ctx->ev_fork, 0));
    TB_TRY(chol_inv_upper_f64(ctx, n, nhin, L.Hfac, L.Uin, L.ftmp, L.fdinv, 0, true, &L.frns));
    // Algorithm 3 line 2: P = ((R U^T) * M_U) U.  Two products of d^3 / 3 flops each per H_in, which few rows do not repay (W_V of a grouped-query
    // block: 128 rows per 8192 x 8192 Hessian, 54 of its 176 ms).  L.lazy: the term that P carries from the columns j to a column k is
    //     sum_{j < k} w_j P[j, k] = sum_{m <= k} v_m U[m, k],    v_m = sum_{j < m} w_j S[j, m] = sum_{k >= m} U[m, k] sum_{j < m} w_j R[j, k],  S = R U^T
    // so a group of SWEEP_SP columns starts from v = r U^T with r = sum of w_j R[j, :] over the columns already done (one product per group), inside the
    // group the block of S on the diagonal takes the place of P, and after it r += w R.  That costs rows d^2 flops more in the sweep and
    // SWEEP_SP d^2 for the blocks: taken when that is less than the products it saves (rows < d / 2 - SWEEP_SP per H_in).
    if (R) {
        TB_TRY(launch_cvt_f32_to_f64(ctx, R, L.Rd, nhin * nn));
        if (L.rC.p) {
            TB_TRY(rns_row_exps(ctx, rows_of(L.Rd, n, n, n), 0, L.rexp));
            TB_TRY(rns_channel_exps(ctx, n, L.wsq, L.kexp, L.rexp, L.rexp));
            RnsSource r = columns_of(L.Rd, n, n, n);
            r.kexp = L.rexp; r.ksign = 1;
            TB_TRY(rns_right_columns(L, r, L.rC));
        }
        if (L.uC.p) TB_TRY(rns_right_columns(L, columns_of(L.Uin, n, n, n), L.uC));
        if (L.uR.p) {
            RnsSource u = rows_of(L.Uin, n, n, n);
            u.kexp = L.kexp; u.ksign = 1;
            TB_TRY(rns_rows(ctx, u, nullptr, 1, RNS_BITS_B, L.uR));
        }
        if (L.lazy) {
            // only the blocks of SWEEP_SP columns on the diagonal of S = R U^T, into L.P
            for (int s0 = 0; s0 < n; s0 += SWEEP_SP) {
                const int w = n - s0 < SWEEP_SP ? n - s0 : SWEEP_SP;
                const long long o = (long long)s0 * n + s0;
                GemmF64 a{};
                a.M = w; a.N = w; a.K = n - s0; a.alpha = 1.0; a.beta = 0.0; a.A = L.Rd + o; a.sam = n; a.sak = 1; a.B = L.Uin + o; a.sbk = 1; a.sbn = n;
                a.C = L.P + o; a.ldc = n; a.batch = nhin; a.strideA = nn; a.strideB = nn; a.strideC = nn; a.tag = TBOA_PROF_F64_FACTOR;
                TB_TRY(gemm_f64(ctx, a));
            }
        } else if (L.rns & RNS_P) {
            TB_TRY(rns_products(L, 1, left_of_channels(L.Rd, n, n, n, L.kexp), {&L.uR, L.Hfac, 0, 1, 0, 1}));      // U[c, k] = 0 for k < c; only above the diagonal
            TB_TRY(rns_products(L, 1, rows_of(L.Hfac, n, n, n), {&L.uC, L.P, 1, 0, 1, 1}));
        } else {
            GemmF64 a{};
            a.M = n; a.N = n; a.K = n; a.alpha = 1.0; a.beta = 0.0;
            a.A = L.Rd; a.sam = n; a.sak = 1; a.B = L.Uin; a.sbk = 1; a.sbn = n; a.klo_n = 1;   // U[c, k] = 0 for k < c
            a.skip_lower = 1;   // only the part above the diagonal survives the mask below
            a.C = L.Hfac; a.ldc = n; a.batch = nhin; a.strideA = nn; a.strideB = nn; a.strideC = nn;
            a.tag = TBOA_PROF_F64_FACTOR;
            TB_TRY(gemm_f64(ctx, a));
            TB_TRY(launch_strict_upper_f64(ctx, L.Hfac, n, nhin));
            GemmF64 b{};
            b.M = n; b.N = n; b.K = n; b.alpha = 1.0; b.beta = 0.0;
            b.A = L.Hfac; b.sam = n; b.sak = 1; b.klo_m = 1;       // (R U^T)_masked[j, m] = 0 for m <= j
            b.B = L.Uin; b.sbk = n; b.sbn = 1; b.khi_n = 1;        // U[m, k] = 0 for m > k
            b.diag_order = 1;                                      // contraction range (row start, column end]: grows with the column
            b.C = L.P; b.ldc = n; b.batch = nhin; b.strideA = nn; b.strideB = nn; b.strideC = nn;
            b.tag = TBOA_PROF_F64_FACTOR;
            TB_TRY(gemm_f64(ctx, b));
        }
    }
    if (L.uS.p) TB_TRY(rns_sweep_columns(L, L.pS.p != nullptr));
    if (H_out) {
        TB_TRY(launch_f32_to_f64_damp(ctx, dh, nh, H_out, d->damp, L.Ho));
        TB_HIP(ctx, hipMemcpyAsync(L.Hofac, L.Ho, (size_t)nh * dh * dh * sizeof(double), hipMemcpyDeviceToDevice, ctx->stream));
        TB_TRY(chol_inv_upper_f64(ctx, dh, nh, L.Hofac, L.Uout, L.ftmp, L.fdinv, 2, true));
    }
    TB_HIP(ctx, hipEventRecord(ctx->ev_join, ctx->aux));
    }
    auto setup_join = [&]() -> int {
        if (joined) return 0;
        TB_HIP(ctx, hipStreamWaitEvent(st, ctx->ev_join, 0));
        joined = true;
        return 0;
    };
    const double* Pp = R ? L.P : nullptr;
    // columns per group of panels: a group-wise grid is searched on the current columns of its group when the sweep enters
    // it, so a group of panels must not straddle a grid group that starts inside it unaligned
    const int sp = (!d->group || SWEEP_SP % L.gsz == 0 || L.gsz % SWEEP_SP == 0) ? SWEEP_SP : L.gsz < 64 ? L.gsz : 64;
    // columns per launch of the sweep: up to where the next grid is searched (and one grid per launch if it has fewer columns than a sub-panel)
    const int pw_max = d->group && (d->adaptive_grid || L.gsz < 16) ? std::min(L.gsz, sp) : sp;

    if (!d->adaptive_grid) {   // BoA: one grid from the original weights
        BlockMap id{dh, dh, 0};
        for (int gi = 0; gi < ng; ++gi) TB_TRY(grid_search(L, L.W64, n, dh, id, gi * L.gsz, L.gsz, gi));
    }
    for (int i0 = 0; i0 < dh; i0 += d->block) {
        const int i1 = (i0 + d->block < dh) ? i0 + d->block : dh;
        const int nbr = i1 - i0, rows = nh * nbr;
        BlockMap map{nbr, dh, i0};
        hipLaunchKernelGGL(gather_rows_kernel, dim3(gx(n), rows), dim3(256), 0, st, L.Wt, L.Wb, L.Wk, map, n);
        TB_KERNEL_CHECK(ctx);
        if (L.lazy) { TB_TRY(launch_fill_f64(ctx, L.nr, (int64_t)rows * n, 0.0)); TB_TRY(launch_fill_f64(ctx, L.nv, (int64_t)rows * n, 0.0)); }
        if (d->adaptive_grid && !d->group) TB_TRY(grid_search(L, L.Wk, n, nbr, map, 0, n, 0));
        // Algorithm 3 in groups of up to SWEEP_SP columns: one launch takes the rows through a group (group-wise grids: through a panel of it, after
        // which the rest of the group follows), and the columns right of the group get the whole update in one product
        for (int s0 = 0; s0 < n; s0 += sp) {
            const int s1 = (n - s0 < sp) ? n : s0 + sp;
            if (L.lazy && s0 > 0)      // -v of the group's columns from what the columns before it have left in -r
                TB_TRY(block_gemm(L, nbr, s1 - s0, n - s0, 1.0, L.nr + s0, n, L.Uin, (long long)s0 * n + s0, 1, n, 0.0, L.nv + s0, n, TBOA_PROF_F64_SWEEP));
            for (int c0 = s0; c0 < s1; c0 += pw_max) {
                const int pw = (s1 - c0 < pw_max) ? s1 - c0 : pw_max, c1 = c0 + pw;
                if (d->group && d->adaptive_grid && c0 % L.gsz == 0) TB_TRY(grid_search(L, L.Wk, n, nbr, map, c0, L.gsz, c0 / L.gsz));
                SweepArgs a;
                a.Wk = L.Wk; a.n = n; a.nbr = nbr; a.map = map; a.U = L.Uin; a.P = Pp; a.per_head = nhin > 1;
                a.c0 = c0; a.width = pw; a.s = L.s64; a.z = L.z64; a.ng = ng; a.gsz = L.gsz; a.maxq = L.maxq;
                a.codes = codes; a.Q = L.Q64; a.Epan = L.Epan + (c0 - s0); a.Wsnap = L.Wsnap + (c0 - s0); a.epitch = SWEEP_SP; a.nv = L.nv;
                TB_TRY(setup_join());
                TB_TRY(launch_sweep(ctx, a, nh, L.lazy));
                if (c1 < s1) {   // group-wise grids: rest of the group of panels, W[:, c1:s1] -= E U[c0:c1, c1:s1] + Wsnap P[c0:c1, c1:s1], both terms in one pass
                    GemmF64 two{};
                    if (Pp) { two.A2 = L.Wsnap + (c0 - s0); two.B2 = L.P + (long long)c0 * n + c1; }
                    TB_TRY(block_gemm(L, nbr, s1 - c1, pw, -1.0, L.Epan + (c0 - s0), SWEEP_SP, L.Uin, (long long)c0 * n + c1, n, 1, 1.0, L.Wk + c1, n,
                                      TBOA_PROF_F64_SWEEP, &two));
                }
            }
            if (s1 < n) {   // columns right of the group: W[:, s1:] -= E U[s0:s1, s1:] + Wsnap P[s0:s1, s1:]
                if (L.lazy) {        // W -= (E + V) U and -R -= Wsnap R
                    TB_TRY(pair_gemm(L, nbr, n - s1, s1 - s0, 0, (long long)s0 * n + s1, L.Rd, s1, L.nr));
                    continue;
                }
                if ((L.rns & RNS_SWEEP) && s1 - s0 == SWEEP_SP) { TB_TRY(rns_sweep_update(L, rows, s0, s1, Pp != nullptr)); continue; }
                GemmF64 two{};
                if (Pp) { two.A2 = L.Wsnap; two.B2 = L.P + (long long)s0 * n + s1; }
                TB_TRY(block_gemm(L, nbr, n - s1, s1 - s0, -1.0, L.Epan, SWEEP_SP, L.Uin, (long long)s0 * n + s1, n, 1, 1.0, L.Wk + s1, n,
                                  TBOA_PROF_F64_SWEEP, &two));
            }
        }
        if (H_out && i1 < dh) {
            const double* S3 = nullptr;
            if (R && (L.rns & RNS_COMP)) {   // W_B R H_in^-1 = ((W_B R) U^T) U
                TB_TRY(rns_products(L, 0, left_of_channels(L.Wb, n, rows, n, L.rexp), {&L.rC, L.S1, 0, 0, 0, 0}));
                TB_TRY(rns_products(L, 0, left_of_channels(L.S1, n, rows, n, L.kexp), {&L.uR, L.S2, 0, 1, 0, 0}));
                TB_TRY(rns_products(L, 0, rows_of(L.S2, n, rows, n), {&L.uC, L.S1, 0, 0, 1, 0}));
                S3 = L.S1;
            } else if (R) {
                GemmF64 f1{}; f1.klo_n = 1;
                GemmF64 f2{}; f2.khi_n = 1;
                TB_TRY(block_gemm(L, nbr, n, n, 1.0, L.Wb, n, L.Rd, 0, n, 1, 0.0, L.S1, n, TBOA_PROF_F64_COMP));
                TB_TRY(block_gemm(L, nbr, n, n, 1.0, L.S1, n, L.Uin, 0, 1, n, 0.0, L.S2, n, TBOA_PROF_F64_COMP, &f1));
                TB_TRY(block_gemm(L, nbr, n, n, 1.0, L.S2, n, L.Uin, 0, n, 1, 0.0, L.S1, n, TBOA_PROF_F64_COMP, &f2));
                S3 = L.S1;
            }
            hipLaunchKernelGGL(comp_error_kernel, dim3(gx(n), rows), dim3(256), 0, st, L.Wb, L.Q64, S3, L.E, map, n);
            const int rem = dh - i1;
            const int t_lds = nbr <= 2048;
            hipLaunchKernelGGL(comp_T_kernel, dim3((rem + 3) / 4, nh), dim3(256), t_lds ? (size_t)4 * nbr * sizeof(double) : 0, st, L.Uout, dh, i0, i1, L.T, d->block,
                               t_lds);
            TB_KERNEL_CHECK(ctx);
            GemmF64 u{};   // W~[i1:, :] -= T E per head
            u.M = rem; u.N = n; u.K = nbr; u.alpha = -1.0; u.beta = 1.0;
            u.A = L.T + (long long)i1 * d->block; u.sam = d->block; u.sak = 1;
            u.B = L.E; u.sbk = n; u.sbn = 1;
            u.C = L.Wt + (long long)i1 * n; u.ldc = n;
            u.batch = nh; u.strideA = (long long)dh * d->block; u.strideB = (long long)nbr * n; u.strideC = (long long)dh * n;
            u.tag = TBOA_PROF_F64_COMP;
            TB_TRY(gemm_f64(ctx, u));
        }
    }

    // Algorithm 2 + outputs + loss
    const int rows_all = d->d_out;
    GemmF64 half{}; half.sym = 1;
    hipLaunchKernelGGL(wbar_kernel, dim3(gx(n), rows_all), dim3(256), 0, st, codes, L.z64, ng, L.gsz, n, L.Wbar);
    TB_KERNEL_CHECK(ctx);
    // products with H_in (without groups its half T in either form, see below)
    const bool rns = L.rns & RNS_REFINE;
    auto rns_with_h = [&](const double* rows, double* to) { return rns_products(L, 0, left_of_channels(rows, n, rows_all, n, L.hexp), {&L.hT, to, 0, 0, d->group ? 0 : 1, 0}); };
    if (rns) {
        if (R) TB_TRY(rns_products(L, 0, left_of_channels(L.W64, n, rows_all, n, L.rexp), {&L.rC, L.WR, 0, 0, 0, 0}));
        if (d->cd_iters > 0) TB_TRY(rns_with_h(L.W64, L.Z));
    } else if (R) TB_TRY(block_gemm(L, dh, n, n, 1.0, L.W64, n, L.Rd, 0, n, 1, 0.0, L.WR, n, TBOA_PROF_F64_CD));
    if (d->cd_iters > 0 && d->group) {
        // Z = W (H_in - R); per group g: AH = Wbar[:, G] H_in[G, :] (into Abar), then the Gram blocks against every group
        const int gsz = L.gsz;
        const long long rr = (long long)dh * dh;
        if (!rns) TB_TRY(block_gemm(L, dh, n, n, 1.0, L.W64, n, L.Hi, 0, n, 1, 0.0, L.Z, n, TBOA_PROF_F64_CD));
        if (R) TB_TRY(launch_sub_f64(ctx, L.Z, L.WR, L.Z, wn));
        if (H_out) {
            GemmF64 f{};   // Fg[h][g] = Wbar_h[:, G] Z_h[:, G]^T
            f.M = dh; f.N = dh; f.K = gsz; f.alpha = 1.0; f.beta = 0.0;
            f.A = L.Wbar; f.sam = n; f.sak = 1; f.B = L.Z; f.sbk = 1; f.sbn = n; f.C = L.Fg; f.ldc = dh;
            f.batch = nh * ng; f.batch_inner = ng;
            f.strideA = (long long)dh * n; f.strideB = f.strideA; f.strideC = ng * rr;
            f.strideA2 = gsz; f.strideB2 = gsz; f.strideC2 = rr;
            TB_TRY(gemm_f64(ctx, f));
        } else {
            hipLaunchKernelGGL(segdot_kernel, dim3((unsigned)(((long long)rows_all * ng + 3) / 4)), dim3(256), 0, st, L.Wbar, L.Z,
                               (long long)rows_all, n, gsz, ng, L.Fg, (long long)ng);
            TB_KERNEL_CHECK(ctx);
        }
        for (int g = 0; g < ng; ++g) {
            // with H_out only the blocks g' <= g: H_in is symmetric, Cg[h][g'][g] = Cg[h][g][g']^T (13B-shaped W_K, 40 groups of 128: the call 88.6 -> 83.8 ms)
            const int gs = H_out ? g + 1 : ng;
            TB_TRY(block_gemm(L, dh, gs * gsz, gsz, 1.0, L.Wbar + (long long)g * gsz, n, L.Hi, (long long)g * gsz * n, n, 1, 0.0, L.Abar, n, TBOA_PROF_F64_CD));
            if (H_out) {
                GemmF64 c{};   // Cg[h][g][g'] = AH_h[:, G'] Wbar_h[:, G']^T
                c.M = dh; c.N = dh; c.K = gsz; c.alpha = 1.0; c.beta = 0.0;
                c.A = L.Abar; c.sam = n; c.sak = 1; c.B = L.Wbar; c.sbk = 1; c.sbn = n; c.C = L.Cg + (long long)g * ng * rr; c.ldc = dh;
                c.batch = nh * gs; c.batch_inner = gs;
                c.strideA = (long long)dh * n; c.strideB = c.strideA; c.strideC = (long long)ng * ng * rr;
                c.strideA2 = gsz; c.strideB2 = gsz; c.strideC2 = rr;
                TB_TRY(gemm_f64(ctx, c));
            } else {   // Cd[row][g][g'] = AH[row, G'] . Wbar[row, G']
                hipLaunchKernelGGL(segdot_kernel, dim3((unsigned)(((long long)rows_all * ng + 3) / 4)), dim3(256), 0, st, L.Abar, L.Wbar,
                                   (long long)rows_all, n, gsz, ng, L.Cg + (long long)g * ng, (long long)ng * ng);
                TB_KERNEL_CHECK(ctx);
            }
        }
        if (H_out) {
            if (ng > 1) {
                const long long tiles = cdiv64(dh, 64) * cdiv64(dh, 64);
                hipLaunchKernelGGL(cd_group_mirror_kernel, dim3((unsigned)(tiles * ng * (ng - 1) / 2), 1, nh), dim3(256), 0, st, L.Cg, dh, ng);
                TB_KERNEL_CHECK(ctx);
            }
            const size_t room = 160 * 1024 / sizeof(double), scales = (size_t)dh * ng;
            if (scales + dh + 8 > room) return tboa_fail(ctx, TBOA_EINVAL, "quantize_layer: %d scales per head exceed the LDS of the group-wise refinement", dh * ng);
            const int pitch = scales + ng <= room ? dh + 1 : dh;      // (an odd pitch: lanes store consecutive groups)
            const int B = (int)std::max<size_t>(1, std::min<size_t>(std::min(CD_ROWS, dh), room / ng - 1));
            const size_t ds = (size_t)B * ng, smem_sums = (size_t)pitch * ng * sizeof(double);
            const int lds = ds + ng + (size_t)ng * ng <= room ? 3 : ds + ng <= room ? 1 : 0;
            const size_t smem = (ds + (lds & 1 ? ng : 0) + (lds & 2 ? (size_t)ng * ng : 0)) * sizeof(double);
            TB_HIP(ctx, hipFuncSetAttribute((const void*)cd_group_sums_kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem_sums));
            TB_HIP(ctx, hipFuncSetAttribute((const void*)cd_group_chain_kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem));
            double* num0 = L.cdnum + (size_t)nh * ng;
            const int shares = (long long)nh * ng < 512 ? 4 : 1;
            for (int it = 0; it < d->cd_iters; ++it)
                for (int j0 = 0; j0 < dh; j0 += B) {
                    const int nj = std::min(B, dh - j0);
                    hipLaunchKernelGGL(cd_group_sums_kernel, dim3(ng, nh, shares), dim3(256), smem_sums, st, L.Fg, L.Cg, L.Ho, dh, ng, j0, nj, pitch, L.s64, num0);
                    hipLaunchKernelGGL(cd_group_chain_kernel, dim3(nh), dim3(1024), smem, st, L.Cg, L.Ho, dh, ng, j0, nj, lds, num0, L.cdnum, L.s64);
                    TB_KERNEL_CHECK(ctx);
                }
        } else {
            const size_t smem = (size_t)4 * ng * sizeof(double);
            hipLaunchKernelGGL(cd_group_diag_kernel, dim3((rows_all + 3) / 4), dim3(256), smem, st, L.Fg, L.Cg, (long long)rows_all, ng,
                               d->cd_iters, L.s64);
        }
        TB_KERNEL_CHECK(ctx);
    } else if (d->cd_iters > 0) {
        // H_in is symmetric and its products only go into symmetric forms: half products A = Wbar T and Z = W T, T + T^T = 2 H_in
        if (rns) TB_TRY(rns_with_h(L.Wbar, L.Abar));
        else {
            TB_TRY(block_gemm(L, dh, n, n, 1.0, L.Wbar, n, L.Hi, 0, n, 1, 0.0, L.Abar, n, TBOA_PROF_F64_CD, &half));
            TB_TRY(block_gemm(L, dh, n, n, 1.0, L.W64, n, L.Hi, 0, n, 1, 0.0, L.Z, n, TBOA_PROF_F64_CD, &half));
        }
        if (H_out) {
            GemmF64 c{};
            c.M = dh; c.N = dh; c.K = n; c.alpha = 1.0; c.beta = 0.0;
            c.A = L.Abar; c.sam = n; c.sak = 1; c.B = L.Wbar; c.sbk = 1; c.sbn = n; c.C = L.Cm; c.ldc = dh;
            c.batch = nh; c.strideA = (long long)dh * n; c.strideB = c.strideA; c.strideC = (long long)dh * dh;
            TB_TRY(gemm_f64(ctx, c));
            // F = Wbar H_in W^T - Wbar (W R)^T = (A W^T + Wbar Z^T) / 2 - Wbar (W R)^T
            c.alpha = 0.5; c.B = L.W64; c.A2 = L.Wbar; c.B2 = L.Z; c.C = L.Fm;
            TB_TRY(gemm_f64(ctx, c));
            if (R) { c.alpha = -1.0; c.beta = 1.0; c.A = L.Wbar; c.B = L.WR; c.A2 = nullptr; c.B2 = nullptr; TB_TRY(gemm_f64(ctx, c)); }
            hipLaunchKernelGGL(cd_head_kernel, dim3(nh), dim3(256), (dh + 8) * sizeof(double), st, L.Fm, L.Cm, L.Ho, dh, d->cd_iters, L.s64);
        } else {
            hipLaunchKernelGGL(cd_row_products_kernel, dim3((rows_all + 3) / 4), dim3(256), 0, st, L.Abar, L.Wbar, L.W64, L.Z, R ? L.WR : nullptr,
                               (long long)rows_all, n, L.dvec, L.dvec + rows_all);
            hipLaunchKernelGGL(cd_diag_kernel, dim3((rows_all + 255) / 256), dim3(256), 0, st, L.dvec + rows_all, L.dvec, rows_all,
                               d->cd_iters, L.s64);
        }
        TB_KERNEL_CHECK(ctx);
    }
    hipLaunchKernelGGL(finalize_kernel, dim3(gx(n), rows_all), dim3(256), 0, st, L.Wbar, L.s64, L.z64, ng, L.gsz, n, L.Q64, W_deq,
                       scales, zeros);
    TB_KERNEL_CHECK(ctx);
    const bool want_loss = loss || loss_per_head;
    if (want_loss) {
        // D = Q - W (into Wbar), D T (into Abar): tr(H_out D H_in D^T) takes the symmetric part of D T D^T
        TB_TRY(launch_sub_f64(ctx, L.Q64, L.W64, L.Wbar, wn));
        if (d->cd_iters > 0 && !d->group) {   // Abar = Wbar T and Z = W T are still those of the scale refinement
            hipLaunchKernelGGL(dh_from_products_kernel, dim3(gx(n), rows_all), dim3(256), 0, st, L.Abar, L.s64, L.Z, n);
            TB_KERNEL_CHECK(ctx);
        } else if (rns) TB_TRY(rns_with_h(L.Wbar, L.Abar));
        else TB_TRY(block_gemm(L, dh, n, n, 1.0, L.Wbar, n, L.Hi, 0, n, 1, 0.0, L.Abar, n, TBOA_PROF_F64_CD, &half));
        double* lq = L.lossbuf; double* lc = L.lossbuf + nh;
        TB_TRY(launch_fill_f64(ctx, L.lossbuf, 2 * nh, 0.0));
        if (H_out) {
            GemmF64 c{};
            c.M = dh; c.N = dh; c.K = n; c.alpha = 1.0; c.beta = 0.0;
            c.A = L.Abar; c.sam = n; c.sak = 1; c.B = L.Wbar; c.sbk = 1; c.sbn = n; c.C = L.Cm; c.ldc = dh;
            c.batch = nh; c.strideA = (long long)dh * n; c.strideB = c.strideA; c.strideC = (long long)dh * dh;
            c.tag = TBOA_PROF_F64_CD;
            TB_TRY(gemm_f64(ctx, c));
            hipLaunchKernelGGL(head_trace_kernel, dim3(nh), dim3(256), 0, st, L.Ho, L.Cm, dh, 1.0, 1, lq);
            if (R) {
                c.A = L.WR; c.B = L.Wbar; c.C = L.Fm;
                TB_TRY(gemm_f64(ctx, c));
                hipLaunchKernelGGL(head_trace_kernel, dim3(nh), dim3(256), 0, st, L.Ho, L.Fm, dh, 2.0, 0, lc);
            }
        } else {
            hipLaunchKernelGGL(rowdot_kernel, dim3((rows_all + 3) / 4), dim3(256), 0, st, L.Abar, (long long)n, L.Wbar, (long long)n,
                               (long long)rows_all, n, L.dvec);
            hipLaunchKernelGGL(head_sum_kernel, dim3(nh), dim3(256), 0, st, L.dvec, dh, 1.0, lq);
            if (R) {
                hipLaunchKernelGGL(rowdot_kernel, dim3((rows_all + 3) / 4), dim3(256), 0, st, L.WR, (long long)n, L.Wbar, (long long)n,
                                   (long long)rows_all, n, L.dvec);
                hipLaunchKernelGGL(head_sum_kernel, dim3(nh), dim3(256), 0, st, L.dvec, dh, 2.0, lc);
            }
        }
        TB_KERNEL_CHECK(ctx);
    }
    // ---- the one place where the call waits for the device: factorisation status, the bookkeeping of the grid search, losses
    TB_TRY(setup_join());      // (a layer with no in-channel sweep at all never joined)
    double* host = nullptr;
    if (want_loss) {
        host = (double*)malloc(2 * (size_t)nh * sizeof(double));
        if (!host) return tboa_fail(ctx, TBOA_ENOMEM, "host buffer");
    }
    hipError_t e = hipMemcpyAsync(ctx->h_status, ctx->d_status, (TB_GSTAT_WORD + GS_WORDS) * sizeof(int), hipMemcpyDeviceToHost, st);
    if (e == hipSuccess && want_loss) e = hipMemcpyAsync(host, L.lossbuf, 2 * (size_t)nh * sizeof(double), hipMemcpyDeviceToHost, st);
    if (e == hipSuccess) e = hipStreamSynchronize(st);
    if (e != hipSuccess) { free(host); return tboa_fail(ctx, TBOA_EHIP, "status and loss copy: %s", hipGetErrorString(e)); }
    for (int slot = 0; slot <= (H_out ? 2 : 0); slot += 2)
        if (ctx->h_status[slot] != 0) {
            free(host);
            return tboa_fail(ctx, TBOA_ENOTSPD, "%s Hessian %d of the batch is not positive definite: pivot %d is not positive",
                             slot ? "out-channel" : "in-channel", ctx->h_status[slot + 1], ctx->h_status[slot] - 1);
        }
    if (L.fast_grid) {
        const int* gs = ctx->h_status + TB_GSTAT_WORD;
        float dev; memcpy(&dev, &gs[GS_MAXDEV], sizeof(float));
        ctx->counters[TBOA_CTR_GRID_SURVIVORS] += gs[GS_SURVIVORS];
        const double guard = d->grid_guard > 0.0 ? d->grid_guard : 0.25;
        // (the guard measures one row in eight at least: where more than that are out of its reach, the approximation is not relied on)
        if (gs[GS_TRIPPED] || 8LL * gs[GS_LOW] > d->d_out) { free(host); return RUN_AGAIN_EXACT; }
        // a cost that its approximation misses by as much as itself (weights that lie on the candidate's grid but for the last bits) is no
        // matter of the bits of H; nor is, with integers, one that it misses by a thousand times what two digits leave out
        const bool delta = grid_delta(d->bits, n);
        if (dev > guard * GRID_TAU) {
            free(host);
            return gs[GS_SHORT] && dev < (delta ? 1.f : 1e-3f) ? RUN_AGAIN_TWO_TERMS : RUN_AGAIN_EXACT;
        }
    }
    if (want_loss) {
        double q = 0.0, c = 0.0;
        for (int h = 0; h < nh; ++h) {
            q += host[h]; c += host[nh + h];
            if (loss_per_head) { loss_per_head[2 * h] = host[h]; loss_per_head[2 * h + 1] = host[nh + h]; }
        }
        if (loss) { loss[0] = q; loss[1] = c; }
        free(host);
        if (!(q == q) || !(c == c)) return tboa_fail(ctx, TBOA_ENAN, "quantize_layer: loss is not finite (non-finite input?)");
    }
    return 0;
}

// right operands that a choice of products needs
struct RnsNeeds { bool hT, rC, uR, uC, uS, pS; };
RnsNeeds rns_needs(int products, bool R) {
    const bool u = R && (products & (RNS_P | RNS_COMP));
    return {(products & (RNS_REFINE | RNS_EXACT)) != 0, R && (products & (RNS_REFINE | RNS_COMP)), u, u, (products & RNS_SWEEP) != 0, R && (products & RNS_SWEEP)};
}

// Which products go to the integer matrix cores: the choice of least modelled time over both forms of every kind and the right operands that it needs (gemm_f64_model_us,
// rns_model_us).  Per-head Hessians keep fp64: their products have the rows of one head, which the preparation of d_in x d_in operands does not repay.
int rns_choice(const Layer& L, bool H_out, bool R) {
    const tboa_layer_desc* d = L.d;
    const int n = L.n, rows = d->d_out;
    if (L.nhin > 1 || n < SWEEP_SP || !rns_takes(8192, n, n)) return 0;
    const int blk = d->block < L.dh ? d->block : L.dh, steps = (L.dh + blk - 1) / blk, step_rows = L.nh * blk;
    const double half = d->group ? 1.0 : 0.5;      // of a product with H_in
    auto fp64 = [](int M, int N, int K) { return 1.15 * gemm_f64_model_us(M, N, K); };      // (one launch among others: 332 us for 2048^3, where the steps alone are 269)
    auto rns = [&](int M, int N, int K, bool tri, bool beta = false) {
        double us = 0.0;
        for (int r = 0; r < M; r += 8192) us += rns_model_us(std::min(8192, M - r), N, K, tri, beta);
        return us;
    };
    double gain[5] = {0.0, 0.0, 0.0, 0.0, 0.0};
    if (R) gain[0] += fp64(rows, n, n) - rns(rows, n, n, false);
    if (d->cd_iters > 0) gain[0] += half * fp64(rows, n, n) - rns(rows, n, n, !d->group);
    if (d->cd_iters > 0 && !d->group) gain[0] += half * fp64(rows, n, n) - rns(rows, n, n, true);
    if (d->cd_iters == 0 || d->group) gain[0] += 0.5 * fp64(rows, n, n) - rns(rows, n, n, !d->group);
    if (L.fast_grid) {      // about one and a half exact costs a row
        const int at_once = std::min(step_rows, L.fast_chunk), m = std::max(1, at_once * 3 / 2);
        gain[1] = (double)steps * step_rows / at_once * (0.5 * fp64(m, n, n) - rns_model_us(m, n, n, true, false));
    }
    if (R && !L.lazy) gain[2] = fp64(n, n, n) - 2.0 * rns(n, n, n, true);
    if (R && H_out) gain[3] = (steps - 1) * (2.0 * fp64(step_rows, n, n) - rns(step_rows, n, n, false) - 2.0 * rns(step_rows, n, n, true));
    const bool whole_groups = !d->group || SWEEP_SP % L.gsz == 0 || L.gsz % SWEEP_SP == 0;
    if (!L.lazy && whole_groups)
        for (int s1 = SWEEP_SP; s1 < n; s1 += SWEEP_SP) gain[4] += steps * (fp64(step_rows, n - s1, (R ? 2 : 1) * SWEEP_SP) - rns(step_rows, n - s1, (R ? 2 : 1) * SWEEP_SP, false, true));
    int best = 0; double most = 150.0;      // us: what the model does not tell apart
    for (int c = 1; c < 32; ++c) {
        if (((c & RNS_P) && (!R || L.lazy)) || ((c & RNS_COMP) && !(R && H_out)) || ((c & RNS_EXACT) && !L.fast_grid) || ((c & RNS_SWEEP) && (L.lazy || !whole_groups))) continue;
        const RnsNeeds need = rns_needs(c, R);
        double g = -(need.hT + need.rC + need.uR + need.uC + need.uS + need.pS) * (rns_prepare_us(n, n) + 8.0);
        for (int k = 0; k < 5; ++k) if (c >> k & 1) g += gain[k];
        if (g > most) { most = g; best = c; }
    }
    return best;
}

// The workspace of a quantize_layer call, carved from `ar` (base == nullptr: only counted).
void plan_layer(Layer& L, bool H_out, bool R, Arena& ar) {
    const tboa_layer_desc* d = L.d;
    const int n = L.n, nh = L.nh, dh = L.dh;
    const int blk = d->block < dh ? d->block : dh;
    const size_t wn = (size_t)d->d_out * n, brows = (size_t)nh * blk;
    const int unit_rows = L.nhin > 1 ? (d->adaptive_grid ? blk : dh) : 1;
    const size_t grows = (size_t)(L.fast_grid ? L.fast_chunk : L.grid_chunk) * unit_rows;
    const bool delta = grid_delta(d->bits, n);
    const size_t np = grid_width(n, delta), mats = L.nhin > 1 ? L.fast_chunk : 1, mat_rows = L.nhin > 1 ? unit_rows : grows;      // of a pass of the two-phase search
    size_t delta_bytes = (size_t)L.grid_chunk * unit_rows * L.ncand * L.gsz * sizeof(double), g_bytes = delta_bytes;
    if (L.fast_grid) {
        const size_t mrows = mats * rows16((long long)mat_rows * L.ncand);
        delta_bytes = std::max(delta_bytes, (delta ? 2 : 1) * mrows * (size_t)grid_pitch((int)np, delta) * sizeof(__half)); g_bytes = std::max(g_bytes, mrows * np * sizeof(float));
    }
    const int fmax = n > dh ? n : dh;
    const int fb = (L.nhin > nh) ? L.nhin : nh;
    const int nblk_f = (fmax + TB_FACT_NB - 1) / TB_FACT_NB;
    L.W64 = ar.get<double>(wn); L.Wt = ar.get<double>(wn); L.Q64 = ar.get<double>(wn);
    L.s64 = ar.get<double>((size_t)d->d_out * L.ng); L.z64 = ar.get<double>((size_t)d->d_out * L.ng);
    L.Hi = ar.get<double>((size_t)L.nhin * L.nn); L.Hfac = ar.get<double>((size_t)L.nhin * L.nn); L.Uin = ar.get<double>((size_t)L.nhin * L.nn);
    L.Rd = R ? ar.get<double>((size_t)L.nhin * L.nn) : nullptr; L.P = R ? ar.get<double>((size_t)L.nhin * L.nn) : nullptr;
    L.Ho = H_out ? ar.get<double>((size_t)nh * dh * dh) : nullptr; L.Hofac = H_out ? ar.get<double>((size_t)nh * dh * dh) : nullptr;
    L.Uout = H_out ? ar.get<double>((size_t)nh * dh * dh) : nullptr;
    // the two factorisations (H_in: nhin matrices of order n; H_out: nh of order dh) share their temporaries
    const size_t t_in = (size_t)L.nhin * n * chol_tmp_pitch(n), t_out = H_out ? (size_t)nh * dh * chol_tmp_pitch(dh) : 0;
    L.ftmp = ar.get<double>(t_in > t_out ? t_in : t_out); L.fdinv = ar.get<double>((size_t)fb * nblk_f * TB_FACT_NB * TB_FACT_NB);
    if (!L.no_rns) chol_rns_plan(n, L.nhin, ar, L.frns);
    else L.frns = CholRns{};
    L.Wb = ar.get<double>(brows * n); L.Wk = ar.get<double>(brows * n);
    L.Epan = ar.get<double>(brows * SWEEP_SP); L.Wsnap = ar.get<double>(brows * SWEEP_SP);
    L.E = H_out ? ar.get<double>(brows * n) : nullptr;
    L.S1 = (H_out && R) ? ar.get<double>(brows * n) : nullptr; L.S2 = (H_out && R) ? ar.get<double>(brows * n) : nullptr;
    // (a group-wise grid is searched on the current columns, which the lazy form does not hold until their turn comes)
    L.lazy = R && !d->group && (L.nhin > 1 ? dh : d->d_out) < n / 2 - SWEEP_SP;
    L.nr = L.lazy ? ar.get<double>(brows * n) : nullptr; L.nv = L.lazy ? ar.get<double>(brows * n) : nullptr;
    L.T = H_out ? ar.get<double>((size_t)nh * dh * d->block) : nullptr;
    L.cand_s = ar.get<double>(grows * L.ncand); L.cand_z = ar.get<double>(grows * L.ncand); L.cost = ar.get<double>(grows * L.ncand);
    L.Delta = ar.get<double>(delta_bytes / sizeof(double) + 1); L.G = ar.get<double>(g_bytes / sizeof(double) + 1);
    L.DeltaS = L.GS = L.costS = nullptr; L.sel = L.list = nullptr; L.Hcat = nullptr;
    if (L.fast_grid) {
        L.DeltaS = ar.get<double>(grows * GRID_KS * n); L.GS = ar.get<double>(grows * GRID_KS * n);
        L.costS = ar.get<double>(grows * GRID_KS); L.sel = ar.get<int>(grows * 3); L.list = ar.get<int>(grows * L.ncand);
        const size_t cols = L.nhin * np;
        L.Hcat = ar.get<__half>((delta ? 2 : 3) * cols * grid_pitch((int)np, delta));
        L.cand_r = ar.get<float>(grows * L.ncand); L.Wf = ar.get<float>(grows * np);
        if (delta) {
            L.gscale.up = ar.get<float>(cols); L.gscale.down = ar.get<double>(cols); L.gscale.dcorr = ar.get<float>(cols);
            L.gscale.off2 = ar.get<double>(cols); L.gscale.scale = ar.get<double>(L.nhin); L.gscale.terms = ar.get<int>(L.nhin);
            L.wdown = ar.get<float>(grows);
        } else {
            L.gint.v = ar.get<double>(cols); L.gint.hd = ar.get<double>(cols); L.gint.v2 = ar.get<double>(cols); L.gint.v3 = ar.get<double>(cols);
            L.gint.e2 = ar.get<double>(cols); L.gint.off2 = ar.get<double>(cols); L.gint.tau = ar.get<double>(L.nhin); L.gint.terms = ar.get<int>(L.nhin);
            const size_t w_rows = mats * rows16(GRID_WD * (long long)mat_rows);
            L.gwt.A = (signed char*)ar.get<__half>(w_rows * grid_pitch((int)np, delta)); L.gwt.wu = ar.get<double>(grows);
            L.gwp = ar.get<int>(3 * w_rows * np); L.gwv = ar.get<double>(grows * np); L.gleast = ar.get<double>(grows);
        }
    }
    L.Wbar = ar.get<double>(wn); L.Abar = ar.get<double>(wn); L.Z = ar.get<double>(wn);
    L.WR = R ? ar.get<double>(wn) : nullptr;
    L.Cm = H_out ? ar.get<double>((size_t)nh * dh * dh) : nullptr; L.Fm = H_out ? ar.get<double>((size_t)nh * dh * dh) : nullptr;
    L.dvec = ar.get<double>(2 * (size_t)d->d_out); L.lossbuf = ar.get<double>(2 * (size_t)nh);
    L.rns = L.no_rns ? 0 : rns_choice(L, H_out, R);
    if (L.rns) {
        const size_t cap = L.fast_grid ? (size_t)L.fast_chunk * GRID_KS : 0;
        auto operand = [&](int rows, int k, bool exps) {
            RnsOperand o{};
            o.kpad = rns_pad(k); o.plane = rns_plane(rows, k); o.p = ar.get<signed char>(TB_RNS_MODULI * o.plane); o.e = exps ? ar.get<int>(rows) : nullptr;
            return o;
        };
        const RnsNeeds need = rns_needs(L.rns, R);
        const bool aux = R && (L.rns & RNS_P);
        L.rns_rows_max = (int)std::max<size_t>((std::min(d->d_out, 8192) + 255) / 256 * 256, (L.rns & RNS_EXACT) ? (cap + 255) / 256 * 256 : 0);
        const int aux_rows = std::min((n + 255) / 256 * 256, L.rns_rows_max);
        if (need.hT) L.hT = operand(n, n, true);
        if (need.rC) L.rC = operand(n, n, true);
        if (need.uR) L.uR = operand(n, n, true);
        if (need.uC) L.uC = operand(n, n, true);
        if (need.uS) L.uS = operand(n, n, true);
        if (need.pS) { L.pS = operand(n, n, false); L.pS.e = L.uS.e; }
        L.left[0] = operand(L.rns_rows_max, std::max(n, 2 * SWEEP_SP), true);
        L.rres[0] = ar.get<unsigned char>(rns_residue_bytes(L.rns_rows_max, n, 1));
        if (aux) { L.left[1] = operand(aux_rows, n, true); L.rres[1] = ar.get<unsigned char>(rns_residue_bytes(aux_rows, n, 1)); }
        L.rsq = ar.get<double>(rns_squares_elems(n)); L.rsq2 = ar.get<double>(rns_squares_elems(n)); L.rpart = ar.get<double>(RNS_CHUNKS * rns_squares_elems(n));
        L.wsq = ar.get<double>(rns_squares_elems(n));
        L.kexp = ar.get<int>(n); L.hexp = ar.get<int>(n); L.rexp = ar.get<int>(n); L.pshift = ar.get<int>(1);
    }
    L.Cg = L.Fg = L.cdnum = nullptr;
    if (d->group && d->cd_iters > 0) {
        const size_t ng = (size_t)L.ng;
        L.Cg = ar.get<double>(H_out ? (size_t)nh * ng * ng * dh * dh : (size_t)d->d_out * ng * ng);
        L.Fg = ar.get<double>(H_out ? (size_t)nh * ng * dh * dh : (size_t)d->d_out * ng);
        L.cdnum = H_out ? ar.get<double>((size_t)nh * ng * (CD_ROWS + 1)) : nullptr;
    }
}

int check_layer_desc(tboa_ctx* ctx, const tboa_layer_desc* d) {
    if (!d) return tboa_fail(ctx, TBOA_EINVAL, "quantize_layer: null descriptor");
    if (d->d_out <= 0 || d->d_in <= 0 || d->n_heads <= 0 || d->d_out % d->n_heads != 0)
        return tboa_fail(ctx, TBOA_EINVAL, "quantize_layer: d_out=%d must be a positive multiple of n_heads=%d", d->d_out, d->n_heads);
    if (!(d->bits == 2 || d->bits == 3 || d->bits == 4 || d->bits == 8)) return tboa_fail(ctx, TBOA_EINVAL, "quantize_layer: bits=%d not in {2,3,4,8}", d->bits);
    if (d->block <= 0) return tboa_fail(ctx, TBOA_EINVAL, "quantize_layer: block must be positive");
    if (d->group < 0 || (d->group > 0 && d->d_in % d->group != 0)) return tboa_fail(ctx, TBOA_EINVAL, "quantize_layer: group=%d must divide d_in=%d", d->group, d->d_in);
    if (d->group > 0 && !(d->group % 64 == 0 || 64 % d->group == 0)) return tboa_fail(ctx, TBOA_EINVAL, "quantize_layer: group=%d must divide or be a multiple of 64", d->group);
    if (d->w_dtype != TBOA_F32 && d->w_dtype != TBOA_BF16) return tboa_fail(ctx, TBOA_EINVAL, "quantize_layer: w_dtype");
    if (d->grid_points <= 0 || !(d->max_shrink > 0.0) || d->max_shrink > 1.0 || d->damp < 0.0 || d->cd_iters < 0 || !(d->grid_guard == d->grid_guard))
        return tboa_fail(ctx, TBOA_EINVAL, "quantize_layer: grid_points/max_shrink/damp/cd_iters/grid_guard out of range");
    return 0;
}

// the quantities of a layer that follow from its descriptor alone
void init_layer(Layer& L, tboa_ctx* ctx, const tboa_layer_desc* d) {
    L.ctx = ctx; L.d = d;
    L.n = d->d_in; L.nh = d->n_heads; L.dh = d->d_out / d->n_heads;
    L.ng = d->group ? d->d_in / d->group : 1; L.gsz = d->group ? d->group : d->d_in;
    L.nhin = d->hin_per_head ? d->n_heads : 1;
    L.ncand = (int)ceil(d->max_shrink * (double)d->grid_points);
    if (L.ncand < 1) L.ncand = 1;
    L.maxq = (double)((1 << d->bits) - 1);
    L.nn = (long long)L.n * L.n;
    const int blk = d->block < L.dh ? d->block : L.dh;
    // grid-search pass size: keep Delta and G near 2 GiB each
    const double cap = 2147483648.0;
    const double per_row = (double)L.ncand * L.gsz * 8.0;
    const int max_rows_block = d->adaptive_grid ? blk : L.dh;
    const int units = L.nhin > 1 ? L.nh : L.nh * max_rows_block;
    const double c = cap / (L.nhin > 1 ? per_row * max_rows_block : per_row);
    L.grid_chunk = c < 1.0 ? 1 : (c > units ? units : (int)c);
    // the two-phase search holds 1 + 4 bytes per entry (codes and products; 4 + 4 with pairs of delta) where the exact one holds 8 + 8: twice the rows in the same buffers
    L.fast_chunk = c < 0.5 ? 1 : (2.0 * c > units ? units : (int)(2.0 * c));
    // per-row grids of wide layers: two-phase search (a negative grid_guard asks for exact costs throughout).  Narrow layers
    // (d_in < 256) keep the exact search: one launch over all candidates, nothing to re-evaluate.  So do steps whose fp64 products take a few
    // microseconds, where a search is 5 launches and not 12.  The line in rows x candidates x d_in^2, a whole step in us, two phases -> exact costs:
    //     2e7 148 -> 111, 8e7 154 -> 121, 3e8 228 -> 198, 7e8 237 -> 221, 1.0e9 252 -> 234, 1.3e9 262 -> 286 (d_in 512), 410 -> 411 (1024), 2.7e9 257 -> 321
    // whatever the rows per head.  Taken below 16 rows a head only, though exact costs would save 10 - 35 us a step up to 1e9 there too (256 columns, 16 rows: 179 -> 146): from 16 rows
    // on the search keeps to two phases at every size, with the counters and the guard that callers of such blocks read and set.
    const bool few = d->adaptive_grid && blk < 16 && (double)L.nh * blk * L.ncand * (double)L.nn <= 1e9;
    L.fast_grid = (!d->group && L.n >= 256 && !few && !(d->grid_guard < 0.0)) ? 1 : 0;
    L.gstat = ctx ? ctx->d_status + TB_GSTAT_WORD : nullptr;
}

size_t layer_bytes(const tboa_layer_desc* d, bool H_out, bool R, bool no_rns) {
    Layer L{};
    init_layer(L, nullptr, d);
    L.no_rns = no_rns;
    Arena ar(nullptr);
    plan_layer(L, H_out, R, ar);
    return ar.off;
}

}  // namespace

extern "C" size_t tboa_quantize_workspace_bytes(const tboa_layer_desc* d, int with_H_out, int with_R) {
    return check_layer_desc(nullptr, d) != 0 ? 0 : layer_bytes(d, with_H_out != 0, with_R != 0, false);
}
extern "C" size_t tboa_quantize_workspace_min_bytes(const tboa_layer_desc* d, int with_H_out, int with_R) {
    return check_layer_desc(nullptr, d) != 0 ? 0 : layer_bytes(d, with_H_out != 0, with_R != 0, true);
}

extern "C" int tboa_quantize_layer(tboa_ctx* ctx, const tboa_layer_desc* d, const void* W, const float* H_in, const float* H_out,
                                   const float* R, uint8_t* codes, float* scales, float* zeros, float* W_deq, double* loss,
                                   double* loss_per_head) {
    if (!ctx) return TBOA_EINVAL;
    if (!d || !W || !H_in || !codes || !scales || !zeros || !W_deq) return tboa_fail(ctx, TBOA_EINVAL, "quantize_layer: null argument");
    TB_TRY(check_layer_desc(ctx, d));
    if (d->hin_per_head && d->n_heads > 1 && !H_out) return tboa_fail(ctx, TBOA_EINVAL, "quantize_layer: per-head H_in needs H_out");

    Layer L{};
    init_layer(L, ctx, d);
    // residues take as much memory again as the fp64 matrices: what fits without them still runs
    bool residues = true;
    TB_TRY(tboa_ws_reserve_either(ctx, layer_bytes(d, H_out != nullptr, R != nullptr, false), layer_bytes(d, H_out != nullptr, R != nullptr, true), residues));
    L.no_rns = !residues;
    Arena ar(ctx->ws);
    plan_layer(L, H_out != nullptr, R != nullptr, ar);
    int rc = run_layer(L, W, H_in, H_out, R, codes, scales, zeros, W_deq, loss, loss_per_head);
    if (rc == RUN_AGAIN_TWO_TERMS) {
        ++ctx->counters[TBOA_CTR_GRID_TWO_TERM_RUNS];
        L.grid_terms = 2;
        rc = run_layer(L, W, H_in, H_out, R, codes, scales, zeros, W_deq, loss, loss_per_head);
    }
    if (rc == RUN_AGAIN_EXACT) {
        // the guard of the two-phase grid search: exact costs for every candidate, same workspace
        ++ctx->counters[TBOA_CTR_GRID_FALLBACKS];
        L.fast_grid = 0;
        rc = run_layer(L, W, H_in, H_out, R, codes, scales, zeros, W_deq, loss, loss_per_head);
    }
    return rc;
}
