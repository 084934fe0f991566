// U = Chol(H^-1)^T (eq. 3) without forming H^-1.
//
// With V upper triangular and H = V V^T (the Cholesky factorisation taken from the last index backwards),
// H^-1 = V^-T V^-1, so U = V^-1 is upper triangular with positive diagonal and U^T U = H^-1: by uniqueness of
// the Cholesky factor it is Chol(H^-1)^T.  One blocked factorisation plus one blocked triangular inverse, all in
// fp64: diagonal blocks are factored and inverted inside LDS by one workgroup per matrix, the panel and trailing
// updates are fp64-MFMA GEMMs batched over the matrices (the per-head Hessians of W_V factor in lockstep).
#include "internal.h"
#include <algorithm>

namespace {

constexpr int NB = TB_FACT_NB;

// v / p for positive p, the quotient to an ulp or two, without the scaling steps and branches of a division
__device__ __forceinline__ double over_pivot(double v, double p) {
    const double m = __builtin_amdgcn_frexp_mant(p);
    double r = __builtin_amdgcn_rcp(m);
#pragma unroll
    for (int i = 0; i < 3; ++i) r = __builtin_fma(__builtin_fma(-m, r, 1.0), r, r);
    return ldexp(v, -__builtin_amdgcn_frexp_exp(p)) * (p < INFINITY ? r : 0.0);
}

// status[0] = 1 + column of the first non-positive pivot (0 = fine), status[1] = batch index
//
// Latency-bound (one workgroup per matrix, between the updates of the factorisation): 64 columns that wait for each other.  The block is taken as 4 x 4 tiles of
// 16 x 16.  A tile on the diagonal is factored by one wavefront in registers, lane = column: a column reaches the other lanes by v_readlane, with
// no LDS and no barrier between two steps, on unscaled columns (V[r][r2] -= c[r] c[r2] / pivot), so that no step waits for a square root.  Then one wavefront
// solves for the tiles above it (lane = row), a second for the 16 rows of the inverse (lane = column), both by substitution, and fp64 MFMAs take what
// they found from the tiles left of and above it.
// 55 -> 28 us per 64 x 64 block (the kernel alone on the GPU) against a step with one barrier for every column of the factorisation and of the inverse.
__global__ __launch_bounds__(256) void diag_factor_kernel(double* __restrict__ H, int n, int j0, int bs,
                                                          double* __restrict__ dinv, int blk, int nblk, int* status, int b0) {
    typedef double v4d __attribute__((ext_vector_type(4)));
    constexpr int TP = NB + 1;                                             // odd pitch: 16 rows fall into different banks
    __shared__ double S[NB][TP], W[NB][TP];                                // the block, then V; the right-hand side I, then W = V^-1
    __shared__ __attribute__((aligned(16))) double Q[16][16], dq[16];      // columns of the tile on the diagonal, 1 / its diagonal
    const int b = blockIdx.x, t = threadIdx.x, lane = t & 63, wave = t >> 6, l16 = lane & 15, lk = lane >> 4;
    double* Hb = H + (long long)b * n * n;
    // the upper triangle, mirrored; beyond bs the identity
    for (int i = t; i < NB * NB; i += 256) {
        const int r = i >> 6, c = i & 63;
        W[r][c] = r == c ? 1.0 : 0.0;
        if (r > c) continue;
        const double v = c < bs ? Hb[(long long)(j0 + r) * n + j0 + c] : (r == c ? 1.0 : 0.0);
        S[r][c] = v; if (r < c) S[c][r] = v;
    }
    __syncthreads();
    const int nt = (bs + 15) / 16;
    // H_jj = V V^T, V upper, and V W = I: 16 columns (rows of W) at a time from the last to the first
    for (int q = nt - 1; q >= 0; --q) {
        if (wave == 0) {
            double v[16], piv = 1.0; int bad = -1;
#pragma unroll
            for (int r = 0; r < 16; ++r) v[r] = S[16 * q + r][16 * q + l16];
#pragma unroll
            for (int c = 15; c >= 0; --c) {
                double p = lane_value(v[c], c);
                bad = p > 0.0 || bad >= 0 ? bad : c;
                p = p > 0.0 ? p : 1.0;
                piv = l16 == c ? p : piv;
                const double f = l16 < c ? over_pivot(v[c], p) : 0.0;      // (the tile is symmetric: V[l16][c] = v[c])
#pragma unroll
                for (int r = 0; r < 16; ++r)
                    if (r < c) v[r] = __builtin_fma(-lane_value(v[r], c), f, v[r]);
            }
            if (bad >= 0 && t == 0) { if (atomicCAS(&status[0], 0, 1 + j0 + 16 * q + bad) == 0) status[1] = b0 + b; }
            const double dv = sqrt(piv), di = 1.0 / dv;
            if (lk == 0) {
                dq[l16] = di;
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    v[r] = r < l16 ? v[r] * di : (r == l16 ? dv : 0.0);    // a non-positive pivot leaves 1 on the diagonal
                    S[16 * q + r][16 * q + l16] = v[r]; Q[l16][r] = v[r];
                }
            }
        }
        __syncthreads();
        // x V_qq^T = h for the rows above (first wavefront), V_qq w = e for the columns from this tile's on (second)
        if (wave < 2) {
            const bool in = wave == 0 ? lane < 16 * q : lane >= 16 * q;
            double x[16];
#pragma unroll
            for (int r = 0; r < 16; ++r) x[r] = wave == 0 ? S[lane][16 * q + r] : W[16 * q + r][lane];
#pragma unroll
            for (int c = 15; c >= 0; --c) {
                x[c] *= dq[c];
#pragma unroll
                for (int r = 0; r < 16; ++r)
                    if (r < c) x[r] = __builtin_fma(-Q[c][r], x[c], x[r]);
            }
            if (in) {
#pragma unroll
                for (int r = 0; r < 16; ++r) if (wave == 0) S[lane][16 * q + r] = x[r]; else W[16 * q + r][lane] = x[r];
            }
        }
        __syncthreads();
        // H[i, j] -= V[i, q] V[j, q]^T, i <= j < q, and I[i, j] -= V[i, q] W[q, j], i < q <= j
        const int nh = q * (q + 1) / 2, nw = q * (nt - q);
        for (int e = wave; e < nh + nw; e += 4) {
            const bool sym = e < nh;
            int j = 0, i = sym ? e : (e - nh) % q;
            if (sym) { while (i > j) { i -= j + 1; ++j; } } else j = q + (e - nh) / q;
            v4d x = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                const int k = 16 * q + 4 * s + lk;
                x = __builtin_amdgcn_mfma_f64_16x16x4f64(S[16 * i + l16][k], sym ? S[16 * j + l16][k] : W[k][16 * j + l16], x, 0, 0, 0);
            }
            double (&T)[NB][TP] = sym ? S : W;
#pragma unroll
            for (int k = 0; k < 4; ++k) T[16 * i + lk + 4 * k][16 * j + l16] -= x[k];
        }
        __syncthreads();
    }
    double* D = dinv + ((long long)b * nblk + blk) * NB * NB;
    for (int i = t; i < NB * NB; i += 256) {
        const int r = i >> 6, c = i & 63;
        const bool in = r < bs && c < bs;
        D[i] = in ? W[r][c] : 0.0;
        if (in) Hb[(long long)(j0 + r) * n + j0 + c] = r <= c ? S[r][c] : 0.0;      // lower part of the block becomes zero
    }
}

__global__ void clear_status_kernel(int* status) { if (threadIdx.x < 2) status[threadIdx.x] = 0; }

__global__ void place_diag_inverse_kernel(double* __restrict__ U, int n, const double* __restrict__ dinv, int nblk) {
    const int b = blockIdx.y, blk = blockIdx.x;
    const int j0 = blk * NB, bs = min(NB, n - j0);
    const double* D = dinv + ((long long)b * nblk + blk) * NB * NB;
    double* Ub = U + (long long)b * n * n;
    for (int i = threadIdx.x; i < bs * bs; i += blockDim.x) {
        const int r = i / bs, c = i % bs;
        Ub[(long long)(j0 + r) * n + j0 + c] = D[r * NB + c];
    }
}

__global__ __launch_bounds__(256) void cvt_damp_kernel(const float* __restrict__ H, double* __restrict__ out, int n, double damp) {
    __shared__ double red[256];
    const int b = blockIdx.x, t = threadIdx.x;
    const float* Hb = H + (long long)b * n * n;
    double* Ob = out + (long long)b * n * n;
    double s = 0.0;
    for (int i = t; i < n; i += 256) s += (double)Hb[(long long)i * n + i];
    red[t] = s;
    __syncthreads();
    for (int o = 128; o > 0; o >>= 1) { if (t < o) red[t] += red[t + o]; __syncthreads(); }
    const double add = damp * (red[0] / (double)n);
    for (int i = t; i < n; i += 256) Ob[(long long)i * n + i] = (double)Hb[(long long)i * n + i] + add;
}

__global__ void cvt_offdiag_kernel(const float* __restrict__ H, double* __restrict__ out, int n, long long total) {
    const long long nn = (long long)n * n;
    for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < total; i += (long long)gridDim.x * blockDim.x) {
        const long long e = i % nn;
        const int r = (int)(e / n), c = (int)(e % n);
        if (r != c) out[i] = (double)H[i];
    }
}

// out = (H + H^T) / 2 off the diagonal, exactly H where H is symmetric; grid.x runs over the pairs of 64 x 64 tiles (tr, tc), tr >= tc, that are each
// other's mirror image, grid.z over the matrices
__global__ __launch_bounds__(256) void cvt_symmetric_kernel(const float* __restrict__ H, double* __restrict__ out, int n) {
    __shared__ float lo[64][65], up[64][65];
    const long long base = (long long)blockIdx.z * n * n;
    int tr = (int)((sqrtf(8.f * (float)blockIdx.x + 1.f) - 1.f) * 0.5f);
    while ((long long)(tr + 1) * (tr + 2) / 2 <= (long long)blockIdx.x) ++tr;
    while ((long long)tr * (tr + 1) / 2 > (long long)blockIdx.x) --tr;
    const int r0 = tr * 64, c0 = (int)(blockIdx.x - (long long)tr * (tr + 1) / 2) * 64;
    for (int i = threadIdx.x; i < 64 * 64; i += 256) {
        const int r = i >> 6, c = i & 63;
        lo[r][c] = (r0 + r < n && c0 + c < n) ? H[base + (long long)(r0 + r) * n + c0 + c] : 0.f;
        up[r][c] = (c0 + r < n && r0 + c < n) ? H[base + (long long)(c0 + r) * n + r0 + c] : 0.f;
    }
    __syncthreads();
    for (int i = threadIdx.x; i < 64 * 64; i += 256) {
        const int r = i >> 6, c = i & 63;
        if (r0 + r < n && c0 + c < n) out[base + (long long)(r0 + r) * n + c0 + c] = 0.5 * ((double)lo[r][c] + (double)up[c][r]);
        if (c0 + r < n && r0 + c < n) out[base + (long long)(c0 + r) * n + r0 + c] = 0.5 * ((double)up[r][c] + (double)lo[c][r]);
    }
}

}  // namespace

int launch_f32_to_f64_damp(tboa_ctx* ctx, int n, int batch, const float* H, double damp, double* out) {
    const long long total = (long long)batch * n * n;
    long long g = (total + 255) / 256; if (g > 16384) g = 16384;
    hipLaunchKernelGGL(cvt_offdiag_kernel, dim3((unsigned)g), dim3(256), 0, ctx->stream, H, out, n, total);
    hipLaunchKernelGGL(cvt_damp_kernel, dim3(batch), dim3(256), 0, ctx->stream, H, out, n, damp);
    TB_KERNEL_CHECK(ctx);
    return 0;
}

int launch_symmetric_f64_damp(tboa_ctx* ctx, int n, int batch, const float* H, double damp, double* out) {
    const long long nt = (n + 63) / 64;
    hipLaunchKernelGGL(cvt_symmetric_kernel, dim3((unsigned)(nt * (nt + 1) / 2), 1, batch), dim3(256), 0, ctx->stream, H, out, n);
    hipLaunchKernelGGL(cvt_damp_kernel, dim3(batch), dim3(256), 0, ctx->stream, H, out, n, damp);
    TB_KERNEL_CHECK(ctx);
    return 0;
}

// Two levels of blocking.  Diagonal blocks of NB columns are factored (and inverted) in LDS; an outer block of OB columns
// is finished block by block with updates confined to its own columns, after which ONE update with an OB-deep
// contraction carries it into the rest of the matrix: the large updates are bound by the matrix cores, not by reading
// and writing the trailing matrix once per NB columns.  The inverse is assembled the same way, OB columns at a time.
int chol_status_f64(tboa_ctx* ctx, int status_slot) {
    TB_HIP(ctx, hipMemcpyAsync(ctx->h_status + status_slot, ctx->d_status + status_slot, 2 * sizeof(int), hipMemcpyDeviceToHost, ctx->stream));
    TB_HIP(ctx, hipStreamSynchronize(ctx->stream));
    if (ctx->h_status[status_slot] != 0)
        return tboa_fail(ctx, TBOA_ENOTSPD, "Hessian %d of the batch is not positive definite: pivot %d is not positive",
                         ctx->h_status[status_slot + 1], ctx->h_status[status_slot] - 1);
    return 0;
}

// Order from which (and number of matrices with which) the updates of 512 columns go to the integer matrix cores; the longest of them contract over n - 512 columns.
// Whole factorisations, fp64 -> residues: 2 of 2048 1.99 -> 2.08 ms, 3 2.45 -> 2.37, 8 3.31 -> 3.30; one of 2048 1.81 -> 1.88, 2560 2.45 -> 2.46, 3008 3.20 -> 3.10, 3072 3.21 -> 3.10,
// 3584 4.03 -> 3.81, 4096 4.85 -> 4.44, 8192 19.0 -> 12.4; below 2048 nothing is gained (4 of 1536 1.59 -> 1.67, 16 2.80 -> 2.92; 8 of 2047 3.67 -> 3.57).
static bool chol_rns_pays(int n, int batch) { return n >= 2048 && (long long)n * n * batch >= 3072LL * 3072 && rns_takes(n, TB_FACT_OB, n - TB_FACT_OB); }

// Matrices at a time: 30 bytes of residues per element, 8 GB or 8 matrices (40 of 5120 at once would take another 31 GB beside the 55 of a layer's fp64 matrices)
static int chol_rns_batch(int n, int batch) {
    const int64_t most = std::max<int64_t>(8, (1LL << 28) / ((long long)n * n));
    return (int)cdiv64(batch, cdiv64(batch, most));
}

void chol_rns_plan(int n, int batch, Arena& ar, CholRns& w) {
    w = CholRns{};
    if (!chol_rns_pays(n, batch)) return;
    batch = chol_rns_batch(n, batch);
    auto operand = [&]() {
        RnsOperand o{};
        o.kpad = rns_pad(n); o.plane = rns_plane(n, n); o.stride = (long long)(TB_RNS_MODULI * o.plane); o.p = ar.get<signed char>(TB_RNS_MODULI * o.plane * batch);
        o.e = ar.get<int>((size_t)n * batch); o.e_stride = n;
        return o;
    };
    w.V = operand(); w.U = operand();
    w.res = ar.get<unsigned char>(rns_residue_bytes(n, TB_FACT_OB, batch));
    w.sq = ar.get<double>(rns_squares_elems(n) * batch); w.panel = ar.get<double>(rns_squares_elems(n) * batch);
    w.part = ar.get<double>(RNS_CHUNKS * rns_squares_elems(n) * batch); w.grown = ar.get<int>((size_t)n * batch);
    if (!ar.base) w.V.p = nullptr;
}

// Inside an outer block a diagonal block's columns either receive what all finished columns of the outer block owe them in one update when their turn comes (left), or every finished
// block updates all columns before it.  The second reads and writes the outer block's columns once per 64; the first writes each once, but has one column of tiles: it needs many rows.
// Whole factorisations, second -> first: one matrix of 1000 0.885 -> 0.921 ms, of 1536 1.26 -> 1.28, of 4096 4.40 -> 4.37, of 8192 12.2 -> 11.9; 4 of 1024 0.937 -> 0.931, 8 of 1024
// 1.14 -> 1.07, 16 of 2048 4.97 -> 4.48, 8 of 8192 47.0 -> 44.3.  (Outer blocks of 256 columns instead: 46.0.)
static bool factor_left(int J1, int batch) { return (long long)J1 * batch >= 4096; }

// The columns J0 .. J1 of V: diagonal blocks of NB columns, the panels above them, and their updates of the other columns of the same outer block
static int factor_columns(tboa_ctx* ctx, int n, int batch, double* H, double* dinv, int J0, int J1, int* status, int b0) {
    const int nblk = (n + NB - 1) / NB;
    const long long nn = (long long)n * n, dstride = (long long)nblk * NB * NB;
    const bool left = factor_left(J1, batch);
    for (int blk = (J1 + NB - 1) / NB - 1; blk >= J0 / NB; --blk) {
        const int j0 = blk * NB, bs = (n - j0 < NB) ? n - j0 : NB, j1 = j0 + bs;
        if (left && j1 < J1) {   // H[0:j1, blk] -= V[0:j1, j1:J1] V[blk, j1:J1]^T
            GemmF64 u{};
            u.M = j1; u.N = bs; u.K = J1 - j1; u.alpha = -1.0; u.beta = 1.0;
            u.A = H + j1; u.sam = n; u.sak = 1;
            u.B = H + (long long)j0 * n + j1; u.sbk = 1; u.sbn = n;
            u.C = H + j0; u.ldc = n;
            u.batch = batch; u.strideA = nn; u.strideB = nn; u.strideC = nn;
            TB_TRY(gemm_f64(ctx, u));
        }
        hipLaunchKernelGGL(diag_factor_kernel, dim3(batch), dim3(256), 0, ctx->stream, H, n, j0, bs, dinv, blk, nblk, status, b0);
        TB_KERNEL_CHECK(ctx);
        if (j0 == 0) break;
        // panel: V[0:j0, blk] = H[0:j0, blk] Vinv_jj^T   (in place: one column tile, each workgroup owns its rows)
        GemmF64 p{};
        p.M = j0; p.N = bs; p.K = bs; p.alpha = 1.0; p.beta = 0.0;
        p.A = H + j0; p.sam = n; p.sak = 1;
        p.B = dinv + (long long)blk * NB * NB; p.sbk = 1; p.sbn = NB;
        p.C = H + j0; p.ldc = n;
        p.batch = batch; p.strideA = nn; p.strideB = dstride; p.strideC = nn;
        TB_TRY(gemm_f64(ctx, p));
        if (!left && j0 > J0) {   // inside the outer block: H[0:j0, J0:j0] -= V[0:j0, blk] V[J0:j0, blk]^T  (upper part)
            GemmF64 s{};
            s.M = j0; s.N = j0 - J0; s.K = bs; s.alpha = -1.0; s.beta = 1.0;
            s.A = H + j0; s.sam = n; s.sak = 1;
            s.B = H + (long long)J0 * n + j0; s.sbk = 1; s.sbn = n;
            s.C = H + J0; s.ldc = n; s.skip_lower = 1; s.skip_col0 = J0;
            s.batch = batch; s.strideA = nn; s.strideB = nn; s.strideC = nn;
            TB_TRY(gemm_f64(ctx, s));
        }
    }
    return 0;
}

// The inverses of the diagonal blocks of V of OB columns, U[J0:J1, J0:J1], from those of their NB columns (placed in U): blocks [ob, ob + count) of full width side by side
static int invert_diagonal_blocks(tboa_ctx* ctx, int n, int batch, const double* H, double* U, double* tmp, const double* dinv, int ob, int count) {
    constexpr int OB = TB_FACT_OB;
    const int nblk = (n + NB - 1) / NB, J0 = ob * OB, J1 = std::min(n, J0 + OB), TL = chol_tmp_pitch(n);
    const long long nn = (long long)n * n, dstride = (long long)nblk * NB * NB, step = (long long)OB * (n + 1);
    for (int blk = J0 / NB + 1; blk <= (J1 + NB - 1) / NB - 1; ++blk) {   // U[J0:j0, blk]
        const int j0 = blk * NB, bs = (n - j0 < NB) ? n - j0 : NB, m = j0 - J0;
        GemmF64 a{};   // tmp = U[J0:j0, J0:j0] V[J0:j0, blk]
        a.M = m; a.N = bs; a.K = m; a.alpha = 1.0; a.beta = 0.0;
        a.A = U + (long long)J0 * (n + 1); a.sam = n; a.sak = 1; a.klo_m = 1;
        a.B = H + (long long)J0 * n + j0; a.sbk = n; a.sbn = 1;
        a.C = tmp + (long long)J0 * TL; a.ldc = TL;
        a.batch = batch * count; a.batch_inner = count; a.strideA = nn; a.strideB = nn; a.strideC = (long long)n * TL;
        a.strideA2 = step; a.strideB2 = step; a.strideC2 = (long long)OB * TL;
        TB_TRY(gemm_f64(ctx, a));
        GemmF64 c{};   // U[J0:j0, blk] = -tmp Vinv_jj
        c.M = m; c.N = bs; c.K = bs; c.alpha = -1.0; c.beta = 0.0;
        c.A = tmp + (long long)J0 * TL; c.sam = TL; c.sak = 1;
        c.B = dinv + (long long)blk * NB * NB; c.sbk = NB; c.sbn = 1;
        c.C = U + (long long)J0 * n + j0; c.ldc = n;
        c.batch = batch * count; c.batch_inner = count; c.strideA = (long long)n * TL; c.strideB = dstride; c.strideC = nn;
        c.strideA2 = (long long)OB * TL; c.strideB2 = (long long)(OB / NB) * NB * NB; c.strideC2 = step;
        TB_TRY(gemm_f64(ctx, c));
    }
    return 0;
}

// With products of residues (CholRns).  They take contractions of any length at 100 - 140 TFLOP/s but write and read 15 bytes per result, so that every block of 512 columns gets ONE
// update over all columns behind it (right-looking updates of 512 terms each run no faster than in fp64: 1.15 ms for 8192 x 8192 x 512 either way):
//     V: H[0:J1, J0:J1] -= V[0:J1, J1:n] V[J0:J1, J1:n]^T, the rows of V in residues once, their norms known from H's diagonal
//     U: U[ob, J1:n] = -U[ob, ob] (V[ob, J1:n] U[J1:n, J1:n]), from the last rows up; the columns of U in residues as they grow
static int chol_inv_rns(tboa_ctx* ctx, int n, int batch, double* H, double* U, double* tmp, double* dinv, int* status, int b0, const CholRns& w) {
    constexpr int OB = TB_FACT_OB;
    const int nblk = (n + NB - 1) / NB, nob = (n + OB - 1) / OB, TL = chol_tmp_pitch(n);
    const long long nn = (long long)n * n;
    TB_TRY(rns_diagonal_exps(ctx, n, batch, H, RNS_BITS_A, w.V.e, w.sq, 3LL * n));
    RnsGemm g{};
    g.batch = batch; g.residues = w.res;
    for (int ob = nob - 1; ob >= 0; --ob) {
        const int J0 = ob * OB, J1 = std::min(n, J0 + OB);
        if (J1 < n) {
            g.A = &w.V; g.B = &w.V; g.a_row = 0; g.b_row = J0; g.a_k = g.b_k = J1; g.M = J1; g.N = J1 - J0; g.K = n - J1;
            g.alpha = -1.0; g.beta = 1.0; g.C = H + J0; g.ldc = n; g.strideC = nn;
            TB_TRY(rns_gemm(ctx, g));
        }
        TB_TRY(factor_columns(ctx, n, batch, H, dinv, J0, J1, status, b0));
        if (J0 > 0) {
            RnsSource v{};
            v.a = H + J0; v.ld = n; v.stride = nn; v.kc = 1; v.rows = J0; v.k = J1 - J0;
            TB_TRY(rns_row_guard(ctx, v, batch, RNS_BITS_A, w.V, w.sq, 3LL * n));
            TB_TRY(rns_rows(ctx, v, nullptr, batch, RNS_GIVEN, w.V, J0));
        }
    }
    TB_TRY(launch_fill_f64(ctx, U, (int64_t)batch * nn, 0.0));
    hipLaunchKernelGGL(place_diag_inverse_kernel, dim3(nblk, batch), dim3(256), 0, ctx->stream, U, n, dinv, nblk);
    TB_KERNEL_CHECK(ctx);
    const int whole = n / OB;
    TB_TRY(invert_diagonal_blocks(ctx, n, batch, H, U, tmp, dinv, 0, whole));
    if (whole < nob) TB_TRY(invert_diagonal_blocks(ctx, n, batch, H, U, tmp, dinv, whole, 1));
    for (int ob = nob - 1; ob >= 0; --ob) {
        const int J0 = ob * OB, J1 = std::min(n, J0 + OB), width = J1 - J0;
        if (J1 < n) {
            // tmp = V[ob, J1:n] U[J1:n, J1:n]; transposed room: width x (n - J1) of tmp's n x TL
            g.A = &w.V; g.B = &w.U; g.a_row = J0; g.b_row = J1; g.a_k = g.b_k = J1; g.M = width; g.N = n - J1; g.K = n - J1; g.khi_n = 1;
            g.alpha = 1.0; g.beta = 0.0; g.C = tmp; g.ldc = n - J1; g.strideC = (long long)n * TL;
            TB_TRY(rns_gemm(ctx, g));
            GemmF64 c{};   // U[ob, J1:n] = -U[ob, ob] tmp   (U[ob, ob] upper: k >= row)
            c.M = width; c.N = n - J1; c.K = width; c.alpha = -1.0; c.beta = 0.0; c.klo_m = 1;
            c.A = U + (long long)J0 * (n + 1); c.sam = n; c.sak = 1;
            c.B = tmp; c.sbk = n - J1; c.sbn = 1;
            c.C = U + (long long)J0 * n + J1; c.ldc = n;
            c.batch = batch; c.strideA = nn; c.strideB = (long long)n * TL; c.strideC = nn;
            TB_TRY(gemm_f64(ctx, c));
        }
        if (J0 == 0) break;
        RnsSource p{};      // the new rows, of the columns J0 ..
        p.a = U + (long long)J0 * (n + 1); p.ld = n; p.stride = nn; p.rows = n - J0; p.k = width;
        TB_TRY(rns_norms(ctx, p, batch, w.panel, 3LL * n, w.part));
        TB_TRY(rns_grow(ctx, n - J0, batch, w.panel, 3LL * n, w.sq + J0, n, 3LL * n, width, RNS_BITS_B, w.U.e + J0, n, w.grown + J0));
        RnsOperand u = w.U;
        u.p += (long long)(J0 >> 4) * u.kpad * 16; u.e += J0;
        p.k = n - J0;
        TB_TRY(rns_columns(ctx, p, batch, u, J0, w.grown + J0, width));
    }
    return 0;
}

int chol_inv_upper_f64(tboa_ctx* ctx, int n, int batch, double* H, double* U, double* tmp, double* dinv, int status_slot, bool defer_status, const CholRns* rns) {
    int* status = ctx->d_status + status_slot;
    constexpr int OB = TB_FACT_OB;
    const int nblk = (n + NB - 1) / NB, nob = (n + OB - 1) / OB;
    const int TL = chol_tmp_pitch(n);     // row pitch of tmp: a matrix of one outer block only ever holds NB columns there
    const long long nn = (long long)n * n;
    hipLaunchKernelGGL(clear_status_kernel, dim3(1), dim3(64), 0, ctx->stream, status);
    TB_KERNEL_CHECK(ctx);
    if (rns && rns->V.p) {
        for (int b0 = 0, per = chol_rns_batch(n, batch); b0 < batch; b0 += per)
            TB_TRY(chol_inv_rns(ctx, n, std::min(per, batch - b0), H + b0 * nn, U + b0 * nn, tmp + (long long)b0 * n * TL, dinv + (long long)b0 * nblk * NB * NB, status, b0, *rns));
        return defer_status ? 0 : chol_status_f64(ctx, status_slot);
    }
    // ---- H = V V^T from the last column to the first
    for (int ob = nob - 1; ob >= 0; --ob) {
        const int J0 = ob * OB, J1 = (J0 + OB < n) ? J0 + OB : n;
        TB_TRY(factor_columns(ctx, n, batch, H, dinv, J0, J1, status, 0));
        if (J0 > 0) {   // H[0:J0, 0:J0] -= V[0:J0, ob] V[0:J0, ob]^T  (upper part)
            GemmF64 s{};
            s.M = J0; s.N = J0; s.K = J1 - J0; s.alpha = -1.0; s.beta = 1.0;
            s.A = H + J0; s.sam = n; s.sak = 1;
            s.B = H + J0; s.sbk = 1; s.sbn = n;
            s.C = H; s.ldc = n; s.skip_lower = 1;
            s.batch = batch; s.strideA = nn; s.strideB = nn; s.strideC = nn;
            TB_TRY(gemm_f64(ctx, s));
        }
    }
    // ---- U = V^-1
    TB_TRY(launch_fill_f64(ctx, U, (int64_t)batch * nn, 0.0));
    hipLaunchKernelGGL(place_diag_inverse_kernel, dim3(nblk, batch), dim3(256), 0, ctx->stream, U, n, dinv, nblk);
    TB_KERNEL_CHECK(ctx);
    const int whole = n / OB;
    if (whole > 0) TB_TRY(invert_diagonal_blocks(ctx, n, batch, H, U, tmp, dinv, 0, whole));
    if (whole < nob) TB_TRY(invert_diagonal_blocks(ctx, n, batch, H, U, tmp, dinv, whole, 1));
    for (int ob = 1; ob < nob; ++ob) {
        const int J0 = ob * OB, J1 = (J0 + OB < n) ? J0 + OB : n, w = J1 - J0;
        GemmF64 a{};   // tmp = U[0:J0, 0:J0] V[0:J0, ob]
        a.M = J0; a.N = w; a.K = J0; a.alpha = 1.0; a.beta = 0.0;
        a.A = U; a.sam = n; a.sak = 1; a.klo_m = 1;
        a.B = H + J0; a.sbk = n; a.sbn = 1;
        a.C = tmp; a.ldc = TL;
        a.batch = batch; a.strideA = nn; a.strideB = nn; a.strideC = (long long)n * TL;
        TB_TRY(gemm_f64(ctx, a));
        GemmF64 c{};   // U[0:J0, ob] = -tmp U[ob, ob]   (U[ob, ob] upper: k <= column)
        c.M = J0; c.N = w; c.K = w; c.alpha = -1.0; c.beta = 0.0;
        c.A = tmp; c.sam = TL; c.sak = 1;
        c.B = U + (long long)J0 * n + J0; c.sbk = n; c.sbn = 1; c.khi_n = 1;
        c.C = U + J0; c.ldc = n;
        c.batch = batch; c.strideA = (long long)n * TL; c.strideB = nn; c.strideC = nn;
        TB_TRY(gemm_f64(ctx, c));
    }
    return defer_status ? 0 : chol_status_f64(ctx, status_slot);
}

extern "C" int tboa_chol_inv_upper(tboa_ctx* ctx, int n, int batch, const float* H, double damp, double* U) {
    if (!ctx) return TBOA_EINVAL;
    if (n <= 0 || batch <= 0 || !H || !U) return tboa_fail(ctx, TBOA_EINVAL, "chol_inv_upper: bad arguments");
    const int nblk = (n + NB - 1) / NB;
    bool residues = true;
    for (int pass = 0; pass < 2; ++pass) {
        Arena ar(pass ? ctx->ws : nullptr);
        double* H64 = ar.get<double>((size_t)batch * n * n);
        double* tmp = ar.get<double>((size_t)batch * n * chol_tmp_pitch(n));
        double* dinv = ar.get<double>((size_t)batch * nblk * NB * NB);
        const size_t plain = ar.off;
        CholRns rns{};
        if (residues) chol_rns_plan(n, batch, ar, rns);
        if (!pass) { TB_TRY(tboa_ws_reserve_either(ctx, ar.off, plain, residues)); continue; }      // what fits without residues still runs
        TB_TRY(launch_f32_to_f64_damp(ctx, n, batch, H, damp, H64));
        TB_TRY(chol_inv_upper_f64(ctx, n, batch, H64, U, tmp, dinv, 0, false, &rns));
    }
    return 0;
}

// ------------------------------------------------------------------------------------------------
// The same factorisation for callers that cannot allocate: its three temporaries (the fp64 copy of H that becomes V,
// the panel buffer of the triangular inverse, the inverted diagonal blocks) live in a file-scope device array instead
// of the context's workspace.  Every GPU the library runs on holds its own copy of the array until the process ends;
// its address on a device is looked up once, by tboa_create with that device current.  All calls on one GPU share the
// array: two calls that overlap in time on the same GPU (different streams, different host threads) race.
namespace {
constexpr size_t STATIC_REGION = (size_t)1 << 20;                    // doubles per temporary: 8 MiB
__device__ __align__(256) double scratch[3 * STATIC_REGION];         // 24 MiB
constexpr int MAX_DEVICES = 64;
double* scratch_on_device[MAX_DEVICES];                              // device address of `scratch`, per device (0 = not looked up)
}  // namespace

int chol_static_init(int device) {
    if (device < 0 || device >= MAX_DEVICES) return TBOA_EINVAL;
    if (scratch_on_device[device]) return 0;
    double* p = nullptr;
    if (hipGetSymbolAddress((void**)&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) { (void)hipGetLastError(); return TBOA_EHIP; }
    scratch_on_device[device] = p;
    return 0;
}

extern "C" size_t tboa_chol_inv_upper_static_max_elems(void) { return STATIC_REGION; }

extern "C" int tboa_chol_inv_upper_static(tboa_ctx* ctx, int n, int batch, const float* H, double damp, double* U) {
    if (!ctx) return TBOA_EINVAL;
    if (n <= 0 || batch <= 0 || !H || !U) return tboa_fail(ctx, TBOA_EINVAL, "chol_inv_upper_static: bad arguments");
    const size_t n64 = (size_t)((n + NB - 1) / NB) * NB;
    if (n > TB_FACT_OB || (size_t)batch * n64 * n64 > STATIC_REGION)
        return tboa_fail(ctx, TBOA_EINVAL, "chol_inv_upper_static: n = %d, batch = %d exceed the static scratch (n <= %d and "
                         "batch * roundup64(n)^2 <= %zu); use tboa_chol_inv_upper", n, batch, TB_FACT_OB, STATIC_REGION);
    double* base = (ctx->device >= 0 && ctx->device < MAX_DEVICES) ? scratch_on_device[ctx->device] : nullptr;
    if (!base) return tboa_fail(ctx, TBOA_EHIP, "chol_inv_upper_static: the static scratch of device %d was not found at tboa_create", ctx->device);
    // H64: batch n^2; tmp: batch n 64 (one outer block: chol_tmp_pitch(n) = 64); dinv: batch ceil(n / 64) 64^2 -- each within a region
    double* H64 = base; double* tmp = base + STATIC_REGION; double* dinv = base + 2 * STATIC_REGION;
    TB_TRY(launch_f32_to_f64_damp(ctx, n, batch, H, damp, H64));
    return chol_inv_upper_f64(ctx, n, batch, H64, U, tmp, dinv);
}
