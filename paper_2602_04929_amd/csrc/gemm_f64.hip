// fp64 GEMM on the CDNA fp64 matrix cores (v_mfma_f64_16x16x4_f64).
//
// C[b] = alpha * A[b] B[b] + beta * C[b].  A(m,k) = A[m*sam + k*sak], B(k,n) = B[k*sbk + n*sbn] with one unit
// stride per operand, so the four transpose cases share one kernel body; the layout of an operand's LDS tile
// follows its contiguous axis so that global loads are coalesced and LDS reads by 16-lane groups are
// (nearly) conflict-free.  Workgroup: 256 threads = 4 wavefronts; global -> register -> LDS software pipeline with two LDS
// buffers, one barrier per k-step.
//
// One v_mfma_f64_16x16x4 occupies its SIMD for 64 cycles, so a 128 x 128 x 16 step takes a workgroup 1.9 us however little
// else it does: a product of few tiles and a long contraction (K_g^T K_g of a head: one tile, k = 8192) ran at the speed of
// a handful of CUs, 1.4 ms for 8 heads.  Four tile shapes and a split of the contraction spread such products over the
// chip; the choice is a cost model over (tiles, k-steps), see choose():
//   128 x 128 x 16  wavefronts 2 x 2, each 64 x 64 (64 fp64 accumulators per lane): the best rate when there are >= 256 tiles
//    64 x  64 x 32  wavefronts 2 x 2, each 32 x 32
//    32 x  32 x 64  wavefronts 2 x 2, each 16 x 16: the shortest step, for the small updates between latency-bound kernels
//    32 x 128 x 16  wavefronts 1 x 4, each 32 x 32: at most 32 rows per batch entry, bound by reading B once from HBM
// With a split every workgroup leaves its part of the sum in a buffer of the context and splitk_sum_kernel adds the parts in
// a fixed order (the results do not depend on timing).
#include "internal.h"
#include <algorithm>

typedef double v4d __attribute__((ext_vector_type(4)));

namespace {

struct Args {
    int M, N, K;
    double alpha, beta;
    const double* A; long long sa_r, sa_k;
    const double* B; long long sb_k, sb_r;
    double* C; long long ldc;
    long long strideA, strideB, strideC, strideA2, strideB2, strideC2;
    int batch_inner;
    int klo_m, klo_n, khi_m, khi_n, skip_lower, skip_upper, skip_col0, diag_order, by_length;
    const int* m_limit;
    const double* A2; const double* B2;
    int sym;
    double* part; int splits;     // splits > 1 or part given: part[(blockIdx.z)][M, N] receives the raw sum of this split
};

constexpr int tile_pitch_kc(int bk) { return bk + 1; }          // [row][k] tile (k-contiguous operand); odd
constexpr int tile_pitch_mc(int rows) { return rows + 16; }     // [k][row] tile (row-contiguous operand): k and k+1 land 32 of the 64 LDS banks apart
constexpr int tile_elems(bool kc, int rows, int bk) { return kc ? rows * tile_pitch_kc(bk) : bk * tile_pitch_mc(rows); }

// Loads the ROWS x BK tile of an operand whose element (r, k) lives at base[r*s_r + k*s_k].
// KC: s_k == 1 (k-contiguous), else s_r == 1.  Indexes beyond the operand are clamped into it: what a row beyond r_lim adds
// only reaches results that are not stored, and store_tile replaces what lies beyond k_lim by zeros (on the way to LDS, so
// that nothing waits for the loads where they are issued).
template <bool KC, int ROWS, int BK>
__device__ __forceinline__ void load_tile(const double* __restrict__ base, long long s_r, long long s_k,
                                          int r0, int k0, int r_lim, int k_lim, double (&reg)[ROWS * BK / 256]) {
    const int t = threadIdx.x;
#pragma unroll
    for (int p = 0; p < ROWS * BK / 512; ++p) {
        const int idx = t + 256 * p;
        const int r = r0 + (KC ? idx / (BK / 2) : (idx % (ROWS / 2)) * 2), k = k0 + (KC ? (idx % (BK / 2)) * 2 : idx / (ROWS / 2));
        const int ra = min(r, r_lim - 1), ka = min(k, k_lim - 1), rb = KC ? ra : min(r + 1, r_lim - 1), kb = KC ? min(k + 1, k_lim - 1) : ka;
        reg[2 * p] = base[(long long)ra * s_r + (long long)ka * s_k];
        reg[2 * p + 1] = base[(long long)rb * s_r + (long long)kb * s_k];
    }
}

// The same for a tile that lies inside the operand, rows 16-byte aligned: no predicates; p0 as tile_origin gives it for the tile
template <bool KC, int ROWS, int BK>
__device__ __forceinline__ const double* tile_origin(const double* __restrict__ base, long long s_r, long long s_k, int r0, int k0) {
    const int t = threadIdx.x;
    return KC ? base + (long long)(r0 + t / (BK / 2)) * s_r + k0 + (t % (BK / 2)) * 2 : base + (long long)(k0 + t / (ROWS / 2)) * s_k + r0 + (t % (ROWS / 2)) * 2;
}
template <bool KC, int ROWS, int BK>
__device__ __forceinline__ void load_tile_inside(const double* __restrict__ p0, long long s_r, long long s_k, double (&reg)[ROWS * BK / 256]) {
    const long long step = KC ? (256 / (BK / 2)) * s_r : (256 / (ROWS / 2)) * s_k;
#pragma unroll
    for (int p = 0; p < ROWS * BK / 512; ++p) {
        const double2 v = *(const double2*)(p0 + p * step);
        reg[2 * p] = v.x; reg[2 * p + 1] = v.y;
    }
}

template <bool KC, int ROWS, int BK>
__device__ __forceinline__ void store_tile(double* __restrict__ lds, const double (&in)[ROWS * BK / 256], int kvalid = BK) {
    const int t = threadIdx.x;
    double reg[ROWS * BK / 256];
#pragma unroll
    for (int i = 0; i < ROWS * BK / 256; ++i) reg[i] = in[i];
    if (kvalid < BK) {      // contraction indices kvalid .. BK - 1 of the tile do not exist
#pragma unroll
        for (int p = 0; p < ROWS * BK / 512; ++p) {
            const int idx = t + 256 * p, k = KC ? (idx % (BK / 2)) * 2 : idx / (ROWS / 2);
            if (k >= kvalid) reg[2 * p] = 0.0;
            if (k + (KC ? 1 : 0) >= kvalid) reg[2 * p + 1] = 0.0;
        }
    }
#pragma unroll
    for (int p = 0; p < ROWS * BK / 512; ++p) {
        const int idx = t + 256 * p;
        if (KC) {
            const int r = idx / (BK / 2), k = (idx % (BK / 2)) * 2;
            lds[r * tile_pitch_kc(BK) + k] = reg[2 * p]; lds[r * tile_pitch_kc(BK) + k + 1] = reg[2 * p + 1];
        } else {
            const int k = idx / (ROWS / 2), r = (idx % (ROWS / 2)) * 2;
            *(double2*)(lds + k * tile_pitch_mc(ROWS) + r) = make_double2(reg[2 * p], reg[2 * p + 1]);
        }
    }
}

template <bool KC, int ROWS, int BK>
__device__ __forceinline__ double lds_at(const double* __restrict__ lds, int r, int k) {
    return KC ? lds[r * tile_pitch_kc(BK) + k] : lds[k * tile_pitch_mc(ROWS) + r];
}

template <bool AKC, bool BKC, int TM, int TN, int BK>
__global__ __launch_bounds__(256) void gemm_f64_kernel(Args g, bool vecA, bool vecB) {
    constexpr int WM = TM == 32 && TN == 128 ? 1 : 2, WN = 4 / WM;      // wavefronts along the rows / columns of the tile
    constexpr int TI = TM / WM / 16, TJ = TN / WN / 16;                 // 16 x 16 MFMA tiles per wavefront
    __shared__ __attribute__((aligned(16))) double As[2][tile_elems(AKC, TM, BK)];
    __shared__ __attribute__((aligned(16))) double Bs[2][tile_elems(BKC, TN, BK)];

    // Workgroups go to the eight XCDs round-robin by linear number, so with a column count that is a multiple of 8 an XCD
    // always gets the same tile columns; where the contraction length grows with the column (diag_order), the columns of
    // each tile row are rotated by the row number so that every XCD sees all lengths.
    int tx = g.diag_order ? (int)((blockIdx.x + blockIdx.y) % gridDim.x) : (int)blockIdx.x, ty = blockIdx.y, tz = blockIdx.z;
    if (g.by_length) {
        // Few rounds of workgroups: the 256 of a round go to the CUs in the same order, so that a CU got the same tile column, and the same length, in every round (8 x 128 rows,
        // 8192 columns, triangular: 2.0 ms, the time of the whole product).  Longest columns first, every other round backwards: long and short ones meet (1.16 ms).
        const int linear = (int)(blockIdx.x + gridDim.x * (blockIdx.y + gridDim.y * blockIdx.z)), total = (int)(gridDim.x * gridDim.y * gridDim.z), first = linear & ~255;
        const int at = linear & 256 ? first + min(256, total - first) - 1 - (linear - first) : linear;
        const int other = (int)(gridDim.y * gridDim.z), rank = at / other, rest = at % other;
        tx = g.khi_n ? (int)gridDim.x - 1 - rank : rank; ty = rest % (int)gridDim.y; tz = rest / (int)gridDim.y;
    }
    const int m0 = ty * TM, n0 = tx * TN;
    const int bz = tz / g.splits, sp = tz % g.splits;
    if (g.m_limit && m0 >= g.m_limit[bz]) return;
    if (g.skip_lower && g.skip_col0 + n0 + TN <= m0) return;
    if (g.skip_upper && m0 + TM <= g.skip_col0 + n0) return;
    const long long b = bz / g.batch_inner, b2 = bz % g.batch_inner;
    const double* A = g.A + b * g.strideA + b2 * g.strideA2;
    const double* B = g.B + b * g.strideB + b2 * g.strideB2;
    const double* A2 = g.A2 ? g.A2 + b * g.strideA + b2 * g.strideA2 : nullptr;
    const double* B2 = g.A2 ? g.B2 + b * g.strideB + b2 * g.strideB2 : nullptr;
    double* C = g.C + b * g.strideC + b2 * g.strideC2;

    int klo = 0, khi = g.K;
    if (g.klo_m) klo = max(klo, m0);
    if (g.klo_n) klo = max(klo, n0);
    if (g.khi_m) khi = min(khi, m0 + TM);
    if (g.khi_n) khi = min(khi, n0 + TN);
    klo = (klo / BK) * BK;
    if (g.splits > 1) {      // this workgroup's run of k-steps
        const int steps = khi > klo ? (khi - klo + BK - 1) / BK : 0, per = (steps + g.splits - 1) / g.splits;
        const int lo = klo + sp * per * BK;
        khi = min(khi, lo + per * BK); klo = lo;
    }
    // a second run of k-steps: the other pair of operands over the same range, or (sym) the diagonal tile after what lies below it
    int klo2 = klo, khi2 = khi;
    if (g.sym) { klo2 = n0; khi2 = min(khi, n0 + TN); klo = min(khi, n0 + TN); A2 = A; B2 = B; }
    const int nk1 = khi > klo ? (khi - klo + BK - 1) / BK : 0;
    const int nk = A2 ? nk1 + (khi2 > klo2 ? (khi2 - klo2 + BK - 1) / BK : 0) : nk1;

    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int wm = (wave / WN) * (TM / WM), wn = (wave % WN) * (TN / WN);
    const int l16 = lane & 15, lk = lane >> 4;

    v4d acc[TI][TJ];
#pragma unroll
    for (int i = 0; i < TI; ++i)
#pragma unroll
        for (int j = 0; j < TJ; ++j) acc[i][j] = (v4d){0.0, 0.0, 0.0, 0.0};

    double ra[TM * BK / 256], rb[TN * BK / 256];
    auto multiply = [&](int cur) {
#pragma unroll
        for (int k4 = 0; k4 < BK / 4; ++k4) {
            double a[TI], bb[TJ];
#pragma unroll
            for (int i = 0; i < TI; ++i) a[i] = lds_at<AKC, TM, BK>(As[cur], wm + 16 * i + l16, 4 * k4 + lk);
#pragma unroll
            for (int j = 0; j < TJ; ++j) bb[j] = lds_at<BKC, TN, BK>(Bs[cur], wn + 16 * j + l16, 4 * k4 + lk);
#pragma unroll
            for (int i = 0; i < TI; ++i)
#pragma unroll
                for (int j = 0; j < TJ; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[i], bb[j], acc[i][j], 0, 0, 0);
        }
    };
    auto stage = [&](int buf, int kvalid = BK) { store_tile<AKC, TM, BK>(As[buf], ra, kvalid); store_tile<BKC, TN, BK>(Bs[buf], rb, kvalid); };
    auto twice = [&]() {
#pragma unroll
        for (int i = 0; i < TI; ++i)
#pragma unroll
            for (int j = 0; j < TJ; ++j) acc[i][j] *= 2.0;
    };
    const int tail = khi > klo ? (khi - klo) % BK : 0, tail2 = A2 && khi2 > klo2 ? (khi2 - klo2) % BK : 0, nfull = tail ? nk - 1 : nk;
    if (vecA && vecB && m0 + TM <= g.M && n0 + TN <= g.N && nfull > 0 && !(A2 && (tail || tail2))) {
        // every whole k-step of this workgroup lies inside the operands: 16-byte loads, one address per load.  (With the edge
        // loads in the same loop the compiler waits for each of them before the next: 58.6 instead of 66.3 TFLOP/s on 8192^3.)
        const double* pa = nk1 ? tile_origin<AKC, TM, BK>(A, g.sa_r, g.sa_k, m0, klo) : tile_origin<AKC, TM, BK>(A2, g.sa_r, g.sa_k, m0, klo2);
        const double* pb = nk1 ? tile_origin<BKC, TN, BK>(B, g.sb_r, g.sb_k, n0, klo) : tile_origin<BKC, TN, BK>(B2, g.sb_r, g.sb_k, n0, klo2);
        const long long da = AKC ? BK : BK * g.sa_k, db = BKC ? BK : BK * g.sb_k;
        load_tile_inside<AKC, TM, BK>(pa, g.sa_r, g.sa_k, ra);
        load_tile_inside<BKC, TN, BK>(pb, g.sb_r, g.sb_k, rb);
        stage(0);
        __syncthreads();
        for (int kt = 0; kt < nfull - 1; ++kt) {
            pa += da; pb += db;
            if (kt + 1 == nk1) {
                pa = tile_origin<AKC, TM, BK>(A2, g.sa_r, g.sa_k, m0, klo2);
                pb = tile_origin<BKC, TN, BK>(B2, g.sb_r, g.sb_k, n0, klo2);
            }
            load_tile_inside<AKC, TM, BK>(pa, g.sa_r, g.sa_k, ra);
            load_tile_inside<BKC, TN, BK>(pb, g.sb_r, g.sb_k, rb);
            if (g.sym && kt == nk1) twice();
            multiply(kt & 1);
            stage((kt & 1) ^ 1);
            __syncthreads();
        }
        if (tail) {
            load_tile<AKC, TM, BK>(A, g.sa_r, g.sa_k, m0, klo + nfull * BK, g.M, khi, ra);
            load_tile<BKC, TN, BK>(B, g.sb_r, g.sb_k, n0, klo + nfull * BK, g.N, khi, rb);
        }
        if (g.sym && nfull - 1 == nk1) twice();
        multiply((nfull - 1) & 1);
        if (tail) {
            stage(nfull & 1, tail);
            __syncthreads();
            multiply(nfull & 1);
        }
    } else if (nk > 0) {
        int lim = khi;
        auto fetch = [&](int kt) {
            const bool second = kt >= nk1;
            const int k0 = second ? klo2 + (kt - nk1) * BK : klo + kt * BK;
            lim = second ? khi2 : khi;
            load_tile<AKC, TM, BK>(second ? A2 : A, g.sa_r, g.sa_k, m0, k0, g.M, lim, ra);
            load_tile<BKC, TN, BK>(second ? B2 : B, g.sb_r, g.sb_k, n0, k0, g.N, lim, rb);
            lim -= k0;
        };
        fetch(0);
        stage(0, min(BK, lim));
        __syncthreads();
        for (int kt = 0; kt < nk; ++kt) {
            if (kt + 1 < nk) fetch(kt + 1);
            if (g.sym && kt == nk1) twice();
            multiply(kt & 1);
            if (kt + 1 < nk) stage((kt & 1) ^ 1, min(BK, lim));
            __syncthreads();
        }
    }

    // accumulator element v of tile (i, j): row 16 i + lane / 16 + 4 v, column 16 j + lane % 16
    double* P = g.part ? g.part + (long long)tz * g.M * g.N : nullptr;
#pragma unroll
    for (int i = 0; i < TI; ++i)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int row = m0 + wm + 16 * i + lk + 4 * v;
            if (row >= g.M) continue;
#pragma unroll
            for (int j = 0; j < TJ; ++j) {
                const int col = n0 + wn + 16 * j + l16;
                if (col >= g.N) continue;
                if (P) { P[(long long)row * g.N + col] = acc[i][j][v]; continue; }
                double* c = C + (long long)row * g.ldc + col;
                double r = g.alpha * acc[i][j][v];
                if (g.beta != 0.0) r += g.beta * (*c);
                *c = r;
            }
        }
}

// C[b][m, n] = alpha * sum_p part[b P + p][m, n] + beta * C[b][m, n], the parts added in increasing p.  `inner` consecutive results
// (b = outer * inner + i) lie at C + outer * sC1 + i * sC2.
__global__ __launch_bounds__(256) void splitk_sum_kernel(const double* __restrict__ part, int P, int M, int N, int nres, int inner, double alpha, double beta,
                                                         double* __restrict__ C, long long ldc, long long sC1, long long sC2) {
    const long long mn = (long long)M * N, total = mn * nres;
    for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < total; i += (long long)gridDim.x * blockDim.x) {
        const long long b = i / mn, e = i - b * mn;
        const double* p = part + b * P * mn + e;
        double s = 0.0;
        for (int k = 0; k < P; ++k) s += p[k * mn];
        double* c = C + (b / inner) * sC1 + (b % inner) * sC2 + (e / N) * ldc + e % N;
        double r = alpha * s;
        if (beta != 0.0) r += beta * (*c);
        *c = r;
    }
}

enum Shape { S128, S64, S32, SKINNY };
struct Choice { Shape shape; int splits; };
constexpr int TILE_M[4] = {128, 64, 32, 32}, TILE_N[4] = {128, 64, 32, 128}, TILE_K[4] = {16, 32, 64, 16};
// microseconds a workgroup takes for 16 contraction indices, measured on contractions of 2048 and more with 256 - 512 tiles in flight:
// the MFMAs bind the large tile (64 of them per SIMD take 1.8 us), loads, LDS and the barrier have a growing part in the small ones
constexpr double STEP_US[4] = {2.1, 0.78, 0.32, 0.8};

// Tile shape and number of splits of least modelled time: rounds of 256 workgroups, each of the contraction's steps, plus the
// second kernel and the traffic of the parts when there is a split.
// own_rows: C takes A's place, row for row: a workgroup reads all of the rows that it writes and no others, with one column of tiles.
// always_parts: the result goes through the parts whatever the split.
Choice choose(const GemmF64& q, bool akc, size_t part_elems, bool always_parts, bool own_rows, double* modelled = nullptr) {
    const double k16 = std::max(1.0, q.K / 16.0 * (q.A2 ? 2.0 : q.sym ? 0.5 : 1.0));
    const bool no_split = q.skip_lower || q.skip_upper || q.m_limit || q.sym || own_rows;
    Choice best{S128, 1}; double best_us = 1e30;
    for (int s = 0; s < 4; ++s) {
        if (s == SKINNY && !(q.M <= 32 && akc)) continue;
        if (own_rows && q.N > TILE_N[s]) continue;
        if (s != S128 && cdiv64(q.M, TILE_M[s]) > 65535) continue;      // rows of tiles that a launch can have
        const double tiles = (double)cdiv64(q.M, TILE_M[s]) * cdiv64(q.N, TILE_N[s]) * q.batch;
        for (int sp = 1; sp <= (no_split ? 1 : 64); sp *= 2) {
            if (sp > 1 && (q.K / TILE_K[s] < 2 * sp || tiles * sp > 1024)) break;
            const bool parts = sp > 1 || always_parts;
            if (parts && (double)q.M * q.N * q.batch * sp > (double)part_elems) break;
            double us = ceil(tiles * sp / 256.0) * (k16 / sp * STEP_US[s] + 2.0);
            if (parts) us += 5.0 + (double)q.M * q.N * q.batch * sp * 16.0 / 3e6;
            if (us < best_us) { best_us = us; best = Choice{(Shape)s, sp}; }
        }
    }
    if (modelled) *modelled = best_us;
    return best;
}

// [first, last] element of an operand of n1 x n2 elements, strides s1 and s2, in b1 x b2 batch entries, strides t1 and t2
struct Span { const double *lo, *hi; };
Span span_of(const double* p, long long n1, long long s1, long long n2, long long s2, long long b1, long long t1, long long b2, long long t2) {
    Span e{p, p};
    for (long long d : {(n1 - 1) * s1, (n2 - 1) * s2, (b1 - 1) * t1, (b2 - 1) * t2}) (d < 0 ? e.lo : e.hi) += d;
    return e;
}
bool meet(Span a, Span b) { return a.lo <= b.hi && b.lo <= a.hi; }

template <int TM, int TN, int BK>
void launch(tboa_ctx* ctx, dim3 grid, bool akc, bool bkc, const Args& a, bool vecA, bool vecB) {
    if (akc && bkc) hipLaunchKernelGGL((gemm_f64_kernel<true, true, TM, TN, BK>), grid, dim3(256), 0, ctx->stream, a, vecA, vecB);
    else if (akc) hipLaunchKernelGGL((gemm_f64_kernel<true, false, TM, TN, BK>), grid, dim3(256), 0, ctx->stream, a, vecA, vecB);
    else if (bkc) hipLaunchKernelGGL((gemm_f64_kernel<false, true, TM, TN, BK>), grid, dim3(256), 0, ctx->stream, a, vecA, vecB);
    else hipLaunchKernelGGL((gemm_f64_kernel<false, false, TM, TN, BK>), grid, dim3(256), 0, ctx->stream, a, vecA, vecB);
}

}  // namespace

double gemm_f64_model_us(int M, int N, int K) {
    GemmF64 q{};
    q.M = M; q.N = N; q.K = K; q.batch = 1;
    double us = 0.0;
    choose(q, true, TB_SPLITK_ELEMS, false, false, &us);
    return us;
}

int gemm_f64(tboa_ctx* ctx, const GemmF64& q) {
    if (q.M <= 0 || q.N <= 0 || q.batch <= 0) return 0;
    if (q.K < 0 || !q.A || !q.B || !q.C) return tboa_fail(ctx, TBOA_EINVAL, "gemm_f64: null operand or negative K");
    const bool akc = (q.sak == 1), bkc = (q.sbk == 1);
    if (!akc && q.sam != 1) return tboa_fail(ctx, TBOA_EINVAL, "gemm_f64: A needs a unit stride");
    if (!bkc && q.sbn != 1) return tboa_fail(ctx, TBOA_EINVAL, "gemm_f64: B needs a unit stride");
    Args a;
    a.M = q.M; a.N = q.N; a.K = q.K; a.alpha = q.alpha; a.beta = q.beta;
    a.A = q.A; a.sa_r = q.sam; a.sa_k = q.sak;
    a.B = q.B; a.sb_k = q.sbk; a.sb_r = q.sbn;
    a.C = q.C; a.ldc = q.ldc;
    a.strideA = q.strideA; a.strideB = q.strideB; a.strideC = q.strideC;
    a.strideA2 = q.strideA2; a.strideB2 = q.strideB2; a.strideC2 = q.strideC2;
    a.batch_inner = q.batch_inner > 0 ? q.batch_inner : 1;
    a.klo_m = q.klo_m; a.klo_n = q.klo_n; a.khi_m = q.khi_m; a.khi_n = q.khi_n;
    a.A2 = q.A2; a.B2 = q.A2 ? q.B2 : nullptr;
    if (q.A2 && (!q.B2 || q.klo_m || q.klo_n || q.khi_m || q.khi_n)) return tboa_fail(ctx, TBOA_EINVAL, "gemm_f64: a second operand pair needs both operands and an unrestricted contraction");
    if (q.sym && (q.N != q.K || q.A2 || q.klo_m || q.klo_n || q.khi_m || q.khi_n || q.skip_lower || q.skip_upper || q.sum_inner))
        return tboa_fail(ctx, TBOA_EINVAL, "gemm_f64: a symmetric right operand is square and goes with no other restriction");
    a.sym = q.sym;
    a.skip_lower = q.skip_lower; a.skip_upper = q.skip_upper; a.skip_col0 = q.skip_col0; a.m_limit = q.m_limit; a.diag_order = q.diag_order || q.sym;
    // sum_inner: the inner batch entries are terms of one result
    const int sum = q.sum_inner ? a.batch_inner : 1;
    if (q.sum_inner && (q.batch % a.batch_inner || q.skip_lower || q.skip_upper || q.m_limit)) return tboa_fail(ctx, TBOA_EINVAL, "gemm_f64: summed batch entries need whole groups and whole results");
    // 16-byte vector loads need every row start and the tile offsets (even) to stay 16-byte aligned
    const bool vecA = ((uintptr_t)q.A % 16 == 0) && ((uintptr_t)q.A2 % 16 == 0) && (q.strideA % 2 == 0) && (q.strideA2 % 2 == 0) && ((akc ? q.sam : q.sak) % 2 == 0);
    const bool vecB = ((uintptr_t)q.B % 16 == 0) && ((uintptr_t)q.B2 % 16 == 0) && (q.strideB % 2 == 0) && (q.strideB2 % 2 == 0) && ((bkc ? q.sbn : q.sbk) % 2 == 0);
    double* part = ctx->splitk[ctx->stream == ctx->aux ? 1 : 0];
    if (sum > 1 && (!part || (size_t)q.M * q.N * q.batch > TB_SPLITK_ELEMS || q.batch > 65535)) {      // the terms one after the other
        GemmF64 one = q;
        one.sum_inner = 0; one.batch = q.batch / a.batch_inner; one.batch_inner = 1;
        for (int r = 0; r < a.batch_inner; ++r) {
            one.A = q.A + r * q.strideA2; one.B = q.B + r * q.strideB2; one.beta = r ? 1.0 : q.beta;
            TB_TRY(gemm_f64(ctx, one));
        }
        return 0;
    }
    // C over an operand: row for row over A with at most 128 columns any shape of one column of tiles does; otherwise workgroups would overwrite
    // what others have yet to read, and the result goes through the parts; where it does not fit them, as one tile does it (128 x 128, no split)
    const bool over_a = q.over_a || q.C == q.A, over_b = q.over_b || q.C == q.B;
    const bool own_rows = !over_b && q.C == q.A && akc && q.sam == q.ldc && q.K <= q.ldc && q.N <= TILE_N[S128] && q.strideA == q.strideC && q.strideA2 == q.strideC2;
    const bool shared = over_b || (over_a && !own_rows), detour = shared && part && (size_t)q.M * q.N * q.batch <= TB_SPLITK_ELEMS &&
                                                                  !(q.skip_lower || q.skip_upper || q.m_limit);
    const Choice ch = shared && !detour ? Choice{S128, 1} : choose(q, akc, part ? TB_SPLITK_ELEMS : 0, sum > 1 || detour, own_rows);
    const int tm = TILE_M[ch.shape], tn = TILE_N[ch.shape];
    // algorithmic flops of a tagged launch: 2 M N K per batch entry over the contraction range each output tile really has;
    // a launch whose row count comes from device memory (m_limit) is timed but not counted
    ProfRec rec{}; bool timed = false;
    if (ctx->prof_on && q.tag >= 0) {
        double macs = 0.0;
        if (!q.m_limit)
            for (int m0 = 0; m0 < q.M; m0 += tm)
                for (int n0 = 0; n0 < q.N; n0 += tn) {
                    if (q.skip_lower && q.skip_col0 + n0 + tn <= m0) continue;
                    if (q.skip_upper && m0 + tm <= q.skip_col0 + n0) continue;
                    int klo = 0, khi = q.K;
                    if (q.klo_m) klo = std::max(klo, m0);
                    if (q.klo_n || q.sym) klo = std::max(klo, n0);
                    if (q.khi_m) khi = std::min(khi, m0 + tm);
                    if (q.khi_n) khi = std::min(khi, n0 + tn);
                    if (khi > klo) macs += (double)std::min(tm, q.M - m0) * std::min(tn, q.N - n0) * (khi - klo) * (q.A2 ? 2.0 : 1.0);
                }
        TB_TRY(prof_begin(ctx, q.tag, 2.0 * macs * q.batch, rec, timed));
    }
    a.splits = ch.splits;
    a.part = (ch.splits > 1 || sum > 1 || detour) ? part : nullptr;
    dim3 grid((unsigned)cdiv64(q.N, tn), (unsigned)cdiv64(q.M, tm), (unsigned)(q.batch * ch.splits));
    if (grid.y > 65535 || cdiv64(q.batch, 1) * ch.splits > 65535) return tboa_fail(ctx, TBOA_EINVAL, "gemm_f64: grid too large");
    const long long wgs = (long long)grid.x * grid.y * grid.z;
    a.by_length = (q.sym || q.klo_n || q.khi_n) && wgs > 256 && wgs <= 2048;      // (many rounds even out by themselves, and neighbours share operands in the other order)
    switch (ch.shape) {
        case S128: launch<128, 128, 16>(ctx, grid, akc, bkc, a, vecA, vecB); break;
        case S64: launch<64, 64, 32>(ctx, grid, akc, bkc, a, vecA, vecB); break;
        case S32: launch<32, 32, 64>(ctx, grid, akc, bkc, a, vecA, vecB); break;
        default: launch<32, 128, 16>(ctx, grid, true, bkc, a, vecA, vecB);
    }
    TB_KERNEL_CHECK(ctx);
    if (a.part) {
        const int nres = q.batch / sum, inner = sum > 1 ? 1 : a.batch_inner;
        const long long total = (long long)q.M * q.N * nres;
        const long long gb = std::min<long long>((total + 255) / 256, 16384);
        hipLaunchKernelGGL(splitk_sum_kernel, dim3((unsigned)gb), dim3(256), 0, ctx->stream, part, sum * ch.splits, q.M, q.N, nres, inner, q.alpha, q.beta,
                           q.C, (long long)q.ldc, (long long)q.strideC, (long long)q.strideC2);
        TB_KERNEL_CHECK(ctx);
    }
    TB_TRY(prof_end(ctx, rec, timed));
    return 0;
}

extern "C" int tboa_gemm_f64(tboa_ctx* ctx, int M, int N, int K, double alpha,
                             const double* A, int64_t sam, int64_t sak, const double* B, int64_t sbk, int64_t sbn,
                             double beta, double* C, int64_t ldc,
                             int batch, int64_t strideA, int64_t strideB, int64_t strideC) {
    if (!ctx) return TBOA_EINVAL;
    GemmF64 g{};
    g.M = M; g.N = N; g.K = K; g.alpha = alpha; g.beta = beta;
    g.A = A; g.sam = sam; g.sak = sak; g.B = B; g.sbk = sbk; g.sbn = sbn;
    g.C = C; g.ldc = ldc; g.batch = batch; g.strideA = strideA; g.strideB = strideB; g.strideC = strideC;
    if (A && B && C && M > 0 && N > 0 && K > 0 && batch > 0) {
        const Span c = span_of(C, M, ldc, N, 1, batch, strideC, 1, 0);
        g.over_a = meet(c, span_of(A, M, sam, K, sak, batch, strideA, 1, 0));
        g.over_b = meet(c, span_of(B, K, sbk, N, sbn, batch, strideB, 1, 0));
    }
    return gemm_f64(ctx, g);
}
