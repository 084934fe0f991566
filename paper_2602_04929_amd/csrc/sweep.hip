// Algorithm 3 (in-channel sweep) over a group of up to SWEEP_SP columns of the rows of a step, in fp64.
//
// Column j of a row is quantized when every earlier column has been taken from it:
//     q_j = clamp(round(w_j / s) + z), e_j = (w_j - s (q_j - z)) / U[j, j],  w_k -= e_j U[j, k] + w_j P[j, k]  for k > j.
// The chain through the columns bounds it: what a step needs from the one before.  A workgroup takes 16 rows through the whole group, in
// sub-panels of 16 columns, with two kinds of wavefronts, one of each on a SIMD:
//   four walk the columns.  16 lanes hold the columns of a row's sub-panel, four rows per wavefront, and hand column j to the others by the DPP operand of the
//     fused multiply-add itself (row_newbcast).  A step is a chain of five instructions: the row is divided by its step s once per sub-panel (decided
//     afterwards for all columns: a sub-panel with a column within rounding of a half-integer is walked again with the division of each column), U's rows are
//     divided by their diagonal beforehand, and what only the results need (codes, e_j) is formed after the walk, one column per lane.  The same steps
//     gather what they take from the next sub-panel's columns, which needs no exchange.
//   four apply the sub-panel before to the columns beyond, kept in LDS, by v_mfma_f64_16x16x4.
// One barrier per sub-panel, which takes 1.1 us where little lies beyond it and 3.4 us with 480 columns beyond, where walk and products take turns on the fp64
// pipe of a SIMD: a group of 512 columns 88 us (16 to 2048 rows), 256 columns 29 us.  Before, a launch per 64 columns (21 us: readlane broadcasts, two rows a
// wavefront) and a product for the rest of the group after it: 330 and 110 us.
#include "internal.h"
#include <type_traits>

typedef double v4d __attribute__((ext_vector_type(4)));

namespace {

constexpr int SUB = 16;

// What a lane of a walking wavefront knows, in units of the row's step: its column, -v of the lazy form, and what the walk takes from the next sub-panel's
struct Walk { double w, v, a, b; };

struct Pieces { double u0[SUB][SUB], u1[SUB][SUB], p0[SUB][SUB], p1[SUB][SUB], ud[SUB], ui[SUB]; };      // -U / its diagonal and -P, nothing on or left of the diagonal; ud: the diagonal, ui: 1 / ud

// four steps' pieces, read from LDS while the four steps before them run (all sixteen at once do not fit the registers)
template <int MODE> struct Four {
    double u0[4], u1[4], p0[4], p1[4];
    __device__ __forceinline__ void load(const Pieces& pc, int j0, int l) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            u0[i] = pc.u0[j0 + i][l]; u1[i] = pc.u1[j0 + i][l];
            if (MODE) { p0[i] = pc.p0[j0 + i][l]; p1[i] = pc.p1[j0 + i][l]; }
        }
    }
};
// Column J of the four rows.  Every lane quantizes its own column; what lane J has is taken from the others (whose pieces are zero up to column J).
template <int MODE, int J>
__device__ __forceinline__ void walk_step(Walk& k, const Four<MODE>& f, double ujj, double lo, double hi) {
    const double wj = MODE == 2 ? __builtin_fma(k.v, ujj, k.w) : k.w;
    const double d = k.w - fmin(fmax(rint(wj), lo), hi);      // lazy: e_j U[j, j] less the part of v that column j itself carries
    // (the value of lane J) x piece, added up.  A value that crosses lanes must have been written two instructions earlier at least: wj was (d follows from it
    // through three instructions), d is by the order here
#define TB_DPP " row_newbcast:%c[j] row_mask:0xf bank_mask:0xf\n\t"
    if (MODE == 0)
        asm("s_nop 1\n\tv_fmac_f64_dpp %[w], %[d], %[u0]" TB_DPP "v_fmac_f64_dpp %[a], %[d], %[u1]" TB_DPP
            : [w] "+&v"(k.w), [a] "+&v"(k.a) : [d] "v"(d), [u0] "v"(f.u0[J % 4]), [u1] "v"(f.u1[J % 4]), [j] "n"(J));
    if (MODE == 1)
        asm("v_fmac_f64_dpp %[a], %[w], %[p1]" TB_DPP "v_fmac_f64_dpp %[w], %[w], %[p0]" TB_DPP "v_fmac_f64_dpp %[w], %[d], %[u0]" TB_DPP "v_fmac_f64_dpp %[a], %[d], %[u1]" TB_DPP
            : [w] "+&v"(k.w), [a] "+&v"(k.a) : [d] "v"(d), [u0] "v"(f.u0[J % 4]), [u1] "v"(f.u1[J % 4]), [p0] "v"(f.p0[J % 4]), [p1] "v"(f.p1[J % 4]), [j] "n"(J));
    if (MODE == 2)
        asm("v_fmac_f64_dpp %[b], %[x], %[p1]" TB_DPP "v_fmac_f64_dpp %[v], %[x], %[p0]" TB_DPP "v_fmac_f64_dpp %[w], %[d], %[u0]" TB_DPP "v_fmac_f64_dpp %[a], %[d], %[u1]" TB_DPP
            : [w] "+&v"(k.w), [a] "+&v"(k.a), [v] "+&v"(k.v), [b] "+&v"(k.b)
            : [x] "v"(wj), [d] "v"(d), [u0] "v"(f.u0[J % 4]), [u1] "v"(f.u1[J % 4]), [p0] "v"(f.p0[J % 4]), [p1] "v"(f.p1[J % 4]), [j] "n"(J));
#undef TB_DPP
    if constexpr (J % 4 < 3) walk_step<MODE, J + 1>(k, f, ujj, lo, hi);
}
template <int MODE, class F>
__device__ __forceinline__ void walk(Walk& k, const Pieces& pc, int l, double ujj, double lo, double hi, F beside) {
    Four<MODE> x, y;
    x.load(pc, 0, l); y.load(pc, 4, l);
    __builtin_amdgcn_sched_barrier(0);
    walk_step<MODE, 0>(k, x, ujj, lo, hi);
    beside();      // independent work for the gaps of the chain
    __builtin_amdgcn_sched_barrier(0);
    x.load(pc, 8, l);
    walk_step<MODE, 4>(k, y, ujj, lo, hi);
    __builtin_amdgcn_sched_barrier(0);
    y.load(pc, 12, l);
    walk_step<MODE, 8>(k, x, ujj, lo, hi);
    __builtin_amdgcn_sched_barrier(0);
    walk_step<MODE, 12>(k, y, ujj, lo, hi);
}

// The same walk not divided by the row's step s, with the quotient w / s where that decides a code.  Columns up to j are left alone by a condition and not
// by zero pieces: an undefined or infinite column (which always comes here) touches later ones only
template <int MODE>
__device__ __forceinline__ void walk_dividing(Walk& k, const Pieces& pc, int l, double s, double lo, double hi) {
#pragma unroll 1
    for (int j = 0; j < SUB; ++j) {
        const int from = (threadIdx.x & 48) + j;
        const double x = __shfl(k.w, from), y = MODE == 2 ? __shfl(k.v, from) : 0.0, wj = MODE == 2 ? __builtin_fma(y, pc.ud[j], x) : x;
        const double d = x - s * fmin(fmax(rint(wj / s), lo), hi);
        const bool later = l > j;
        if (MODE == 1) { k.a = __builtin_fma(wj, pc.p1[j][l], k.a); k.w = later ? __builtin_fma(wj, pc.p0[j][l], k.w) : k.w; }
        if (MODE == 2) { k.b = __builtin_fma(wj, pc.p1[j][l], k.b); k.v = later ? __builtin_fma(wj, pc.p0[j][l], k.v) : k.v; }
        k.w = later ? __builtin_fma(d, pc.u0[j][l], k.w) : k.w; k.a = __builtin_fma(d, pc.u1[j][l], k.a);
    }
}

// MODE 0: no deviation term; 1: through P; 2 (lazy): through S = R U^T in P's place, nv holding -v (see run_layer).
// Grid: (tiles of 16 block rows, heads if each has its own U, else 1).
template <int MODE>
__global__ __launch_bounds__(512) void sweep_kernel(SweepArgs a, int rows_per_tile_set, int pitch) {
    extern __shared__ double sh[];
    double* Wl = sh;                                              // [16][pitch]: the group's columns of the 16 rows
    double* Nl = Wl + (MODE == 2 ? 16 * pitch : 0);               // the same of nv
    double* Es = Nl + 16 * pitch;                                 // [2][16][17]: e of a sub-panel
    double* Ss = Es + 2 * 16 * 17;                                // [2][16][17]: the columns as they were quantized
    Pieces* pc = (Pieces*)(Ss + 2 * 16 * 17);                     // [2]
    const int h = blockIdx.y, n = a.n, c0 = a.c0, width = a.width, np = (width + SUB - 1) / SUB;
    const double* U = a.U + (a.per_head ? (long long)h * n * n : 0) + (long long)c0 * n + c0;
    const double* P = MODE ? a.P + (a.per_head ? (long long)h * n * n : 0) + (long long)c0 * n + c0 : nullptr;
    const int t = threadIdx.x, lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6), l = lane & 15, g = lane >> 4;
    const int r0 = blockIdx.x * 16, rbase = h * rows_per_tile_set;
    auto block_row = [&](int r) { return rbase + min(r0 + r, rows_per_tile_set - 1); };
    for (int i = t; i < 16 * np * SUB; i += 512) {
        const int r = i / (np * SUB), c = i - r * (np * SUB);
        const long long o = (long long)block_row(r) * n + c0 + min(c, width - 1);
        Wl[r * pitch + c] = c < width ? a.Wk[o] : 0.0;
        if (MODE == 2) Nl[r * pitch + c] = c < width ? a.nv[o] : 0.0;
    }
    // pieces of sub-panel p: thread (k, l) of 256 takes row k, columns l and 16 + l; in two halves so that the loads are in flight meanwhile
    double raw[5];
    auto fetch = [&](int p, int k, int col) {
        const int kr = min(SUB * p + k, width - 1), ca = min(SUB * p + col, width - 1), cb = min(SUB * p + SUB + col, width - 1);
        const double* u = U + (long long)kr * n;
        raw[0] = u[ca]; raw[1] = u[cb]; raw[4] = u[kr];
        if (MODE) { const double* q = P + (long long)kr * n; raw[2] = q[ca]; raw[3] = q[cb]; }
    };
    auto place = [&](int p, int k, int col) {
        Pieces& o = pc[p & 1];
        const bool row = SUB * p + k < width, in0 = row && col > k && SUB * p + col < width, in1 = row && SUB * p + SUB + col < width;
        const double inv = 1.0 / raw[4];
        o.u0[k][col] = in0 ? -raw[0] * inv : 0.0; o.u1[k][col] = in1 ? -raw[1] * inv : 0.0;
        if (MODE) { o.p0[k][col] = in0 ? -raw[2] : 0.0; o.p1[k][col] = in1 ? -raw[3] : 0.0; }
        if (col == k) { o.ud[k] = row ? raw[4] : 1.0; o.ui[k] = row ? inv : 1.0; }
    };
    if (wave < 4) {
        const int row = 4 * wave + g;                                // of this lane
        const int R = block_row(row);
        const long long lr = layer_row(a.map, R);
        int next_grid = 0;                                           // sub-panel at which the next grid begins
        double s = 1.0, si = 1.0, z = 0.0, ca = 0.0, cb = 0.0;       // ca, cb: what the walk of the sub-panel before takes from this one
        const long long eo = (long long)R * a.epitch + l, qo = lr * n + c0 + l;
        double *to_e = a.Epan + eo, *to_s = a.Wsnap + eo, *to_q = a.Q + qo;
        uint8_t* to_c = a.codes + qo;
        const double *at_w = Wl + row * pitch + l, *at_v = Nl + row * pitch + l;
        fetch(0, t >> 4, l);
        place(0, t >> 4, l);
        fetch(1, t >> 4, l);      // (rows and columns beyond the group are clamped into it)
        asm volatile("" : : "v"(raw[0]), "v"(raw[1]), "v"(raw[4]));
        if (MODE) asm volatile("" : : "v"(raw[2]), "v"(raw[3]));
        __syncthreads();
        // Rows of the tile that do not exist repeat the last one, results included.  Only the last sub-panel can have columns that do not exist: nothing is
        // conditional in the loop over the whole ones, so that a wait for the loads of pieces does not become one for the stores after them
        auto sub_panel = [&](int p, bool whole) {
            const Pieces& pp = pc[p & 1];
            if (p == next_grid) {
                const int gi = (c0 + SUB * p) / a.gsz;
                next_grid = ((gi + 1) * a.gsz - c0) / SUB;
                s = a.s[lr * a.ng + gi]; z = a.z[lr * a.ng + gi]; si = 1.0 / s;
                asm volatile("" : : "v"(si), "v"(z));      // waits here, not in every sub-panel
            }
            const double lo = -z, hi = a.maxq - z;
            const double w0 = at_w[SUB * p] + ca, v0 = MODE == 2 ? at_v[SUB * p] + cb : 0.0;
            const double ujj = pp.ud[l];
            Walk k{w0 * si, v0 * si, 0.0, 0.0};
            walk<MODE>(k, pp, l, ujj, lo, hi, [&]() { place(p + 1, t >> 4, l); });
            fetch(p + 2, t >> 4, l);
            // column l of the row as it stood at its turn: no later step changes it
            double tt = MODE == 2 ? __builtin_fma(k.v, ujj, k.w) : k.w, r = rint(tt), wv, vv;
            if (__any(!(0.5 - fabs(tt - r) > fabs(tt) * 1e-15))) {
                // some quotient rounds to a half-integer as far as the product with 1 / s (within 4 ulp of it) can tell
                k = Walk{w0, v0, 0.0, 0.0};
                walk_dividing<MODE>(k, pp, l, s, lo, hi);
                vv = k.v; ca = k.a; cb = k.b;
                wv = MODE == 2 ? __builtin_fma(vv, ujj, k.w) : k.w;
                r = rint(wv / s);
            } else { vv = k.v * s; ca = k.a * s; cb = k.b * s; wv = tt * s; }
            const double q = fmin(fmax(r, lo), hi), Qj = s * q, d = wv - Qj, uinv = pp.ui[l], e0 = d * uinv;
            double e = __builtin_fma(__builtin_fma(-e0, ujj, d), uinv, e0);      // d / ujj
            if (MODE == 2) e -= vv;
            Es[(p & 1) * 272 + row * 17 + l] = e;
            if (MODE) Ss[(p & 1) * 272 + row * 17 + l] = wv;
            __syncthreads();
            if (whole || SUB * p + l < width) {
                to_e[SUB * p] = e;
                if (MODE) to_s[SUB * p] = wv;
                to_c[SUB * p] = (uint8_t)(q + z);
                to_q[SUB * p] = Qj;
            }
        };
        const int nwhole = width / SUB;
        for (int p = 0; p < nwhole; ++p) sub_panel(p, true);
        if (nwhole < np) sub_panel(nwhole, false);
        return;
    }
    // applying wavefronts: wavefront fw takes sub-panel p - 1 out of the tiles p + 1 + fw + 4 i (i = 0, 1, ..) while sub-panel p is walked.  The fragments of U
    // and P of all of its tiles are loaded a sub-panel ahead, each as soon as the one before it is used up.  The number of tiles M falls by one every four
    // sub-panels and is a constant of each of the loops below: nothing in a loop is conditional, so the compiler knows which loads are in flight and waits for
    // the oldest only (with a branch around a tile it waits for all of them, 1 us per tile).
    const int fw = wave - 4;
    constexpr int SLOTS = (SWEEP_SP / SUB + 1) / 4;
    double bu[SLOTS][4], bp[SLOTS][4];
    auto fragments = [&](int i, int p, int tile) {
        const int col = min(SUB * tile + l, width - 1);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const long long o = (long long)(SUB * p + 4 * q + g) * n + col;
            bu[i][q] = U[o];
            if (MODE) bp[i][q] = P[o];
        }
    };
    double *at_w = Wl + g * pitch + l, *at_v = Nl + g * pitch + l;
    v4d acc, acn;      // columns of the next tile
    auto columns = [&](int tile) {
#pragma unroll
        for (int v = 0; v < 4; ++v) { acc[v] = at_w[4 * v * pitch + SUB * tile]; if (MODE == 2) acn[v] = at_v[4 * v * pitch + SUB * tile]; }
    };
    auto tiles = [&](int p) { return (np + 2 - p - fw) / 4; };      // of wavefront fw when sub-panel p is walked
    if (np > 1) {
#pragma unroll
        for (int i = 0; i < SLOTS; ++i) fragments(i, 0, 2 + fw + 4 * i);
    }
    __syncthreads();
    __syncthreads();      // sub-panel 0
    int p = 1;
    auto apply = [&](auto count) {
        constexpr int M = decltype(count)::value;
        for (; p < np && tiles(p) == M; ++p) {
            if constexpr (M > 0) {
                const double* E = Es + ((p - 1) & 1) * 272; const double* S = Ss + ((p - 1) & 1) * 272;
                double ae[4], as[4];
#pragma unroll
                for (int q = 0; q < 4; ++q) { ae[q] = -E[l * 17 + 4 * q + g]; if (MODE) as[q] = -S[l * 17 + 4 * q + g]; }
                columns(p + 1 + fw);
#pragma unroll
                for (int i = 0; i < M; ++i) {
                    const int tile = p + 1 + fw + 4 * i;
                    const v4d cur = acc, cun = acn;
                    if (i + 1 < M) columns(tile + 4);
                    v4d o = cur, on = cun;
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        o = __builtin_amdgcn_mfma_f64_16x16x4f64(ae[q], bu[i][q], o, 0, 0, 0);
                        if (MODE == 1) o = __builtin_amdgcn_mfma_f64_16x16x4f64(as[q], bp[i][q], o, 0, 0, 0);
                        if (MODE == 2) on = __builtin_amdgcn_mfma_f64_16x16x4f64(as[q], bp[i][q], on, 0, 0, 0);
                    }
#pragma unroll
                    for (int v = 0; v < 4; ++v) { at_w[4 * v * pitch + SUB * tile] = o[v]; if (MODE == 2) at_v[4 * v * pitch + SUB * tile] = on[v]; }
                    fragments(i, p, tile + 1);
                }
            }
            __syncthreads();
        }
    };
    using std::integral_constant;
    apply(integral_constant<int, 8>()); apply(integral_constant<int, 7>()); apply(integral_constant<int, 6>()); apply(integral_constant<int, 5>());
    apply(integral_constant<int, 4>()); apply(integral_constant<int, 3>()); apply(integral_constant<int, 2>()); apply(integral_constant<int, 1>());
    apply(integral_constant<int, 0>());
}

}  // namespace

int launch_sweep(tboa_ctx* ctx, const SweepArgs& a, int nh, bool lazy) {
    const int np = (a.width + SUB - 1) / SUB, mode = !a.P ? 0 : lazy ? 2 : 1;
    const int pitch = SUB * (np + 1 + (np & 1));      // an odd multiple of 128 bytes: rows 0 and 1 of a 16 x 16 tile lie in different LDS banks
    const size_t smem = ((size_t)(mode == 2 ? 32 : 16) * pitch + 4 * 16 * 17) * sizeof(double) + 2 * sizeof(Pieces);
    const int set = a.per_head ? a.nbr : a.nbr * nh;
    const dim3 grid((unsigned)((set + 15) / 16), a.per_head ? nh : 1);
    void (*kern)(SweepArgs, int, int) = mode == 0 ? sweep_kernel<0> : mode == 1 ? sweep_kernel<1> : sweep_kernel<2>;
    TB_HIP(ctx, hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem));
    hipLaunchKernelGGL(kern, grid, dim3(512), smem, ctx->stream, a, set, pitch);
    TB_KERNEL_CHECK(ctx);
    return 0;
}
