// fp64 products as products of residues on the integer matrix cores (v_mfma_i32_32x32x32_i8).
//
// The fp64 matrix cores give 66 TFLOP/s; signed bytes run at 2.6 POP/s.  A row a of the left operand and a row b of the right one (C = A B^T) are scaled by powers of
// two and rounded to integers with |a| <= 2^57, |b| <= 2^58 (2-norms), so that their product is an integer below 2^115 (Cauchy-Schwarz) and is known from its residues
// modulo 15 coprime numbers of 8 bits whose product is 2^116.8 (the Chinese remainder theorem; the scheme is that of Ozaki, Uchino and Imamura, "Ozaki Scheme II: A
// GEMM-oriented emulation of floating-point matrix multiplication using an integer modular technique", 2025).  Each residue of C is one exact product of bytes.
//
// Error.  The sums are exact, what is rounded is the operands: half a unit an entry at most, 0.29 as root mean square, with norms of 2^56 and 2^57 units at least.  C is off by
// 0.32 - 0.65 x 2^-57 |a| |b| (root mean square, by where the norms lie within their powers of two) and 0.75 sqrt(K) 2^-56 |a| |b| at most, plus the rounding of the result.  An fp64 product rounds every partial sum: 0.3 x 2^-53 |a| |b| over terms of random sign whatever
// their number, more where they have one sign.
// What the error is measured against are norms, not sum |a_k b_k|: contractions over channels of very different size take the sizes out by powers of two per channel, half of
// them on either side (rns_channel_exps), and what no product reads does not count in a norm (RnsSource::before).
//
//   rns_rows, rns_columns  powers of two of the rows, residues: one plane of signed bytes per modulus in the blocks of 16 rows x 64 bytes that the product copies into LDS
//   rns_gemm_kernel        one output tile through all (or some) moduli per workgroup
//   rns_result_kernel      residues of C -> alpha C + beta C0
#include "internal.h"
#include <algorithm>

namespace {

typedef int i32x4 __attribute__((ext_vector_type(4)));
typedef int i32x16 __attribute__((ext_vector_type(16)));

constexpr int NMAX = TB_RNS_MODULI;
// coprime: 237 = 3 79, 235 = 5 47, 221 = 13 17, 217 = 7 31, 209 = 11 19, 256 = 2^8, the others prime.  None but 256 above 239: see the epilogue of rns_gemm_kernel
constexpr int MODULI[NMAX] = {256, 239, 237, 235, 233, 229, 227, 223, 221, 217, 211, 209, 199, 197, 193};
constexpr int BM = 256, BN = 256, SK = 64, NS = 4;      // output tile; bytes of the contraction per stage; stages in the LDS ring
constexpr int STAGE_BYTES = (BM + BN) * SK;
constexpr int KPAD = SK * NS;                           // contraction lengths and limits are whole turns of the ring
constexpr int UNDEFINED = 0x7fffffff;                   // exponent of a row that holds an infinity or NaN
constexpr int NOTHING = -(1 << 28);                     // and of one that is zero: smaller than any other

// Sums of squares in three ranges, so that squares neither overflow nor vanish: entries beyond 2^400, below 2^-400, and the others
struct Squares { double mid = 0.0, big = 0.0, tiny = 0.0; };
constexpr double HUGE_ENTRY = 0x1p400, TINY_ENTRY = 0x1p-400, DOWN = 0x1p-600, UP = 0x1p600;
__device__ __forceinline__ void add_square(Squares& s, double v) {
    const double a = fabs(v);
    const bool b = a > HUGE_ENTRY, t = a < TINY_ENTRY;
    const double w = v * (b ? DOWN : t ? UP : 1.0), q = w * w;
    s.mid += b || t ? 0.0 : q; s.big += b ? q : 0.0; s.tiny += t ? q : 0.0;      // (an undefined entry is none of the two)
}

// what an element that is stored as v counts, and its power of two
__device__ __forceinline__ double counted(const RnsSource& s, double v, int r, int k) {
    if (s.half) v = k > r ? 0.0 : k < r ? v + v : v;
    if (s.before && k >= r - r % s.before) v = 0.0;
    return v;
}
__device__ __forceinline__ int power(const RnsSource& s, int k, int shift) { return s.kexp ? shift + s.ksign * s.kexp[k] : shift; }
__device__ __forceinline__ double scaled(const RnsSource& s, double v, int r, int k, int shift) {
    v = counted(s, v, r, k);
    return (s.kexp || s.exp_shift) ? ldexp(v, power(s, k, shift)) : v;
}
__device__ __forceinline__ int shift_of(const RnsSource& s) { return s.exp_shift ? s.ksign * s.exp_shift[0] : 0; }

// row-contiguous source: blockIdx.y takes a share of the contraction, part[chunks][3][rows]
__global__ __launch_bounds__(256) void rns_col_squares_kernel(RnsSource s, int per, double* __restrict__ part, long long part_stride) {
    const int r = blockIdx.x * 256 + threadIdx.x, k0 = blockIdx.y * per, k1 = min(s.k, k0 + per);
    if (r >= s.rows) return;
    const double* a = s.a + blockIdx.z * s.stride + r;
    const int shift = shift_of(s);
    Squares q;
    for (int k = k0; k < k1; ++k) add_square(q, scaled(s, a[(long long)k * s.ld], r, k, shift));
    double* p = part + blockIdx.z * part_stride + 3LL * blockIdx.y * s.rows + r;
    p[0] = q.mid; p[s.rows] = q.big; p[2 * s.rows] = q.tiny;
}
__global__ __launch_bounds__(256) void rns_sum_squares_kernel(int rows, int chunks, const double* __restrict__ part, long long part_stride, double* __restrict__ out, long long out_stride) {
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i >= 3 * rows) return;
    const double* p = part + blockIdx.z * part_stride + i;
    double* o = out + blockIdx.z * out_stride + i;
    double v = 0.0;
    for (int c = 0; c < chunks; ++c) v += p[3LL * c * rows];
    *o = v;
}

// e with sqrt(sum of squares) < 2^(e + bits)
__device__ __forceinline__ int row_exponent(double mid, double big, double tiny, int bits) {
    if (!(mid + big + tiny < INFINITY)) return UNDEFINED;
    double v = mid + tiny * DOWN * DOWN; int e = 0;
    if (big > 0.0) { v = big + mid * DOWN * DOWN; e = 600; }
    else if (mid == 0.0) { v = tiny; e = -600; }
    return v > 0.0 ? (ilogb(v) >> 1) + 1 + e - bits : NOTHING;
}
__global__ __launch_bounds__(256) void rns_exps_kernel(int rows, const double* __restrict__ sq, long long sq_stride, int bits, int* __restrict__ e, long long e_stride) {
    const int r = blockIdx.x * 256 + threadIdx.x;
    if (r >= rows) return;
    const double* p = sq + blockIdx.z * sq_stride + r;
    e[blockIdx.z * e_stride + r] = row_exponent(p[0], p[rows], p[2 * rows], bits);
}

// size[k]: half the exponent of H_kk, the size of channel k
__global__ __launch_bounds__(256) void rns_channel_sizes_kernel(const double* __restrict__ H, int n, int* __restrict__ size) {
    const int k = blockIdx.x * 256 + threadIdx.x;
    if (k >= n) return;
    const double v = H[(long long)k * n + k];
    size[k] = v > 0.0 && v < INFINITY ? ilogb(v) >> 1 : v == 0.0 ? NOTHING : 0;
}
// Powers of two for a contraction over channels k between a weight's columns (sq: their squares in the three ranges) and rows of size 2^right[k]: the right operand times 2^x[k] and the
// left one times 2^-x[k] are of one size in every channel, where |a| |b| is least and next to sum |a_k b_k|.  Later rows and columns of a layer also carry what compensation for the
// others has added, which goes with 1 / 2^size[k], the channel's size: a column counts as no less than 2^-6 of the root mean square of column x size, over its own size.
// (Weights falling from 1e2 to 1e-2 as the channels grow from 1e-2 to 1e2: 2^-55 of sum |w h| instead of 2^-48, from 1e4 and 1e-4: 2^-55 instead of 2^-36; fp64 products 2^-51 - 2^-54.)
// One workgroup: n words in, n words out.
__global__ __launch_bounds__(1024) void rns_channel_exps_kernel(int n, const double* __restrict__ sq, const int* __restrict__ size, const int* right, int* x) {      // (right may be x)
    __shared__ double red[16];
    __shared__ int top_s;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    auto left_of = [&](int k) {
        const double m = sq[k], b = sq[n + k], t = sq[2LL * n + k];
        const int e = row_exponent(m, b, t, 0);
        return e != UNDEFINED ? e : NOTHING;
    };
    if (threadIdx.x == 0) top_s = NOTHING;
    __syncthreads();
    int top = NOTHING;
    for (int k = threadIdx.x; k < n; k += 1024) { const int l = left_of(k); if (l != NOTHING && size[k] != NOTHING) top = max(top, l + size[k]); }
    atomicMax(&top_s, top);
    __syncthreads();
    top = top_s;
    double sum = 0.0;
    for (int k = threadIdx.x; k < n; k += 1024) { const int l = left_of(k); if (l != NOTHING && size[k] != NOTHING) sum += ldexp(1.0, 2 * (l + size[k] - top)); }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) sum += __shfl_xor(sum, o, 64);
    if (lane == 0) red[wave] = sum;
    __syncthreads();
    sum = 0.0;
    for (int w = 0; w < 16; ++w) sum += red[w];
    const int least = top == NOTHING ? NOTHING : top + (ilogb(sum / n) >> 1) - 6;
    for (int k = threadIdx.x; k < n; k += 1024) {
        const int r = right[k], l = top == NOTHING || size[k] == NOTHING ? left_of(k) : max(left_of(k), least - size[k]);
        // (a channel that is zero on the right must not count on the left, whatever its size there)
        x[k] = r == NOTHING ? 900 : l == NOTHING || r == UNDEFINED ? 0 : min(max((l - r) >> 1, -900), 900);
    }
}

// Two pairs of operands of one product, A1 B1 + A2 B2, share the powers of two of their rows: B2 times 2^f (A2 times 2^-f), which brings its Frobenius norm to that of B1, so
// that neither product is rounded in units of the other's operands.  sq1 <- sum of squares of the rows of [B1 | 2^f B2]
__global__ __launch_bounds__(1024) void rns_balance_kernel(int rows, double* __restrict__ sq1, const double* __restrict__ sq2, int* __restrict__ f_out) {
    __shared__ double red[6][16];
    __shared__ int f_s;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    double t[6] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
    for (int r = threadIdx.x; r < rows; r += 1024)
        for (int c = 0; c < 3; ++c) { t[c] += sq1[(long long)c * rows + r]; t[3 + c] += sq2[(long long)c * rows + r]; }
#pragma unroll
    for (int c = 0; c < 6; ++c) {
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) t[c] += __shfl_xor(t[c], o, 64);
        if (lane == 0) red[c][wave] = t[c];
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int c = 0; c < 6; ++c) { t[c] = 0.0; for (int w = 0; w < 16; ++w) t[c] += red[c][w]; }
        const int e1 = row_exponent(t[0], t[1], t[2], 0), e2 = row_exponent(t[3], t[4], t[5], 0);
        const bool none = e1 == UNDEFINED || e2 == UNDEFINED || t[0] + t[1] + t[2] == 0.0 || t[3] + t[4] + t[5] == 0.0;
        f_s = none ? 0 : e1 - e2;
        f_out[0] = f_s;
    }
    __syncthreads();
    const int f = f_s;
    for (int r = threadIdx.x; r < rows; r += 1024) {
        double v[3];
        for (int c = 0; c < 3; ++c) v[c] = sq2[(long long)c * rows + r];
        // the three ranges of the second operand's squares, moved by 2 f, into those of the first
        for (int c = 0; c < 3; ++c) {
            if (v[c] == 0.0) continue;
            if (!(v[c] < INFINITY)) { sq1[r] = v[c]; continue; }
            const int e = ilogb(v[c]) + (c == 1 ? 1200 : c == 2 ? -1200 : 0) + 2 * f;      // of the moved square
            const int to = e > 800 ? 1 : e < -800 ? 2 : 0;
            sq1[(long long)to * rows + r] += ldexp(v[c], 2 * f + (c == 1 ? 1200 : c == 2 ? -1200 : 0) - (to == 1 ? 1200 : to == 2 ? -1200 : 0));
        }
    }
}

// Columns that are completed panel by panel: sq += the panel's squares; a column that has outgrown its power of two gets one with room for twice its norm, and is marked
__global__ __launch_bounds__(256) void rns_grow_kernel(int rows, const double* __restrict__ panel, long long panel_stride, double* __restrict__ sq, int sq_rows, long long sq_stride, int fresh_below,
                                                       int bits, int* __restrict__ e, long long e_stride, int* __restrict__ grown) {
    const int r = blockIdx.x * 256 + threadIdx.x;
    if (r >= rows) return;
    const double* p = panel + blockIdx.z * panel_stride + r;
    double* q = sq + blockIdx.z * sq_stride + r;
    const bool fresh = r < fresh_below;      // the panel's own columns begin here
    double v[3];
    for (int c = 0; c < 3; ++c) { v[c] = p[(long long)c * rows] + (fresh ? 0.0 : q[(long long)c * sq_rows]); q[(long long)c * sq_rows] = v[c]; }
    int* ep = e + blockIdx.z * e_stride + r;
    const int now = row_exponent(v[0], v[1], v[2], bits), had = *ep;
    const bool more = fresh || now > had;      // (UNDEFINED is the largest)
    if (more) *ep = fresh || now == UNDEFINED ? now : now + 1;
    grown[blockIdx.z * e_stride + r] = more && !fresh;
}
// powers of two of the rows of V, H = V V^T: a row's norm is the root of H's diagonal entry.  None for an entry that is not positive; sum: nothing so far.
// (An infinite entry makes the damping and with it the whole diagonal infinite: V then has nothing beside its diagonal, as in fp64)
__global__ __launch_bounds__(256) void rns_diagonal_exps_kernel(int n, const double* __restrict__ H, long long stride, int bits, int* __restrict__ e, double* __restrict__ sum, long long sum_stride) {
    const int r = blockIdx.x * 256 + threadIdx.x;
    if (r >= n) return;
    const double v = H[blockIdx.z * stride + (long long)r * (n + 1)];
    e[blockIdx.z * (long long)n + r] = !(v > 0.0) ? UNDEFINED : v < INFINITY ? row_exponent(v, 0.0, 0.0, bits) : 0;
    sum[blockIdx.z * sum_stride + r] = 0.0;
}
// The norms above are those of a positive definite H only.  A row whose squares so far (a wavefront sums those of the panel, in units of its power of two) are more than twice as many
// as H's diagonal entry allows, or undefined, no longer fits its residues: it is marked undefined, so that its own pivot is, as the negative one would be that fp64 products leave.
// Rows up to twice too long are held exactly (|a| |b| <= 2^115) and their pivots come out negative.
__global__ __launch_bounds__(256) void rns_row_guard_kernel(RnsSource s, int bits, int* __restrict__ e, long long e_stride, double* __restrict__ sum, long long sum_stride) {
    const int lane = threadIdx.x & 63, r = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (r >= s.rows) return;
    int* er = e + blockIdx.z * e_stride + r;
    if (*er == UNDEFINED) return;
    const double* a = s.a + blockIdx.z * s.stride + (long long)r * s.ld;
    const int down = -*er - bits;
    double q = 0.0;
    for (int k = lane; k < s.k; k += 64) { const double v = ldexp(a[k], down); q = __builtin_fma(v, v, q); }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) q += __shfl_xor(q, o, 64);
    if (lane == 0) {
        double* sr = sum + blockIdx.z * sum_stride + r;
        q += *sr; *sr = q;
        if (!(q <= 2.0)) *er = UNDEFINED;
    }
}

struct Moduli { float inv[NMAX]; int m[NMAX]; };
struct Residue { double inv[NMAX], c[NMAX]; int m[NMAX], ci[NMAX]; };      // c = 2^29 mod m, centred

// Residues of 16 consecutive elements of a row, scaled and rounded: one 16-byte piece of every plane.  The integers have up to 58 bits: x = h 2^29 + l, and x mod m from
// y = h (2^29 mod m) + l, 37 bits, so that the quotient is off by nothing that matters.  Of y - quotient m only the low byte is wanted: 32-bit integers do.
__device__ __forceinline__ void store_residues(const double (&x)[16], const Residue& q, signed char* __restrict__ o, long long plane) {
    constexpr double MAGIC = 0x1.8p52;
    double h[16], l[16];
    int hi[16], li[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) { h[i] = rint(x[i] * 0x1p-29); l[i] = __builtin_fma(h[i], -0x1p29, x[i]); hi[i] = (int)h[i]; li[i] = (int)l[i]; }
#pragma unroll
    for (int p = 0; p < NMAX; ++p) {
        unsigned w[4];
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            unsigned b[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int i = 4 * g + j;
                const int n = __double2loint(__builtin_fma(__builtin_fma(h[i], q.c[p], l[i]), q.inv[p], MAGIC));
                b[j] = (unsigned)(__mul24(hi[i], q.ci[p]) + li[i] - __mul24(n, q.m[p]));      // (24 bits of the factors: the low byte is right)
            }
            const unsigned lo = __builtin_amdgcn_perm(b[1], b[0], 0x0c0c0400), up = __builtin_amdgcn_perm(b[3], b[2], 0x0c0c0400);
            w[g] = lo | (up << 16);
        }
        *(uint4*)(o + p * plane) = make_uint4(w[0], w[1], w[2], w[3]);
    }
}

// Row-contiguous source, exponents given: a wavefront makes one block of 16 rows x 64 contraction indices of every plane.  Bound by memory: 8 bytes read and 15 written per
// element, 8192 x 8192 in 0.35 ms.
__global__ __launch_bounds__(256) void rns_columns_kernel(RnsSource s, const int* __restrict__ exps, long long e_stride, Residue q, signed char* __restrict__ out,
                                                          long long plane, long long out_stride, int kpad, int koff, int kblocks, const int* __restrict__ grown, int kpanel) {
    const int lane = threadIdx.x & 63, kb = blockIdx.x * 4 + (threadIdx.x >> 6), r0 = blockIdx.y * 16;
    if (kb >= kblocks) return;
    if (grown && kb >= kpanel && !__any(r0 + (lane & 15) < s.rows && grown[blockIdx.z * e_stride + r0 + (lane & 15)])) return;      // beyond the panel only rows of a new power of two
    const int ri = lane & 15, piece = lane >> 4, r = r0 + ri, k0 = kb * SK + 16 * piece, shift = shift_of(s);
    const double* a = s.a + blockIdx.z * s.stride + r;
    const int e = r < s.rows ? exps[blockIdx.z * e_stride + r] : UNDEFINED;
    double x[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) x[i] = e != UNDEFINED && k0 + i < s.k ? a[(long long)(k0 + i) * s.ld] : 0.0;
#pragma unroll
    for (int i = 0; i < 16; ++i) x[i] = e != UNDEFINED && k0 + i < s.k ? rint(ldexp(counted(s, x[i], r, k0 + i), power(s, k0 + i, shift - e))) : 0.0;
    store_residues(x, q, out + blockIdx.z * out_stride + ((long long)(r0 >> 4) * (kpad >> 6) + (koff >> 6) + kb) * 1024 + ri * 64 + ((piece ^ (ri >> 2)) << 4), plane);
}

// Exponents of rows whose elements are contiguous, over one or two sources: a wavefront per row
__global__ __launch_bounds__(256) void rns_row_exps_kernel(RnsSource s0, RnsSource s1, int two, int bits, int* __restrict__ exps, long long e_stride) {
    const int lane = threadIdx.x & 63, r = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (r >= s0.rows || (s0.row_limit && r >= s0.row_limit[0])) return;
    Squares t;
    for (int u = 0; u <= two; ++u) {
        const RnsSource& s = u ? s1 : s0;
        const double* a = s.a + blockIdx.z * s.stride + (long long)r * s.ld;
        const int shift = shift_of(s), kend = s.half ? min(s.k, r + 1) : s.k;
        int k = lane;
        for (; k + 7 * 64 < kend; k += 512) {      // eight loads in flight
            double v[8]; int p[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) { v[i] = a[k + 64 * i]; p[i] = power(s, k + 64 * i, shift); }
#pragma unroll
            for (int i = 0; i < 8; ++i) add_square(t, ldexp(counted(s, v[i], r, k + 64 * i), p[i]));
        }
        for (; k < kend; k += 64) add_square(t, scaled(s, a[k], r, k, shift));
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) { t.mid += __shfl_xor(t.mid, o, 64); t.big += __shfl_xor(t.big, o, 64); t.tiny += __shfl_xor(t.tiny, o, 64); }
    if (lane == 0) exps[blockIdx.z * e_stride + r] = row_exponent(t.mid, t.big, t.tiny, bits);
}

// Residues of rows whose elements are contiguous, one or two sources one after the other along the contraction.  A block of 16 rows x 64 indices passes through LDS (a
// wavefront's own part) to 16 consecutive elements a lane; read that way from memory each lane would walk a line of its own.
constexpr int ROW_PITCH = 66;
__global__ __launch_bounds__(256) void rns_rows_kernel(RnsSource s0, RnsSource s1, const int* __restrict__ exps, long long e_stride, Residue q, signed char* __restrict__ out,
                                                       long long plane, long long out_stride, int kpad, int koff, int kblocks0, int kblocks1) {
    __shared__ __attribute__((aligned(16))) double lds[4][16 * ROW_PITCH];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, r0 = blockIdx.y * 16, kb = blockIdx.x * 4 + wave;
    if (kb >= kblocks0 + kblocks1 || (s0.row_limit && r0 >= s0.row_limit[0])) return;
    const bool second = kb >= kblocks0;
    const RnsSource& s = second ? s1 : s0;
    const int k0 = (second ? kb - kblocks0 : kb) * SK, shift = shift_of(s), kk = 2 * (lane & 31), k = k0 + kk;
    const double* a = s.a + blockIdx.z * s.stride + k;
    double v0[8], v1[8]; int e[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        const int r = r0 + 2 * j + (lane >> 5);
        e[j] = r >= s.rows ? UNDEFINED : exps[blockIdx.z * e_stride + r];
        const bool live = r < s.rows && !(s.half && k > r);
        v0[j] = live && k < s.k ? a[(long long)r * s.ld] : 0.0; v1[j] = live && k + 1 < s.k ? a[(long long)r * s.ld + 1] : 0.0;
    }
    double* mine = lds[wave];
    const int p0 = k < s.k ? power(s, k, shift) : 0, p1 = k + 1 < s.k ? power(s, k + 1, shift) : 0;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        const int ri = 2 * j + (lane >> 5), r = r0 + ri;
        *(double2*)(mine + ri * ROW_PITCH + kk) = e[j] == UNDEFINED ? make_double2(0.0, 0.0)
                                                                    : make_double2(rint(ldexp(counted(s, v0[j], r, k), p0 - e[j])), rint(ldexp(counted(s, v1[j], r, k + 1), p1 - e[j])));
    }
    __builtin_amdgcn_wave_barrier();
    const int ri = lane >> 2, piece = lane & 3;
    double x[16];
#pragma unroll
    for (int i = 0; i < 8; ++i) { const double2 v = *(const double2*)(mine + ri * ROW_PITCH + 16 * piece + 2 * i); x[2 * i] = v.x; x[2 * i + 1] = v.y; }
    store_residues(x, q, out + blockIdx.z * out_stride + ((long long)(r0 >> 4) * (kpad >> 6) + (koff >> 6) + kb) * 1024 + ri * 64 + ((piece ^ (ri >> 2)) << 4), plane);
}

// ---------------------------------------------------------------------------------------------- the product
struct Args {
    const char *A, *B;                       // first row, first contraction index
    long long planeA, planeB, strideA, strideB, termB;      // termB: from B to the second term's right operand (its left operand follows the first's along k)
    int pitchA, pitchB;                      // bytes from one row of blocks to the next
    int M, N, K, terms;                      // K: multiple of KPAD
    int row0, klo_m, klo_n, khi_n, upper, wide;
    const int* m_limit;
    unsigned char* C;
    int tiles_m, tiles_n, batch, splits, per, chunk;      // per: moduli a workgroup takes
    Moduli q;
};

struct Range { int lo, hi; };
__device__ __forceinline__ Range k_range(int K, int klo_m, int klo_n, int khi_n, int m0, int n0) {
    Range r{0, K};
    if (klo_m) r.lo = max(r.lo, m0);
    if (klo_n) r.lo = max(r.lo, n0);
    if (khi_n) r.hi = min(r.hi, n0 + BN);
    return r;
}

__device__ __forceinline__ i32x4 read_frag(const signed char* __restrict__ t, int row, int chunk) {
    return *(const i32x4*)(t + row * SK + ((chunk ^ ((row >> 2) & 3)) << 4));
}

// A workgroup takes one 256 x 256 tile through a run of moduli: the pipeline of gemm_bf16_nt_stream_kernel (8 wavefronts of 128 x 64, LDS-direct loads into a ring of four
// stages) with the planes as one stream of stages, so that the ring never drains between two products.  After a plane the accumulators become residues: 4 operations
// each, 16 bytes a lane and store, in the order in which the MFMA leaves them (rns_result_kernel reads them the same way).  A dispatched workgroup per tile and
// plane would pay the ring's filling and draining 15 times, as much as the products themselves where K is 1024.
// Residue: q = round(acc / m) from the rounding of a float sum; |acc| 2^-23 / m is its error in units, which for contractions up to 4096 leaves
// |acc - q m| <= 239 / 2 + 7.5 < 128 (the moduli are below 240 for that; modulo 256 the low byte needs no reduction); longer ones are brought back by one step (wide).
__global__ __launch_bounds__(512) void rns_gemm_kernel(Args g) {
    constexpr int TJ = 2, LPW = 2;
    extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
    signed char* ring = (signed char*)smem;

    const int loc = blockIdx.x >> 3, item = ((loc / g.chunk) * 8 + (blockIdx.x & 7)) * g.chunk + loc % g.chunk, tiles = g.tiles_m * g.tiles_n;
    if (item >= tiles * g.batch * g.splits) return;
    const int sp = __builtin_amdgcn_readfirstlane(item / (tiles * g.batch)), zt = item - sp * tiles * g.batch, z = __builtin_amdgcn_readfirstlane(zt / tiles), t = zt - z * tiles;
    // bands of 8 rows of tiles, column by column; the longest contractions first
    const int band = t / (8 * g.tiles_n), rows = min(8, g.tiles_m - 8 * band), in = t - band * 8 * g.tiles_n;
    const int tm = __builtin_amdgcn_readfirstlane(8 * band + in % rows), tc = __builtin_amdgcn_readfirstlane(in / rows), tn = g.khi_n ? g.tiles_n - 1 - tc : tc;
    const int m0 = tm * BM, n0 = tn * BN;
    if (g.m_limit && m0 >= g.m_limit[z]) return;
    if (g.upper && n0 + BN <= g.row0 + m0) return;
    const Range kr = k_range(g.K, g.klo_m, g.klo_n, g.khi_n, g.row0 + m0, n0);
    if (kr.hi <= kr.lo) return;
    const int p0 = sp * g.per, p1 = min(NMAX, p0 + g.per);
    if (p0 >= p1) return;
    const int nk = (kr.hi - kr.lo) / SK * g.terms;      // stages of a plane: a multiple of NS

    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, wave_s = __builtin_amdgcn_readfirstlane(wave);
    const int wm = (wave / 4) * 128, wn = (wave % 4) * 64, l32 = lane & 31, lh = lane >> 5;
    unsigned offA[LPW], offB[LPW];
#pragma unroll
    for (int i = 0; i < LPW; ++i) {      // blocks beyond the operands are read again from the last one (their products are never used)
        offA[i] = (unsigned)(min(wave * LPW + i, (g.M - 1 - m0) >> 4) * g.pitchA + lane * 16);
        offB[i] = (unsigned)(min(wave * LPW + i, (g.N - 1 - n0) >> 4) * g.pitchB + lane * 16);
    }
    const char* Ap = g.A + z * g.strideA + p0 * g.planeA + (long long)(m0 >> 4) * g.pitchA + (long long)kr.lo * 16;
    const char* Bp = g.B + z * g.strideB + p0 * g.planeB + (long long)(n0 >> 4) * g.pitchB + (long long)kr.lo * 16;
    // position of the stream of stages: byte offsets from Ap and Bp (64 contraction indices are one block of 1 KB)
    const int klen = kr.hi - kr.lo;
    long long ka = 0, kb = 0; int kin = 0, term = 0, left = nk * (p1 - p0);
    auto advance = [&]() {      // after the loads of a stage have been issued; beyond the last stage the stream re-reads it
        if (--left <= 0) { left = 0; return; }
        ka += 1024; kb += 1024; kin += SK;
        if (kin < klen) return;
        kin = 0;
        if (++term < g.terms) { ka += (long long)(g.K - klen) * 16; kb += g.termB - (long long)klen * 16; return; }
        term = 0; Ap += g.planeA; Bp += g.planeB; ka = 0; kb = 0;
    };
    const unsigned ring_lds = (unsigned)(unsigned long long)((__attribute__((address_space(3))) void*)ring);
    i32x16 acc[4][TJ];
    i32x4 fa[2][4], fb[2][TJ];
#define TB_LOAD_FRAGS(SET, SLOT, KS)                                                                        \
    {                                                                                                       \
        const signed char* a_s = ring + (SLOT) * STAGE_BYTES;                                               \
        const signed char* b_s = a_s + BM * SK;                                                             \
        _Pragma("unroll") for (int i = 0; i < 4; ++i) fa[SET][i] = read_frag(a_s, wm + 32 * i + l32, 2 * (KS) + lh); \
        _Pragma("unroll") for (int i = 0; i < TJ; ++i) fb[SET][i] = read_frag(b_s, wn + 32 * i + l32, 2 * (KS) + lh); \
    }
#define TB_STAGE(SLOT, NEXTSLOT, WAIT, FIRST)                                                               \
    {                                                                                                       \
        __builtin_amdgcn_sched_barrier(0);                                                                  \
        const char* pa_ = Ap + ka; const char* pb_ = Bp + kb;                                               \
        const unsigned st_ = ring_lds + (unsigned)((SLOT) * STAGE_BYTES);                                   \
        TB_LOAD_FRAGS(1, SLOT, 1)                                                                           \
        _Pragma("unroll") for (int i = 0; i < 4; ++i)                                                       \
            _Pragma("unroll") for (int jj = 0; jj < TJ; ++jj)                                               \
                acc[i][jj] = __builtin_amdgcn_mfma_i32_32x32x32_i8(fa[0][i], fb[0][jj], (FIRST) ? zero16 : acc[i][jj], 0, 0, 0); \
        __builtin_amdgcn_sched_group_barrier(0x100, 4 + TJ, 0);                                             \
        __builtin_amdgcn_sched_group_barrier(0x008, 4 * TJ, 0);                                             \
        __builtin_amdgcn_sched_barrier(0);                                                                  \
        if (WAIT) wait_loads_but<(NS - 2) * 2 * LPW>();                                                     \
        else asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");                                             \
        __syncthreads();                                                                                    \
        __builtin_amdgcn_sched_barrier(0);                                                                  \
        TB_LOAD_FRAGS(0, NEXTSLOT, 0)                                                                       \
        _Pragma("unroll") for (int i = 0; i < 4; ++i) {                                                     \
            _Pragma("unroll") for (int jj = 0; jj < TJ; jj += 2) {                                          \
                acc[i][jj] = __builtin_amdgcn_mfma_i32_32x32x32_i8(fa[1][i], fb[1][jj], acc[i][jj], 0, 0, 0); \
                acc[i][jj + 1] = __builtin_amdgcn_mfma_i32_32x32x32_i8(fa[1][i], fb[1][jj + 1], acc[i][jj + 1], 0, 0, 0); \
                const int q_ = (i * TJ + jj) / 2;              /* 0 .. 2 LPW - 1 */                           \
                const unsigned blk_ = (unsigned)(wave_s * LPW + q_ / 2) * 1024u;                            \
                __builtin_amdgcn_sched_barrier(0);                                                          \
                if (q_ % 2 == 0) lds_direct_16(offA[q_ / 2], pa_, st_ + blk_);                              \
                else lds_direct_16(offB[q_ / 2], pb_, st_ + (unsigned)(BM * SK) + blk_);                    \
                __builtin_amdgcn_sched_barrier(0);                                                          \
            }                                                                                               \
        }                                                                                                   \
        advance();                                                                                          \
    }
#pragma unroll
    for (int s = 0; s < NS; ++s) {
        const unsigned st = ring_lds + (unsigned)(s * STAGE_BYTES);
#pragma unroll
        for (int i = 0; i < LPW; ++i) {
            const unsigned blk = (unsigned)(wave_s * LPW + i) * 1024u;
            lds_direct_16(offA[i], Ap + ka, st + blk);
            lds_direct_16(offB[i], Bp + kb, st + (unsigned)(BM * SK) + blk);
        }
        advance();
    }
    wait_loads_but<0>();
    __syncthreads();
    TB_LOAD_FRAGS(0, 0, 0)
    const i32x16 zero16 = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
    for (int p = p0; p < p1; ++p) {
#pragma unroll
        for (int u = 0; u < NS; ++u) TB_STAGE(u, (u + 1) % NS, u == NS - 1, u == 0)
        for (int kt = NS; kt < nk; kt += NS) {
#pragma unroll
            for (int u = 0; u < NS; ++u) TB_STAGE(u, (u + 1) % NS, true, false)
        }
        // the loads issued so far land before the first store (see gemm_bf16_nt_stream_kernel)
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        const int m = g.q.m[p];
        const float inv = g.q.inv[p];
        unsigned char* o = g.C + (((long long)p * g.batch + z) * tiles + tm * g.tiles_n + tn) * (BM * BN) + ((wave_s * 8) * 64 + lane) * 16;
        constexpr float MAGIC = 12582912.f;      // 1.5 x 2^23: the low 24 bits of the sum are 2^22 plus the rounded quotient
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int j = 0; j < TJ; ++j) {
                unsigned w[4];
#pragma unroll
                for (int b = 0; b < 4; ++b) {
                    unsigned r[4];
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const int a = acc[i][j][4 * b + e];
                        int v = a;
                        if (p > 0) {
                            const int n = __float_as_int(__builtin_fmaf((float)a, inv, MAGIC));
                            v = a - __mul24(n, m);      // (2^22 m more than the residue: nothing modulo 256)
                            if (g.wide) { v += m << 22; v += v < -128 ? m : 0; v -= v > 127 ? m : 0; }
                        }
                        r[e] = (unsigned)v;
                    }
                    const unsigned lo = __builtin_amdgcn_perm(r[1], r[0], 0x0c0c0400), hi = __builtin_amdgcn_perm(r[3], r[2], 0x0c0c0400);
                    w[b] = lo | (hi << 16);
                }
                *(uint4*)(o + (i * TJ + j) * 1024) = make_uint4(w[0], w[1], w[2], w[3]);
            }
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");      // the re-read stages still in flight write LDS
#undef TB_STAGE
#undef TB_LOAD_FRAGS
}

// X = M frac(sum_p r_p w_p), w_p = ((M / m_p)^-1 mod m_p) / m_p.  w_p as 40 bits, whose sum with the residues is exact, and the rest: X to 2^-80 M and to the 53 bits of the
// result.  |X| < 2^115 < 0.3 M, so that the fraction never wraps.
struct Crt { double hi[NMAX], lo[NMAX], M; };
struct ResultArgs {
    const unsigned char* R;
    const int *ea, *eb; long long strideEa, strideEb;
    double *C; long long ldc, strideC; double alpha, beta;
    int M, N, K, row0, klo_m, klo_n, khi_n, upper, tiles_m, tiles_n, batch;
    const int* m_limit;
    Crt c;
};
// One wavefront per 32 x 32 results.  Bound by memory: 15 bytes of residues and 8 or 16 of C.
__global__ __launch_bounds__(256) void rns_result_kernel(ResultArgs g) {
    const int lane = threadIdx.x & 63, s = blockIdx.x * 4 + (threadIdx.x >> 6), w = s >> 3, ij = s & 7;
    const int tile = blockIdx.y, z = blockIdx.z, tm = tile / g.tiles_n, tn = tile - tm * g.tiles_n, m0 = tm * BM, n0 = tn * BN;
    const int row0 = m0 + (w / 4) * 128 + 32 * (ij >> 1), col = n0 + (w % 4) * 64 + 32 * (ij & 1) + (lane & 31), rl = row0 + 4 * (lane >> 5);
    if (row0 >= g.M || (g.m_limit && row0 >= g.m_limit[z])) return;
    const Range kr = k_range(g.K, g.klo_m, g.klo_n, g.khi_n, g.row0 + m0, n0);
    double hi[16], lo[16];
#pragma unroll
    for (int v = 0; v < 16; ++v) hi[v] = lo[v] = 0.0;
    if (kr.hi > kr.lo && !(g.upper && n0 + BN <= g.row0 + m0)) {
        const unsigned char* src = g.R + ((long long)z * g.tiles_m * g.tiles_n + tile) * (BM * BN) + (s * 64 + lane) * 16;
        const long long step = (long long)g.batch * g.tiles_m * g.tiles_n * (BM * BN);
        uint4 x[NMAX];
#pragma unroll
        for (int p = 0; p < NMAX; ++p) x[p] = *(const uint4*)(src + p * step);
#pragma unroll
        for (int p = 0; p < NMAX; ++p) {
            const unsigned q[4] = {x[p].x, x[p].y, x[p].z, x[p].w};
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const double r = (double)(int)(signed char)(q[v >> 2] >> (8 * (v & 3)));
                hi[v] = __builtin_fma(r, g.c.hi[p], hi[v]); lo[v] = __builtin_fma(r, g.c.lo[p], lo[v]);
            }
        }
    }
    if (col >= g.N) return;
    const int eb = g.eb[z * g.strideEb + col];
    double* C = g.C + z * g.strideC + col;
#pragma unroll
    for (int v = 0; v < 16; ++v) {
        const int row = rl + 8 * (v >> 2) + (v & 3);
        if (row >= g.M) continue;
        const int ea = g.ea[z * g.strideEa + row];
        double x = ldexp(((hi[v] - rint(hi[v])) + lo[v]) * g.c.M, ea + eb);
        if (ea == UNDEFINED || eb == UNDEFINED) x = NAN;
        if (g.upper && col <= g.row0 + row) x = 0.0;
        double* c = C + (long long)row * g.ldc;
        double r = g.alpha * x;
        if (g.beta != 0.0) r += g.beta * *c;
        *c = r;
    }
}

int mulmod_all_but(int l) {      // the product of the other moduli modulo the l-th
    int r = 1;
    for (int p = 0; p < NMAX; ++p) if (p != l) r = r * (MODULI[p] % MODULI[l]) % MODULI[l];
    return r;
}
Crt crt_constants() {
    Crt c{};
    unsigned __int128 M = 1;
    for (int p = 0; p < NMAX; ++p) M *= (unsigned)MODULI[p];
    c.M = (double)M;
    for (int p = 0; p < NMAX; ++p) {
        const int m = MODULI[p], o = mulmod_all_but(p);
        long long inv = 1;
        while (inv * o % m != 1) ++inv;
        const long long h = ((inv << 40) + m / 2) / m;
        c.hi[p] = (double)h * 0x1p-40;
        c.lo[p] = (double)((inv << 40) - h * m) / (double)m * 0x1p-40;
    }
    return c;
}

}  // namespace

bool rns_takes(int M, int N, int K) { return K <= 32768 && cdiv64(M, BM) * cdiv64(N, BN) <= 65535; }
int rns_pad(int k) { return (k + KPAD - 1) / KPAD * KPAD; }
size_t rns_plane(int rows, int k) { return (size_t)((rows + 15) / 16 * 16) * rns_pad(k); }
size_t rns_squares_elems(int rows) { return (size_t)3 * rows; }
static int col_chunks(int rows, int k) { return (int)std::max<int64_t>(1, std::min<int64_t>(std::min<int64_t>(RNS_CHUNKS, cdiv64(k, 32)), cdiv64(2048, cdiv64(rows, 256)))); }
size_t rns_residue_bytes(int M, int N, int batch) { return (size_t)cdiv64(M, BM) * cdiv64(N, BN) * batch * NMAX * BM * BN; }

int rns_norms(tboa_ctx* ctx, const RnsSource& s, int batch, double* sq, long long sq_stride, double* part) {
    if (s.kc) return tboa_fail(ctx, TBOA_EINVAL, "rns_norms: rows that are contiguous have theirs from rns_rows");
    const int chunks = col_chunks(s.rows, s.k), per = (int)cdiv64(s.k, chunks);
    const long long ps = 3LL * chunks * s.rows;
    hipLaunchKernelGGL(rns_col_squares_kernel, dim3((unsigned)cdiv64(s.rows, 256), chunks, batch), dim3(256), 0, ctx->stream, s, per, part, ps);
    hipLaunchKernelGGL(rns_sum_squares_kernel, dim3((unsigned)cdiv64(3LL * s.rows, 256), 1, batch), dim3(256), 0, ctx->stream, s.rows, chunks, part, ps, sq, sq_stride);
    TB_KERNEL_CHECK(ctx);
    return 0;
}
int rns_grow(tboa_ctx* ctx, int rows, int batch, const double* panel, long long panel_stride, double* sq, int sq_rows, long long sq_stride, int fresh_below, int bits, int* e, long long e_stride,
             int* grown) {
    hipLaunchKernelGGL(rns_grow_kernel, dim3((unsigned)cdiv64(rows, 256), 1, batch), dim3(256), 0, ctx->stream, rows, panel, panel_stride, sq, sq_rows, sq_stride, fresh_below, bits, e, e_stride,
                       grown);
    TB_KERNEL_CHECK(ctx);
    return 0;
}
int rns_diagonal_exps(tboa_ctx* ctx, int n, int batch, const double* H, int bits, int* e, double* sum, long long sum_stride) {
    hipLaunchKernelGGL(rns_diagonal_exps_kernel, dim3((unsigned)cdiv64(n, 256), 1, batch), dim3(256), 0, ctx->stream, n, H, (long long)n * n, bits, e, sum, sum_stride);
    TB_KERNEL_CHECK(ctx);
    return 0;
}
int rns_row_guard(tboa_ctx* ctx, const RnsSource& s, int batch, int bits, const RnsOperand& o, double* sum, long long sum_stride) {
    if (!s.kc || !o.e || s.kexp || s.exp_shift || s.half) return tboa_fail(ctx, TBOA_EINVAL, "rns_row_guard: source must be plain rows");
    hipLaunchKernelGGL(rns_row_guard_kernel, dim3((unsigned)cdiv64(s.rows, 4), 1, batch), dim3(256), 0, ctx->stream, s, bits, o.e, o.e_stride, sum, sum_stride);
    TB_KERNEL_CHECK(ctx);
    return 0;
}
int rns_balance(tboa_ctx* ctx, int rows, double* sq1, const double* sq2, int* f) {
    hipLaunchKernelGGL(rns_balance_kernel, dim3(1), dim3(1024), 0, ctx->stream, rows, sq1, sq2, f);
    TB_KERNEL_CHECK(ctx);
    return 0;
}
int rns_exps(tboa_ctx* ctx, int rows, int batch, const double* sq, long long sq_stride, int bits, int* e, long long e_stride) {
    hipLaunchKernelGGL(rns_exps_kernel, dim3((unsigned)cdiv64(rows, 256), 1, batch), dim3(256), 0, ctx->stream, rows, sq, sq_stride, bits, e, e_stride);
    TB_KERNEL_CHECK(ctx);
    return 0;
}
int rns_channel_sizes(tboa_ctx* ctx, int n, const double* H, int* size) {
    hipLaunchKernelGGL(rns_channel_sizes_kernel, dim3((unsigned)cdiv64(n, 256)), dim3(256), 0, ctx->stream, H, n, size);
    TB_KERNEL_CHECK(ctx);
    return 0;
}
int rns_channel_exps(tboa_ctx* ctx, int n, const double* sq, const int* size, const int* right, int* x) {
    hipLaunchKernelGGL(rns_channel_exps_kernel, dim3(1), dim3(1024), 0, ctx->stream, n, sq, size, right, x);
    TB_KERNEL_CHECK(ctx);
    return 0;
}
int rns_row_exps(tboa_ctx* ctx, const RnsSource& s, int bits, int* e) {
    if (!s.kc) return tboa_fail(ctx, TBOA_EINVAL, "rns_row_exps: rows must be contiguous");
    hipLaunchKernelGGL(rns_row_exps_kernel, dim3((unsigned)cdiv64(s.rows, 4), 1, 1), dim3(256), 0, ctx->stream, s, s, 0, bits, e, 0LL);
    TB_KERNEL_CHECK(ctx);
    return 0;
}
static Residue residue_constants() {
    Residue q;
    for (int p = 0; p < NMAX; ++p) {
        int c = (int)((1LL << 29) % MODULI[p]);
        if (2 * c > MODULI[p]) c -= MODULI[p];
        q.m[p] = MODULI[p]; q.inv[p] = 1.0 / MODULI[p]; q.c[p] = q.ci[p] = c;
    }
    return q;
}
int rns_columns(tboa_ctx* ctx, const RnsSource& s, int batch, const RnsOperand& o, int koff, const int* grown, int panel) {
    const int kblocks = (int)(std::min<int64_t>(rns_pad(s.k), o.kpad - koff) / SK);
    const unsigned rb = (unsigned)cdiv64(s.rows, 16);
    if (s.kc || !o.e || koff % SK || kblocks * SK < s.k || rb > 65535 || (size_t)rb * 16 * o.kpad > o.plane) return tboa_fail(ctx, TBOA_EINVAL, "rns_columns: source does not fit the operand");
    hipLaunchKernelGGL(rns_columns_kernel, dim3((unsigned)cdiv64(kblocks, 4), rb, batch), dim3(256), 0, ctx->stream, s, o.e, o.e_stride, residue_constants(), o.p, (long long)o.plane,
                       o.stride, o.kpad, koff, kblocks, grown, (panel + SK - 1) / SK);
    TB_KERNEL_CHECK(ctx);
    return 0;
}
int rns_rows(tboa_ctx* ctx, const RnsSource& s, const RnsSource* second, int batch, int bits, const RnsOperand& o, int koff) {
    const int kb0 = rns_pad(s.k) / SK, kb1 = second ? rns_pad(second->k) / SK : 0;
    const unsigned rb = (unsigned)cdiv64(s.rows, 16);
    if (!s.kc || (second && (!second->kc || second->rows != s.rows || s.k % KPAD)) || !o.e || koff % SK || koff + (kb0 + kb1) * SK > o.kpad || rb > 65535 || (size_t)rb * 16 * o.kpad > o.plane)
        return tboa_fail(ctx, TBOA_EINVAL, "rns_rows: source does not fit the operand");
    const RnsSource& s1 = second ? *second : s;
    if (bits >= 0) hipLaunchKernelGGL(rns_row_exps_kernel, dim3((unsigned)cdiv64(s.rows, 4), 1, batch), dim3(256), 0, ctx->stream, s, s1, second ? 1 : 0, bits, o.e, o.e_stride);
    hipLaunchKernelGGL(rns_rows_kernel, dim3((unsigned)cdiv64(kb0 + kb1, 4), rb, batch), dim3(256), 0, ctx->stream, s, s1, o.e, o.e_stride, residue_constants(), o.p, (long long)o.plane,
                       o.stride, o.kpad, koff, kb0, kb1);
    TB_KERNEL_CHECK(ctx);
    return 0;
}

// Microseconds of a launch and its best number of runs of moduli.  A plane of a tile takes 11.6 us for 1024 contraction indices and 6 for its residues, a workgroup 8 to fill and
// drain its ring (measured at 256 - 8192); tiles of unequal length (triangular operands, half of it on average) go longest first, so that what counts is the sum of the
// work and, at the end, half of the longest workgroup.
static double gemm_us(long long tiles, int K, bool triangular, int* splits) {
    auto plane = [](double k) { return k / 1024.0 * 11.6 + 6.0; };
    double best = 1e300;
    for (int s = 1; s <= NMAX; ++s) {
        const int per = (NMAX + s - 1) / s;
        if ((NMAX + per - 1) / per != s) continue;
        const double us = triangular ? (double)tiles * s / 256.0 * (per * plane(0.5 * K) + 8.0) + 0.5 * (per * plane(K) + 8.0) : (double)cdiv64(tiles * s, 256) * (per * plane(K) + 8.0);
        if (us < best) { best = us; if (splits) *splits = s; }
    }
    return best;
}
// Microseconds of a product with its left operand's preparation; of the preparation of an operand (4.5 TB/s, launches of 5 us)
double rns_model_us(int M, int N, int K, bool triangular, bool beta) {
    return rns_prepare_us(M, K) + gemm_us(cdiv64(M, BM) * cdiv64(N, BN), rns_pad(K), triangular, nullptr) + 10.0 + (double)M * N * (NMAX + (beta ? 16.0 : 8.0)) / 4.5e6;
}
double rns_prepare_us(int rows, int k) { return 12.0 + (double)rows * k * (16.0 + TB_RNS_MODULI) / 4.5e6; }

int rns_gemm(tboa_ctx* ctx, const RnsGemm& q) {
    if (q.M <= 0 || q.N <= 0) return 0;
    const int K = rns_pad(q.K);
    if (!q.A || !q.B || !q.C || !q.residues || q.K <= 0 || !rns_takes(q.M, q.N, K) || !q.A->e || !q.B->e || q.a_row % 16 || q.b_row % 16 || q.a_k % SK || q.b_k % SK ||
        q.a_k + (q.B2 ? 2 : 1) * K > q.A->kpad || q.b_k + K > q.B->kpad || (size_t)(q.a_row + cdiv64(q.M, 16) * 16) * q.A->kpad > q.A->plane ||
        (size_t)(q.b_row + cdiv64(q.N, 16) * 16) * q.B->kpad > q.B->plane || (q.B2 && (q.K % KPAD || q.B2->kpad != q.B->kpad || q.B2->plane != q.B->plane || q.B2->stride != q.B->stride)))
        return tboa_fail(ctx, TBOA_EINVAL, "rns_gemm: unsupported product");
    Args a{};
    a.pitchA = q.A->kpad * 16; a.pitchB = q.B->kpad * 16;
    a.A = (const char*)q.A->p + (long long)(q.a_row >> 4) * a.pitchA + (long long)q.a_k * 16;
    a.B = (const char*)q.B->p + (long long)(q.b_row >> 4) * a.pitchB + (long long)q.b_k * 16;
    a.planeA = (long long)q.A->plane; a.planeB = (long long)q.B->plane; a.strideA = q.A->stride; a.strideB = q.B->stride;
    a.M = q.M; a.N = q.N; a.K = K; a.terms = q.B2 ? 2 : 1; a.termB = q.B2 ? (long long)(q.B2->p - q.B->p) : 0;
    a.klo_m = q.klo_m; a.klo_n = q.klo_n; a.khi_n = q.khi_n; a.upper = q.upper; a.row0 = q.row0; a.wide = K * a.terms > 4096; a.m_limit = q.m_limit;
    a.C = q.residues; a.tiles_m = (int)cdiv64(q.M, BM); a.tiles_n = (int)cdiv64(q.N, BN); a.batch = q.batch;
    for (int p = 0; p < NMAX; ++p) { a.q.m[p] = MODULI[p]; a.q.inv[p] = 1.0f / (float)MODULI[p]; }
    const long long tiles = (long long)a.tiles_m * a.tiles_n * q.batch;
    gemm_us(tiles, K * a.terms, q.klo_m || q.klo_n || q.khi_n || q.upper, &a.splits); a.per = (NMAX + a.splits - 1) / a.splits;
    const long long items = tiles * a.splits;
    a.chunk = (int)std::max<long long>(1, std::min<long long>(32, cdiv64(items, 8)));
    const long long wgs = cdiv64(items, 8LL * a.chunk) * 8 * a.chunk;
    if (wgs > 0x7fffffffLL || q.batch > 65535) return tboa_fail(ctx, TBOA_EINVAL, "rns_gemm: grid too large");
    ProfRec rec{}; bool timed = false;
    if (ctx->prof_on) {
        double macs = 0.0;
        if (!q.m_limit)      // (how many rows there are only the device knows)
            for (int m0 = 0; m0 < q.M; m0 += BM)
                for (int n0 = 0; n0 < q.N; n0 += BN) {
                    if (q.upper && n0 + BN <= q.row0 + m0) continue;
                    const int lo = std::max(q.klo_m ? q.row0 + m0 : 0, q.klo_n ? n0 : 0), hi = q.khi_n ? std::min(q.K, n0 + BN) : q.K;
                    if (hi > lo) macs += (double)std::min(BM, q.M - m0) * std::min(BN, q.N - n0) * (hi - lo) * a.terms;
                }
        TB_TRY(prof_begin(ctx, q.m_limit ? TBOA_PROF_F64_GRID : TBOA_PROF_RESIDUES, 2.0 * macs * q.batch, rec, timed));
    }
    constexpr int smem = NS * STAGE_BYTES;
    TB_HIP(ctx, hipFuncSetAttribute((const void*)rns_gemm_kernel, hipFuncAttributeMaxDynamicSharedMemorySize, smem));
    hipLaunchKernelGGL(rns_gemm_kernel, dim3((unsigned)wgs), dim3(512), smem, ctx->stream, a);
    TB_KERNEL_CHECK(ctx);
    ResultArgs r{};
    r.R = q.residues; r.ea = q.A->e + q.a_row; r.eb = q.B->e + q.b_row; r.strideEa = q.A->e_stride; r.strideEb = q.B->e_stride;
    r.C = q.C; r.ldc = q.ldc; r.strideC = q.strideC; r.alpha = q.alpha; r.beta = q.beta; r.M = q.M; r.N = q.N; r.K = K; r.klo_m = q.klo_m; r.klo_n = q.klo_n; r.khi_n = q.khi_n;
    r.row0 = q.row0; r.upper = q.upper; r.tiles_m = a.tiles_m; r.tiles_n = a.tiles_n; r.batch = q.batch; r.m_limit = q.m_limit;
    r.c = crt_constants();
    hipLaunchKernelGGL(rns_result_kernel, dim3(16, (unsigned)(a.tiles_m * a.tiles_n), q.batch), dim3(256), 0, ctx->stream, r);
    TB_KERNEL_CHECK(ctx);
    return prof_end(ctx, rec, timed);
}

// C = alpha A B^T + beta C with operands in fp64, through the context's workspace: the building block on its own.
extern "C" int tboa_gemm_f64_residues(tboa_ctx* ctx, int M, int N, int K, double alpha, const double* A, int64_t lda, const double* B, int64_t sbk, int64_t sbn, double beta, double* C,
                                      int64_t ldc) {
    if (!ctx) return TBOA_EINVAL;
    if (M <= 0 || N <= 0 || K <= 0 || !rns_takes(M, N, K) || !A || !B || !C || lda < K || ldc < N || !((sbk == 1 && sbn >= K) || (sbn == 1 && sbk >= N)))
        return tboa_fail(ctx, TBOA_EINVAL, "gemm_f64_residues: bad arguments");
    for (int pass = 0; pass < 2; ++pass) {
        Arena ar(pass ? ctx->ws : nullptr);
        RnsOperand a{}, b{};
        a.kpad = b.kpad = rns_pad(K); a.plane = rns_plane(M, K); b.plane = rns_plane(N, K);
        a.p = ar.get<signed char>(a.plane * NMAX); b.p = ar.get<signed char>(b.plane * NMAX);
        a.e = ar.get<int>(M); b.e = ar.get<int>(N);
        double* sq = ar.get<double>(rns_squares_elems(N));
        double* part = ar.get<double>(RNS_CHUNKS * rns_squares_elems(N));
        unsigned char* res = ar.get<unsigned char>(rns_residue_bytes(M, N, 1));
        if (!pass) { TB_TRY(tboa_ws_reserve(ctx, ar.off)); continue; }
        RnsSource sa{}, sb{};
        sa.a = A; sa.ld = lda; sa.kc = 1; sa.rows = M; sa.k = K;
        sb.a = B; sb.kc = sbk == 1; sb.ld = sb.kc ? sbn : sbk; sb.rows = N; sb.k = K;
        TB_TRY(rns_rows(ctx, sa, nullptr, 1, RNS_BITS_A, a));
        if (sb.kc) TB_TRY(rns_rows(ctx, sb, nullptr, 1, RNS_BITS_B, b));
        else { TB_TRY(rns_norms(ctx, sb, 1, sq, 0, part)); TB_TRY(rns_exps(ctx, N, 1, sq, 0, RNS_BITS_B, b.e, 0)); TB_TRY(rns_columns(ctx, sb, 1, b, 0)); }
        RnsGemm g{};
        g.A = &a; g.B = &b; g.M = M; g.N = N; g.K = K; g.batch = 1; g.alpha = alpha; g.beta = beta; g.C = C; g.ldc = ldc; g.residues = res;
        TB_TRY(rns_gemm(ctx, g));
    }
    return 0;
}
