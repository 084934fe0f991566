// Attention outputs O_h = softmax(Q_h K_g^T / sqrt(d_h)) V_g of whole sequences in one kernel: scores, probabilities and the product with the values of a block of keys stay
// in the registers of one wavefront.  (Probabilities by attn_probs_t_kernel, which forms the scores twice and writes 8 bytes per probability and path, and a product that
// reads them again took 4.4 + 2.5 ms of the 7B-shaped W_O Hessian over 8 x 2048 tokens, both paths.)
//
// One workgroup per (path, sequence, head, 256 queries); each of its eight wavefronts keeps the Q^ fragments of 32 queries (as attn_probs_t_kernel does) and all
// d_h outputs of them.  Blocks of 32 keys of K^ (segments k_hi, k_lo) and V^T (hi, lo) are copied global -> LDS into a ring of four.  For each:
//     S^T = K^ Q^T              a lane holds one query and 16 of the keys, 8 b + 4 (lane / 32) + j for b, j < 4
//     r = running maximum of the query less 14 (0 for bf16), p = 2^(S - r) as (hi, lo) pair: half values below 2^14, whose low parts are normal numbers down to 2^-17 of the largest;
//                               O^T and the sum are rescaled where a maximum has grown.  Beyond |r| = 2^20 the difference to the maximum is taken before the
//                               scale: r is rounded, and p would be 2^14 times up to half a unit of r, infinite as half from r = 2^25 on
//     O^T += V^T P^T            the lane's 16 probabilities ARE the right operand of two 16-deep steps, if step s contracts over the keys 16 s + 4 (lane / 32) + {0 .. 3, 8 .. 11}:
//                               V^T is stored with its keys in that order (vt_blocks_kernel), so that nothing is exchanged between lanes
// The scores of block i + 1 and the product of block i are one run of MFMAs, the exponentials one run of vector instructions, with a barrier after each; of the two wavefronts of a
// SIMD one is a run behind, so that one multiplies while the other exponentiates.  (Both paths of 8 sequences x 32 heads x 2048 x 128: 2.2 ms, with all in step 2.44; the MFMAs
// take 0.75 of it, the rest is the exponentials' and the pairs' vector instructions, which the two wavefronts of a SIMD share.  A ring of five blocks or priorities: no gain.
// Four wavefronts and 128 queries are not better for short sequences either, though half of the eight have nothing to do up to 128 tokens: 16 sequences x 32 heads x 128, forward pass, 4 -> 8
// wavefronts, 72 tokens 0.237 -> 0.221 ms, 128 0.248 -> 0.242, 136 0.287 -> 0.259, 256 0.489 -> 0.451; 2 x 4 heads of 128 tokens 0.099 -> 0.098.)
// Operands as for the stored probabilities: scores q_hi k_hi + q_lo k_hi + q_hi k_lo of half pairs (22 bits) or bf16 pairs, probabilities and values as pairs of 16-bit values in
// three products, fp32 sums.
#include "internal.h"
#include <algorithm>
#include <type_traits>

typedef __hip_bfloat16 bf16;
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

namespace {

__device__ __forceinline__ float ex2(float x) { return __builtin_amdgcn_exp2f(x); }

template <bool F16>
__device__ __forceinline__ f32x16 mma(bf16x8 a, bf16x8 b, f32x16 c) {
    if constexpr (F16) return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x8, b), c, 0, 0, 0);
    else return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}
template <bool F16>
__device__ __forceinline__ unsigned short enc(float v) {
    if constexpr (F16) return __builtin_bit_cast(unsigned short, (_Float16)v);
    else return __builtin_bit_cast(unsigned short, (__bf16)v);
}
template <bool F16>
__device__ __forceinline__ float dec(unsigned short b) {
    if constexpr (F16) return (float)__builtin_bit_cast(_Float16, b);
    else return (float)__builtin_bit_cast(__bf16, b);
}

struct Args {
    AttnPath path[2];
    int paths, S, L, Hq, rep, blocked, causal, nqb, f16;
    float scale2;
    long long vseq, vpath, vlo;      // V^T blocks: elements from one sequence, path, part to the next
    int vkb;                         // 16 x 32 blocks per block row of V^T
    const bf16* V;
    bf16 *OT[2], *OTl[2]; long long ldo;      // [Hq dh][ldo] pairs per path
    bf16* rows; long long ldr;                 // or token-major bf16 rows of path 0
    long long total; int runs;
};

constexpr int NS = 4;      // blocks of 32 keys in the LDS ring
constexpr int W = 8;       // wavefronts
template <int DH> constexpr int ring_slot() { return 4 * 32 * 2 * DH; }

__device__ __forceinline__ void phase_end() {      // nothing is moved across
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("s_barrier" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
}

template <int DH, bool F16>
__global__ __launch_bounds__(64 * W, 2) void attn_output_kernel(Args g) {
    constexpr int NKS = DH / 16, NCB = DH / 32, KB = 3 * DH / 32, BQ = 32 * W;
    constexpr int KSEG = 32 * 2 * DH, KBYTES = 2 * KSEG, VPART = 32 * 2 * DH, SLOT = ring_slot<DH>(), NBLK = SLOT / 1024, LPW = NBLK / W;
    static_assert(NBLK % W == 0, "every wavefront copies as many blocks");
    extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
    // an XCD takes consecutive items: the blocks of a head, longest first, walk the same keys side by side, and so do the heads of a group
    int item = blockIdx.x;
    if (g.runs) item = (blockIdx.x & 7) * (int)(g.total / 8) + (blockIdx.x >> 3);
    const int qb = g.nqb - 1 - item % g.nqb, rem = item / g.nqb;
    const int h = __builtin_amdgcn_readfirstlane(rem % g.Hq), ps = rem / g.Hq, p = __builtin_amdgcn_readfirstlane(ps / g.S), sq = __builtin_amdgcn_readfirstlane(ps % g.S);
    const int t0 = __builtin_amdgcn_readfirstlane(qb) * BQ, L = g.L, grp = __builtin_amdgcn_readfirstlane(h / g.rep), Hkv = __builtin_amdgcn_readfirstlane(g.Hq / g.rep);
    const AttnPath& pa = g.path[p];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, wave_s = __builtin_amdgcn_readfirstlane(wave), l32 = lane & 31, lh = lane >> 5;
    const int tq = t0 + 32 * wave_s, t = tq + l32;

    bool half_ops = false;
    float sc2 = g.scale2;
    if (pa.qa && pa.ka) {
        const int bq = __builtin_amdgcn_readfirstlane(pa.qa[sq]), bk = __builtin_amdgcn_readfirstlane(pa.ka[sq]);
        if (bq >= 0 && bk >= 0) { half_ops = true; sc2 = ldexpf(g.scale2, -(tboa_half_exp(bq) + tboa_half_exp(bk))); }
    }
    // Q^ and K^ of a (sequence, head): [L, 3 dh] in blocks, or rows of all heads
    const bool blocked = __builtin_amdgcn_readfirstlane(g.blocked) != 0;
    const long long mat = (long long)L * 3 * DH, pq = (long long)g.Hq * 3 * DH, pk = (long long)Hkv * 3 * DH;
    const bf16* Qp = pa.Q + (blocked ? ((long long)sq * g.Hq + h) * mat : (long long)sq * L * pq + (long long)h * 3 * DH);
    const bf16* Kp = pa.K + (blocked ? ((long long)sq * Hkv + grp) * mat : (long long)sq * L * pk + (long long)grp * 3 * DH);
    const bf16* Vp = g.V + p * g.vpath + sq * g.vseq + (long long)grp * (DH / 16) * g.vkb * 512;

    bf16x8 qh[NKS], ql[NKS];
    {
        const int tc = min(t, L - 1);
#pragma unroll
        for (int ks = 0; ks < NKS; ++ks) {
            const int c = 16 * ks + 8 * lh;
            qh[ks] = *(const bf16x8*)(blocked ? Qp + tboa_blocked_offset(tc, c, KB) : Qp + tc * pq + c);
            ql[ks] = *(const bf16x8*)(blocked ? Qp + tboa_blocked_offset(tc, DH + c, KB) : Qp + tc * pq + DH + c);
        }
    }

    const unsigned lds0 = (unsigned)(unsigned long long)((__attribute__((address_space(3))) void*)smem);
    // block of 32 keys into its slot of the ring.  K: 1 KB blocks ((seg NCB + cb) 2 + rb), 16 keys x 64 bytes, pieces swizzled; V: (part DH / 16 + rb).  Keys
    // beyond the sequence are read from earlier rows (their probabilities are zero); V^T is there, zeros, up to whole 64s.  This wavefront's LPW of them:
    // address of the next block, bytes to the one after it, the last there is.
    const char* src[LPW]; unsigned step[LPW], voff[LPW]; int last[LPW];
#pragma unroll
    for (int j = 0; j < LPW; ++j) {
        const int b = wave_s + W * j;
        voff[j] = (unsigned)lane * 16u;
        if (b < KBYTES / 1024) {
            const int rb = b & 1, sc = b >> 1, cb = sc % NCB, seg = sc / NCB;
            if (blocked) { src[j] = (const char*)(Kp + ((long long)rb * KB + (seg ? 2 * NCB : 0) + cb) * 512); step[j] = 2 * KB * 1024; last[j] = (((L - 1) >> 4) - rb) >> 1; }
            else {
                const int row = 16 * rb + (lane >> 2), piece = (lane & 3) ^ ((row >> 2) & 3);
                src[j] = (const char*)(Kp + (seg ? 2 * DH : 0) + cb * 32); step[j] = (unsigned)(32 * pk * 2); last[j] = (L - 1) >> 5;
                voff[j] = (unsigned)((row * pk + piece * 8) * 2);
            }
            if (last[j] < 0) { last[j] = 0; src[j] = (const char*)(Kp + ((seg ? 2 * NCB : 0) + cb) * 512); }      // (one block row in all)
        } else {
            const int v = b - KBYTES / 1024, rb = v % (DH / 16), part = v / (DH / 16);
            src[j] = (const char*)(Vp + part * g.vlo + (long long)rb * g.vkb * 512); step[j] = 1024; last[j] = g.vkb - 1;
        }
    }
    auto issue = [&](int i) __attribute__((always_inline)) {      // blocks in order
        const unsigned to = lds0 + (unsigned)((i % NS) * SLOT);
        const bool ragged = !blocked && 32 * i + 32 > L;
#pragma unroll
        for (int j = 0; j < LPW; ++j) {
            const int b = wave_s + W * j;
            unsigned vo = voff[j];
            if (ragged && b < KBYTES / 1024) {
                const int row = 16 * (b & 1) + (lane >> 2), piece = (lane & 3) ^ ((row >> 2) & 3);
                vo = (unsigned)((min(row, L - 1 - 32 * i) * pk + piece * 8) * 2);
            }
            lds_direct_16(vo, src[j], to + (unsigned)b * 1024u);
            if (i < last[j]) src[j] += step[j];
        }
    };
    const f32x16 zero16 = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    f32x16 O[NCB], acc = zero16, low = zero16;      // acc, low: q_hi k_hi and what the low parts add to it
#pragma unroll
    for (int c = 0; c < NCB; ++c) O[c] = zero16;
    union { unsigned short h[8]; bf16x8 x; } ph[2], pl[2];
    constexpr float UP = F16 ? 14.f : 0.f, LARGE = 0x1p20f;
    static_assert(ATTN_PROBS_HALF_SCALE == 16384.f, "2^14");
    // m: the maximum; r: what the exponents are taken from, m times the scale less UP; large: of this wavefront's r some are, and p = 2^((S - m) scale + UP)
    float m = -INFINITY, r = -INFINITY, s[4] = {0.f, 0.f, 0.f, 0.f};      // (four sums: one over all keys is off by as much as the rest together)
    bool large = false;

    const int kend = g.causal ? min(L, t0 + BQ) : L, nblk = __builtin_amdgcn_readfirstlane((kend + 31) / 32);
    const int mine = __builtin_amdgcn_readfirstlane(tq >= L ? 0 : g.causal ? min(nblk, tq / 32 + 1) : nblk);      // this wavefront's blocks
    auto scores_step = [&](const unsigned char* kt, int ks, auto hs) __attribute__((always_inline)) {
        constexpr bool HS = decltype(hs)::value;
        const int c8 = 2 * ks + lh, off = (c8 >> 2) * 2048 + l32 * 64 + (((c8 & 3) ^ ((l32 >> 2) & 3)) << 4);
        const bf16x8 kh = *(const bf16x8*)(kt + off), kl = *(const bf16x8*)(kt + KSEG + off);
        low = mma<HS>(kh, ql[ks], ks ? low : zero16); acc = mma<HS>(kh, qh[ks], ks ? acc : zero16); low = mma<HS>(kl, qh[ks], low);
    };
    auto values_step = [&](const unsigned char* vt, int u) __attribute__((always_inline)) {      // u: step 2 c + st
        const int st = u / NCB, c = u % NCB, vr = 32 * c + l32, off = (vr >> 4) * 1024 + (vr & 15) * 64 + (((2 * st + lh) ^ ((vr >> 2) & 3)) << 4);
        const bf16x8 vh = *(const bf16x8*)(vt + off), vl = *(const bf16x8*)(vt + VPART + off);
        O[c] = mma<F16>(vl, ph[st].x, O[c]); O[c] = mma<F16>(vh, pl[st].x, O[c]); O[c] = mma<F16>(vh, ph[st].x, O[c]);
    };
    auto exponentials = [&](int i) __attribute__((always_inline)) {
        const int k0 = 32 * i;
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[e] += low[e];
        if (k0 + 31 > (g.causal ? tq : L - 1)) {
            asm volatile("s_nop 0");      // (a branch, not sixteen selections in every block)
            const int ib = k0 + 4 * lh, limit = g.causal ? t : L - 1;
#pragma unroll
            for (int e = 0; e < 16; ++e) if (ib + 8 * (e >> 2) + (e & 3) > limit) acc[e] = -INFINITY;
        }
        float vm = acc[0];
#pragma unroll
        for (int e = 1; e < 16; ++e) vm = fmaxf(vm, acc[e]);
        vm = fmaxf(vm, __shfl_xor(vm, 32, 64));
        if (__any(vm > m)) {
            const float mn = fmaxf(m, vm), rn = mn * sc2 - UP;
            const bool was = large;
            large = was || __any(fabsf(rn) > LARGE);
            const float f = m == -INFINITY ? 0.f : ex2(was ? (m - mn) * sc2 : large ? __builtin_fmaf(-mn, sc2, r) + UP : r - rn);
#pragma unroll
            for (int e = 0; e < 4; ++e) s[e] *= f;
#pragma unroll
            for (int c = 0; c < NCB; ++c)
#pragma unroll
                for (int e = 0; e < 16; ++e) O[c][e] *= f;
            m = mn; r = rn;
        }
        float ref = m == -INFINITY ? 0.f : -r;
        if (large) {
            asm volatile("s_nop 0");
            const float from = m == -INFINITY ? 0.f : m;
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[e] -= from;
            ref = UP;
        }
#pragma unroll
        for (int e = 0; e < 16; ++e) {
            const float a = ex2(__builtin_fmaf(acc[e], sc2, ref));
            s[e & 3] += a;
            const unsigned short hi = enc<F16>(a);
            ph[e >> 3].h[e & 7] = hi; pl[e >> 3].h[e & 7] = enc<F16>(a - dec<F16>(hi));
        }
    };
    auto walk = [&](auto hs) __attribute__((always_inline)) {      // (the encoding of the scores' operands decided once, outside the loop)
#pragma unroll
        for (int i = 0; i < NS - 1; ++i) if (i < nblk) issue(i);
        wait_loads_but<0>();
        phase_end();
        if (mine > 0) {
#pragma unroll
            for (int ks = 0; ks < NKS; ++ks) scores_step(smem, ks, hs);
            exponentials(0);
        }
        const bool behind = wave_s >= 4;
        if (behind) phase_end();
        auto multiply_end = [&](int i) __attribute__((always_inline)) {
            if (i + NS - 1 < nblk) wait_loads_but<LPW>();      // all but the newest block's
            else wait_loads_but<0>();
            phase_end();
        };
        int i = 0;
        for (; i + 1 < mine; ++i) {
            if (i + NS - 1 < nblk) issue(i + NS - 1);
            const unsigned char* kt = smem + ((i + 1) % NS) * SLOT;
            const unsigned char* vt = smem + (i % NS) * SLOT + KBYTES;
            __builtin_amdgcn_s_setprio(1);
#pragma unroll
            for (int u = 0; u < NKS; ++u) { scores_step(kt, u, hs); values_step(vt, u); }      // (as many steps of the one as of the other: d_h / 16)
            __builtin_amdgcn_sched_group_barrier(0x100, 4, 0);      // the fragments of one step ahead
#pragma unroll
            for (int u = 1; u < NKS; ++u) { __builtin_amdgcn_sched_group_barrier(0x100, 4, 0); __builtin_amdgcn_sched_group_barrier(0x008, 6, 0); }
            __builtin_amdgcn_sched_group_barrier(0x008, 6, 0);
            __builtin_amdgcn_sched_barrier(0);
            __builtin_amdgcn_s_setprio(0);
            multiply_end(i);
            exponentials(i + 1);
            phase_end();
        }
        for (; i < nblk; ++i) {      // this wavefront's last block; the copies and barriers of the others'
            if (i + NS - 1 < nblk) issue(i + NS - 1);
            if (i < mine) {
                const unsigned char* vt = smem + (i % NS) * SLOT + KBYTES;
#pragma unroll
                for (int u = 0; u < NKS; ++u) values_step(vt, u);
            }
            multiply_end(i);
            phase_end();
        }
        if (!behind) phase_end();
    };
    if (half_ops) walk(std::true_type{});
    else walk(std::false_type{});
    float sum = (s[0] + s[1]) + (s[2] + s[3]);
    sum += __shfl_xor(sum, 32, 64);
    const float inv = 1.f / sum;
    __syncthreads();
    // results through LDS, BQ queries a row: 64 bytes and more to every row of O^T, whole rows of a head to O
    if (g.rows) {
        constexpr int P = DH + 8;      // elements per query
        unsigned short* x = (unsigned short*)smem;
#pragma unroll
        for (int c = 0; c < NCB; ++c)
#pragma unroll
            for (int b = 0; b < 4; ++b) {
                union { unsigned short h[4]; uint2 u; } o;
#pragma unroll
                for (int j = 0; j < 4; ++j) o.h[j] = enc<false>(O[c][4 * b + j] * inv);
                *(uint2*)(x + (32 * wave + l32) * P + 32 * c + 8 * b + 4 * lh) = o.u;
            }
        __syncthreads();
        for (int i = threadIdx.x; i < BQ * DH / 8; i += 64 * W) {
            const int r = i / (DH / 8), c8 = i % (DH / 8);
            if (t0 + r < L) *(uint4*)(g.rows + ((long long)sq * L + t0 + r) * g.ldr + (long long)h * DH + 8 * c8) = *(const uint4*)(x + r * P + 8 * c8);
        }
        return;
    }
    constexpr int P = BQ + 8;
    unsigned short* x = (unsigned short*)smem;
    bf16* dst[2] = {g.OT[p], g.OTl[p]};
#pragma unroll
    for (int part = 0; part < 2; ++part) {
        if (part) __syncthreads();
#pragma unroll
        for (int c = 0; c < NCB; ++c)
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                float o = O[c][e] * inv;
                asm volatile("" : "+v"(o));      // (as in vt_blocks_kernel)
                const unsigned short hi = enc<F16>(o);
                x[(32 * c + 8 * (e >> 2) + 4 * lh + (e & 3)) * P + 32 * wave + l32] = part ? enc<F16>(o - dec<F16>(hi)) : hi;
            }
        __syncthreads();
        for (int i = threadIdx.x; i < DH * BQ / 8; i += 64 * W) {
            const int r = i / (BQ / 8), c8 = i % (BQ / 8);      // (sequences are whole 8s)
            if (t0 + 8 * c8 < L) *(uint4*)(dst[part] + ((long long)h * DH + r) * g.ldo + (long long)sq * L + t0 + 8 * c8) = *(const uint4*)(x + r * P + 8 * c8);
        }
    }
}

// V^T fp32 [rows, S L] (times a factor per row, or as it is) -> (hi, lo) in 16 x 32 blocks per sequence, zeros from L to whole 64s; inside 16 keys the order
// 0-3, 8-11, 4-7, 12-15.  Four consecutive keys a thread.
template <bool F16>
__global__ __launch_bounds__(256) void vt_blocks_kernel(const float* __restrict__ in, const float* __restrict__ scale, int rows, int S, int L, int kb, bf16* __restrict__ hi, long long vseq,
                                                        long long vlo) {
    const int k4s = kb * 8;
    const long long tot = (long long)rows * S * k4s;
    for (long long i = blockIdx.x * 256LL + threadIdx.x; i < tot; i += (long long)gridDim.x * 256) {
        const int k = (int)(i % k4s) * 4, r = (int)(i / k4s % rows), sq = (int)(i / k4s / rows);
        float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
        if (k < L) v = *(const float4*)(in + (long long)r * S * L + (long long)sq * L + k);
        const float f = scale ? scale[r] : 1.f;
        float x[4] = {v.x * f, v.y * f, v.z * f, v.w * f};
        union { unsigned short h[4]; uint2 u; } a, b;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            // the product is rounded to fp32 here: folded into one of the two conversions (one rounding instead of two) the stored high part and the one that the low part
            // is taken from differ now and then, by a unit of the high part
            asm volatile("" : "+v"(x[j]));
            a.h[j] = enc<F16>(x[j]); b.h[j] = enc<F16>(x[j] - dec<F16>(a.h[j])); }
        const int q = (k >> 2) & 3, pos = (k & ~15) + (q == 1 ? 8 : q == 2 ? 4 : 4 * q);
        const long long o = sq * vseq + tboa_blocked_offset(r, pos, kb);
        *(uint2*)(hi + o) = a.u; *(uint2*)(hi + vlo + o) = b.u;
    }
}

template <int DH, bool F16>
int launch(tboa_ctx* ctx, const Args& a) {
    constexpr int buf = NS * ring_slot<DH>(), rows = 32 * W * (DH + 8) * 2, cols = DH * (32 * W + 8) * 2, smem = buf > rows ? (buf > cols ? buf : cols) : rows > cols ? rows : cols;
    TB_HIP(ctx, hipFuncSetAttribute((const void*)attn_output_kernel<DH, F16>, hipFuncAttributeMaxDynamicSharedMemorySize, smem));
    hipLaunchKernelGGL((attn_output_kernel<DH, F16>), dim3((unsigned)a.total), dim3(64 * W), smem, ctx->stream, a);
    TB_KERNEL_CHECK(ctx);
    return 0;
}
int dispatch(tboa_ctx* ctx, int dh, const Args& a) {
    switch (dh) {
        case 32: return a.f16 ? launch<32, true>(ctx, a) : launch<32, false>(ctx, a);
        case 64: return a.f16 ? launch<64, true>(ctx, a) : launch<64, false>(ctx, a);
        case 96: return a.f16 ? launch<96, true>(ctx, a) : launch<96, false>(ctx, a);
        default: return a.f16 ? launch<128, true>(ctx, a) : launch<128, false>(ctx, a);
    }
}

}  // namespace

bool attn_output_supported(int L, int dh) { return L % 8 == 0 && (dh == 32 || dh == 64 || dh == 96 || dh == 128); }

size_t attn_output_v_elems(int dkv, int S, int L, int paths) { return (size_t)2 * paths * S * dkv * cdiv64(L, 64) * 64; }

int attn_output(tboa_ctx* ctx, const AttnOutput& q) {
    if (!attn_output_supported(q.L, q.dh) || q.Hq % q.rep || q.S <= 0 || !q.V || q.paths < 1 || q.paths > 2 || !q.VT32[0] || (q.paths > 1 && !q.VT32[1]) ||
        (q.rows ? q.paths != 1 || q.ldr % 8 || ((uintptr_t)q.rows & 15) : q.ldo % 8 != 0))
        return tboa_fail(ctx, TBOA_EINVAL, "attn_output: unsupported shape or missing buffer");
    const int Hkv = q.Hq / q.rep, dkv = Hkv * q.dh;
    Args a{};
    a.paths = q.paths; a.S = q.S; a.L = q.L; a.Hq = q.Hq; a.rep = q.rep; a.blocked = q.blocked; a.causal = q.causal; a.f16 = q.f16;
    a.scale2 = (float)(1.4426950408889634 / sqrt((double)q.dh));
    a.vkb = (int)cdiv64(q.L, 64) * 2; a.vseq = (long long)dkv * a.vkb * 32; a.vlo = a.vseq * q.S; a.vpath = 2 * a.vlo;
    a.V = q.V; a.rows = q.rows; a.ldr = q.ldr; a.ldo = q.ldo;
    for (int p = 0; p < q.paths; ++p) {
        a.path[p] = q.path[p]; a.OT[p] = q.OT[p]; a.OTl[p] = q.OTl[p];
        if (!q.path[p].Q || !q.path[p].K || (!q.rows && (!q.OT[p] || !q.OTl[p] || (((uintptr_t)q.OT[p] | (uintptr_t)q.OTl[p]) & 15))))
            return tboa_fail(ctx, TBOA_EINVAL, "attn_output: missing or misaligned buffer");
        // (row-major K^: byte offsets within a block of 32 keys, of 32 bits)
        if (!q.blocked && 32LL * Hkv * 3 * q.dh * 2 >= (1LL << 32)) return tboa_fail(ctx, TBOA_EINVAL, "attn_output: a sequence's keys exceed 4 GiB");
        const long long n4 = (long long)dkv * q.S * a.vkb * 8;
        const unsigned wgs = (unsigned)std::min<long long>(cdiv64(n4, 256), 16384);
        if (q.f16) hipLaunchKernelGGL(vt_blocks_kernel<true>, dim3(wgs), dim3(256), 0, ctx->stream, q.VT32[p], q.v_scale[p], dkv, q.S, q.L, a.vkb, q.V + p * a.vpath, a.vseq, a.vlo);
        else hipLaunchKernelGGL(vt_blocks_kernel<false>, dim3(wgs), dim3(256), 0, ctx->stream, q.VT32[p], q.v_scale[p], dkv, q.S, q.L, a.vkb, q.V + p * a.vpath, a.vseq, a.vlo);
        TB_KERNEL_CHECK(ctx);
    }
    const long long heads = (long long)q.paths * q.S * q.Hq;
    a.nqb = (int)cdiv64(q.L, 32 * W);
    a.total = heads * a.nqb; a.runs = a.total % 8 == 0;
    if (a.total > 0x7fffffffLL) return tboa_fail(ctx, TBOA_EINVAL, "attn_output: grid too large");
    ProfRec rec{}; bool timed = false;
    if (ctx->prof_on) TB_TRY(prof_begin(ctx, TBOA_PROF_PV, 2.0 * 6.0 * heads * q.dh * (q.causal ? 0.5 * q.L * (q.L + 1.0) : (double)q.L * q.L), rec, timed));
    TB_TRY(dispatch(ctx, q.dh, a));
    return prof_end(ctx, rec, timed);
}
