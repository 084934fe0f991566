// Table 1 Hessians for fp32 inputs: every contraction on the fp64 matrix cores (small problems, reference-grade
// accuracy).  Literal order of Table 1: projections, A_h = softmax(Q_h K_h^T / sqrt(d_h)) per sequence and head,
// Y = A_h X_s, sums of outer products over tokens.  These calls are bound by launches: the products of a chunk of sequences and KV
// groups are one launch each (per query head of a group where the operands' layout asks for it), and the sums over the chunk's
// sequences and heads are one long contraction: the tiny configuration (8 sequences, 4 heads) takes 40 launches instead of 350.  The bf16 path for large blocks lives in hessian_bf16.hip.
#include "internal.h"
#include <algorithm>
#include <math.h>

namespace {

// in place: every row t of the [L, L] matrices becomes softmax(row[:k_end]) with k_end = t+1 (causal) or L; zeros elsewhere.  One wavefront per row.
__global__ __launch_bounds__(256) void softmax_f64_kernel(double* __restrict__ S, long long rows, int L, int causal) {
    const int lane = threadIdx.x & 63;
    const long long row = (long long)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (row >= rows) return;
    const int t = (int)(row % L);
    double* s = S + row * L;
    const int kend = causal ? t + 1 : L;
    double m = -INFINITY;
    for (int k = lane; k < kend; k += 64) m = fmax(m, s[k]);
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) m = fmax(m, __shfl_xor(m, o, 64));
    double sum = 0.0;
    for (int k = lane; k < kend; k += 64) sum += exp(s[k] - m);
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) sum += __shfl_xor(sum, o, 64);
    for (int k = lane; k < L; k += 64) s[k] = (k < kend) ? exp(s[k] - m) / sum : 0.0;
}

struct F64Attn {
    tboa_ctx* ctx; const tboa_attn_desc* d;
    int T, dm, Hq, Hkv, dh, L, S, rep, dq, dkv;
};

inline GemmF64 mk(int M, int N, int K, double alpha, const double* A, int64_t sam, int64_t sak, const double* B, int64_t sbk,
                  int64_t sbn, double beta, double* C, int64_t ldc) {
    GemmF64 g{};
    g.M = M; g.N = N; g.K = K; g.alpha = alpha; g.beta = beta; g.A = A; g.sam = sam; g.sak = sak; g.B = B; g.sbk = sbk; g.sbn = sbn;
    g.C = C; g.ldc = ldc; g.batch = 1;
    return g;
}

// Sequences, KV groups and query heads of a group taken together: as many as keep the probabilities and two [L, width] results per head within
// 1 GiB, but one head at least.  The same for every set of outputs (a build without the full-precision path needs one result only), so that no
// call needs more than the one that asks for everything.
struct Chunk { int G, gc, rc; };
Chunk pick_chunk(const F64Attn& a, int width) {
    const double per_head = (double)a.L * (a.L + 2.0 * width) * 8.0, per_group = a.rep * per_head, room = 1073741824.0;
    if (per_group > room) return Chunk{1, 1, (int)std::min<double>(a.rep, std::max(1.0, floor(room / per_head)))};
    int gc = (int)std::min<double>(a.Hkv, floor(room / per_group));
    int G = gc < a.Hkv ? 1 : (int)std::min<double>(a.S, std::max(1.0, floor(room / (per_group * a.Hkv))));
    if ((long long)G * gc > 32768) { G = 32768 / gc; if (G < 1) { G = 1; gc = 32768; } }
    return Chunk{G, gc, a.rep};
}

// probabilities P[g][s][r][L, L] of the sequences s0 .. s0 + Gc - 1, the KV groups g0 .. g0 + gc - 1 and rc of their query heads (g rep + r0 + r)
// from the projected activations Qa [T, dq], Ka [T, dkv]
int attn_probs(const F64Attn& a, const double* Qa, const double* Ka, int s0, int Gc, int g0, int gc, int r0, int rc, double* P) {
    const long long L = a.L, LL = L * L;
    for (int r = 0; r < rc; ++r) {
        GemmF64 g = mk(a.L, a.L, a.dh, 1.0 / sqrt((double)a.dh), Qa + s0 * L * a.dq + ((long long)g0 * a.rep + r0 + r) * a.dh, a.dq, 1,
                       Ka + s0 * L * a.dkv + (long long)g0 * a.dh, 1, a.dkv, 0.0, P + r * LL, L);
        g.batch = gc * Gc; g.batch_inner = Gc;
        g.strideA = (long long)a.rep * a.dh; g.strideA2 = L * a.dq; g.strideB = a.dh; g.strideB2 = L * a.dkv;
        g.strideC = (long long)Gc * rc * LL; g.strideC2 = rc * LL;
        TB_TRY(gemm_f64(a.ctx, g));
    }
    const long long rows = (long long)gc * Gc * rc * L;
    hipLaunchKernelGGL(softmax_f64_kernel, dim3((unsigned)((rows + 3) / 4)), dim3(256), 0, a.ctx->stream, P, rows, a.L, a.d->causal);
    TB_HIP(a.ctx, hipGetLastError());
    return 0;
}

}  // namespace

int build_hessians_f64(tboa_ctx* ctx, const tboa_attn_desc* d, const void* X, const void* X_fp, const void* Wq, const void* Wk,
                       const void* Wv, const void* Wo, float* Hin_qk, float* R_qk, float* Hout_q, float* Hout_k, float* Hin_v,
                       float* R_v, float* Hout_v) {
    (void)Wv;
    F64Attn a{ctx, d, d->n_seqs * d->seq_len, d->d_model, d->n_q_heads, d->n_kv_heads, d->head_dim, d->seq_len, d->n_seqs,
              d->n_q_heads / d->n_kv_heads, d->n_q_heads * d->head_dim, d->n_kv_heads * d->head_dim};
    const int T = a.T, dm = a.dm, Hq = a.Hq, Hkv = a.Hkv, dh = a.dh, L = a.L, dq = a.dq, dkv = a.dkv;
    const bool fp = X_fp != nullptr;
    const bool rv = fp && R_v;
    const Chunk ck = pick_chunk(a, dm);
    double *X64, *Xf64, *dX, *Wq64, *Wk64, *Wo64, *Qa, *Ka, *Qf, *Kf, *P, *Y, *Yf, *Hin, *Rq, *Hoq, *Hok, *Hiv, *Rv, *Hov;
    for (int pass = 0; pass < 2; ++pass) {
        Arena ar(pass ? ctx->ws : nullptr);
        X64 = ar.get<double>((size_t)T * dm); Xf64 = fp ? ar.get<double>((size_t)T * dm) : nullptr; dX = fp ? ar.get<double>((size_t)T * dm) : nullptr;
        Wq64 = ar.get<double>((size_t)dq * dm); Wk64 = ar.get<double>((size_t)dkv * dm); Wo64 = ar.get<double>((size_t)dm * dq);
        Qa = ar.get<double>((size_t)T * dq); Ka = ar.get<double>((size_t)T * dkv);
        Qf = rv ? ar.get<double>((size_t)T * dq) : nullptr; Kf = rv ? ar.get<double>((size_t)T * dkv) : nullptr;
        const size_t mats = (size_t)ck.gc * ck.G * ck.rc;
        P = ar.get<double>(mats * L * L); Y = ar.get<double>(mats * L * dm); Yf = rv ? ar.get<double>(mats * L * dm) : nullptr;
        Hin = ar.get<double>((size_t)dm * dm); Rq = fp ? ar.get<double>((size_t)dm * dm) : nullptr;
        Hoq = ar.get<double>((size_t)Hq * dh * dh); Hok = ar.get<double>((size_t)Hkv * dh * dh); Hov = ar.get<double>((size_t)Hkv * dh * dh);
        Hiv = ar.get<double>((size_t)Hkv * dm * dm); Rv = rv ? ar.get<double>((size_t)Hkv * dm * dm) : nullptr;
        if (!pass) TB_TRY(tboa_ws_reserve(ctx, ar.off));
    }
    TB_TRY(launch_cvt_to_f64(ctx, X, TBOA_F32, X64, (int64_t)T * dm));
    TB_TRY(launch_cvt_to_f64(ctx, Wq, TBOA_F32, Wq64, (int64_t)dq * dm));
    TB_TRY(launch_cvt_to_f64(ctx, Wk, TBOA_F32, Wk64, (int64_t)dkv * dm));
    TB_TRY(launch_cvt_to_f64(ctx, Wo, TBOA_F32, Wo64, (int64_t)dm * dq));
    // H_in = X X^T (paper's X is channels x tokens) and R = alpha dX X^T
    TB_TRY(gemm_f64(ctx, mk(dm, dm, T, 1.0, X64, 1, dm, X64, dm, 1, 0.0, Hin, dm)));
    if (fp) {
        TB_TRY(launch_cvt_to_f64(ctx, X_fp, TBOA_F32, Xf64, (int64_t)T * dm));
        TB_TRY(launch_sub_f64(ctx, X64, Xf64, dX, (int64_t)T * dm));
        TB_TRY(gemm_f64(ctx, mk(dm, dm, T, d->alpha, dX, 1, dm, X64, dm, 1, 0.0, Rq, dm)));
    }
    // projections
    TB_TRY(gemm_f64(ctx, mk(T, dq, dm, 1.0, X64, dm, 1, Wq64, 1, dm, 0.0, Qa, dq)));
    TB_TRY(gemm_f64(ctx, mk(T, dkv, dm, 1.0, X64, dm, 1, Wk64, 1, dm, 0.0, Ka, dkv)));
    if (rv) {
        TB_TRY(gemm_f64(ctx, mk(T, dq, dm, 1.0, Xf64, dm, 1, Wq64, 1, dm, 0.0, Qf, dq)));
        TB_TRY(gemm_f64(ctx, mk(T, dkv, dm, 1.0, Xf64, dm, 1, Wk64, 1, dm, 0.0, Kf, dkv)));
    }
    // H_out of W_Q,h: K_g^T K_g ; of W_K,g: sum_h Q_h^T Q_h ; of W_V,g: sum_h W_out,h^T W_out,h
    // (a launch has at most 65535 batch entries: as many KV groups at a time as that allows)
    const int per = std::max(1, std::min(Hkv, 65535 / a.rep)), rc = std::min(a.rep, 65535);
    for (int g0 = 0; g0 < Hkv; g0 += per) {
        const long long hh = (long long)dh * dh, h0 = (long long)g0 * a.rep;
        const int gc = std::min(per, Hkv - g0);
        GemmF64 q = mk(dh, dh, T, 1.0, Ka + (long long)g0 * dh, 1, dkv, Ka + (long long)g0 * dh, dkv, 1, 0.0, nullptr, dh);
        q.strideA = dh; q.strideB = dh; q.strideC = a.rep * hh; q.strideC2 = hh;
        for (int r0 = 0; r0 < a.rep; r0 += rc) {
            q.batch_inner = std::min(rc, a.rep - r0); q.batch = gc * q.batch_inner; q.C = Hoq + (h0 + r0) * hh;
            TB_TRY(gemm_f64(ctx, q));
        }
        GemmF64 k = mk(dh, dh, T, 1.0, Qa + h0 * dh, 1, dq, Qa + h0 * dh, dq, 1, 0.0, Hok + g0 * hh, dh);
        k.batch = gc * a.rep; k.batch_inner = a.rep; k.sum_inner = 1; k.strideA = (long long)a.rep * dh; k.strideB = k.strideA; k.strideA2 = dh; k.strideB2 = dh; k.strideC = hh;
        TB_TRY(gemm_f64(ctx, k));
        k.K = dm; k.A = Wo64 + h0 * dh; k.B = k.A; k.C = Hov + g0 * hh;
        TB_TRY(gemm_f64(ctx, k));
    }
    // H_in of W_V,g: sum over heads of the group and sequences of (A_h X_s)^T (A_h X_s)
    const long long LL = (long long)L * L, Ld = (long long)L * dm, dd = (long long)dm * dm;
    for (int s0 = 0; s0 < a.S; s0 += ck.G)
        for (int g0 = 0; g0 < Hkv; g0 += ck.gc)
        for (int r0 = 0; r0 < a.rep; r0 += ck.rc) {
            const int Gc = std::min(ck.G, a.S - s0), gc = std::min(ck.gc, Hkv - g0), rc = std::min(ck.rc, a.rep - r0);
            const long long kk = (long long)Gc * rc * L;         // rows of Y of one KV group
            auto outputs = [&](const double* X, double* out) -> int {      // Y[g][s][r] = A X_s
                for (int r = 0; r < rc; ++r) {
                    GemmF64 y = mk(L, dm, L, 1.0, P + r * LL, L, 1, X + s0 * Ld, dm, 1, 0.0, out + r * Ld, dm);
                    y.batch = gc * Gc; y.batch_inner = Gc; y.strideA = Gc * rc * LL; y.strideA2 = rc * LL; y.strideB2 = Ld;
                    y.strideC = Gc * rc * Ld; y.strideC2 = rc * Ld;
                    TB_TRY(gemm_f64(ctx, y));
                }
                return 0;
            };
            if (kk > 2147483647LL) return tboa_fail(ctx, TBOA_EINVAL, "build_hessians: a KV group's rows exceed the range of int");
            TB_TRY(attn_probs(a, Qa, Ka, s0, Gc, g0, gc, r0, rc, P));
            TB_TRY(outputs(X64, Y));
            GemmF64 h = mk(dm, dm, (int)kk, 1.0, Y, 1, dm, Y, dm, 1, s0 || r0 ? 1.0 : 0.0, Hiv + g0 * dd, dm);
            h.batch = gc; h.strideA = kk * dm; h.strideB = h.strideA; h.strideC = dd;
            TB_TRY(gemm_f64(ctx, h));
            if (rv) {
                TB_TRY(attn_probs(a, Qf, Kf, s0, Gc, g0, gc, r0, rc, P));
                TB_TRY(outputs(Xf64, Yf));
                TB_TRY(launch_sub_f64(ctx, Y, Yf, Yf, gc * kk * dm));
                h.A = Yf; h.alpha = d->alpha; h.C = Rv + g0 * dd;
                TB_TRY(gemm_f64(ctx, h));
            }
        }
    if (Hin_qk) TB_TRY(launch_cvt_f64_to_f32(ctx, Hin, Hin_qk, (int64_t)dm * dm));
    if (fp && R_qk) TB_TRY(launch_cvt_f64_to_f32(ctx, Rq, R_qk, (int64_t)dm * dm));
    if (Hout_q) TB_TRY(launch_cvt_f64_to_f32(ctx, Hoq, Hout_q, (int64_t)Hq * dh * dh));
    if (Hout_k) TB_TRY(launch_cvt_f64_to_f32(ctx, Hok, Hout_k, (int64_t)Hkv * dh * dh));
    if (Hout_v) TB_TRY(launch_cvt_f64_to_f32(ctx, Hov, Hout_v, (int64_t)Hkv * dh * dh));
    if (Hin_v) TB_TRY(launch_cvt_f64_to_f32(ctx, Hiv, Hin_v, (int64_t)Hkv * dm * dm));
    if (rv) TB_TRY(launch_cvt_f64_to_f32(ctx, Rv, R_v, (int64_t)Hkv * dm * dm));
    return 0;
}

// attention output concat_h(A_h V_g(h)) [T, dq] for weights Wq/Wk/Wv (fp64) on activations Xa (fp64)
static int attn_output_f64(const F64Attn& a, Chunk ck, const double* Xa, const double* Wq64, const double* Wk64, const double* Wv64,
                           double* Qa, double* Ka, double* Va, double* P, double* O) {
    tboa_ctx* ctx = a.ctx;
    const int T = a.T, dm = a.dm, dq = a.dq, dkv = a.dkv, L = a.L, dh = a.dh;
    const long long LL = (long long)L * L;
    TB_TRY(gemm_f64(ctx, mk(T, dq, dm, 1.0, Xa, dm, 1, Wq64, 1, dm, 0.0, Qa, dq)));
    TB_TRY(gemm_f64(ctx, mk(T, dkv, dm, 1.0, Xa, dm, 1, Wk64, 1, dm, 0.0, Ka, dkv)));
    TB_TRY(gemm_f64(ctx, mk(T, dkv, dm, 1.0, Xa, dm, 1, Wv64, 1, dm, 0.0, Va, dkv)));
    for (int s0 = 0; s0 < a.S; s0 += ck.G)
        for (int g0 = 0; g0 < a.Hkv; g0 += ck.gc)
        for (int r0 = 0; r0 < a.rep; r0 += ck.rc) {
            const int Gc = std::min(ck.G, a.S - s0), gc = std::min(ck.gc, a.Hkv - g0), rc = std::min(ck.rc, a.rep - r0);
            TB_TRY(attn_probs(a, Qa, Ka, s0, Gc, g0, gc, r0, rc, P));
            for (int r = 0; r < rc; ++r) {
                GemmF64 o = mk(L, dh, L, 1.0, P + r * LL, L, 1, Va + (long long)s0 * L * dkv + (long long)g0 * dh, dkv, 1, 0.0,
                               O + (long long)s0 * L * dq + ((long long)g0 * a.rep + r0 + r) * dh, dq);
                o.batch = gc * Gc; o.batch_inner = Gc; o.strideA = Gc * rc * LL; o.strideA2 = rc * LL;
                o.strideB = dh; o.strideB2 = (long long)L * dkv; o.strideC = (long long)a.rep * dh; o.strideC2 = (long long)L * dq;
                TB_TRY(gemm_f64(ctx, o));
            }
        }
    return 0;
}

int build_hessian_out_proj_f64(tboa_ctx* ctx, const tboa_attn_desc* d, const void* X, const void* X_fp, const float* Wq_deq,
                               const float* Wk_deq, const float* Wv_deq, const void* Wq, const void* Wk, const void* Wv,
                               float* Hin_o, float* R_o) {
    F64Attn a{ctx, d, d->n_seqs * d->seq_len, d->d_model, d->n_q_heads, d->n_kv_heads, d->head_dim, d->seq_len, d->n_seqs,
              d->n_q_heads / d->n_kv_heads, d->n_q_heads * d->head_dim, d->n_kv_heads * d->head_dim};
    const int T = a.T, dm = a.dm, L = a.L, dq = a.dq, dkv = a.dkv;
    const bool fp = X_fp && R_o;
    const Chunk ck = pick_chunk(a, 0);
    double *X64, *Wq64, *Wk64, *Wv64, *Qa, *Ka, *Va, *P, *O, *Of, *H;
    for (int pass = 0; pass < 2; ++pass) {
        Arena ar(pass ? ctx->ws : nullptr);
        X64 = ar.get<double>((size_t)T * dm);
        Wq64 = ar.get<double>((size_t)dq * dm); Wk64 = ar.get<double>((size_t)dkv * dm); Wv64 = ar.get<double>((size_t)dkv * dm);
        Qa = ar.get<double>((size_t)T * dq); Ka = ar.get<double>((size_t)T * dkv); Va = ar.get<double>((size_t)T * dkv);
        P = ar.get<double>((size_t)ck.gc * ck.G * ck.rc * L * L);
        O = ar.get<double>((size_t)T * dq); Of = fp ? ar.get<double>((size_t)T * dq) : nullptr;
        H = ar.get<double>((size_t)dq * dq);
        if (!pass) TB_TRY(tboa_ws_reserve(ctx, ar.off));
    }
    TB_TRY(launch_cvt_to_f64(ctx, X, TBOA_F32, X64, (int64_t)T * dm));
    TB_TRY(launch_cvt_to_f64(ctx, Wq_deq, TBOA_F32, Wq64, (int64_t)dq * dm));
    TB_TRY(launch_cvt_to_f64(ctx, Wk_deq, TBOA_F32, Wk64, (int64_t)dkv * dm));
    TB_TRY(launch_cvt_to_f64(ctx, Wv_deq, TBOA_F32, Wv64, (int64_t)dkv * dm));
    TB_TRY(attn_output_f64(a, ck, X64, Wq64, Wk64, Wv64, Qa, Ka, Va, P, O));
    TB_TRY(gemm_f64(ctx, mk(dq, dq, T, 1.0, O, 1, dq, O, dq, 1, 0.0, H, dq)));
    TB_TRY(launch_cvt_f64_to_f32(ctx, H, Hin_o, (int64_t)dq * dq));
    if (fp) {
        TB_TRY(launch_cvt_to_f64(ctx, X_fp, TBOA_F32, X64, (int64_t)T * dm));
        TB_TRY(launch_cvt_to_f64(ctx, Wq, TBOA_F32, Wq64, (int64_t)dq * dm));
        TB_TRY(launch_cvt_to_f64(ctx, Wk, TBOA_F32, Wk64, (int64_t)dkv * dm));
        TB_TRY(launch_cvt_to_f64(ctx, Wv, TBOA_F32, Wv64, (int64_t)dkv * dm));
        TB_TRY(attn_output_f64(a, ck, X64, Wq64, Wk64, Wv64, Qa, Ka, Va, P, Of));
        TB_TRY(launch_sub_f64(ctx, O, Of, Of, (int64_t)T * dq));
        TB_TRY(gemm_f64(ctx, mk(dq, dq, T, d->alpha, Of, 1, dq, O, dq, 1, 0.0, H, dq)));
        TB_TRY(launch_cvt_f64_to_f32(ctx, H, R_o, (int64_t)dq * dq));
    }
    return 0;
}

// attention output concat_h(A_h V_g(h)) [T, Hq dh] (fp32) of fp32 activations and weights, on the fp64 matrix cores
int attention_forward_f64(tboa_ctx* ctx, const tboa_attn_desc* d, const float* X, const float* Wq, const float* Wk, const float* Wv, float* O) {
    F64Attn a{ctx, d, d->n_seqs * d->seq_len, d->d_model, d->n_q_heads, d->n_kv_heads, d->head_dim, d->seq_len, d->n_seqs,
              d->n_q_heads / d->n_kv_heads, d->n_q_heads * d->head_dim, d->n_kv_heads * d->head_dim};
    const int T = a.T, dm = a.dm, L = a.L, dq = a.dq, dkv = a.dkv;
    const Chunk ck = pick_chunk(a, 0);
    double *X64, *Wq64, *Wk64, *Wv64, *Qa, *Ka, *Va, *P, *O64;
    for (int pass = 0; pass < 2; ++pass) {
        Arena ar(pass ? ctx->ws : nullptr);
        X64 = ar.get<double>((size_t)T * dm);
        Wq64 = ar.get<double>((size_t)dq * dm); Wk64 = ar.get<double>((size_t)dkv * dm); Wv64 = ar.get<double>((size_t)dkv * dm);
        Qa = ar.get<double>((size_t)T * dq); Ka = ar.get<double>((size_t)T * dkv); Va = ar.get<double>((size_t)T * dkv);
        P = ar.get<double>((size_t)ck.gc * ck.G * ck.rc * L * L);
        O64 = ar.get<double>((size_t)T * dq);
        if (!pass) TB_TRY(tboa_ws_reserve(ctx, ar.off));
    }
    TB_TRY(launch_cvt_to_f64(ctx, X, TBOA_F32, X64, (int64_t)T * dm));
    TB_TRY(launch_cvt_to_f64(ctx, Wq, TBOA_F32, Wq64, (int64_t)dq * dm));
    TB_TRY(launch_cvt_to_f64(ctx, Wk, TBOA_F32, Wk64, (int64_t)dkv * dm));
    TB_TRY(launch_cvt_to_f64(ctx, Wv, TBOA_F32, Wv64, (int64_t)dkv * dm));
    TB_TRY(attn_output_f64(a, ck, X64, Wq64, Wk64, Wv64, Qa, Ka, Va, P, O64));
    return launch_cvt_f64_to_f32(ctx, O64, O, (int64_t)T * dq);
}

namespace {
__global__ void add_cvt_kernel(const double* __restrict__ Y, const float* __restrict__ Res, float* __restrict__ out, long long n) {
    for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < n; i += (long long)gridDim.x * blockDim.x)
        out[i] = (float)(Res ? Y[i] + (double)Res[i] : Y[i]);
}
}  // namespace

// Y = X W^T (+ Res), fp32 in and out, on the fp64 matrix cores
int linear_forward_f64(tboa_ctx* ctx, long long T, int din, int dout, const float* X, const float* W, const float* Res, float* Y) {
    double *X64, *W64, *Y64;
    for (int pass = 0; pass < 2; ++pass) {
        Arena ar(pass ? ctx->ws : nullptr);
        X64 = ar.get<double>((size_t)T * din); W64 = ar.get<double>((size_t)dout * din); Y64 = ar.get<double>((size_t)T * dout);
        if (!pass) TB_TRY(tboa_ws_reserve(ctx, ar.off));
    }
    TB_TRY(launch_cvt_to_f64(ctx, X, TBOA_F32, X64, (int64_t)T * din));
    TB_TRY(launch_cvt_to_f64(ctx, W, TBOA_F32, W64, (int64_t)dout * din));
    TB_TRY(gemm_f64(ctx, mk((int)T, dout, din, 1.0, X64, din, 1, W64, 1, din, 0.0, Y64, dout)));
    long long n = T * dout, gb = (n + 255) / 256; if (gb > 16384) gb = 16384;
    hipLaunchKernelGGL(add_cvt_kernel, dim3((unsigned)gb), dim3(256), 0, ctx->stream, Y64, Res, Y, n);
    TB_HIP(ctx, hipGetLastError());
    return 0;
}

namespace {
__global__ void swiglu_f64_kernel(const double* __restrict__ G, const double* __restrict__ U, float* __restrict__ out, long long n) {
    for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < n; i += (long long)gridDim.x * blockDim.x) {
        const double g = G[i];
        out[i] = (float)((g / (1.0 + exp(-g))) * U[i]);
    }
}
}  // namespace

// fp32 inputs: H = X^T X and R = alpha (X - X~)^T X on the fp64 matrix cores
int build_hessian_linear_f64(tboa_ctx* ctx, long long T, int n, double alpha, const float* X, const float* X_fp, float* H_in, float* R) {
    const bool fp = X_fp && R;
    double *X64, *Xf64, *H64;
    for (int pass = 0; pass < 2; ++pass) {
        Arena ar(pass ? ctx->ws : nullptr);
        X64 = ar.get<double>((size_t)T * n); Xf64 = fp ? ar.get<double>((size_t)T * n) : nullptr; H64 = ar.get<double>((size_t)n * n);
        if (!pass) TB_TRY(tboa_ws_reserve(ctx, ar.off));
    }
    TB_TRY(launch_cvt_to_f64(ctx, X, TBOA_F32, X64, (int64_t)T * n));
    TB_TRY(gemm_f64(ctx, mk(n, n, (int)T, 1.0, X64, 1, n, X64, n, 1, 0.0, H64, n)));
    TB_TRY(launch_cvt_f64_to_f32(ctx, H64, H_in, (int64_t)n * n));
    if (fp) {
        TB_TRY(launch_cvt_to_f64(ctx, X_fp, TBOA_F32, Xf64, (int64_t)T * n));
        TB_TRY(launch_sub_f64(ctx, X64, Xf64, Xf64, (int64_t)T * n));
        TB_TRY(gemm_f64(ctx, mk(n, n, (int)T, alpha, Xf64, 1, n, X64, n, 1, 0.0, H64, n)));
        TB_TRY(launch_cvt_f64_to_f32(ctx, H64, R, (int64_t)n * n));
    }
    return 0;
}

int swiglu_forward_f64(tboa_ctx* ctx, long long T, int d, int dff, const float* X, const float* Wg, const float* Wu, float* Act) {
    double *X64, *Wg64, *Wu64, *G, *U;
    for (int pass = 0; pass < 2; ++pass) {
        Arena ar(pass ? ctx->ws : nullptr);
        X64 = ar.get<double>((size_t)T * d); Wg64 = ar.get<double>((size_t)dff * d); Wu64 = ar.get<double>((size_t)dff * d);
        G = ar.get<double>((size_t)T * dff); U = ar.get<double>((size_t)T * dff);
        if (!pass) TB_TRY(tboa_ws_reserve(ctx, ar.off));
    }
    TB_TRY(launch_cvt_to_f64(ctx, X, TBOA_F32, X64, (int64_t)T * d));
    TB_TRY(launch_cvt_to_f64(ctx, Wg, TBOA_F32, Wg64, (int64_t)dff * d));
    TB_TRY(launch_cvt_to_f64(ctx, Wu, TBOA_F32, Wu64, (int64_t)dff * d));
    TB_TRY(gemm_f64(ctx, mk((int)T, dff, d, 1.0, X64, d, 1, Wg64, 1, d, 0.0, G, dff)));
    TB_TRY(gemm_f64(ctx, mk((int)T, dff, d, 1.0, X64, d, 1, Wu64, 1, d, 0.0, U, dff)));
    long long n = T * dff, gb = (n + 255) / 256; if (gb > 16384) gb = 16384;
    hipLaunchKernelGGL(swiglu_f64_kernel, dim3((unsigned)gb), dim3(256), 0, ctx->stream, G, U, Act, n);
    TB_HIP(ctx, hipGetLastError());
    return 0;
}
