// Internal declarations shared by the translation units of libturboboa (not part of the ABI).
#pragma once
#include <hip/hip_runtime.h>
#include <hip/hip_bf16.h>
#include <stdint.h>
#include <stdio.h>
#include <stdarg.h>
#include <string.h>
#include <vector>
#include "../../include/turboboa.h"

struct ProfRec { hipEvent_t a, b; int tag; double flops; };

struct TileOrder { int tiles_m, tiles_n, flags, tile_rows, tile_cols; int* dev; int count; };   // gemm_bf16: launch order of the output tiles
// gemm_bf16, persistent kernel: per workgroup the list of (batch entry, tm << 16 | tn) it works through, `rounds` entries each
struct TileSchedule { int tiles_m, tiles_n, flags, batch, seg_len; int2* dev; int rounds, wgs; };

struct tboa_ctx {
    int device;
    hipStream_t stream;
    char err[768];
    void* ws;            // context-owned workspace
    size_t ws_bytes;
    int* d_status;       // device status words: [0..3] factorisation breakdown (two slots), [4] integer-form check,
                         // [TB_GSTAT_WORD ..] bookkeeping of the two-phase grid search
    int* h_status;       // pinned host mirror
    hipStream_t aux;     // second stream (default priority) for work of one call that is independent of what `stream` does
    hipEvent_t ev_fork, ev_join;
    double* splitk[2];   // partial sums of split fp64 contractions, TB_SPLITK_ELEMS each: launches on `stream`, launches on `aux`
    int prof_on;         // record HIP events around tagged GEMM launches
    std::vector<ProfRec> prof;
    long long counters[8];   // tboa_counter_id
    int plan_only = 0;       // a host-only context of the workspace queries: tboa_ws_reserve records the request and stops the call
    size_t plan_bytes = 0, plan_plain = 0;
    size_t no_room = (size_t)-1;   // a workspace from this size on is not asked for again: the device has refused one (tboa_reserve_workspace)
    std::vector<TileOrder> tile_orders;   // device tables owned by the context
    std::vector<TileSchedule> tile_schedules;
};

#define TB_GSTAT_WORD 8
#define TB_SPLITK_ELEMS ((size_t)1 << 22)     // 32 MiB
int tboa_fail(tboa_ctx* ctx, int code, const char* fmt, ...);

#define TB_HIP(ctx, call)                                                                          \
    do {                                                                                           \
        hipError_t e_ = (call);                                                                    \
        if (e_ != hipSuccess)                                                                      \
            return tboa_fail(ctx, TBOA_EHIP, "%s:%d %s: %s", __FILE__, __LINE__, #call,            \
                             hipGetErrorString(e_));                                               \
    } while (0)

#define TB_TRY(expr)                                                                               \
    do {                                                                                           \
        int rc_ = (expr);                                                                          \
        if (rc_ != 0) return rc_;                                                                  \
    } while (0)

#define TB_KERNEL_CHECK(ctx) TB_HIP(ctx, hipGetLastError())

// Bump allocator over the context workspace.  With base == nullptr it only counts bytes, so the same
// planning code sizes the workspace and then carves it.
struct Arena {
    char* base;
    size_t off;
    explicit Arena(void* b) : base((char*)b), off(0) {}
    template <typename T>
    T* get(size_t n) {
        size_t bytes = (n * sizeof(T) + 255) & ~(size_t)255;
        T* p = base ? (T*)(base + off) : nullptr;
        off += bytes;
        return p;
    }
};
// returns TB_PLAN_STOP (not an error) on a plan-only context, after recording `bytes`
#define TB_PLAN_STOP 1000
int tboa_ws_reserve(tboa_ctx* ctx, size_t bytes);
// for a call that has a form with residues (`full` bytes) and one without (`plain`): the first unless it is known or found not to fit
int tboa_ws_reserve_either(tboa_ctx* ctx, size_t full, size_t plain, bool& take_full);

static inline int64_t cdiv64(int64_t a, int64_t b) { return (a + b - 1) / b; }

// ---------------------------------------------------------------- gemm_f64.hip
struct GemmF64 {
    int M, N, K;
    double alpha, beta;
    const double* A; int64_t sam, sak;
    const double* B; int64_t sbk, sbn;
    double* C; int64_t ldc;
    int batch; int64_t strideA, strideB, strideC;
    // two-level batch: b -> (b / batch_inner, b % batch_inner); the *2 strides apply to the inner index
    int batch_inner = 1; int64_t strideA2 = 0, strideB2 = 0, strideC2 = 0;
    // optional restriction of the contraction range per output tile (operands with triangular zeros):
    // k_lo = max(klo_m ? tile row start : 0, klo_n ? tile col start : 0)
    // k_hi = min(khi_m ? tile row end : K, khi_n ? tile col end : K); tiles with k_lo >= k_hi write beta*C.
    int klo_m = 0, klo_n = 0, khi_m = 0, khi_n = 0;
    int skip_lower = 0;  // skip tiles entirely below the diagonal (col end <= row start): left untouched
    int skip_upper = 0;  // skip tiles entirely above the diagonal (row end <= col start)
    int skip_col0 = 0;   // column of C's first column relative to its first row, for the two tests above
    int diag_order = 0;  // rotate the tile columns of tile row r by r: spreads column-dependent contraction lengths over the XCDs
    const int* m_limit = nullptr;   // device array [batch]: rows m >= m_limit[b] of batch entry b are not computed
    // optional second pair of operands with the shapes, strides and batch strides of the first:
    // C = alpha (A B + A2 B2) + beta C in one pass (not combined with the contraction-range restrictions)
    const double* A2 = nullptr; const double* B2 = nullptr;
    // B symmetric (K == N): C = A T with T = twice the part of B below the diagonal tiles, the diagonal tiles once and nothing above
    // (T + T^T = 2 B): half the work where C only goes into symmetric forms, A B A'^T = (C A'^T + A C'^T) / 2 with C' = A' T.  The tile
    // width is the launch's own: two launches of the same shape (M, N, batch) have the same T.
    int sym = 0;
    int over_a = 0, over_b = 0;      // C may share memory with A / with B (C == A and C == B are seen without)
    int sum_inner = 0;   // C[outer] = alpha * sum over the batch_inner entries of A B + beta * C[outer] (strideC2 unused)
    int tag = -1;   // tboa_prof_tag of this launch (timed with HIP events when profiling is on)
};
int gemm_f64(tboa_ctx* ctx, const GemmF64& g);
double gemm_f64_model_us(int M, int N, int K);      // what a product without restrictions takes, as gemm_f64's choice of tiles models it
// brackets a tagged launch with HIP events on the context's current stream when profiling is on
int prof_begin(tboa_ctx* ctx, int tag, double flops, ProfRec& rec, bool& timed);
int prof_end(tboa_ctx* ctx, const ProfRec& rec, bool timed);

// ---------------------------------------------------------------- gemm_rns.hip
// fp64 products as products of residues (signed bytes).  An operand is prepared once (norms -> exponents -> residues) and may serve many products.
#define TB_RNS_MODULI 15
constexpr int RNS_BITS_A = 57, RNS_BITS_B = 58;      // bits of the rows' 2-norms: together with the sign and half a bit of room, what 15 moduli hold
constexpr int RNS_CHUNKS = 64;                       // partial sums of rns_norms over a row-contiguous source: RNS_CHUNKS * rns_squares_elems(rows) doubles
struct RnsSource {
    const double* a; long long ld, stride;      // element (r, k): a[r ld + k] (kc), else a[k ld + r]; stride: batch entries
    int kc, rows, k;
    int half;                                    // symmetric source: twice what is before the diagonal, the diagonal once (as GemmF64::sym)
    int before;                                  // > 0: only what lies before the row's own block of that many indices (k < r - r % before) counts, the rest is zero
    const int* kexp; int ksign;                  // column k times 2^(ksign kexp[k])
    const int* exp_shift;                        // everything times 2^(ksign exp_shift[0])
    const int* row_limit;                        // device word: rows from there on are not needed
};
struct RnsOperand { signed char* p; size_t plane; long long stride; int kpad; int* e; long long e_stride; };      // p: [batch][planes]
struct RnsGemm {
    const RnsOperand *A, *B; const RnsOperand* B2 = nullptr;      // C = alpha (A B^T [+ A' B2^T, A' = the K columns of A after the first K]) + beta C
    int a_row = 0, b_row = 0, a_k = 0, b_k = 0;                    // first row (multiple of 16) and first contraction index (multiple of 64)
    int M, N, K, batch = 1;
    int row0 = 0;      // of C within the matrix that the limits below speak of (multiple of 256)
    int klo_m = 0, klo_n = 0, khi_n = 0;      // as in GemmF64, with tiles of 256
    int upper = 0;     // C is only wanted above its diagonal: zero on and below it
    const int* m_limit = nullptr;
    double alpha, beta; double* C; long long ldc, strideC = 0;
    unsigned char* residues;      // rns_residue_bytes
};
int rns_pad(int k);
size_t rns_plane(int rows, int k);
size_t rns_squares_elems(int rows);
size_t rns_residue_bytes(int M, int N, int batch);
bool rns_takes(int M, int N, int K);      // what rns_gemm can do: sums of K terms (two operands' worth of them) within 32 bits and the quotients' 22, tiles within a grid
// operand whose rows are contiguous (second: a second source right after the first along k): exponents, `bits` below the norm each, and residues; bits RNS_GIVEN:
// the operand's exponents stand already
constexpr int RNS_GIVEN = -1;
int rns_rows(tboa_ctx* ctx, const RnsSource& s, const RnsSource* second, int batch, int bits, const RnsOperand& o, int koff = 0);
// operand whose rows are strided: sums of squares, exponents, residues
int rns_norms(tboa_ctx* ctx, const RnsSource& s, int batch, double* sq, long long sq_stride, double* part);
int rns_exps(tboa_ctx* ctx, int rows, int batch, const double* sq, long long sq_stride, int bits, int* e, long long e_stride);
int rns_columns(tboa_ctx* ctx, const RnsSource& s, int batch, const RnsOperand& o, int koff, const int* grown = nullptr, int panel = 0);
// columns that grow by panels (of `rows` columns whose squares are `panel`; the first fresh_below of them begin with it): sq, exponents, and which have a new one; rns_columns
// then makes the first `panel` indices of every row, the others of the rows that have grown
int rns_grow(tboa_ctx* ctx, int rows, int batch, const double* panel, long long panel_stride, double* sq, int sq_rows, long long sq_stride, int fresh_below, int bits, int* e, long long e_stride,
             int* grown);
// exponents of the rows of V, H = V V^T, from H's diagonal; before rns_rows with them: which rows are longer than H's diagonal says (sum: their squares over all panels)
int rns_diagonal_exps(tboa_ctx* ctx, int n, int batch, const double* H, int bits, int* e, double* sum, long long sum_stride);
int rns_row_guard(tboa_ctx* ctx, const RnsSource& s, int batch, int bits, const RnsOperand& o, double* sum, long long sum_stride);
// exponents of rows that are contiguous (norm < 2^(e + bits)); powers of two per channel for a contraction between columns of a weight (sq: their squares, of rns_norms) and rows of size
// 2^right[k] (size: exponents of the channels' sizes, half those of H's diagonal; x may be right).  The right operand takes x as kexp with ksign 1, the left one with -1
int rns_channel_sizes(tboa_ctx* ctx, int n, const double* H, int* size);
int rns_row_exps(tboa_ctx* ctx, const RnsSource& s, int bits, int* e);
int rns_channel_exps(tboa_ctx* ctx, int n, const double* sq, const int* size, const int* right, int* x);
int rns_balance(tboa_ctx* ctx, int rows, double* sq1, const double* sq2, int* f);
int rns_gemm(tboa_ctx* ctx, const RnsGemm& q);
double rns_model_us(int M, int N, int K, bool triangular, bool beta);
double rns_prepare_us(int rows, int k);

// ---------------------------------------------------------------- gemm_bf16.hip
struct GemmBf16 {
    int M, N, K;
    float alpha;
    const __hip_bfloat16* A; int64_t lda;
    const __hip_bfloat16* B; int64_t ldb;
    void* C; int64_t ldc; int c_dtype; int accumulate; int flags;
    void* C2 = nullptr;   // with TBOA_GEMM_C_HILO: second 16-bit result buffer (the low parts), laid out as C
    float lo_scale = 1.f; // with TBOA_GEMM_C_HILO_HALF: the low parts are stored times this (a power of two that keeps them normal numbers)
    int batch; int64_t strideA, strideB, strideC;
    // two-level batch: z -> (z / batch_inner, z % batch_inner); the *2 strides apply to the inner index
    int batch_inner = 1; int64_t strideA2 = 0, strideB2 = 0, strideC2 = 0;
    int tag = -1;   // tboa_prof_tag of this launch (timed with HIP events when profiling is on)
    int kseg = 0;   // > 0: K is a concatenation of K/kseg segments; TBOA_GEMM_CAUSAL_K then limits each segment
    // nterms > 1: the contraction runs over nterms operand pairs, K / nterms columns each, the t-th pair read from termA[t], termB[t]
    // (laid out and strided as A and B; A = termA[0], B = termB[0]): C = sum_t termA[t] termB[t]^T in one pass over the accumulators
    // (LDS-direct kernels; kseg only with the persistent one).
    int nterms = 1; const __hip_bfloat16* termA[4] = {}; const __hip_bfloat16* termB[4] = {};
    // dispatched kernel: the sum of the terms before the last is multiplied by this power of two when the last term begins (low parts stored with a
    // factor of their own go first)
    float last_scale = 1.f;
    // dispatched LDS-direct kernel, a single bf16 result: C = round(A B^T * col_scale[column] + residual) (each or NULL; residual laid out as C)
    const float* col_scale = nullptr; const __hip_bfloat16* residual = nullptr;
    // B holds gate rows, then as many up rows (N = 2 N', N' a multiple of 32, all of B below 4 GiB); the result has N' columns:
    // C = round(silu(A B_gate^T * col_scale) * (A B_up^T * up_scale))
    bool gate_up = false; const float* up_scale = nullptr;
    // dispatched kernel: device array, one int per batch entry: only its first min(segs, nterms) terms are taken; K is then the length of
    // ONE term and the flops counted are those of one
    const int* segs = nullptr;
};
// internal flag: a 16-bit result leaves as an exact-to-16-bit pair of bf16 values (hi into C, lo into C2), whatever the operands
#define TBOA_GEMM_C_HILO 0x10000
#define TBOA_GEMM_C_HILO_HALF 0x20000     // (with C_HILO) the pair is IEEE half, 22 significant bits, instead of bf16, 16: for values known to fit half
// internal flag: A and B hold signed bytes, two in every 16-bit element (K, lda, ldb and strides count elements; 16 x 32 blocks hold 64 bytes of a row), C receives
// 32-bit integers.  Several terms are digits of B to the base 256, the highest first: C = sum_t 256^(terms - 1 - t) A termB[t]^T, modulo 2^32.
#define TBOA_GEMM_I8 0x40000
int gemm_bf16_nt(tboa_ctx* ctx, const GemmBf16& g);
// C = scale * sum_t termA[t] termB[t]^T as one fp32 matrix whose sums round as those of `chunk` (a multiple of 128) contraction indices do (gemm_128x256_kernel); nterms pairs of K / nterms
// columns each, K / nterms a multiple of 32, no batch, C fp32; flags: LOWER (only the tiles on or below the diagonal are written), F16, A_TILED and B_TILED together.
// gemm_gram_tiles: how many workgroups such a launch has.
int gemm_gram(tboa_ctx* ctx, const GemmBf16& g, double scale, int chunk);
long long gemm_gram_tiles(int M, int N, int lower);

// Transposed causal attention probabilities of all heads of one sequence as (hi, lo) pairs of 16-bit values (IEEE half
// when f16, else bf16): Pt[g][i][r L + t] = A_h[t, i], h = g rep + r, every [L, ldp] matrix of a KV group in 16 x 32 blocks,
// rows i up to the end of the 256-tile that holds t written (zeros beyond the diagonal).  dhi, dlo: A - A~ of a second
// score matrix (nullptr without one).
struct PtOut { __hip_bfloat16 *hi, *lo, *dhi, *dlo; };
// factor on the probabilities attn_probs_t writes as IEEE half (f16 set), and that attn_output holds as such; bf16 ones are unscaled
#define ATTN_PROBS_HALF_SCALE 16384.f
// How the (hi, lo) pairs of Q^ and K^ are encoded, per score matrix: a device word per operand that holds the bits of the
// largest magnitude of that operand's fp32 values, in which case the pairs are IEEE half values of the operand times
// 2^tboa_half_exp(word) (22 significant bits wherever the magnitude is within 2^-17 of the largest), or a negative word / a
// null pointer: pairs of bf16, unscaled (16 significant bits).
struct QkScale { const int *qa, *ka, *qb, *kb; };
// e such that amax 2^e lies in [2^13, 2^14) (amax: the bits of a non-negative float); 0 for zero, denormal or non-finite amax
__host__ __device__ __forceinline__ int tboa_half_exp(int amax_bits) {
    const int E = (amax_bits >> 23) & 0xff;
    return (E < 13 || E == 255) ? 0 : 140 - E;
}
// straight from the blocked 3-term operands Q^ [Hq][L, 3 dh], K^ [Hkv][L, 3 dh] of the score product (second pair Qb, Kb or
// nullptr); attn_probs_t_supported tells which shapes the kernel takes
bool attn_probs_t_supported(int L, int dh);
int attn_probs_t(tboa_ctx* ctx, const __hip_bfloat16* Qa, const __hip_bfloat16* Ka, const __hip_bfloat16* Qb, const __hip_bfloat16* Kb, int L,
                 int Hq, int rep, int dh, PtOut out, long long ldp, long long group_stride, int f16, QkScale qs);

// ---------------------------------------------------------------- attn_output.hip
// Attention outputs of S whole sequences of L tokens, one or two paths (operands of their own, the same shapes).  Q, K: the 3-term operands of the score product of all
// sequences (blocked: one [L, 3 dh] matrix in 16 x 32 blocks per sequence and head, else rows [S L][heads][3 dh]); qa, ka: words of their encoding (QkScale), one per sequence,
// or null; VT32: V^T [Hkv dh][S L] in fp32, v_scale: a factor per row or null; V: room for attn_output_v_elems 16-bit elements.
// Results: rows (one path): token-major bf16 [S L][ldr]; else O^T [Hq dh][ldo] per path as (hi, lo) pairs in OT, OTl (half when f16, else bf16).
struct AttnPath { const __hip_bfloat16 *Q, *K; const int *qa, *ka; };
struct AttnOutput {
    int S, L, Hq, rep, dh, paths, blocked, causal, f16;
    AttnPath path[2];
    const float *VT32[2], *v_scale[2];
    __hip_bfloat16* V;
    __hip_bfloat16 *OT[2], *OTl[2]; long long ldo;
    __hip_bfloat16* rows; long long ldr;
};
bool attn_output_supported(int L, int dh);
size_t attn_output_v_elems(int dkv, int S, int L, int paths);
int attn_output(tboa_ctx* ctx, const AttnOutput& q);

// ---------------------------------------------------------------- device code that several files use
// One 1 KB block global -> LDS: lane l moves the 16 bytes at base + voff to lds_addr + 16 l.  Written as inline assembly so that the compiler does not pair every later LDS read with a wait for
// ALL outstanding loads (it cannot tell that the ring slot being filled is not the one being read); the explicit wait_loads_but + barrier of the main loops is the
// synchronisation.
__device__ __forceinline__ void lds_direct_16(unsigned voff, const char* base, unsigned lds_addr) {
    asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %2" ::"v"(voff), "s"(lds_addr), "s"(base) : "memory", "m0");
}
// waits until no more than the N newest loads are in flight, and for all LDS reads
template <int N>
__device__ __forceinline__ void wait_loads_but() { asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"(N) : "memory"); }
__device__ __forceinline__ double lane_value(double v, int lane) {      // of a lane that is the same for the wavefront
    const int lo = __builtin_amdgcn_readlane(__double2loint(v), lane), hi = __builtin_amdgcn_readlane(__double2hiint(v), lane);
    return __hiloint2double(hi, lo);
}
// element offset of (r, c) in a matrix kept in the 16 x 32 blocks the bf16 GEMM can read and write (TBOA_GEMM_*_TILED);
// kb = leading dimension / 32
__device__ __forceinline__ long long tboa_blocked_offset(long long r, long long c, long long kb) {
    const int ri = (int)(r & 15), ci = (int)(c & 31);
    return ((r >> 4) * kb + (c >> 5)) * 512 + ri * 32 + (((ci >> 3) ^ (ri >> 2)) << 3) + (ci & 7);
}

// ---------------------------------------------------------------- factor.hip
// H64 [batch, n, n] fp64, overwritten; U [batch, n, n] fp64 out.  Checks the device status and
// returns TBOA_ENOTSPD on breakdown (synchronises).  tmp: workspace of batch * n * chol_tmp_pitch(n) doubles,
// dinv: batch * ceil(n / TB_FACT_NB) * TB_FACT_NB^2 doubles.
#define TB_FACT_NB 64     // diagonal blocks factored inside LDS
#define TB_FACT_OB 512    // outer blocks: width of the large trailing updates
static inline int chol_tmp_pitch(int n) { return n <= TB_FACT_OB ? TB_FACT_NB : TB_FACT_OB; }
// status_slot: which pair of device status words records a breakdown (0 or 2); defer_status: do not wait for them here,
// the caller checks with chol_status_f64 once the work has been joined.
// rns: workspace of the form that takes the large updates to the integer matrix cores (chol_rns_plan; its V.p null: fp64 throughout).
struct CholRns { RnsOperand V, U; unsigned char* res; double *sq, *panel, *part; int* grown; };
void chol_rns_plan(int n, int batch, Arena& ar, CholRns& w);
int chol_inv_upper_f64(tboa_ctx* ctx, int n, int batch, double* H64, double* U, double* tmp, double* dinv, int status_slot = 0,
                       bool defer_status = false, const CholRns* rns = nullptr);
int chol_status_f64(tboa_ctx* ctx, int status_slot);
int chol_static_init(int device);   // looks up the device address of the static scratch of tboa_chol_inv_upper_static (device current)
int launch_f32_to_f64_damp(tboa_ctx* ctx, int n, int batch, const float* H, double damp, double* out);
int launch_symmetric_f64_damp(tboa_ctx* ctx, int n, int batch, const float* H, double damp, double* out);      // of (H + H^T) / 2

// ---------------------------------------------------------------- sweep.hip
// the rows of a step: block row R = h nbr + r is layer row h dh + i0 + r
struct BlockMap { int nbr, dh, i0; };
__device__ __forceinline__ long long layer_row(const BlockMap& m, int R) {
    return (long long)(R / m.nbr) * m.dh + m.i0 + (R % m.nbr);
}
constexpr int SWEEP_SP = 512;      // columns whose updates of the columns further right are applied in one product: the widest sweep launch
struct SweepArgs {
    const double* Wk; int n; int nbr; BlockMap map;
    const double* U; const double* P; int per_head;   // U, P: [n, n] or [n_heads, n, n]; P null: no deviation term
    const double* nv;                // lazy: block array [rows, n], P holds S (see run_layer)
    int c0, width;                   // columns c0 .. c0 + width - 1, width <= SWEEP_SP; more than 16 only where the grid groups are whole 16s
    const double* s; const double* z; int ng, gsz; double maxq;      // grids per layer row and group of gsz columns
    uint8_t* codes; double* Q;       // layer arrays [d_out, n]
    double* Epan; double* Wsnap;     // block arrays [rows, epitch], already offset to the first column
    int epitch;
};
int launch_sweep(tboa_ctx* ctx, const SweepArgs& a, int nh, bool lazy);

// ---------------------------------------------------------------- misc elementwise (elementwise.hip)
int launch_fill_f64(tboa_ctx* ctx, double* p, int64_t n, double v);
int launch_fill_f32(tboa_ctx* ctx, float* p, int64_t n, float v);
int launch_cvt_to_f64(tboa_ctx* ctx, const void* src, int dtype, double* dst, int64_t n);
int launch_cvt_f64_to_f32(tboa_ctx* ctx, const double* src, float* dst, int64_t n);
int launch_cvt_f32_to_f64(tboa_ctx* ctx, const float* src, double* dst, int64_t n);
// out[r, c] = in[r, c] for c > r else 0 (square n x n, batch)
int launch_strict_upper_f64(tboa_ctx* ctx, double* a, int n, int batch);
// symmetrise: upper <- lower (fp32, n x n, batch)
int launch_mirror_lower_f32(tboa_ctx* ctx, float* a, int n, int batch);
int launch_sub_f64(tboa_ctx* ctx, const double* a, const double* b, double* out, int64_t n);

// ---------------------------------------------------------------- hessian_f64.hip
int build_hessians_f64(tboa_ctx* ctx, const tboa_attn_desc* d, const void* X, const void* X_fp, const void* Wq, const void* Wk,
                       const void* Wv, const void* Wo, float* Hin_qk, float* R_qk, float* Hout_q, float* Hout_k, float* Hin_v,
                       float* R_v, float* Hout_v);
int build_hessian_out_proj_f64(tboa_ctx* ctx, const tboa_attn_desc* d, const void* X, const void* X_fp, const float* Wq_deq,
                               const float* Wk_deq, const float* Wv_deq, const void* Wq, const void* Wk, const void* Wv,
                               float* Hin_o, float* R_o);
int build_hessian_linear_f64(tboa_ctx* ctx, long long T, int n, double alpha, const float* X, const float* X_fp, float* H_in, float* R);
int attention_forward_f64(tboa_ctx* ctx, const tboa_attn_desc* d, const float* X, const float* Wq, const float* Wk, const float* Wv, float* O);
int linear_forward_f64(tboa_ctx* ctx, long long T, int din, int dout, const float* X, const float* W, const float* Res, float* Y);
int swiglu_forward_f64(tboa_ctx* ctx, long long T, int d, int dff, const float* X, const float* Wg, const float* Wu, float* Act);
