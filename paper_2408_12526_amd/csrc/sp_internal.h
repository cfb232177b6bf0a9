// Internal declarations shared by the translation units of libsp_mi355x.so.
// Nothing here is part of the C ABI (that is include/sp.h).
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include <mutex>

#include "sp.h"

namespace sp {

// SP_DTYPE_FP8 is the bf16 path with fp8 copies of the four projection matrices: everything that asks "bf16 or fp32
// storage" treats the two alike.
inline bool bf16_path(const sp_config& c) { return c.dtype != SP_DTYPE_FP32; }

typedef __bf16 bf16;
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

#if defined(__HIPCC__)
// ---- device helpers shared by the projection kernels ---------------------------------------------
// GELU (erf form) for outputs that are rounded to bf16 afterwards, written with the complementary error function:
//   gelu(x) = x (1 + erf(x / sqrt 2)) / 2 = max(x, 0) - |x| erfc(|x| / sqrt 2) / 2,
//   log2 erfc(z) = z Q(z) on [0, 4.3], Q a degree-5 minimax fit (weighted for the absolute error of gelu);
//   erfc(4.3) = 1.2e-9, so |x| is clamped at 4.3 sqrt 2 (in the erfc term only: beyond it the term stays below 4e-9
//   instead of growing with |x|).
// Evaluated in fp32 the result is within 3.2e-7 of the exact function for every x (0.03 bf16 ulp at most where
// |gelu| > 1e-3).  One quarter-rate instruction (exp2) and nine full-rate ones: the epilogue of the FFN
// up-projection is bound by these vector instructions while the matrix cores wait (libm's erff costs several times
// more; the rational-exponential formula 7.1.26 of Abramowitz & Stegun needs a reciprocal as well).  To get there:
//   * the polynomial is in a = |x| directly (coefficient i carries 2^(-(i + 1) / 2)), so z is never formed, and the
//     halving of erfc rides in the exponent: |x| erfc / 2 = a 2^(a Q'(a) - 1), the -1 being the addend of the
//     multiply-add that forms the exponent;
//   * clamps are median-of-three instructions (one each for the clamp of x and for max(x, 0), the latter with the
//     largest finite float as its upper bound: fminf / fmaxf, and a median with an infinite bound, which the
//     compiler rewrites as one of them, cost a second instruction that quiets signalling NaNs first); |.| is an
//     operand modifier.
__device__ inline float gelu_erf_fast(float x)
{
    const float a = __builtin_fabsf(__builtin_amdgcn_fmed3f(x, -6.0811f, 6.0811f));
    float q = __builtin_fmaf(2.992383634e-05f, a, -7.398715825e-04f);
    q = __builtin_fmaf(q, a, 7.977455854e-03f);
    q = __builtin_fmaf(q, a, -5.323817581e-02f);
    q = __builtin_fmaf(q, a, -4.589156806e-01f);
    q = __builtin_fmaf(q, a, -1.151147127e+00f);
    const float e = __builtin_amdgcn_exp2f(__builtin_fmaf(q, a, -1.0f));
    return __builtin_fmaf(-a, e, __builtin_amdgcn_fmed3f(x, 0.0f, 3.402823466e+38f));
}

// The same function where the result is stored as an e4m3 code (three mantissa bits: steps of 2^-4 relative): the
// exponent is a cubic, log2(erfc(a / sqrt 2) / 2) ~ -1 + a (c0 + a (c1 + a c2)), fitted (minimax in the error of
// the function value) on [0, 4.5]; all three coefficients are negative, so it keeps falling beyond the fitted range and
// needs no clamp.  Within 8.6e-5 of the erf form everywhere, a thirtieth of the e4m3 step at the function's minimum
// (-0.17): four multiply-adds, one median and the exponential.
// The scaled form returns s gelu(y / s) for y = s x, with the coefficients divided by s, s^2, s^3 by the caller
// (gelu_q8_coefficients): the scale of the quantised output then costs no instruction per value.
constexpr float kGeluQ8C0 = -1.140919014e+00f, kGeluQ8C1 = -4.882554528e-01f, kGeluQ8C2 = -2.763128887e-02f;
__device__ inline float gelu_erf_q8_scaled(float y, float k0, float k1, float k2)
{
    const float a = __builtin_fabsf(y);
    float q = __builtin_fmaf(k2, a, k1);
    q = __builtin_fmaf(q, a, k0);
    const float e = __builtin_amdgcn_exp2f(__builtin_fmaf(q, a, -1.0f));
    return __builtin_fmaf(-a, e, __builtin_amdgcn_fmed3f(y, 0.0f, 3.402823466e+38f));
}
__device__ inline float gelu_erf_q8(float x) { return gelu_erf_q8_scaled(x, kGeluQ8C0, kGeluQ8C1, kGeluQ8C2); }

// ---- reductions over the 64 lanes of a wave, result in every lane -------------------------------------------------
// Inside a row of 16 lanes the second operand of each step comes through the data-parallel-primitive path of the
// instruction itself (neighbour in the pair, other pair of the quad, mirror image in the half row, mirror image in the
// row: after each step every lane of the growing group holds the group's result); rows 0|1 and 2|3, then the two halves
// of the wave, are exchanged by the row / half swap instructions (both operands hold the value; afterwards one has the
// even rows' (lower half's) data in every row (half), the other the odd rows' (upper half's)).  Eight instructions
// where six general lane permutations through LDS (`__shfl_xor`) take about forty, and no LDS round trips on the
// critical path.  Every lane of the wave must be active.  (The swaps are inline assembly with the two idle issue slots
// the hardware wants after a vector write of their operands: this toolchain's builtins return their first result
// twice.)
template <int CTRL>
__device__ inline float dpp_moved(float v)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, 0xf, 0xf, true));
}
__device__ inline void swap_rows(float& a, float& b)       // odd rows of a <-> even rows of b
{
    asm volatile("s_nop 1\n\tv_permlane16_swap_b32 %0, %1\n\ts_nop 1" : "+v"(a), "+v"(b));
}
__device__ inline void swap_halves(float& a, float& b)     // lanes 32-63 of a <-> lanes 0-31 of b
{
    asm volatile("s_nop 1\n\tv_permlane32_swap_b32 %0, %1\n\ts_nop 1" : "+v"(a), "+v"(b));
}
constexpr int kDppPair = 0xB1, kDppQuad = 0x4E, kDppHalfRowMirror = 0x141, kDppRowMirror = 0x140;
__device__ inline float wave_sum(float v)
{
    v += dpp_moved<kDppPair>(v);           // quad_perm [1, 0, 3, 2]
    v += dpp_moved<kDppQuad>(v);           // quad_perm [2, 3, 0, 1]
    v += dpp_moved<kDppHalfRowMirror>(v);
    v += dpp_moved<kDppRowMirror>(v);
    float a = v, b = v;
    swap_rows(a, b);
    v = a + b;
    a = v;
    b = v;
    swap_halves(a, b);
    return a + b;
}
__device__ inline float wave_max(float v)
{
    v = __builtin_fmaxf(v, dpp_moved<kDppPair>(v));
    v = __builtin_fmaxf(v, dpp_moved<kDppQuad>(v));
    v = __builtin_fmaxf(v, dpp_moved<kDppHalfRowMirror>(v));
    v = __builtin_fmaxf(v, dpp_moved<kDppRowMirror>(v));
    float a = v, b = v;
    swap_rows(a, b);
    v = __builtin_fmaxf(a, b);
    a = v;
    b = v;
    swap_halves(a, b);
    return __builtin_fmaxf(a, b);
}

typedef __attribute__((address_space(3))) void lds_void;
typedef __attribute__((address_space(1))) const void gbl_void;

// Sixteen bytes per lane straight into LDS: from base + soff (uniform) + voff to dst (uniform) + 16 lane.  The buffer form of the
// instruction, not the global one: the compiler counts it among the loads in flight, where behind a global one it
// waits for all of them (vmcnt(0)) before it uses the result of any.
__device__ __forceinline__ void load_lds16(const void* base, lds_void* dst, int voff, int soff)
{
#if defined(__HIP_DEVICE_COMPILE__)                         // (the host pass does not know the resource type)
    const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), 0, -1, 0x00020000);   // (raw, no bound)
    __builtin_amdgcn_raw_ptr_buffer_load_lds(r, dst, 16, voff, soff, 0, 0);
#endif
}

// Sixteen bytes per lane from base + soff (uniform) + voff to registers: one register of address per lane.
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ u32x4 load16(const void* base, int voff, int soff)
{
#if defined(__HIP_DEVICE_COMPILE__)
    return __builtin_amdgcn_raw_buffer_load_b128(__builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), 0, -1, 0x00020000), voff, soff, 0);
#else
    return u32x4{};
#endif
}

// Stores of a projection's output, which the next launch reads.  Written through the L2 (sc1): nothing is left there for the end of the
// launch to write back.  STREAM (nt): neither is it kept behind the L2, for outputs that the memory-side cache does not hold until
// they are read (kStreamBytes).  (The idle slots around the instruction are those that the hardware wants between it and writes of its data.)
template <bool STREAM>
__device__ __forceinline__ void store16_through(void* p, u32x4 v)
{
    if (STREAM) __builtin_nontemporal_store(v, (u32x4*)p);
#if defined(__HIP_DEVICE_COMPILE__)
    else asm volatile("s_nop 0\n\tglobal_store_dwordx4 %0, %1, off sc1\n\ts_nop 0" ::"v"(p), "v"(v));   // (nothing here reads it back)
#endif
}

template <int N>
__device__ inline void wait_vmcnt() { asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory"); }

// Workgroup barrier that waits for this wave's LDS traffic only.  (__syncthreads() also waits for every
// outstanding global load, which would serialise the loads that are deliberately left in flight across it.)
__device__ inline void barrier_lds()
{
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

// The last sequence b for which in(b, cu[b]) holds (true up to some b, at least for 0), and its boundaries.  The whole wave looks at
// 64 boundaries at once, so 64 sequences take one round trip to memory and 4096 take two, where halving takes six and twelve.
template <class In>
__device__ __forceinline__ int last_sequence(const int32_t* __restrict__ cu, int B, int lane, In in, int& c0, int& c1)
{
    int base = 0, span = B;
    for (;;) {
        const int step = (span + 63) >> 6, off = lane * step;
        const int at = base + (off < span ? off : 0), v0 = cu[at], v1 = cu[at + 1];
        const int n = __popcll(__ballot(off < span && in(at, v0))), last = n > 0 ? n - 1 : 0;
        base += last * step;
        if (step == 1) {
            c0 = __builtin_amdgcn_readlane(v0, last);
            c1 = __builtin_amdgcn_readlane(v1, last);
            return base;
        }
        span = step < span - last * step ? step : span - last * step;
    }
}

#endif  // __HIPCC__

constexpr int kRowPad = 256;  // activation rows per student are padded to a multiple of this
constexpr int kRowsMaxTokens = 256;   // largest call whose all-token layers run on the few-row projections
// Most elements (rows of all students x hidden width) that the fused LayerNorm + projection kernels take: every workgroup
// repeats the statistics of its rows, and beyond this a LayerNorm launch and the tile kernel are faster (hidden 768: 256 rows
// 35.4 us for a layer's embedding, q|k|v and FFN up against 38, 352 rows 40 against 38; hidden 256: 528 rows 17.5 against 26).
constexpr long kRowsLnMaxElems = 262144;
// First-token rows (elements as above) beyond which all their projections take the tile kernel, whose bare sums the LayerNorm
// launches finish: where no width loses by it.  us a call, few-row kernels / this, by 2^20 elements: hidden 256, three students: 1.0 511 /
// 515, 2.0 955 / 958, 2.9 1419 / 1418, 5.9 2728 / 2719; the wider ones break even earlier: 512, four: 1.0 547 / 533, 2.4 1223 / 1202; 768, two: 0.4
// 447 / 455, 0.75 801 / 798, 1.5 1455 / 1435, 2.2 2106 / 2056; eight: 0.75 504 / 508, 1.5 898 / 889, 3.0 3329 / 3249; 1024, two: 0.8 925 / 915, 1.6
// 1817 / 1793.
constexpr long kRowsTilesElems = 1L << 21;
constexpr int kRowsU = 1024;          // fp32 rows per student of the few-row projections' scratch
constexpr int kFirstOnlyMinTokens = 1024;   // smallest call whose first-token rows have buffers of their own
// fp8 projections: activations are quantised as e4m3(value * kActQuantScale) by the kernel that produces them
// (LayerNorm outputs and GELU outputs are of order one: 448 / 16 = 28 before saturation, 2^-6 / 16 = 1e-3 before the
// subnormal range), and only calls that compute at least kFp8MinRows rows use them
constexpr float kActQuantScale = 16.f;
constexpr int kFp8MinRows = 2048;

// Outputs of a projection (bytes, all students) from which they are streamed.  us a call, hidden 768, 14653 tokens, kept / streamed, by
// MiB: q|k|v 129 613 / 612, 193 901 / 898, 257 1176 / 1166, 515 2135 / 2125; FFN up 172 613 / 618, 258 901 / 894, 343 1176 / 1162, 687 2135 / 2118; hidden 1024:
// q|k|v 108 594 / 595, 215 1202 / 1197, 322 1659 / 1645; FFN up 144 594 / 602, 160 694 / 697, 287 1202 / 1199.  The hidden-wide outputs: no difference at
// any size up to 215.  Both kinds together, both sides three times in turn on another card: hidden 768, students 3 869 / 859, 6 1643 / 1592, 8 2119 / 2071;
// hidden 1024, 18.4 k tokens, 3 1577 / 1536, 6 3096 / 3038; runs of one side within 0.3 %.
constexpr size_t kStreamBytes = (size_t)192 << 20;

// Byte offsets of every tensor inside one student's slab of the weight arena.
// The encoder matrices are stored transposed with respect to the host blob, reduction index innermost: fp32 as
// [out][in], bf16 in blocks of 16 outputs x 8 inputs, [out / 16][in / 8][16][8] (what a matrix instruction takes is then
// contiguous); wp and the classifier matrix keep the blob's [in][out] order.
struct ArenaLayout {
    size_t tok, pos, emb_g, emb_b;
    size_t layer0, layer_stride;
    // relative to the start of a layer
    size_t wqkv, bqkv, wo, bo, ln1g, ln1b, w1, b1, w2, b2, ln2g, ln2b;
    size_t wk_io;                  // the key projection once more with the roles exchanged: rows in, reduction index out (folded first-token queries)
    // SP_DTYPE_FP8 only (0 otherwise), relative to the start of a layer: the fused q|k|v, attention-output, FFN-up and
    // FFN-down matrices once more as e4m3 codes and their per-output-feature scales (fp32).  Codes lie in blocks of 32
    // outputs x 64 inputs, [out / 32][in / 64][c % 2][c / 2][out % 32][in % 16] with c = in / 16 % 4: the two wave-loads of
    // one matrix-instruction operand, 1 KB in a row each
    size_t wqkv8, sqkv, wo8, so, w18, s1, w28, s2;
    size_t wp, wp_t, bp, wc, bc;   // wp: [in][out] (column-parallel head kernel); wp_t: projection operand
    size_t student_stride;
};

ArenaLayout make_arena_layout(const sp_config& c);

// Workspace carve-up for one call.
struct WsLayout {
    size_t x, qkv, vt, att, u, x1, g, z, zpart, end;
    size_t qkv2;                         // second q|k|v of fp32 calls in few launches, [K][rows][3H]: all of vt, att and u
    size_t cu0, cq, catt, cx1, cg;       // first-token rows only: [K][crows][H] (cu0: fp32; cg: [F]), last layer
    size_t cqt, cxb;                     // folded queries / weighted mean rows: [K][crows][heads][H]
    size_t part;                         // fp32 rows between the few-row projections: [K][kRowsU][H]
    size_t lpart;                        // per-group logit sums when two groups of students run side by side: [2][B][C]
    size_t xq, x1q, attq, gq;            // SP_DTYPE_FP8 only: fp8 copies of x, x1 and att ([K][rows][H] bytes), fp8 g ([K][rows][F])
    int rows, crows;
    int act_bytes;
};
WsLayout make_ws_layout(const sp_config& c, int total_tokens, int batch);

}  // namespace sp

struct sp_model {
    sp_config cfg;
    char* arena;
    sp::ArenaLayout L;
    // for calls that run two groups of students side by side (null: never)
    hipStream_t aux = nullptr;
    hipEvent_t ev_fork = nullptr, ev_join = nullptr;
    std::mutex* mu = nullptr;
};

namespace sp {

// Where element (row r, column c) of an activation buffer sits: (r / 16) rb + (r % 16) rs + (c / 8) cs + c % 8 (elements).
struct RowsLayout { size_t rb; int rs, cs; };
inline RowsLayout rows_layout(int width) { return {(size_t)16 * width, width, 8}; }           // row after row
inline RowsLayout packed_layout(int width) { return {(size_t)16 * width, 8, 128}; }          // matrix-operand blocks of 16 rows x 8

// ---- launchers (each returns the hipError_t of its launch) ------------------

// X[m][row][:] = LN(tok[id[row]] + pos[row - cu[seq(row)]]) for row < T; zero rows up to `rows`.
// Rows T..mrows of x and of att are zeroed.
// xq (may be null): the rows once more as fp8 (e4m3) codes of value * qscale, [m][rows][H] bytes; attq (may be
// null): fp8 attention output buffer of the same shape, whose rows T..mrows are zeroed like those of att.
hipError_t launch_embed_ln(const sp_model* M, const int32_t* ids, const int32_t* cu, int B, int T, int rows,
                           int mrows, int k, void* x, void* att, hipStream_t s, void* xq = nullptr, float qscale = 1.f,
                           void* attq = nullptr);

// out[m][row][:] = LN(u[m][row][:]; g, b); g/b are byte offsets into the student slab.
hipError_t launch_layernorm(const sp_model* M, const void* u, void* out, int rows, int mrows, int k, size_t g_off,
                            size_t b_off, hipStream_t s, void* outq = nullptr, float qscale = 1.f);

// out[m][b][:] = LN(u[m][cu[b]][:]; g, b) for b < B (bf16 path; the same arithmetic)
hipError_t launch_layernorm_first(const sp_model* M, const void* u, void* out, int rows, const int32_t* cu, int B, int T, int k,
                                  size_t g_off, size_t b_off, hipStream_t s);

// EPI_QKV (bf16 path only): bias; output columns >= n_split (the value projection) are written transposed,
// out2[m][column - n_split][row], so that attention reads key-contiguous value tiles.
enum Epilogue { EPI_BIAS = 0, EPI_BIAS_GELU = 1, EPI_BIAS_RESIDUAL = 2, EPI_QKV = 3, EPI_BIAS_TANH = 4, EPI_PARTIAL = 5 };

// out[m][row][0..N) = epi(A[m][row][0..Kd) . W^T + bias), W stored [N][Kd] at w_off of each student.
// lda / ldo / ldr are row strides in elements; residual may be null unless EPI_BIAS_RESIDUAL;
// mrows (a multiple of 64, <= the padded row count) is how many rows are computed.
hipError_t launch_gemm(const sp_model* M, const void* A, int lda, size_t w_off, size_t b_off, void* out, int ldo,
                       const void* residual, int ldr, int mrows, int N, int Kd, int k, Epilogue epi,
                       size_t a_student_stride, size_t o_student_stride, size_t r_student_stride, hipStream_t s,
                       void* out2 = nullptr, int n_split = 0, int ld2 = 0, size_t o2_student_stride = 0,
                       bool packed_out = false);   // packed_out (bf16): out in packed_layout(ldo)

// Split reduction for launches of few tiles: part[sp][m][row][0..N) = A[m][row][sp*Kd/splits ..) . W^T (fp32, no bias), sp <
// splits; slice: elements from slice to slice, p_student_stride from student to student.
hipError_t launch_gemm_split(const sp_model* M, const void* A, int lda, size_t w_off, float* part, size_t slice, int mrows,
                             int N, int Kd, int k, int splits, size_t a_student_stride, size_t p_student_stride, hipStream_t s);
// out[m][row][:] = LN(sum_sp part[sp][m][row][:] + bias + residual[m][row][:]; g, b) for row < T, zero for T <= row < mrows
hipError_t launch_ln_slices(const sp_model* M, const float* part, size_t slice, size_t p_ss, int splits, size_t bias_off,
                            const void* residual, void* out, int rows, int T, int mrows, int k, size_t g_off, size_t b_off,
                            hipStream_t s);

// Tile height in blocks of 32 tokens (1 to 4) for a projection of mrows rows onto N features (a multiple of 256) of k students.  cost[h]:
// what a token costs in a tile of height h, of one in the tallest; gemm_token_cost: of a bf16 projection from Kd.
int gemm_tile_height(int mrows, int N, int k, const double* cost);
const double* gemm_token_cost(int Kd);

// The same projection on fp8 operands (SP_DTYPE_FP8: mrows a multiple of 64, N and Kd of 256).
// A8: e4m3 codes of activation * a_qscale, [m][row][lda] bytes; weights at w_off (e4m3, operand blocks) with fp32
// scales at s_off; epi is EPI_QKV (bf16 out, value third transposed into out2), EPI_BIAS_GELU (out: e4m3 codes of
// gelu(.) * out_qscale, ldo bytes per row) or EPI_BIAS_RESIDUAL (bf16 out).  Student strides in bytes.
hipError_t launch_gemm_fp8(const sp_model* M, const void* A8, int lda, size_t w_off, size_t s_off, size_t b_off,
                           float a_qscale, void* out, int ldo, const void* residual, int ldr, int mrows, int N, int Kd,
                           int k, Epilogue epi, size_t a_student_stride, size_t o_student_stride,
                           size_t r_student_stride, hipStream_t s, void* out2, int n_split, int ld2,
                           size_t o2_student_stride, float out_qscale);

// y[i] = GELU as the bf16 FFN up-projection's epilogue evaluates it, in fp32 (i < n).  Test aid.
hipError_t launch_gelu_probe(const float* x, float* y, long n, hipStream_t s);
hipError_t launch_gelu_q8_probe(const float* x, float* y, long n, hipStream_t s);

// ---- students of hidden width 256 (sp_layer.hip; bf16 path): out = LN(x1 + FFN(x1)), x1 = LN(x + att Wo + bo), of mrows
// rows per student (a multiple of 64; all three buffers [m][rows][256]; out may be x)
bool layer_supported(const sp_config& c);
bool layer_pays(const sp_config& c, int64_t rows_of_all_students);
hipError_t launch_layer(const sp_model* M, size_t lo, const void* att, const void* x, void* out, int rows, int mrows, int k,
                        hipStream_t s);

// x = LN(embedding) of T rows per student and q|k|v of the layer at lo from them (values transposed into vt); rows T..mrows: x and att
// become zero
hipError_t launch_embed_qkv(const sp_model* M, size_t lo, const int32_t* ids, const int32_t* cu, int B, int T, void* x, void* att, void* qkv,
                            void* vt, int rows, int mrows, int k, hipStream_t s);

// ---- projections of few rows (sp_rows.hip; bf16 path).  u: fp32 rows before a LayerNorm, [student][u_ss], row stride H.
// Student strides (_ss) are in elements.
// q|k|v of all T tokens (values transposed into vt) from the embedding rows (u null; g_off / b_off: the embedding
// LayerNorm) or from LN(u); the normalised rows go to x as well.
hipError_t launch_rows_qkv(const sp_model* M, size_t lo, const float* u, size_t u_ss, size_t g_off, size_t b_off,
                           const int32_t* ids, const int32_t* cu, int B, int T, void* x, void* qkv, void* vt, int rows,
                           int k, hipStream_t s);
// g = gelu(LN(u; ln1) W1^T + b1), the normalised rows to x1 (row stride H)
hipError_t launch_rows_ffn_up(const sp_model* M, size_t lo, const float* u, size_t u_ss, int nrows, void* x1, size_t x1_ss,
                              void* g, size_t g_ss, RowsLayout gl, int k, hipStream_t s);
// zpart[m][n][r][c] = sum over the n-th 64 features of tanh(LN(u; ln2) Wp + bp) Wc (for launch_head_sum)
hipError_t launch_rows_pooler(const sp_model* M, size_t lo, const float* u, size_t u_ss, int nrows, float* zpart, int k,
                              hipStream_t s);
// out[r] (fp32, H wide) = A[r or cu[r]] W^T + bias + res[r or cu[r]]; Kd columns of A
hipError_t launch_rows_residual(const sp_model* M, size_t w_off, size_t b_off, const bf16* A, size_t a_ss, RowsLayout al,
                                int Kd, bool a_first, const bf16* res, size_t r_ss, bool r_first, float* out, size_t o_ss,
                                const int32_t* cu, int T, int nrows, int k, hipStream_t s);
// att[b][h*64..] = Wv_h xbar[b][h] + bv_h
hipError_t launch_rows_head_values(const sp_model* M, size_t lo, const void* xbar, size_t xb_ss, void* att, size_t att_ss,
                                   int nrows, int k, hipStream_t s);
// q[b] = x[cu[b]] Wq^T + bq; qt[b][h] = Wk_h q[b][h]  (cu null: x[b]).  scaled: qt times the scales at g_off, feature by feature
hipError_t launch_fold_query(const sp_model* M, size_t lo, const void* x, int rows, const int32_t* cu, int T, int B,
                             void* q, size_t q_ss, void* qt, size_t qt_ss, int k, hipStream_t s, bool scaled, size_t g_off);
// attention output of the first token of every sequence, at its token row
hipError_t launch_attention_first(const sp_model* M, const void* qkv, const void* vt, void* att, const int32_t* cu, int B,
                                  int T, int max_seqlen, int rows, int k, hipStream_t s);
// out = LN(u), bf16 rows
hipError_t launch_rows_ln_out(const sp_model* M, size_t g_off, size_t b_off, const float* u, size_t u_ss, void* out,
                              size_t o_ss, int nrows, int k, hipStream_t s);

// out = LN(u + bias + residual), bf16 rows; the residual of row r is row r of res, or row cu[r] of T (cu not null)
hipError_t launch_rows_ln_add(const sp_model* M, size_t g_off, size_t b_off, const float* u, size_t u_ss, size_t bias_off,
                              const void* res, size_t r_ss, const int32_t* cu, int T, void* out, size_t o_ss, int nrows, int k,
                              hipStream_t s);

// ---- fp32 path, calls of few rows (sp_rows_f32.hip), a launch each:
bool f32_layer_supported(const sp_config& c, long rows_of_all_students);
// x = LN(embedding) of T rows per student, and q|k|v of the layer at lo from them
hipError_t launch_f32_embed(const sp_model* M, size_t lo, const int32_t* ids, const int32_t* cu, int B, int T, void* x, void* qkv,
                            int rows, int k, hipStream_t s);
// x = LN(x1 + FFN(x1)), x1 = LN(x + att Wo + bo), att the attention over qkv, of T rows per student, and q|k|v of the next layer from the
// new x (qkv_next, not qkv; null: there is none, and the attention output is kept in att)
hipError_t launch_f32_layer(const sp_model* M, size_t lo, const void* qkv, void* x, void* qkv_next, void* att, const int32_t* cu, int B, int T,
                            int max_seqlen, int rows, int k, hipStream_t s);
// the same of the first token of every sequence (att: their rows alone), then z[m][b][c] = tanh(x Wp + bp) Wc + bc and (not null, one student) the same as logits
hipError_t launch_f32_last(const sp_model* M, size_t lo, const void* qkv, void* x, void* att, const int32_t* cu, int B, int T, int max_seqlen, int rows,
                           int k, float* z, float* logits, hipStream_t s);

// att[m][t][h*64..] = softmax(q k^T / 8) v inside each sequence; qkv rows are [q | k | v] of width 3H.
// bf16 path: the values are read from vt[m][H][rows] (transposed) instead of the third slice of qkv.
// attq (may be null, bf16 path only): the output once more as e4m3 codes of value * qscale, [m][rows][H] bytes.
hipError_t launch_attention(const sp_model* M, const void* qkv, const void* vt, void* att, const int32_t* cu, int B,
                            int T, int max_seqlen, int rows, int k, hipStream_t s, void* attq = nullptr,
                            float qscale = 1.f);

// Attention of the first token of each sequence with folded queries: for sequence b and head h,
// p = softmax_t(qt[m][b][h] . x[m][t] / 8) over the tokens t of the sequence and xbar[m][b][h][:] = sum_t p_t x[m][t][:].
// qt and xbar are [m][.._ss elements], rows of [heads][H].  raw: x holds rows before their LayerNorm (g_off, b_off), and qt carries
// its scale.
// parts (may be null): scratch for sequences split over workgroups, p_ss floats per student (fold_splits says whether it pays and suffices).
bool attention_first_fold_supported(const sp_config& c, int max_seqlen);
bool fold_splits(const sp_config& c, int B, int T, long work, size_t bytes);
hipError_t launch_attention_first_fold(const sp_model* M, const void* x, const void* qt, size_t qt_ss, void* xbar,
                                       size_t xb_ss, const int32_t* cu, int B, int T, int max_seqlen, int rows, int k,
                                       hipStream_t s, bool raw, size_t g_off, size_t b_off, float* parts, size_t p_ss);

// Head on the pooler's sums without bias (fp32 rows, p_ss elements from student to student): z[m][b][c] = tanh(sums + bp) . Wc + bc;
// logits[b][c] = sum_{m<k} z[m][b][c] (m ascending; not written if null).
hipError_t launch_head_classify(const sp_model* M, const float* sums, size_t p_ss, int B, int k, float* z, float* logits,
                                hipStream_t s);
// z[m][b][c] = bc + sum over the H / 64 slices n of zpart[m][n][b][c]; logits as above
hipError_t launch_head_sum(const sp_model* M, const float* zpart, int B, int k, float* z, float* logits, hipStream_t s);

// flags[0] |= SP_BAD_* bits for the inputs of a forward (flags[0] is cleared first, on the same stream).
hipError_t launch_check_inputs(const int32_t* ids, const int32_t* cu, int B, int T, int max_seqlen, int vocab,
                               unsigned* flags, hipStream_t s);

// logits[i] = sum_{m<k} z[m][i], m ascending (i < n).
hipError_t launch_sum_students(const float* z, int n, int k, float* logits, hipStream_t s);

// z[m][b][c] = tanh(x[m][cu[b]] Wp + bp) Wc + bc ; logits[b][c] = sum_{m<k} z[m][b][c] (m ascending).
hipError_t launch_head(const sp_model* M, const void* x, const int32_t* cu, int B, int T, int rows, int k, float* z,
                       float* zpart, float* logits, hipStream_t s);

}  // namespace sp
