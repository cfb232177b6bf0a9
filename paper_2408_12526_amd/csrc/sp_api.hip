// C ABI of libsp_mi355x.so: argument checks, weight upload, workspace carve-up
// and the order in which the kernels of one forward pass are enqueued.
#include <cmath>
#include <cstdlib>
#include <cstring>
#include <new>
#include <mutex>
#include <thread>
#include <vector>

#include "sp_dispatch.h"
#include "sp_internal.h"

namespace sp {

static size_t align_up(size_t v, size_t a) { return (v + a - 1) / a * a; }

static bool config_ok(const sp_config* c)
{
    if (!c) return false;
    if (c->K < 1 || c->layers < 1 || c->hidden < 1 || c->heads < 1 || c->ffn < 1 || c->vocab < 1 || c->max_pos < 1 ||
        c->classes < 1)
        return false;
    if (c->dtype != SP_DTYPE_FP32 && c->dtype != SP_DTYPE_BF16 && c->dtype != SP_DTYPE_FP8) return false;
    if (!(c->ln_eps >= 0.f)) return false;
    return true;
}

// what the kernels support
static bool config_supported(const sp_config& c)
{
    if (c.hidden % c.heads || c.hidden / c.heads != 64) return false;
    if (c.classes > 16 || c.hidden > 1024 || c.K > 64) return false;
    if (c.hidden % 128 || c.ffn % 128) return false;   // reduction depth of every projection: whole 64-wide k-tiles, at least two
    return true;
}

ArenaLayout make_arena_layout(const sp_config& c)
{
    const size_t H = c.hidden, F = c.ffn, C = c.classes;
    const size_t wb = bf16_path(c) ? 2 : 4;  // bytes per matrix / table element
    const size_t q8 = c.dtype == SP_DTYPE_FP8 ? 1 : 0;     // fp8 copies of three matrices
    ArenaLayout L{};
    size_t o = 0;
    auto take = [&](size_t bytes) { size_t at = o; o = align_up(o + bytes, 256); return at; };
    L.tok = take((size_t)c.vocab * H * wb);
    L.pos = take((size_t)c.max_pos * H * wb);
    L.emb_g = take(H * 4);
    L.emb_b = take(H * 4);
    L.layer0 = o;
    {
        size_t base = o;
        L.wqkv = take(3 * H * H * wb) - base;
        L.bqkv = take(3 * H * 4) - base;
        L.wo = take(H * H * wb) - base;
        L.bo = take(H * 4) - base;
        L.ln1g = take(H * 4) - base;
        L.ln1b = take(H * 4) - base;
        L.w1 = take(F * H * wb) - base;
        L.b1 = take(F * 4) - base;
        L.w2 = take(H * F * wb) - base;
        L.b2 = take(H * 4) - base;
        L.ln2g = take(H * 4) - base;
        L.ln2b = take(H * 4) - base;
        L.wk_io = take(H * H * wb) - base;
        if (q8) {
            L.wqkv8 = take(3 * H * H) - base;
            L.sqkv = take(3 * H * 4) - base;
            L.wo8 = take(H * H) - base;
            L.so = take(H * 4) - base;
            L.w18 = take(F * H) - base;
            L.s1 = take(F * 4) - base;
            L.w28 = take(H * F) - base;
            L.s2 = take(H * 4) - base;
        }
        L.layer_stride = o - base;
        o = base + L.layer_stride * (size_t)c.layers;
    }
    L.wp = take(H * H * wb);
    L.wp_t = take(H * H * wb);
    L.bp = take(H * 4);
    L.wc = take(C * H * wb);
    L.bc = take(C * 4);
    L.student_stride = align_up(o, 4096);
    return L;
}

WsLayout make_ws_layout(const sp_config& c, int total_tokens, int batch)
{
    WsLayout W{};
    const size_t ab = bf16_path(c) ? 2 : 4;
    const size_t rows = align_up((size_t)total_tokens, kRowPad);
    const size_t K = c.K, H = c.hidden, F = c.ffn;
    size_t o = 0;
    auto take = [&](size_t bytes) { size_t at = o; o = align_up(o + bytes, 256); return at; };
    W.x = take(K * rows * H * ab);
    W.qkv = take(K * rows * 3 * H * ab);
    W.vt = take(K * rows * H * ab);
    W.att = take(K * rows * H * ab);
    W.u = take(K * rows * H * ab);
    W.qkv2 = W.vt;                       // (the three above: taken one behind another, with x1 behind them)
    W.x1 = take(K * rows * H * ab);
    W.g = take(K * rows * F * ab);
    W.z = take(K * (size_t)batch * c.classes * 4);
    W.zpart = take(K * (size_t)(H / 64) * batch * c.classes * 4);
    // compact buffers for the first-token rows of the last layer (never used by calls of fewer than
    // kFirstOnlyMinTokens tokens: those get none)
    const size_t crows = total_tokens >= kFirstOnlyMinTokens ? align_up((size_t)batch, kRowPad) : 0;
    W.cu0 = take(K * crows * H * 2 * ab);
    W.cq = take(K * crows * H * ab);
    W.catt = take(K * crows * H * ab);
    W.cx1 = take(K * crows * H * ab);
    W.cg = take(K * crows * F * ab);
    W.cqt = take(K * crows * (size_t)c.heads * H * ab);
    W.cxb = take(K * crows * (size_t)c.heads * H * ab);
    W.part = take(K * (size_t)kRowsU * H * 4);
    W.lpart = take(2 * (size_t)batch * c.classes * 4);
    if (c.dtype == SP_DTYPE_FP8 && rows >= (size_t)kFp8MinRows) {
        W.xq = take(K * rows * H);
        W.x1q = take(K * rows * H);
        W.attq = take(K * rows * H);
        W.gq = take(K * rows * F);
    }
    W.crows = (int)crows;
    W.end = o;
    W.rows = (int)rows;
    W.act_bytes = (int)ab;
    return W;
}

static size_t student_blob_floats(const sp_config& c)
{
    const size_t H = c.hidden, F = c.ffn, C = c.classes;
    const size_t layer = 4 * (H * H + H) + 2 * H + (H * F + F) + (F * H + H) + 2 * H;
    return (size_t)c.vocab * H + (size_t)c.max_pos * H + 2 * H + (size_t)c.layers * layer + H * H + H + H * C + C;
}

// ---- host-side conversion into the arena image --------------------------------

static inline uint16_t f32_to_bf16_rne(float f)
{
    uint32_t u;
    memcpy(&u, &f, 4);
    if ((u & 0x7fffffffu) > 0x7f800000u) return (uint16_t)((u >> 16) | 0x0040u);  // NaN stays NaN
    u += 0x7fffu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}

// OCP e4m3 (4 exponent bits, bias 7, 3 mantissa bits, no infinities, largest finite value 448): round to nearest
// even, saturating.
static inline uint8_t f32_to_e4m3(float f)
{
    const uint8_t sign = std::signbit(f) ? 0x80 : 0;
    const float a = std::fabs(f);
    if (a != a) return (uint8_t)(sign | 0x7f);
    if (a >= 448.f) return (uint8_t)(sign | 0x7e);
    if (a < 0.015625f) {                                   // below 2^-6: multiples of 2^-9
        const int q = (int)std::nearbyint(a * 512.f);     // 0..8 (8 = the smallest normal number)
        return (uint8_t)(sign | q);
    }
    int e;
    const float mant = std::frexp(a, &e);                  // a = mant * 2^e, mant in [0.5, 1)
    int q = (int)std::nearbyint((mant * 2.f - 1.f) * 8.f); // 0..8
    int ex = e - 1;                                        // a = (1 + q / 8) * 2^ex
    if (q == 8) { q = 0; ++ex; }
    const int code = ((ex + 7) << 3) | q;
    return (uint8_t)(sign | (code > 0x7e ? 0x7e : code));
}

// code (o, i) = e4m3(src[i][o] / scale[o]), scale[o] = max_i |src[i][o]| / 448 (1 for an all-zero column), in the operand
// blocks of ArenaLayout; src is [n_in][n_out], n_in a multiple of 64 and n_out of 32
static void quantize_transposed(uint8_t* dst8, float* scale, const float* src, size_t n_in, size_t n_out)
{
    std::vector<float> amax(n_out, 0.f);
    for (size_t i = 0; i < n_in; ++i)
        for (size_t o = 0; o < n_out; ++o) {
            const float a = std::fabs(src[i * n_out + o]);
            if (a > amax[o]) amax[o] = a;
        }
    for (size_t o = 0; o < n_out; ++o) scale[o] = amax[o] > 0.f ? amax[o] / 448.f : 1.f;
    const size_t T = 32;
    for (size_t i0 = 0; i0 < n_in; i0 += T)
        for (size_t o0 = 0; o0 < n_out; o0 += T) {
            const size_t i1 = i0 + T < n_in ? i0 + T : n_in, o1 = o0 + T < n_out ? o0 + T : n_out;
            for (size_t o = o0; o < o1; ++o)
                for (size_t i = i0; i < i1; ++i) {
                    const size_t c = i >> 4 & 3;
                    dst8[((o >> 5) * (n_in >> 6) + (i >> 6)) * 2048 + (c & 1) * 1024 + (c >> 1) * 512 + (o & 31) * 16 + (i & 15)] =
                        f32_to_e4m3(src[i * n_out + o] / scale[o]);
                }
        }
}

struct Writer {
    bool bf16;
    // copy n values as the arena's matrix element type
    void copy(char* dst, const float* src, size_t n) const
    {
        if (bf16) {
            uint16_t* d = (uint16_t*)dst;
            for (size_t i = 0; i < n; ++i) d[i] = f32_to_bf16_rne(src[i]);
        } else {
            memcpy(dst, src, n * 4);
        }
    }
    // The matrix of rows o (o < n_o) and reduction index i (i < n_i) whose element (o, i) is src[i * si + o * so], as a
    // projection operand.  fp32: [o][i].  bf16: blocks of 16 rows x 8 elements, [o / 16][i / 8][o % 16][i % 8], so that the
    // sixteen rows by 32 elements (or 32 by 16) one matrix instruction takes are whole 256-byte runs, lane after lane.
    void operand(char* dst, const float* src, size_t n_o, size_t n_i, size_t so, size_t si) const
    {
        const size_t T = 32;
        for (size_t i0 = 0; i0 < n_i; i0 += T)
            for (size_t o0 = 0; o0 < n_o; o0 += T) {
                const size_t i1 = i0 + T < n_i ? i0 + T : n_i, o1 = o0 + T < n_o ? o0 + T : n_o;
                for (size_t o = o0; o < o1; ++o)
                    for (size_t i = i0; i < i1; ++i) {
                        const float v = src[i * si + o * so];
                        if (bf16) ((uint16_t*)dst)[((o >> 4) * (n_i >> 3) + (i >> 3)) * 128 + (o & 15) * 8 + (i & 7)] = f32_to_bf16_rne(v);
                        else ((float*)dst)[o * n_i + i] = v;
                    }
            }
    }
    // src is [n_in][n_out]: rows = outputs
    void transpose(char* dst, const float* src, size_t n_in, size_t n_out) const { operand(dst, src, n_out, n_in, 1, n_out); }
};

static void fill_student(const sp_config& c, const ArenaLayout& L, const float* src, char* dst)
{
    const size_t H = c.hidden, F = c.ffn, C = c.classes, wb = bf16_path(c) ? 2 : 4;
    const bool q8 = c.dtype == SP_DTYPE_FP8;
    Writer w{bf16_path(c)};
    const float* p = src;
    w.copy(dst + L.tok, p, (size_t)c.vocab * H); p += (size_t)c.vocab * H;
    w.copy(dst + L.pos, p, (size_t)c.max_pos * H); p += (size_t)c.max_pos * H;
    memcpy(dst + L.emb_g, p, H * 4); p += H;
    memcpy(dst + L.emb_b, p, H * 4); p += H;
    for (int l = 0; l < c.layers; ++l) {
        char* lb = dst + L.layer0 + (size_t)l * L.layer_stride;
        for (int part = 0; part < 3; ++part) {  // Wq bq Wk bk Wv bv -> rows [part*H, part*H+H) of the fused matrix
            if (part == 1) w.operand(lb + L.wk_io, p, H, H, H, 1);
            if (q8) quantize_transposed((uint8_t*)(lb + L.wqkv8) + (size_t)part * H * H, (float*)(lb + L.sqkv) + part * H, p, H, H);
            w.transpose(lb + L.wqkv + (size_t)part * H * H * wb, p, H, H); p += H * H;
            memcpy(lb + L.bqkv + (size_t)part * H * 4, p, H * 4); p += H;
        }
        if (q8) quantize_transposed((uint8_t*)(lb + L.wo8), (float*)(lb + L.so), p, H, H);
        w.transpose(lb + L.wo, p, H, H); p += H * H;
        memcpy(lb + L.bo, p, H * 4); p += H;
        memcpy(lb + L.ln1g, p, H * 4); p += H;
        memcpy(lb + L.ln1b, p, H * 4); p += H;
        if (q8) quantize_transposed((uint8_t*)(lb + L.w18), (float*)(lb + L.s1), p, H, F);
        w.transpose(lb + L.w1, p, H, F); p += H * F;
        memcpy(lb + L.b1, p, F * 4); p += F;
        if (q8) quantize_transposed((uint8_t*)(lb + L.w28), (float*)(lb + L.s2), p, F, H);
        w.transpose(lb + L.w2, p, F, H); p += F * H;
        memcpy(lb + L.b2, p, H * 4); p += H;
        memcpy(lb + L.ln2g, p, H * 4); p += H;
        memcpy(lb + L.ln2b, p, H * 4); p += H;
    }
    w.copy(dst + L.wp, p, H * H);
    w.transpose(dst + L.wp_t, p, H, H); p += H * H;
    memcpy(dst + L.bp, p, H * 4); p += H;
    w.copy(dst + L.wc, p, H * C); p += H * C;
    memcpy(dst + L.bc, p, C * 4); p += C;
}

// Optional per-phase timing: an event is recorded after every launch and tagged with its phase.
struct PhaseTimer {
    std::vector<hipEvent_t> ev;      // grows with the launch count (a dozen per layer)
    std::vector<int> phase;
    int n = 0;
    bool ok = true;
    void mark(int ph, hipStream_t s)
    {
        hipEvent_t e;
        if (hipEventCreate(&e) != hipSuccess) { ok = false; return; }
        try { ev.push_back(e); phase.push_back(ph); } catch (...) { (void)hipEventDestroy(e); ok = false; return; }
        ++n;
        if (hipEventRecord(e, s) != hipSuccess) ok = false;
    }
    void release() { for (int i = 0; i < n; ++i) (void)hipEventDestroy(ev[i]); ev.clear(); phase.clear(); n = 0; }
};

// Calls of at least this many tokens choose their kernels by the model's students, not by how many are active, and split no
// reduction, so that a student's term has the same bits whatever k.  (Smaller calls go by the active ones: a call pruned to one student
// would otherwise run on kernels for eight.)
constexpr int kLargeTokens = 8192;

// The forward of students [m0, m0 + k) of the model (k >= 1), all of it enqueued on stream s.  Every buffer of the
// workspace is sliced per student, so groups of students can run side by side on different streams.  With
// with_head the group's z rows are written; logits (the group's own sum, in student order) only if non-null.
// k_rule, may_split: what the rules that choose between kernels of different rounding go by, never the group's own k.
static int run_students(const sp_model* M0, const WsLayout& W, const int32_t* ids, const int32_t* cu, int B, int T,
                        int max_seqlen, int m0, int k, int k_rule, bool may_split, int stop_layers, bool with_head, char* w,
                        float* logits, hipStream_t s, PhaseTimer* pt)
{
    const sp_config& c = M0->cfg;
    sp_model shifted = *M0;                 // launchers address student i of the group as arena + i * stride
    shifted.arena = M0->arena + (size_t)m0 * M0->L.student_stride;
    const sp_model* M = &shifted;
    const int H = c.hidden, F = c.ffn, rows = W.rows;
    // quantised students: the four projections of the all-token layers on fp8 operands (large calls only)
    // (the fp8 kernel's tiles are 256 features wide: widths that are not multiples of it stay on the bf16 path)
    const bool fp8 = c.dtype == SP_DTYPE_FP8 && rows >= kFp8MinRows && W.xq && H % 256 == 0 && F % 256 == 0;
    // rows actually computed
    const int mtile = !bf16_path(c) ? 256 : 64;
    const int mrows = !bf16_path(c) && T <= 256 ? (T + (T > 64 ? 127 : 63)) / (T > 64 ? 128 : 64) * (T > 64 ? 128 : 64)
                                                : (T + mtile - 1) / mtile * mtile;
    const size_t ab = W.act_bytes;
    const size_t sH = (size_t)rows * H * ab, s3H = 3 * sH, sF = (size_t)rows * F * ab;
    char *x = w + W.x + m0 * sH, *qkv = w + W.qkv + m0 * s3H, *vt = w + W.vt + m0 * sH, *att = w + W.att + m0 * sH;
    char *u = w + W.u + m0 * sH, *x1 = w + W.x1 + m0 * sH, *g = w + W.g + m0 * sF;
    float* z = (float*)(w + W.z) + (size_t)m0 * B * c.classes;
    float* zpart = (float*)(w + W.zpart) + (size_t)m0 * (H / 64) * B * c.classes;
    const ArenaLayout& L = M->L;

#define SP_TRY(expr) do { if ((expr) != hipSuccess) return SP_EHIP; } while (0)
#define SP_MARK(ph) do { if (pt) pt->mark(ph, s); } while (0)
    const size_t qH = (size_t)rows * H, qF = (size_t)rows * F;       // bytes per student of the fp8 buffers
    char *xq = fp8 ? w + W.xq + m0 * qH : nullptr, *x1q = fp8 ? w + W.x1q + m0 * qH : nullptr;
    char *gq = fp8 ? w + W.gq + m0 * qF : nullptr, *attq = fp8 ? w + W.attq + m0 * qH : nullptr;
    SP_MARK(-1);
    // Last layer on the first-token rows only (see sp_config.last_layer_all_tokens).  Not used by the partial
    // forwards of the tests unless they stop before the last layer.
    // Calls of fewer than kFirstOnlyMinTokens tokens have no compact buffers: their first-token rows use the q|k|v and FFN
    // buffers, which the folded layer leaves free, where those are large enough.
    const bool first_only = !c.last_layer_all_tokens && with_head && attention_first_fold_supported(c, max_seqlen) &&
                            (T >= kFirstOnlyMinTokens ||
                             ((size_t)B * c.heads <= (size_t)3 * rows && (size_t)B * c.heads * H <= (size_t)rows * F));
    const int crows = W.crows;
    // fp32 rows of the few-row projections: after the attention-output projection, after the FFN, and (many first tokens) the
    // pooler's sums.  Calls of up to kRowsMaxTokens tokens: regions of kRowsMaxTokens rows of the scratch.  The folded last layer has
    // as many rows as sequences: the first rows in its own buffer (fewer than kFirstOnlyMinTokens tokens: the scratch, which holds
    // that many rows), the second over the folded queries, which nobody reads any more, and the sums over the first.
    struct FirstRows { float *o, *d, *pooled; size_t o_ss, d_ss; };
    float* const part = (float*)(w + W.part) + (size_t)m0 * kRowsU * H;
    const size_t part_ss = (size_t)kRowsU * H;
    const FirstRows small{part, part + (size_t)kRowsMaxTokens * H, nullptr, part_ss, part_ss};
    // Projection onto the hidden width, residual and LayerNorm of the T token rows (bf16): out = LN(A W^T + b + res).  A launch
    // of fewer than a tile per compute unit splits the reduction range over workgroups; the fp32 slices go into the buffers
    // that are free at that point (q|k|v and values, and behind them the attention output and the pre-LayerNorm rows once
    // the output projection is done), and the LayerNorm adds them.
    // raw (not null): the caller can do with the rows before the LayerNorm (in u); set if that is what it gets.
    auto project_ln = [&](const char* A, int Kd, size_t a_ss, size_t w_off, size_t b_off, const char* res, char* out, size_t g_off,
                          size_t be_off, int phase, bool* raw = nullptr) -> int {
        int splits = 1;
        const long tiles = (long)((mrows + 63) / 64) * (H / (H % 256 ? 128 : 256)) * k;
        // Tiles of half the features: only reductions that are deep for their tiles gain (hidden 384, depth 1536, 33 tiles: 14.7 us
        // against 7.3 and 1 for the slices; hidden 128, depth 512: 16 tiles 8.2 against 4.1, 116 tiles 7.0 against 7.5).
        const long most = H % 256 && Kd < 2048 ? Kd / 8 : 256;
        // (calls that may run as two groups have no room for slices; partial forwards keep the buffers for the tests)
        if (may_split && with_head && tiles < most) {
            const int room = (A == att ? 2 : 3) * c.K / k;
            for (int sp : {2, 3, 4, 6, 8})
                if (sp <= room && (Kd / 64) % (2 * sp) == 0 && Kd / sp >= 256) {
                    splits = sp;
                    if (tiles * sp >= 224) break;
                }
        }
        if (splits > 1) {
            float* ps = (float*)(w + W.qkv);
            const size_t p_ss = (size_t)rows * H, slice = p_ss * k;
            SP_TRY(launch_gemm_split(M, A, Kd, w_off, ps, slice, mrows, H, Kd, k, splits, a_ss, p_ss, s));
            SP_MARK(phase);
            SP_TRY(launch_ln_slices(M, ps, slice, p_ss, splits, b_off, res, out, rows, T, mrows, k, g_off, be_off, s));
        } else {
            SP_TRY(launch_gemm(M, A, Kd, w_off, b_off, u, H, res, H, mrows, H, Kd, k, EPI_BIAS_RESIDUAL, a_ss, sH, sH, s));
            SP_MARK(phase);
            if (raw) { *raw = true; return SP_OK; }
            SP_TRY(launch_layernorm(M, u, out, rows, mrows, k, g_off, be_off, s));
        }
        SP_MARK(SP_PHASE_LAYERNORM);
        return SP_OK;
    };
    // g = gelu(LN(u; ln1) W1^T + b1) of n rows: fused while the rows of all students are few, else a LayerNorm launch and
    // the tile kernel
    auto ffn_up = [&](size_t lo, int n, const float* uo, size_t u_ss, void* x1r, size_t x1_ss, void* gr, size_t g_ss,
                      bool packed) -> hipError_t {
        if ((long)n * k_rule * H <= kRowsLnMaxElems)
            return launch_rows_ffn_up(M, lo, uo, u_ss, n, x1r, x1_ss, gr, g_ss, packed ? packed_layout(F) : rows_layout(F), k, s);
        const hipError_t e = launch_rows_ln_out(M, lo + L.ln1g, lo + L.ln1b, uo, u_ss, x1r, x1_ss, n, k, s);
        if (e != hipSuccess) return e;
        return launch_gemm(M, x1r, H, lo + L.w1, lo + L.b1, gr, F, nullptr, 0, (n + 63) / 64 * 64, F, H, k, EPI_BIAS_GELU,
                           x1_ss * ab, g_ss * ab, 0, s, nullptr, 0, 0, 0, packed);
    };
    // Last layer from the attention output of the first tokens: A and x hold token rows (a_first, x_first) or one row per
    // sequence; x1c and gc are scratch of one row per sequence.  ss: student strides, elements.
    auto first_rows_tail = [&](size_t lo, const FirstRows& f, const bf16* A, size_t a_ss, bool a_first, bool x_first, bf16* x1c,
                               size_t x1c_ss, bf16* gc, size_t gc_ss) -> int {
        const size_t sT = (size_t)rows * H;
        SP_TRY(launch_rows_residual(M, lo + L.wo, lo + L.bo, A, a_ss, rows_layout(H), H, a_first, (const bf16*)x, sT, x_first, f.o,
                                    f.o_ss, cu, T, B, k, s));
        SP_MARK(SP_PHASE_LAST_FIRST);
        SP_TRY(ffn_up(lo, B, f.o, f.o_ss, x1c, x1c_ss, gc, gc_ss, true));
        SP_MARK(SP_PHASE_LAST_FIRST);
        SP_TRY(launch_rows_residual(M, lo + L.w2, lo + L.b2, gc, gc_ss, packed_layout(F), F, false, x1c, x1c_ss, false, f.d,
                                    f.d_ss, cu, T, B, k, s));
        SP_MARK(SP_PHASE_LAST_FIRST);
        SP_TRY(launch_rows_pooler(M, lo, f.d, f.d_ss, B, zpart, k, s));
        SP_TRY(launch_head_sum(M, zpart, B, k, z, logits, s));
        SP_MARK(SP_PHASE_HEAD);
        return SP_OK;
    };
    // The same from one row per sequence where the rows are many: the tile kernels, whose bare sums the LayerNorm launches
    // (and the classifier) finish.  xf: scratch like x1c.  Rows behind the last sequence are computed and never read.
    auto first_rows_tail_tiles = [&](size_t lo, const FirstRows& f, const bf16* A, size_t a_ss, bool x_first, bf16* x1c, size_t x1c_ss,
                                     bf16* gc, size_t gc_ss, bf16* xf, size_t xf_ss) -> int {
        const int mr = (B + 63) / 64 * 64;
        SP_TRY(launch_gemm_split(M, A, H, lo + L.wo, f.o, 0, mr, H, H, k, 1, a_ss * ab, f.o_ss, s));
        SP_TRY(launch_rows_ln_add(M, lo + L.ln1g, lo + L.ln1b, f.o, f.o_ss, lo + L.bo, x, (size_t)rows * H, x_first ? cu : nullptr, T, x1c,
                                  x1c_ss, B, k, s));
        SP_MARK(SP_PHASE_LAST_FIRST);
        SP_TRY(launch_gemm(M, x1c, H, lo + L.w1, lo + L.b1, gc, F, nullptr, 0, mr, F, H, k, EPI_BIAS_GELU, x1c_ss * ab, gc_ss * ab,
                           0, s));
        SP_MARK(SP_PHASE_LAST_FIRST);
        SP_TRY(launch_gemm_split(M, gc, F, lo + L.w2, f.d, 0, mr, H, F, k, 1, gc_ss * ab, f.d_ss, s));
        SP_TRY(launch_rows_ln_add(M, lo + L.ln2g, lo + L.ln2b, f.d, f.d_ss, lo + L.b2, x1c, x1c_ss, nullptr, T, xf, xf_ss, B, k, s));
        SP_MARK(SP_PHASE_LAST_FIRST);
        SP_TRY(launch_gemm_split(M, xf, H, L.wp_t, f.pooled, 0, mr, H, H, k, 1, xf_ss * ab, f.o_ss, s));
        SP_TRY(launch_head_classify(M, f.pooled, f.o_ss, B, k, z, logits, s));
        SP_MARK(SP_PHASE_HEAD);
        return SP_OK;
    };
    if (bf16_path(c) && T <= kRowsMaxTokens) {
        const size_t sT = (size_t)rows * H, sG = (size_t)rows * F, u_ss = part_ss;
        float *uo = small.o, *ud = small.d;
        // Many rows over all students: the tile kernel with a split reduction for the two projections onto the hidden width as
        // well (hidden 768, 960 rows, us for both projections of a layer and their LayerNorms: 31.4 against 34.7; 352 rows 22.6
        // against 23.1; hidden 1024, 768 rows: 43.4 against 50.9)
        const bool tiles_from_here = H % 256 == 0 && (long)T * k_rule * H > 2 * kRowsLnMaxElems;
        // (the partial forwards of the tests read the FFN activations row by row)
        const RowsLayout gl = with_head ? packed_layout(F) : rows_layout(F);
        if (stop_layers == 0) {
            SP_TRY(launch_embed_ln(M, ids, cu, B, T, rows, mrows, k, x, att, s));
            SP_MARK(SP_PHASE_EMBED);
        }
        for (int l = 0; l < stop_layers; ++l) {
            const size_t lo = L.layer0 + (size_t)l * L.layer_stride, pl = lo - L.layer_stride;
            if ((long)T * k_rule * H <= kRowsLnMaxElems) {
                SP_TRY(launch_rows_qkv(M, lo, l ? ud : nullptr, u_ss, l ? pl + L.ln2g : L.emb_g, l ? pl + L.ln2b : L.emb_b,
                                       ids, cu, B, T, x, qkv, vt, rows, k, s));
            } else {
                // (the embedding kernel zeroes the padding rows of x, and nothing writes them afterwards)
                if (l == 0) SP_TRY(launch_embed_ln(M, ids, cu, B, T, rows, mrows, k, x, att, s));
                else if (!tiles_from_here) SP_TRY(launch_rows_ln_out(M, pl + L.ln2g, pl + L.ln2b, ud, u_ss, x, sT, T, k, s));
                SP_MARK(l == 0 ? SP_PHASE_EMBED : SP_PHASE_LAYERNORM);
                SP_TRY(launch_gemm(M, x, H, lo + L.wqkv, lo + L.bqkv, qkv, 3 * H, nullptr, 0, mrows, 3 * H, H, k, EPI_QKV, sH,
                                   s3H, 0, s, vt, 2 * H, rows, sH));
            }
            SP_MARK(SP_PHASE_QKV);
            if (with_head && !c.last_layer_all_tokens && l == c.layers - 1) {
                SP_TRY(launch_attention_first(M, qkv, vt, att, cu, B, T, max_seqlen, rows, k, s));
                SP_MARK(SP_PHASE_LAST_FIRST);
                return first_rows_tail(lo, small, (const bf16*)att, sT, true, true, (bf16*)x1, sT, (bf16*)g, sG);
            }
            SP_TRY(launch_attention(M, qkv, vt, att, cu, B, T, max_seqlen, rows, k, s));
            SP_MARK(SP_PHASE_ATTENTION);
            if (tiles_from_here) {
                int rc = project_ln(att, H, sH, lo + L.wo, lo + L.bo, x, x1, lo + L.ln1g, lo + L.ln1b, SP_PHASE_OPROJ);
                if (rc != SP_OK) return rc;
                SP_TRY(launch_gemm(M, x1, H, lo + L.w1, lo + L.b1, g, F, nullptr, 0, mrows, F, H, k, EPI_BIAS_GELU, sH, sF, 0, s));
                SP_MARK(SP_PHASE_FFN_UP);
                rc = project_ln(g, F, sF, lo + L.w2, lo + L.b2, x1, x, lo + L.ln2g, lo + L.ln2b, SP_PHASE_FFN_DOWN);
                if (rc != SP_OK) return rc;
                continue;
            }
            SP_TRY(launch_rows_residual(M, lo + L.wo, lo + L.bo, (const bf16*)att, sT, rows_layout(H), H, false,
                                        (const bf16*)x, sT, false, uo, u_ss, cu, T, T, k, s));
            SP_MARK(SP_PHASE_OPROJ);
            SP_TRY(ffn_up(lo, T, uo, u_ss, x1, sT, g, sG, with_head));
            SP_MARK(SP_PHASE_FFN_UP);
            SP_TRY(launch_rows_residual(M, lo + L.w2, lo + L.b2, (const bf16*)g, sG, gl, F, false, (const bf16*)x1, sT, false,
                                        ud, u_ss, cu, T, T, k, s));
            SP_MARK(SP_PHASE_FFN_DOWN);
            if (l == stop_layers - 1) {
                SP_TRY(launch_rows_ln_out(M, lo + L.ln2g, lo + L.ln2b, ud, u_ss, x, sT, T, k, s));
                SP_MARK(SP_PHASE_LAYERNORM);
            }
        }
        if (with_head) {
            SP_TRY(launch_head(M, x, cu, B, T, rows, k, z, zpart, logits, s));
            SP_MARK(SP_PHASE_HEAD);
        }
        return SP_OK;
    }
    // (the partial forwards of the tests read the buffers between the projections: not these either)
    const bool f32_layer = with_head && f32_layer_supported(c, (long)T * k_rule);
    // Their rows' q|k|v alternate between two buffers: other workgroups read those of a layer while the next one's are written.  The last
    // layer's are in qkv.
    if (f32_layer && W.x1 - W.qkv2 < c.K * s3H) return SP_EINVAL;
    auto f32_qkv = [&](int l) { return (c.layers - 1 - l) & 1 ? w + W.qkv2 + m0 * s3H : qkv; };
    // Students of hidden width 256: two launches a layer, the attention between them, where the rows are enough (see layer_pays).  Embedding and
    // the first q|k|v in one from 8192 rows on; below, the more workgroups of two launches are quicker to look up their rows.  us a call, FFN 1024,
    // eight launches a layer / embedding and q|k|v apart / in one, by tokens: one student 2718 82.5 / 73.8 / 75.2, 5475 93.1 / 78.7 / 78.7, 9143 98.0 / 82.7 /
    // 81.1, 14653 112.8 / 96.9 / 86.9; three 658 79.0 / 71.2 / 73.4, 2718 98.5 / 79.8 / 79.2, 5475 119.8 / 107.1 / 102.4, 9143 155.6 / 128.2 / 117.2, 14653 220.0 /
    // 175.1 / 166.0.
    const bool narrow = with_head && !fp8 && layer_pays(c, (int64_t)T * k_rule);
    const bool narrow_qkv = narrow && (int64_t)T * k_rule >= 8192 && !(first_only && c.layers == 1);
    if (narrow_qkv) SP_TRY(launch_embed_qkv(M, L.layer0, ids, cu, B, T, x, att, qkv, vt, rows, mrows, k, s));
    else if (f32_layer) SP_TRY(launch_f32_embed(M, L.layer0, ids, cu, B, T, x, f32_qkv(0), rows, k, s));
    else SP_TRY(launch_embed_ln(M, ids, cu, B, T, rows, mrows, k, x, att, s, xq, kActQuantScale, attq));
    SP_MARK(SP_PHASE_EMBED);
    // Where the folded last layer follows, the rows stay as they are before the LayerNorm (see attention_first_fold_kernel) and only
    // the first tokens' are normalised, into the first B rows of x: a read and a write of every row less, for a longer fold and one more
    // launch.  By tokens x students x hidden width (Mi), and not for sequences so short that the fold's tiles of 32 tokens are mostly
    // empty.  us a call, with the LayerNorm of all rows / this.  768 wide: 5 236 / 240; 9 330 / 331; 11 383 / 381; 14 435 / 441; 18 569 / 566; 21
    // 637 / 628; 22 629 / 620; 88 2290 / 2251, quantised 1588 / 1524; eight sequences of 512 tokens: 6 242 / 253, 12 414 / 421, 24 696 / 690.
    // 1024 wide: 7 305 / 308, 12 463 / 465, 21 743 / 739, 29 978 / 966.  512 wide: 15 361 / 363, 16 396 / 402, 18 463 / 457.  256 wide (those of one
    // launch behind the attention never take it; an FFN of 1280, three students): 3.0 117 / 119, 6.0 159 / 159, 8.8 213 / 211, 12 268 / 264, 18 358 / 351;
    // quantised, FFN 1024: 6.0 144 / 142, 8.8 180 / 177, 12 205 / 198, 47 651 / 635.  Sequences of 4 tokens: 24 1021 / 1031 (768 wide), 1212 / 1263 (1024); of 16: 24 742 / 731, 875 / 872.
    // (In calls of kLargeTokens and more by the model's students, not by those that are active: the two round differently.  One of three
    // or of eight pays for that: 256 wide, 11 of long sequences 123 / 124; 768 wide, 88 365 / 367.)
    const int64_t fold_work = (int64_t)T * (T >= kLargeTokens ? c.K : k_rule) * H;
    const bool raw_pays = fold_work > (int64_t)(H == 256 ? 10 : 16) << 20 && T >= (int64_t)16 * B;
    bool raw = false;
    for (int l = 0; l < stop_layers; ++l) {
        const size_t lo = L.layer0 + (size_t)l * L.layer_stride, pl = lo - L.layer_stride;
        const bool fold_next = first_only && raw_pays && !narrow && l == c.layers - 2;
        if (first_only && l == c.layers - 1) {
            const bool own = T >= kFirstOnlyMinTokens;
            const size_t sT = (size_t)rows * H, sC = (size_t)crows * H;
            const size_t s1 = own ? sC : sT, sq = own ? sC * c.heads : 3 * sT, sx = own ? sC * c.heads : (size_t)rows * F;
            const size_t sg = (size_t)(own ? crows : rows) * F;
            bf16* q1 = own ? (bf16*)(w + W.cq) + m0 * sC : (bf16*)vt;
            bf16* att1 = own ? (bf16*)(w + W.catt) + m0 * sC : (bf16*)att;
            bf16* qt1 = own ? (bf16*)(w + W.cqt) + m0 * sq : (bf16*)qkv;
            bf16* xb1 = own ? (bf16*)(w + W.cxb) + m0 * sx : (bf16*)g;
            bf16* x11 = own ? (bf16*)(w + W.cx1) + m0 * sC : (bf16*)x1;
            bf16* g1 = own ? (bf16*)(w + W.cg) + m0 * sg : (bf16*)g;
            const FirstRows f = own ? FirstRows{(float*)(w + W.cu0) + m0 * sC, (float*)qt1, (float*)(w + W.cu0) + m0 * sC, sC, sq / 2}
                                    : FirstRows{part, (float*)qt1, part, part_ss, sq / 2};
            if (raw) {
                SP_TRY(launch_layernorm_first(M, u, x, rows, cu, B, T, k, pl + L.ln2g, pl + L.ln2b, s));
                SP_MARK(SP_PHASE_LAST_FIRST);
            }
            SP_TRY(launch_fold_query(M, lo, x, rows, raw ? nullptr : cu, T, B, q1, s1, qt1, sq, k, s, raw, pl + L.ln2g));
            SP_MARK(SP_PHASE_LAST_FIRST);
            // (scratch: the FFN's activations, which the last layer of such a call has elsewhere)
            const bool split = own && fold_splits(c, B, T, (long)B * (T >= kLargeTokens ? c.K : k_rule), sF);
            SP_TRY(launch_attention_first_fold(M, raw ? u : x, qt1, sq, xb1, sx, cu, B, T, max_seqlen, rows, k, s, raw, pl + L.ln2g,
                                               pl + L.ln2b, split ? (float*)g : nullptr, sF / 4));
            SP_MARK(SP_PHASE_LAST_FIRST);
            SP_TRY(launch_rows_head_values(M, lo, xb1, sx, att1, s1, B, k, s));
            SP_MARK(SP_PHASE_LAST_FIRST);
            if (own && (long)B * k_rule * H > kRowsTilesElems)
                return first_rows_tail_tiles(lo, f, att1, s1, !raw, x11, s1, g1, sg, xb1, sx);
            return first_rows_tail(lo, f, att1, s1, false, !raw, x11, s1, g1, sg);
        }
        const bool left = f32_layer || (narrow_qkv && l == 0);          // the launch before has left q|k|v
        if (fp8)
            SP_TRY(launch_gemm_fp8(M, xq, H, lo + L.wqkv8, lo + L.sqkv, lo + L.bqkv, kActQuantScale, qkv, 3 * H, nullptr, 0,
                                   mrows, 3 * H, H, k, EPI_QKV, qH, s3H, 0, s, vt, 2 * H, rows, sH, 1.f));
        else if (bf16_path(c) && !left)
            SP_TRY(launch_gemm(M, x, H, lo + L.wqkv, lo + L.bqkv, qkv, 3 * H, nullptr, 0, mrows, 3 * H, H, k, EPI_QKV,
                               sH, s3H, 0, s, vt, 2 * H, rows, sH));
        else if (!left)
            SP_TRY(launch_gemm(M, x, H, lo + L.wqkv, lo + L.bqkv, qkv, 3 * H, nullptr, 0, mrows, 3 * H, H, k, EPI_BIAS,
                               sH, s3H, 0, s));
        if (!left) SP_MARK(SP_PHASE_QKV);
        if (f32_layer) {
            if (l == c.layers - 1 && !c.last_layer_all_tokens) {
                SP_TRY(launch_f32_last(M, lo, f32_qkv(l), x, att, cu, B, T, max_seqlen, rows, k, z, k == 1 ? logits : nullptr, s));
                SP_MARK(SP_PHASE_LAST_FIRST);
                if (k == 1 || !logits) return SP_OK;
                SP_TRY(launch_sum_students(z, B * c.classes, k, logits, s));
                SP_MARK(SP_PHASE_HEAD);
                return SP_OK;
            }
            SP_TRY(launch_f32_layer(M, lo, f32_qkv(l), x, l + 1 < stop_layers ? f32_qkv(l + 1) : nullptr, att, cu, B, T, max_seqlen, rows, k, s));
            SP_MARK(SP_PHASE_FFN_DOWN);
            continue;
        }
        // (quantised students: the output projection reads the fp8 copy only, so a whole forward skips the bf16 one;
        // the partial forwards of the tests keep it)
        SP_TRY(launch_attention(M, qkv, vt, fp8 && with_head ? nullptr : att, cu, B, T, max_seqlen, rows, k, s, attq,
                                kActQuantScale));
        SP_MARK(SP_PHASE_ATTENTION);
        if (narrow) {
            SP_TRY(launch_layer(M, lo, att, x, x, rows, mrows, k, s));
            SP_MARK(SP_PHASE_FFN_DOWN);
            continue;
        }
        if (bf16_path(c) && !fp8) {
            int rc = project_ln(att, H, sH, lo + L.wo, lo + L.bo, x, x1, lo + L.ln1g, lo + L.ln1b, SP_PHASE_OPROJ);
            if (rc != SP_OK) return rc;
            SP_TRY(launch_gemm(M, x1, H, lo + L.w1, lo + L.b1, g, F, nullptr, 0, mrows, F, H, k, EPI_BIAS_GELU, sH, sF, 0, s));
            SP_MARK(SP_PHASE_FFN_UP);
            rc = project_ln(g, F, sF, lo + L.w2, lo + L.b2, x1, x, lo + L.ln2g, lo + L.ln2b, SP_PHASE_FFN_DOWN,
                            fold_next ? &raw : nullptr);
            if (rc != SP_OK) return rc;
            continue;
        }
        if (fp8)
            SP_TRY(launch_gemm_fp8(M, attq, H, lo + L.wo8, lo + L.so, lo + L.bo, kActQuantScale, u, H, x, H, mrows, H, H, k,
                                   EPI_BIAS_RESIDUAL, qH, sH, sH, s, nullptr, 0, 0, 0, 1.f));
        else
            SP_TRY(launch_gemm(M, att, H, lo + L.wo, lo + L.bo, u, H, x, H, mrows, H, H, k, EPI_BIAS_RESIDUAL, sH, sH, sH, s));
        SP_MARK(SP_PHASE_OPROJ);
        SP_TRY(launch_layernorm(M, u, x1, rows, mrows, k, lo + L.ln1g, lo + L.ln1b, s, x1q, kActQuantScale));
        SP_MARK(SP_PHASE_LAYERNORM);
        if (fp8)
            SP_TRY(launch_gemm_fp8(M, x1q, H, lo + L.w18, lo + L.s1, lo + L.b1, kActQuantScale, gq, F, nullptr, 0, mrows, F,
                                   H, k, EPI_BIAS_GELU, qH, qF, 0, s, nullptr, 0, 0, 0, kActQuantScale));
        else
            SP_TRY(launch_gemm(M, x1, H, lo + L.w1, lo + L.b1, g, F, nullptr, 0, mrows, F, H, k, EPI_BIAS_GELU, sH, sF, 0,
                               s));
        SP_MARK(SP_PHASE_FFN_UP);
        if (fp8)
            SP_TRY(launch_gemm_fp8(M, gq, F, lo + L.w28, lo + L.s2, lo + L.b2, kActQuantScale, u, H, x1, H, mrows, H, F, k,
                                   EPI_BIAS_RESIDUAL, qF, sH, sH, s, nullptr, 0, 0, 0, 1.f));
        else
            SP_TRY(launch_gemm(M, g, F, lo + L.w2, lo + L.b2, u, H, x1, H, mrows, H, F, k, EPI_BIAS_RESIDUAL, sF, sH, sH, s));
        SP_MARK(SP_PHASE_FFN_DOWN);
        if (fold_next) { raw = true; continue; }
        SP_TRY(launch_layernorm(M, u, x, rows, mrows, k, lo + L.ln2g, lo + L.ln2b, s, xq, kActQuantScale));
        SP_MARK(SP_PHASE_LAYERNORM);
    }
    if (with_head) {
        SP_TRY(launch_head(M, x, cu, B, T, rows, k, z, zpart, logits, s));
        SP_MARK(SP_PHASE_HEAD);
    }
#undef SP_MARK
#undef SP_TRY
    return SP_OK;
}

// Whole call: argument checks, then either all active students on the caller's stream, or, where that pays (two_groups_pay), two
// halves of them side by side: the first on the caller's stream, the second on the model's auxiliary stream (forked
// and joined with events, so the call stays asynchronous and capturable).  The matrix-core phases run at the
// package power limit while the bandwidth-bound phases leave most of it unused; two groups of students drift out
// of phase and fill each other's gaps (starting the second group late, after the first group's first projection, measured no
// better).  The logits are summed over all students in ascending order after the join, so the result does not depend on the
// grouping.
//

// Two groups only in calls of kLargeTokens and more: smaller ones share nothing with other streams' calls on the same model.  By work, in
// Mi = 2^20 tokens x active students x hidden width; one stream / two, us a call, both on one card in turn:
//   * From 20: fork and join cost about 20 us, and half the students fill the chip less well.  768 wide, 2 students: 12.1 399 / 417, 16.7
//     507 / 505, 20.9 606 / 603, 29 801 / 789; 4: 24 723 / 682; quantised, 2: 12.1 307 / 321, 20.8 451 / 441; 512 wide, 2: 13.9 351 / 363, 4:
//     27.9 637 / 607; 256 wide, 3: 10.4 226 / 253, 20.5 408 / 402, 6: 20.9 412 / 381.  The cost is paid once, the gain per
//     layer: six layers 768 wide, 2 students: 12.1 1626 / 1612, 16.8 2156 / 2106; 256 wide, 2: 4.0 483 / 471, 7.0 668 / 609.  Not so for an odd number
//     of students, of which one group is done before the other: six layers 256 wide, 3: 10.4 898 / 974.  With a layer of 256 in two launches (FFN
//     1024) the same lines, at which some numbers of tiles lose a few per cent and others gain: 2: 20.0 269 / 269, 29 400 / 400, 3: 20.1 274 / 272,
//     29 403 / 399, 43 559 / 551, 58 726 / 698, 4: 20.0 285 / 280, 23.4 301 / 315, 34 438 / 437, 58 719 / 707, 6: 21.5 287 / 292, 35 453 / 446, 87 1028 / 1006;
//     six layers, 2: 4.0 379 / 358, 7.2 460 / 472, 4: 8.0 580 / 515, 14 809 / 762, 3: 20.5 1124 / 1076.
//   * bf16 of hidden 512 and more, whose projections reach the power limit by themselves: even numbers of students only (768 wide, 3:
//     31 852 / 858, 61 1635 / 1675; 5: 52 1421 / 1432; 512 wide, 3: 20.9 492 / 506), and up to 64, beyond which a group alone fills the chip as
//     well (768 wide, 8: 49 1302 / 1288, 58 1567 / 1555, 70 1850 / 1918, 84 2136-2200 / 2196-2220, 328 8196 / 8329; 4: 42 1141 / 1103, 58.5 1576 /
//     1558, 82 2156 / 2220; six layers, 2: 41 5092 / 4897, 59 7306 / 7255, 82 9953 / 10314; 1024 wide, 6: 48 1501 / 1501, 107 3201 / 3226).
//     Quantised and narrow students have no such limit (quantised, 8: 84 1498 / 1472, 164 2878 / 2853; 256 wide, 6: 161 2569 / 2539).
constexpr int64_t kTwoGroupsWork = 20 << 20, kTwoGroupsMostWork = 64 << 20;
static bool two_groups_pay(const sp_config& c, int T, int k)
{
    if (k < 2 || T < kLargeTokens) return false;
    const int64_t work = (int64_t)T * k * c.hidden;
    const bool even = k % 2 == 0;
    if (work * (even && c.layers > 2 ? c.layers - 1 : 1) < kTwoGroupsWork) return false;
    return c.dtype == SP_DTYPE_FP8 || c.hidden < 512 || (even && work <= kTwoGroupsMostWork);
}

// Whether work on s can be continued on the model's stream.  A capture that forked to it keeps it until the capture ends, and other
// streams' calls can neither join that capture nor wait for it: they stay on their own stream meanwhile (the same bits).
static bool aux_may_follow(const sp_model* M, hipStream_t s)
{
    hipStreamCaptureStatus aux = hipStreamCaptureStatusNone, own = hipStreamCaptureStatusNone;
    unsigned long long aux_id = 0, own_id = 0;
    const bool known = hipStreamGetCaptureInfo(M->aux, &aux, &aux_id) == hipSuccess;
    if (known && aux == hipStreamCaptureStatusNone) return true;
    const bool same = known && aux == hipStreamCaptureStatusActive && hipStreamGetCaptureInfo(s, &own, &own_id) == hipSuccess &&
                      own == hipStreamCaptureStatusActive && own_id == aux_id;
    if (!same) (void)hipGetLastError();             // (a query that was refused is not an error of the call)
    return same;
}

static int run_forward(const sp_model* M, const int32_t* ids, const int32_t* cu, int B, int T, int max_seqlen, int k,
                       int stop_layers, bool with_head, void* ws, size_t ws_bytes, float* logits, hipStream_t s,
                       PhaseTimer* pt = nullptr)
{
    if (!M || !ids || !cu || !ws || (with_head && !logits)) return SP_EINVAL;
    if (((uintptr_t)ws & 255) || ((uintptr_t)ids & 3) || ((uintptr_t)cu & 3) || ((uintptr_t)logits & 3)) return SP_EINVAL;
    const sp_config& c = M->cfg;
    if (B < 1 || T < B || max_seqlen < 1 || max_seqlen > c.max_pos || (int64_t)B * max_seqlen < T) return SP_ESHAPE;
    if (k < 1 || k > c.K) return SP_EKACTIVE;
    if (stop_layers < 0 || stop_layers > c.layers) return SP_EINVAL;
    const WsLayout W = make_ws_layout(c, T, B);
    if (ws_bytes < W.end) return SP_ENOMEM;
    char* w = (char*)ws;

    const bool large = T >= kLargeTokens;
    const int ka = (k + 1) / 2, k_rule = large ? (c.K + 1) / 2 : k;
    std::unique_lock<std::mutex> hold;              // one fork/join at a time on the model's stream and events
    bool two_groups = with_head && !pt && !c.single_stream && M->aux && two_groups_pay(c, T, k);
    if (two_groups) {
        hold = std::unique_lock<std::mutex>(*M->mu);
        two_groups = aux_may_follow(M, s);
        if (!two_groups) hold.unlock();
    }
    if (!two_groups)
        return run_students(M, W, ids, cu, B, T, max_seqlen, 0, k, k_rule, !large, stop_layers, with_head, w, logits, s, pt);

    float* lpart = (float*)(w + W.lpart);
    const size_t n = (size_t)B * c.classes;
    if (hipEventRecord(M->ev_fork, s) != hipSuccess || hipStreamWaitEvent(M->aux, M->ev_fork, 0) != hipSuccess)
        return SP_EHIP;
    int rc = run_students(M, W, ids, cu, B, T, max_seqlen, 0, ka, k_rule, false, stop_layers, true, w, lpart, s, nullptr);
    const int rc2 = run_students(M, W, ids, cu, B, T, max_seqlen, ka, k - ka, k_rule, false, stop_layers, true, w, lpart + n,
                                 M->aux, nullptr);
    // join even after an error, so that the auxiliary stream never runs on beyond the call
    if (hipEventRecord(M->ev_join, M->aux) != hipSuccess || hipStreamWaitEvent(s, M->ev_join, 0) != hipSuccess)
        return SP_EHIP;
    if (rc == SP_OK) rc = rc2;
    if (rc != SP_OK) return rc;
    if (launch_sum_students((const float*)(w + W.z), (int)n, k, logits, s) != hipSuccess) return SP_EHIP;
    return SP_OK;
}

// ---- workspace for callers that cannot allocate ---------------------------------------------------
// One array per GPU, part of the library's device image: every GPU the library runs on holds it until the process
// ends.  In host code the array's name is only a stand-in for the symbol; the device address is looked up once per
// device and everything on the host (kernel arguments included) goes through that pointer.
constexpr size_t kStaticScratchBytes = (size_t)SP_STATIC_SCRATCH_MIB << 20;
constexpr int kMaxDevices = 64;
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];
static std::mutex scratch_mu;
static void* scratch_ptr[kMaxDevices];      // per device; null until looked up

// The current device's copy of the array (looked up on the first request for that device).
static int static_scratch(void** out)
{
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess) return SP_EHIP;
    if (dev < 0 || dev >= kMaxDevices) return SP_EINVAL;
    std::lock_guard<std::mutex> hold(scratch_mu);
    if (!scratch_ptr[dev]) {
        void* p = nullptr;
        if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return SP_EHIP;
        scratch_ptr[dev] = p;
    }
    *out = scratch_ptr[dev];
    return SP_OK;
}

}  // namespace sp

using namespace sp;

extern "C" {

size_t sp_blob_floats(const sp_config* cfg)
{
    if (!config_ok(cfg)) return 0;
    return (size_t)cfg->K * student_blob_floats(*cfg);
}

size_t sp_arena_bytes(const sp_config* cfg)
{
    if (!config_ok(cfg)) return 0;
    return make_arena_layout(*cfg).student_stride * (size_t)cfg->K;
}

size_t sp_workspace_bytes(const sp_config* cfg, int32_t max_tokens, int32_t max_batch)
{
    if (!config_ok(cfg) || max_tokens < 1 || max_batch < 1) return 0;
    return make_ws_layout(*cfg, max_tokens, max_batch).end;
}

int sp_workspace_layout(const sp_config* cfg, int32_t total_tokens, int32_t batch, sp_ws_layout* out)
{
    if (!config_ok(cfg) || !out) return SP_EINVAL;
    if (total_tokens < 1 || batch < 1) return SP_ESHAPE;
    const WsLayout W = make_ws_layout(*cfg, total_tokens, batch);
    out->x = W.x; out->qkv = W.qkv; out->vt = W.vt; out->att = W.att; out->x1 = W.x1; out->g = W.g; out->z = W.z;
    out->rows = W.rows; out->act_bytes = W.act_bytes;
    out->first_q = W.cq; out->first_att = W.catt; out->first_rows = W.crows;
    out->xq = W.xq; out->x1q = W.x1q; out->gq = W.gq; out->attq = W.attq;
    return SP_OK;
}

int sp_load_students(const sp_config* cfg, const float* host_weights, size_t nfloats, void* device_arena,
                     size_t arena_bytes, void* hip_stream, sp_model** out)
{
    if (!config_ok(cfg) || !host_weights || !device_arena || !out) return SP_EINVAL;
    if ((uintptr_t)device_arena & 255) return SP_EINVAL;
    if (!config_supported(*cfg)) return SP_ESHAPE;
    const size_t per = student_blob_floats(*cfg);
    if (nfloats < per * (size_t)cfg->K) return SP_ENOMEM;
    const ArenaLayout L = make_arena_layout(*cfg);
    if (arena_bytes < L.student_stride * (size_t)cfg->K) return SP_ENOMEM;

    sp_model* m = new (std::nothrow) sp_model;
    if (!m) return SP_ENOMEM;
    m->cfg = *cfg; m->arena = (char*)device_arena; m->L = L;

    // Build the arena image on the host, a few students at a time, then upload.
    const int K = cfg->K;
    const int group = K < 4 ? K : 4;
    char* stage = (char*)calloc((size_t)group, L.student_stride);
    if (!stage) { delete m; return SP_ENOMEM; }
    hipStream_t s = (hipStream_t)hip_stream;
    int rc = SP_OK;
    for (int m0 = 0; m0 < K && rc == SP_OK; m0 += group) {
        const int n = m0 + group <= K ? group : K - m0;
        std::thread th[4];                  // (group <= 4); a thread that cannot be started is replaced by a plain call
        for (int i = 0; i < n; ++i) {
            try {
                th[i] = std::thread(fill_student, std::cref(*cfg), std::cref(L), host_weights + (size_t)(m0 + i) * per,
                                    stage + (size_t)i * L.student_stride);
            } catch (...) {
                fill_student(*cfg, L, host_weights + (size_t)(m0 + i) * per, stage + (size_t)i * L.student_stride);
            }
        }
        for (int i = 0; i < n; ++i)
            if (th[i].joinable()) th[i].join();
        if (hipMemcpyAsync((char*)device_arena + (size_t)m0 * L.student_stride, stage, (size_t)n * L.student_stride,
                           hipMemcpyHostToDevice, s) != hipSuccess || hipStreamSynchronize(s) != hipSuccess)
            rc = SP_EHIP;
    }
    free(stage);
    if (rc != SP_OK) { delete m; return rc; }
    // Auxiliary stream (default priority) and events for calls that run two groups of students side by side; without
    // them every call stays on the caller's stream.
    m->mu = new (std::nothrow) std::mutex;
    if (m->mu && hipStreamCreateWithFlags(&m->aux, hipStreamNonBlocking) == hipSuccess) {
        if (hipEventCreateWithFlags(&m->ev_fork, hipEventDisableTiming) != hipSuccess ||
            hipEventCreateWithFlags(&m->ev_join, hipEventDisableTiming) != hipSuccess) {
            if (m->ev_fork) (void)hipEventDestroy(m->ev_fork);
            (void)hipStreamDestroy(m->aux);
            m->aux = nullptr; m->ev_fork = m->ev_join = nullptr;
        }
    } else {
        m->aux = nullptr;
    }
    // this device's copy of the static workspace (sp_forward_static): looked up now, with the device current, so
    // that the calls themselves do nothing but enqueue kernels
    void* unused = nullptr;
    (void)static_scratch(&unused);
    *out = m;
    return SP_OK;
}

size_t sp_static_scratch_bytes(void) { return kStaticScratchBytes; }

int sp_forward_static(const sp_model* model, const int32_t* token_ids, const int32_t* cu_seqlens, int32_t batch,
                      int32_t total_tokens, int32_t max_seqlen, int32_t k_active, float* logits_out, void* hip_stream)
{
    if (!model) return SP_EINVAL;
    if (batch < 1 || total_tokens < batch) return SP_ESHAPE;
    // too large for the static array: refuse before anything is enqueued
    if (make_ws_layout(model->cfg, total_tokens, batch).end > kStaticScratchBytes) return SP_ETOOBIG;
    void* ws = nullptr;
    const int rc = static_scratch(&ws);
    if (rc != SP_OK) return rc;
    return run_forward(model, token_ids, cu_seqlens, batch, total_tokens, max_seqlen, k_active, model->cfg.layers,
                       true, ws, kStaticScratchBytes, logits_out, (hipStream_t)hip_stream);
}

int sp_forward(const sp_model* model, const int32_t* token_ids, const int32_t* cu_seqlens, int32_t batch,
               int32_t total_tokens, int32_t max_seqlen, int32_t k_active, void* workspace, size_t workspace_bytes,
               float* logits_out, void* hip_stream)
{
    if (!model) return SP_EINVAL;
    return run_forward(model, token_ids, cu_seqlens, batch, total_tokens, max_seqlen, k_active, model->cfg.layers,
                       true, workspace, workspace_bytes, logits_out, (hipStream_t)hip_stream);
}

int sp_forward_partial(const sp_model* model, const int32_t* token_ids, const int32_t* cu_seqlens, int32_t batch,
                       int32_t total_tokens, int32_t max_seqlen, int32_t k_active, int32_t stop_after_layers,
                       void* workspace, size_t workspace_bytes, void* hip_stream)
{
    if (!model) return SP_EINVAL;
    return run_forward(model, token_ids, cu_seqlens, batch, total_tokens, max_seqlen, k_active, stop_after_layers,
                       false, workspace, workspace_bytes, nullptr, (hipStream_t)hip_stream);
}

int sp_forward_profiled(const sp_model* model, const int32_t* token_ids, const int32_t* cu_seqlens, int32_t batch,
                        int32_t total_tokens, int32_t max_seqlen, int32_t k_active, void* workspace,
                        size_t workspace_bytes, float* logits_out, void* hip_stream, float* phase_ms_host)
{
    if (!model || !phase_ms_host) return SP_EINVAL;
    PhaseTimer pt;
    hipStream_t s = (hipStream_t)hip_stream;
    int rc = run_forward(model, token_ids, cu_seqlens, batch, total_tokens, max_seqlen, k_active, model->cfg.layers,
                         true, workspace, workspace_bytes, logits_out, s, &pt);
    if (hipStreamSynchronize(s) != hipSuccess || !pt.ok) rc = rc == SP_OK ? SP_EHIP : rc;
    for (int i = 0; i < SP_PHASE_COUNT; ++i) phase_ms_host[i] = 0.f;
    if (rc == SP_OK)
        for (int i = 1; i < pt.n; ++i) {
            float ms = 0.f;
            if (hipEventElapsedTime(&ms, pt.ev[i - 1], pt.ev[i]) != hipSuccess) { rc = SP_EHIP; break; }
            phase_ms_host[pt.phase[i]] += ms;
        }
    pt.release();
    return rc;
}

int sp_probe_e4m3(const float* x_host, int64_t n, uint8_t* codes_host)
{
    if (!x_host || !codes_host) return SP_EINVAL;
    if (n < 0) return SP_ESHAPE;
    for (int64_t i = 0; i < n; ++i) codes_host[i] = f32_to_e4m3(x_host[i]);
    return SP_OK;
}

int sp_probe_gelu(const float* x_device, float* y_device, int64_t n, void* hip_stream)
{
    if (!x_device || !y_device) return SP_EINVAL;
    if (n < 1 || n > ((int64_t)1 << 31)) return SP_ESHAPE;
    return launch_gelu_probe(x_device, y_device, (long)n, (hipStream_t)hip_stream) == hipSuccess ? SP_OK : SP_EHIP;
}

int sp_probe_gelu_fp8(const float* x_device, float* y_device, int64_t n, void* hip_stream)
{
    if (!x_device || !y_device) return SP_EINVAL;
    if (n < 1 || n > ((int64_t)1 << 31)) return SP_ESHAPE;
    return launch_gelu_q8_probe(x_device, y_device, (long)n, (hipStream_t)hip_stream) == hipSuccess ? SP_OK : SP_EHIP;
}

void sp_free(sp_model* model)
{
    if (!model) return;
    if (model->aux) {
        (void)hipStreamSynchronize(model->aux);
        (void)hipEventDestroy(model->ev_fork);
        (void)hipEventDestroy(model->ev_join);
        (void)hipStreamDestroy(model->aux);
    }
    delete model->mu;
    delete model;
}

const char* sp_strerror(int code)
{
    switch (code) {
        case SP_OK: return "ok";
        case SP_EINVAL: return "invalid argument (null or misaligned pointer, malformed config)";
        case SP_ESHAPE: return "unsupported or inconsistent shape";
        case SP_EKACTIVE: return "k_active outside 1..K";
        case SP_ENOMEM: return "buffer smaller than required";
        case SP_EHIP: return "HIP runtime error";
        case SP_ETOOBIG: return "call too large for the library's static workspace (use sp_forward with a workspace of your own)";
        case SP_EFULL: return "length-aware buffer storage full";
        case SP_EEMPTY: return "length-aware buffer empty";
        default: return "unknown error code";
    }
}

int sp_check_inputs(const sp_model* model, const int32_t* token_ids, const int32_t* cu_seqlens, int32_t batch,
                    int32_t total_tokens, int32_t max_seqlen, void* scratch, void* hip_stream, int32_t* problems_host)
{
    if (!model || !token_ids || !cu_seqlens || !scratch || !problems_host || ((uintptr_t)scratch & 3)) return SP_EINVAL;
    if (batch < 1 || total_tokens < batch || max_seqlen < 1 || max_seqlen > model->cfg.max_pos) return SP_ESHAPE;
    hipStream_t s = (hipStream_t)hip_stream;
    if (sp::launch_check_inputs(token_ids, cu_seqlens, batch, total_tokens, max_seqlen, model->cfg.vocab,
                                (unsigned*)scratch, s) != hipSuccess)
        return SP_EHIP;
    unsigned flags = 0;
    if (hipMemcpyAsync(&flags, scratch, sizeof flags, hipMemcpyDeviceToHost, s) != hipSuccess ||
        hipStreamSynchronize(s) != hipSuccess)
        return SP_EHIP;
    *problems_host = (int32_t)flags;
    return SP_OK;
}

int sp_pack(const int32_t* lengths_host, int32_t batch, int32_t* cu_seqlens_host)
{
    if (!lengths_host || !cu_seqlens_host) return SP_EINVAL;
    if (batch < 1) return SP_ESHAPE;
    int64_t acc = 0;
    cu_seqlens_host[0] = 0;
    for (int32_t i = 0; i < batch; ++i) {
        if (lengths_host[i] < 1) return SP_ESHAPE;
        acc += lengths_host[i];
        if (acc > INT32_MAX) return SP_ESHAPE;
        cu_seqlens_host[i + 1] = (int32_t)acc;
    }
    return SP_OK;
}

}  // extern "C"
