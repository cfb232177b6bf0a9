// fp32 path, calls of few rows: a launch per layer.  What it starts with is the embedding, or the attention over the queries, keys and values
// that the launch before left; what it ends with is the q|k|v projection of the next layer, or, in the last layer, which then has the first
// token of every sequence as its rows, pooler and classifier.
//
// Such a call is a chain of dependent launches of 4-6 us that leave the chip idle: six per layer and one for the attention.  All but the
// keys and values of the other rows is row-wise, so a workgroup takes two rows through the whole chain with the rows in LDS and reads
// the layer's weights (768 KB at 128 x 512) from the L2, which is what bounds it: about 64 bytes per cycle and compute unit.
//   * attention (RowAttention): two waves per row and head; its loads are requested first, then the first four blocks of weights, then it
//     is computed.  The rows' q|k|v alternate between two buffers: other workgroups read a layer's while the next one's are written.
//   * sixteen lanes share an output feature and read 256 bytes in a row of its weights ([out][in]); eight waves x four
//     features x four make a block of 128 features x 128 reduction elements, eight wave-loads per wave; the next three blocks are
//     in flight, also across the barriers between the projections (one in flight: twice the time, a block waits for its
//     memory round trip).  The order of the blocks is fixed at compile time, an instance per FFN width.
//   * a lane's partial sums are added over the sixteen lanes by four data-parallel-primitive adds; then one lane per output
//     applies bias, GELU or residual.  Biases and LayerNorm parameters come through LDS, so nothing waits behind the weights.
// us a call, two students of 2 layers x 128 wide on 86 tokens: separate launches, 19 of them, 83.6; one launch per layer after
// the attention, a block of weights in flight, and embedding, first q|k|v, pooler and classifier apart, 8 launches, 51; these as now, the
// attention apart, 6 launches, 38.8; this, 4 launches, 30.9 (30.8 with the last layer's q|k|v in the other buffer where layers are even).  One
// of 256 tokens 90.9 / 40.8, one student on one of 512 147 / 49.6.
#include <type_traits>
#include <utility>

#include "sp_internal.h"

namespace sp {

namespace {

constexpr int kWaves = 8, kRows = 2, H = 128;             // (see f32_layer_supported)
constexpr int kAhead = 4;                                   // blocks of weights in registers

constexpr int kPart = 68;                                   // floats of LDS per wave: its sums of a row's and head's values, maximum, sum

enum { FROM_EMBEDDING, FROM_ATTENTION };                   // what the rows come from
enum { TO_QKV, TO_ROWS, TO_CLASSES };                       // and what is made of them: q|k|v, x alone, the students' classifier outputs

struct F32LayerArgs {
    const char* arena;
    size_t ss, wo, bo, g1, be1, w1, b1, w2, b2, g2, be2;    // byte offsets into a student slab (FROM_EMBEDDING: g2, be2 alone)
    size_t wn, bn;                    // what follows the last LayerNorm: q|k|v or the pooler, [out][in]
    size_t wc, bc, tok, pos;
    const float* qkv;                 // FROM_ATTENTION: queries, keys and values of the rows
    float *x, *qkv_out, *z, *att;     // student strides: rows x H, rows x 3 H, M x C, rows x H (att: last layer only)
    float* logits;                    // one student: its classifier outputs once more (null: somebody adds the students' up)
    const int32_t *ids, *cu;
    int M, Tn, rows, B, C, V, P;      // M: rows to compute (tokens, or first tokens of sequences)
    int max_seqlen;
    float eps;
};

// A block of a matrix with reduction depth K: features f0 + 32 i + 4 wave + lane / 16 (i < 4), reduction elements k0 + 4 (lane % 16)
// and 64 more
__device__ __forceinline__ void load_block(f32x4 (&w)[8], const float* W, int K, int f0, int k0, int lane, int wave)
{
    const float* p = W + (size_t)(f0 + wave * 4 + (lane >> 4)) * K + k0 + (lane & 15) * 4;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        w[2 * i] = *(const f32x4*)(p + (size_t)i * 32 * K);
        w[2 * i + 1] = *(const f32x4*)(p + (size_t)i * 32 * K + 64);
    }
}

__device__ __forceinline__ void multiply_block(const f32x4 (&w)[8], const float* xs, int pitch, int lane, float (&acc)[kRows][4])
{
    const int l16 = lane & 15;
#pragma unroll
    for (int r = 0; r < kRows; ++r) {
        const f32x4 xa = *(const f32x4*)(xs + r * pitch + l16 * 4), xb = *(const f32x4*)(xs + r * pitch + 64 + l16 * 4);
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                acc[r][i] = fmaf(w[2 * i][e], xa[e], acc[r][i]);
                acc[r][i] = fmaf(w[2 * i + 1][e], xb[e], acc[r][i]);
            }
    }
}

// emit(feature - f0, row, sum over the sixteen lanes) and zero the sums
template <class Emit>
__device__ __forceinline__ void finish_block(float (&acc)[kRows][4], int lane, int wave, Emit emit)
{
    const int l16 = lane & 15;
    float out = 0.f;                                        // lane l16 = 4 r + i of the group takes row r, step i
#pragma unroll
    for (int r = 0; r < kRows; ++r)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            float v = acc[r][i];
            v += dpp_moved<kDppPair>(v);
            v += dpp_moved<kDppQuad>(v);
            v += dpp_moved<kDppHalfRowMirror>(v);
            v += dpp_moved<kDppRowMirror>(v);
            out = l16 == 4 * r + i ? v : out;
            acc[r][i] = 0.f;
        }
    if (l16 < 4 * kRows) emit((l16 & 3) * 32 + wave * 4 + (lane >> 4), l16 >> 2, out);
}

// LayerNorm of a row in LDS, in place, by one wave; dst (may be null): the row once more
__device__ inline void layernorm_row(float* v, const float* g, const float* b, float eps, int lane, float* dst)
{
    const float x0 = v[lane], x1 = v[lane + 64];
    const float inv_h = 1.0f / H, mean = wave_sum(x0 + x1) * inv_h;
    const float d0 = x0 - mean, d1 = x1 - mean, inv = __builtin_amdgcn_rsqf(wave_sum(d0 * d0 + d1 * d1) * inv_h + eps);
    const float o0 = g[lane] * (d0 * inv) + b[lane], o1 = g[lane + 64] * (d1 * inv) + b[lane + 64];
    v[lane] = o0;
    v[lane + 64] = o1;
    if (dst) {
        dst[lane] = o0;
        dst[lane + 64] = o1;
    }
}

// f(0) ... f(N - 1), the number as a constant
template <class Fn, int... I>
__device__ __forceinline__ void each_of(std::integer_sequence<int, I...>, Fn f) { (f(std::integral_constant<int, I>{}), ...); }
template <int N, class Fn>
__device__ __forceinline__ void each(Fn f) { each_of(std::make_integer_sequence<int, N>{}, f); }

template <int FROM, int TO, int FB>
constexpr int f32_layer_floats()                            // of LDS; see the kernel's carve-up
{
    return kRows * H + 2 * H + (TO == TO_QKV ? 3 : 1) * H + (FROM == FROM_EMBEDDING ? 0 : kRows * (H + 128 * FB) + 4 * H + 128 * FB + kWaves * kPart);
}

// Attention of one row and head by two waves, every other 32 keys each: sixteen lanes share a key (four dimensions each), four keys side
// by side, 64 keys of both waves per step; the first step's keys and values are requested together by begin().  Running softmax with
// exact exponentials; the wave's sums (unscaled), maximum and sum of the weights go to LDS, and a wave without keys leaves none.
struct RowAttention {
    const float* keys;                                      // of the sequence's first token, this lane's dimensions; values: H behind
    int L, first;                                           // first: the wave's first key
    f32x4 q, k[8], v[8];

    __device__ __forceinline__ int key(int s0, int i, int lane) const { return s0 + first + 4 * i + (lane >> 4); }
    __device__ __forceinline__ void request(int s0, int lane)
    {
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const int t = key(s0, i, lane) < L ? key(s0, i, lane) : L - 1;
            k[i] = *(const f32x4*)(keys + (size_t)t * 3 * H);
            v[i] = *(const f32x4*)(keys + (size_t)t * 3 * H + H);
        }
    }
    // row: index of the sequence (of_first), else of the token
    __device__ __forceinline__ void begin(const F32LayerArgs& p, const float* qkv, bool of_first, int row, int token, int head, int half, int lane)
    {
        int t0, t1;
        if (of_first) { t0 = p.cu[row]; t1 = p.cu[row + 1]; }
        else last_sequence(p.cu, p.B, lane, [&](int, int c) { return c <= row; }, t0, t1);
        t0 = t0 < 0 ? 0 : (t0 > p.Tn - 1 ? p.Tn - 1 : t0);
        L = t1 - t0;
        L = L < 1 ? 1 : L;
        L = L > p.max_seqlen ? p.max_seqlen : L;
        L = L > p.Tn - t0 ? p.Tn - t0 : L;
        first = 32 * half;
        const int d = head * 64 + (lane & 15) * 4;
        q = *(const f32x4*)(qkv + (size_t)token * 3 * H + d);
        keys = qkv + (size_t)t0 * 3 * H + H + d;
        request(0, lane);
    }
    __device__ __forceinline__ void run(float* out, int lane)
    {
        float mrun = -INFINITY, lrun = 0.f;
        f32x4 o = {0.f, 0.f, 0.f, 0.f};
        for (int s0 = 0;;) {
            float s[8], mx = mrun;
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                float a = q[0] * k[i][0];
#pragma unroll
                for (int e = 1; e < 4; ++e) a = fmaf(q[e], k[i][e], a);
                a += dpp_moved<kDppPair>(a);
                a += dpp_moved<kDppQuad>(a);
                a += dpp_moved<kDppHalfRowMirror>(a);
                a += dpp_moved<kDppRowMirror>(a);
                s[i] = key(s0, i, lane) < L ? a * 0.125f : -INFINITY;
                mx = fmaxf(mx, s[i]);
            }
            float a = mx, b = mx;
            swap_rows(a, b);
            mx = fmaxf(a, b);
            a = mx;
            b = mx;
            swap_halves(a, b);
            mx = fmaxf(a, b);
            const float ref = mx == -INFINITY ? 0.f : mx, alpha = expf(mrun - ref);     // (no key of the wave's yet: weights of zero)
            mrun = mx;
            lrun *= alpha;
            o *= alpha;
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const float w = expf(s[i] - ref);
                lrun += w;
                o += w * v[i];
            }
            s0 += 64;
            if (s0 >= L) break;
            request(s0, lane);
        }
        auto over_keys = [](float x) {                      // over the four keys side by side
            float a = x, b = x;
            swap_rows(a, b);
            x = a + b;
            a = x;
            b = x;
            swap_halves(a, b);
            return a + b;
        };
#pragma unroll
        for (int e = 0; e < 4; ++e) o[e] = over_keys(o[e]);
        lrun = over_keys(lrun);
        if (lane < 16) *(f32x4*)(out + 4 * lane) = o;
        if (lane == 0) {
            out[64] = mrun;
            out[65] = lrun;
        }
    }
};

// FB: FFN width / 128
template <int FROM, int TO, int FB>
__global__ __launch_bounds__(64 * kWaves) void f32_layer_kernel(F32LayerArgs p)
{
    __shared__ __attribute__((aligned(16))) float lds[f32_layer_floats<FROM, TO, FB>()];
    constexpr int F = 128 * FB, NB = TO == TO_QKV ? 3 * H : H;         // NB: biases of what follows the last LayerNorm
    constexpr int BODY = FROM == FROM_EMBEDDING ? 0 : 1 + 2 * FB, BLOCKS = BODY + (TO == TO_QKV ? 3 : TO == TO_CLASSES ? 1 : 0);
    const int m = blockIdx.y, r0 = blockIdx.x * kRows;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    float *xa = lds, *g2 = xa + kRows * H, *be2 = g2 + H, *bn = be2 + H, *xr = bn + NB, *bo = xr + kRows * H, *g1 = bo + H;
    float *be1 = g1 + H, *b2 = be1 + H, *b1 = b2 + H, *xg = b1 + F, *part = xg + kRows * F;
    const char* sb = p.arena + (size_t)m * p.ss;

    // token row of row r (rows beyond the last one repeat it)
    auto token = [&](int r) {
        r = r < p.M ? r : p.M - 1;
        if (TO != TO_CLASSES) return r;
        const int t = p.cu[r];
        return t < 0 ? 0 : (t < p.Tn ? t : p.Tn - 1);
    };
    f32x4 w[kAhead][8];
    float acc[kRows][4] = {};
    // blocks in order: Wo; W1 feature block by feature block; W2 along its reduction; then q|k|v or the pooler
    auto request = [&](auto i_c) {
        constexpr int i = decltype(i_c)::value;
        if constexpr (i >= BLOCKS) return;
        else if constexpr (i >= BODY) load_block(w[i % kAhead], (const float*)(sb + p.wn), H, (i - BODY) * 128, 0, lane, wave);
        else if constexpr (i == 0) load_block(w[0], (const float*)(sb + p.wo), H, 0, 0, lane, wave);
        else if constexpr (i <= FB) load_block(w[i % kAhead], (const float*)(sb + p.w1), H, (i - 1) * 128, 0, lane, wave);
        else load_block(w[i % kAhead], (const float*)(sb + p.w2), F, 0, (i - 1 - FB) * 128, lane, wave);
    };
    auto multiply = [&](auto i_c, const float* xs, int pitch) {
        constexpr int i = decltype(i_c)::value;
        multiply_block(w[i % kAhead], xs, pitch, lane, acc);
        request(std::integral_constant<int, i + kAhead>{});
    };

    RowAttention at;
    if constexpr (FROM == FROM_ATTENTION) {                 // (its loads in front of the weights': they are waited for first)
        const int row = r0 + (wave >> 2) < p.M ? r0 + (wave >> 2) : p.M - 1;
        at.begin(p, p.qkv + (size_t)m * p.rows * 3 * H, TO == TO_CLASSES, row, token(row), wave >> 1 & 1, wave & 1, lane);
    }
    if constexpr (FROM == FROM_EMBEDDING) {
        if (wave < kRows) {                                 // a wave per row: its sequence starts at the last boundary up to it
            const int row = token(r0 + wave), id = p.ids[row];
            int start = 0;
            for (int b0 = 0; b0 < p.B; b0 += 64) {
                const int cv = b0 + lane < p.B ? p.cu[b0 + lane] : 0x7fffffff, n = __popcll(__ballot(cv <= row));
                if (n > 0) start = __builtin_amdgcn_readlane(cv, n - 1);
            }
            int at = row - start;
            at = at < 0 ? 0 : (at < p.P ? at : p.P - 1);
            const float* te = (const float*)(sb + p.tok) + (size_t)(id < 0 ? 0 : (id < p.V ? id : p.V - 1)) * H;
            const float* pe = (const float*)(sb + p.pos) + (size_t)at * H;
#pragma unroll
            for (int c = lane; c < H; c += 64) xa[wave * H + c] = te[c] + pe[c];
        }
    }
    // Biases, LayerNorm parameters and residual rows: requested here, put down behind the attention (a wait for them in between would keep the
    // weights' requests back).
    constexpr int NT = 64 * kWaves, NB1 = (F + NT - 1) / NT;
    auto element = [&](size_t off, int n, int i) { return ((const float*)(sb + off))[i < n ? i : n - 1]; };
    const float v_g2 = element(p.g2, H, tid), v_be2 = element(p.be2, H, tid), v_bn = TO == TO_ROWS ? 0.f : element(p.bn, NB, tid);
    float v_bo, v_g1, v_be1, v_b2, v_x, v_b1[NB1];
    size_t own = 0;                                         // this thread's element of the rows (of the first kRows * H threads)
    if constexpr (FROM == FROM_ATTENTION) {
        v_bo = element(p.bo, H, tid);
        v_g1 = element(p.g1, H, tid);
        v_be1 = element(p.be1, H, tid);
        v_b2 = element(p.b2, H, tid);
#pragma unroll
        for (int i = 0; i < NB1; ++i) v_b1[i] = element(p.b1, F, tid + NT * i);
        own = ((size_t)m * p.rows + token(r0 + (tid / H) % kRows)) * H + tid % H;
        v_x = p.x[own];
    }
    __builtin_amdgcn_sched_barrier(0);
    each<kAhead>(request);
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (FROM == FROM_ATTENTION) {
        at.run(part + wave * kPart, lane);
        if (tid < kRows * H) xr[tid] = v_x;
        if (tid < H) {
            bo[tid] = v_bo;
            g1[tid] = v_g1;
            be1[tid] = v_be1;
            b2[tid] = v_b2;
        }
#pragma unroll
        for (int i = 0; i < NB1; ++i)
            if (tid + NT * i < F) b1[tid + NT * i] = v_b1[i];
    }
    if (tid < H) {
        g2[tid] = v_g2;
        be2[tid] = v_be2;
    }
    if (TO != TO_ROWS && tid < NB) bn[tid] = v_bn;
    if constexpr (FROM == FROM_ATTENTION) {
        barrier_lds();
        if (tid < kRows * H) {                              // the halves of the keys, waves 2 n and 2 n + 1
            const float *a = part + (tid >> 6) * 2 * kPart, *b = a + kPart;
            const float mx = fmaxf(a[64], b[64]), wa = expf(a[64] - mx), wb = expf(b[64] - mx);
            const float v = (a[tid & 63] * wa + b[tid & 63] * wb) / (a[65] * wa + b[65] * wb);
            xa[tid] = v;
            if (TO != TO_QKV) p.att[own] = v;
        }
    }
    barrier_lds();
    if constexpr (FROM == FROM_ATTENTION) {
        multiply(std::integral_constant<int, 0>{}, xa, H);
        finish_block(acc, lane, wave, [&](int f, int r, float v) { xr[r * H + f] = v + bo[f] + xr[r * H + f]; });
        barrier_lds();
        if (wave < kRows) layernorm_row(xr + wave * H, g1, be1, p.eps, lane, nullptr);
        barrier_lds();
        each<FB>([&](auto i) {
            multiply(std::integral_constant<int, 1 + decltype(i)::value>{}, xr, H);
            finish_block(acc, lane, wave, [&](int f, int r, float v) {
                const float u = v + b1[i() * 128 + f];
                xg[r * F + i() * 128 + f] = 0.5f * u * (1.0f + erff(u * 0.70710678118654752f));
            });
        });
        barrier_lds();
        each<FB>([&](auto i) { multiply(std::integral_constant<int, 1 + FB + decltype(i)::value>{}, xg + i() * 128, F); });
        finish_block(acc, lane, wave, [&](int f, int r, float v) { xa[r * H + f] = v + b2[f] + xr[r * H + f]; });
        barrier_lds();
    }
    if (wave < kRows)
        layernorm_row(xa + wave * H, g2, be2, p.eps, lane,
                      r0 + wave < p.M ? p.x + ((size_t)m * p.rows + token(r0 + wave)) * H : nullptr);
    if constexpr (TO == TO_ROWS) return;
    barrier_lds();
    if constexpr (TO == TO_QKV) {
        each<3>([&](auto i) {
            multiply(std::integral_constant<int, BODY + decltype(i)::value>{}, xa, H);
            finish_block(acc, lane, wave, [&](int f, int r, float v) {
                if (r0 + r < p.M) p.qkv_out[((size_t)m * p.rows + r0 + r) * 3 * H + i() * 128 + f] = v + bn[i() * 128 + f];
            });
        });
    }
    if constexpr (TO == TO_CLASSES) {
        multiply(std::integral_constant<int, BODY>{}, xa, H);
        finish_block(acc, lane, wave, [&](int f, int r, float v) { xr[r * H + f] = tanhf(v + bn[f]); });
        barrier_lds();
        if (wave < kRows && r0 + wave < p.M)
            for (int c = 0; c < p.C; ++c) {
                const float* wc = (const float*)(sb + p.wc) + c;
                const float v = wave_sum(xr[wave * H + lane] * wc[(size_t)lane * p.C] + xr[wave * H + lane + 64] * wc[(size_t)(lane + 64) * p.C]) +
                                ((const float*)(sb + p.bc))[c];
                if (lane == 0) {
                    p.z[((size_t)m * p.M + r0 + wave) * p.C + c] = v;
                    if (p.logits) p.logits[(size_t)(r0 + wave) * p.C + c] = v;
                }
            }
    }
}

template <int FROM, int TO>
hipError_t launch(const sp_model* M, const F32LayerArgs& a, int k, hipStream_t s)
{
    const dim3 grid((a.M + kRows - 1) / kRows, k);
#define SP_GO(FB) case FB: hipLaunchKernelGGL((f32_layer_kernel<FROM, TO, FB>), grid, dim3(64 * kWaves), 0, s, a); break
    switch (FROM == FROM_EMBEDDING ? 1 : M->cfg.ffn / 128) {
        SP_GO(1);
        default: return hipErrorInvalidValue;
        case 2: case 3: case 4: case 5: case 6:
            if constexpr (FROM != FROM_EMBEDDING)
                switch (M->cfg.ffn / 128) { SP_GO(2); SP_GO(3); SP_GO(4); SP_GO(5); SP_GO(6); }
    }
#undef SP_GO
    return hipGetLastError();
}

F32LayerArgs layer_args(const sp_model* M, size_t lo, const void* qkv, void* x, const int32_t* cu, int B, int T, int max_seqlen, int rows)
{
    const sp_config& c = M->cfg;
    const ArenaLayout& L = M->L;
    F32LayerArgs a{};
    a.arena = M->arena; a.ss = L.student_stride;
    a.wo = lo + L.wo; a.bo = lo + L.bo; a.g1 = lo + L.ln1g; a.be1 = lo + L.ln1b; a.w1 = lo + L.w1; a.b1 = lo + L.b1;
    a.w2 = lo + L.w2; a.b2 = lo + L.b2; a.g2 = lo + L.ln2g; a.be2 = lo + L.ln2b;
    a.qkv = (const float*)qkv; a.x = (float*)x; a.cu = cu; a.max_seqlen = max_seqlen;
    a.M = T; a.Tn = T; a.rows = rows; a.B = B; a.C = c.classes; a.V = c.vocab; a.P = c.max_pos; a.eps = c.ln_eps;
    return a;
}

}  // namespace

// Every workgroup reads the layer's weights, so the kernel is for narrow students (hidden 128 with an FFN of up to 768, 1 MB of
// weights: 7 us at the L2's rate; the separate launches spread them over the chip) and for calls of at most one workgroup per
// compute unit.
bool f32_layer_supported(const sp_config& c, long rows_of_all_students)
{
    return !bf16_path(c) && c.hidden == H && c.ffn % 128 == 0 && c.ffn <= 768 && rows_of_all_students <= 256 * kRows;
}

hipError_t launch_f32_embed(const sp_model* M, size_t lo, const int32_t* ids, const int32_t* cu, int B, int T, void* x, void* qkv,
                            int rows, int k, hipStream_t s)
{
    const ArenaLayout& L = M->L;
    F32LayerArgs a = layer_args(M, lo, nullptr, x, cu, B, T, 0, rows);
    a.g2 = L.emb_g; a.be2 = L.emb_b; a.wn = lo + L.wqkv; a.bn = lo + L.bqkv; a.tok = L.tok; a.pos = L.pos; a.ids = ids;
    a.qkv_out = (float*)qkv;
    return launch<FROM_EMBEDDING, TO_QKV>(M, a, k, s);
}

hipError_t launch_f32_layer(const sp_model* M, size_t lo, const void* qkv, void* x, void* qkv_next, void* att, const int32_t* cu, int B, int T, int max_seqlen,
                            int rows, int k, hipStream_t s)
{
    F32LayerArgs a = layer_args(M, lo, qkv, x, cu, B, T, max_seqlen, rows);
    a.att = (float*)att;
    if (!qkv_next) return launch<FROM_ATTENTION, TO_ROWS>(M, a, k, s);
    if (qkv_next == qkv) return hipErrorInvalidValue;       // (other workgroups read it)
    a.wn = lo + M->L.layer_stride + M->L.wqkv; a.bn = lo + M->L.layer_stride + M->L.bqkv; a.qkv_out = (float*)qkv_next;
    return launch<FROM_ATTENTION, TO_QKV>(M, a, k, s);
}

hipError_t launch_f32_last(const sp_model* M, size_t lo, const void* qkv, void* x, void* att, const int32_t* cu, int B, int T, int max_seqlen, int rows, int k,
                           float* z, float* logits, hipStream_t s)
{
    F32LayerArgs a = layer_args(M, lo, qkv, x, cu, B, T, max_seqlen, rows);
    a.M = B; a.wn = M->L.wp_t; a.bn = M->L.bp; a.wc = M->L.wc; a.bc = M->L.bc; a.z = z; a.att = (float*)att;
    if (logits && k > 1) return hipErrorInvalidValue;       // (their sum takes all students' outputs)
    a.logits = logits;
    return launch<FROM_ATTENTION, TO_CLASSES>(M, a, k, s);
}

}  // namespace sp
