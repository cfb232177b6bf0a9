// Students of hidden width 256 (bf16 path): two launches make an encoder layer, with the attention between them.
//   layer_kernel: x1 = LN(att Wo + bo + x),  out = LN(x1 + gelu(x1 W1 + b1) W2 + b2)
//   embed_qkv_kernel: x = LN(embedding), q|k|v = x Wqkv + bqkv (first layer)
// As separate launches a layer writes and reads the rows before each LayerNorm, x1 and the FFN's activations (F wide), and at a depth of
// 256 a projection has four k-tiles between its first loads and its epilogue.  Here a workgroup takes 64 tokens through all of it: four
// waves, each with all the tokens and 64 of the 256 features (of the FFN's, 64 of every 256), so that sums of whole rows stay in
// registers; x1 and 256 FFN activations at a time pass from wave to wave in LDS, in the tile layout of the projections (rows of eight 16-byte
// slots, slot = chunk ^ ((row / 2) % 8): no bank conflicts, and a wave's 64 features are one k-tile).  The weights go from memory (L2) to
// registers, two k-tiles ahead, across the barriers as well.  76 KB of LDS and 256 registers: two workgroups per compute unit, so that one's
// GELU and statistics run under the other's products.
// What bounds layer_kernel: the products (2048 matrix-core cycles for each of 1 + 2 F / 256 of them and workgroup), the GELU's vector
// instructions (about as many cycles) and the weights' way from the L2 (all of them once per workgroup, 1.2 MB at F = 1024), none
// saturated.  embed_qkv_kernel: the write of its outputs.
// us per launch, three students on 14653 tokens, F = 1024: output projection 16.0, LayerNorm 12.5, FFN up 42.9 and down 32.4 before, layer_kernel
// 69 (750 TFLOP/s); embedding 16.4 and q|k|v 30.1, embed_qkv_kernel 36.4.  (Three of its workgroups to a compute unit, their outputs staged by
// halves: 36.8.)
// Roundings: x1 and the activations to bf16 as in the separate launches; the sums before a LayerNorm are not rounded.
#include <atomic>

#include "sp_internal.h"

namespace sp {

namespace {

constexpr int kH = 256, kTok = 64, kMaxF = 1024, kTileUnits = kTok * 8;     // kTileUnits: 16-byte units of 64 tokens x 64 features
constexpr size_t kLayerLds = (size_t)8 * kTileUnits * 16 + (6 * kH + kMaxF + 2 * 4 * kTok) * 4;
static_assert(2 * kLayerLds <= 160 * 1024, "two workgroups per compute unit");

struct LayerArgs {
    const char* arena;
    size_t ss, wo, bo, g1, be1, w1, b1, w2, b2, g2, be2;    // byte offsets into a student slab
    const bf16 *att, *x;
    bf16* out;
    size_t t_ss;                      // student stride of the three, elements
    int F, mtiles, total;
    float eps;
};

// Accumulators of a wave: element v of lane l in block (i, t) is token 32 t + l % 32, feature 64 wave + 32 i + 8 (v / 4) + 4 (l / 32) + v % 4.
typedef f32x16 Acc[2][2];
typedef bf16x8 Weights[2][4][2];                            // two k-tiles of 64: [slot][step of 16][block of 32 features]

// step s of a k-tile at kt_off bytes behind base, depth Kd: lane -> row l % 32 of a 32-feature block, chunk l / 32 (operand blocks, see ArenaLayout)
__device__ __forceinline__ int weights_lane(int j31, int g, int Kd) { return 2 * ((j31 >> 4) * 16 * Kd + g * 128 + (j31 & 15) * 8); }
__device__ __forceinline__ void load_weights(Weights& w, int slot, int s, const char* base, int lane_off, int Kd, int kt_off)
{
#pragma unroll
    for (int i = 0; i < 2; ++i) w[slot][s][i] = __builtin_bit_cast(bf16x8, load16(base, lane_off + s * 512, kt_off + i * 64 * Kd));
}
// a += W rows^T over four k-tiles; request(kt, s): the step that takes the place of step s of k-tile kt, two k-tiles on
template <class Request>
__device__ __forceinline__ void multiply(Acc& a, const Weights& w, const uint4* rows, int j31, int g, Request request)
{
    const int xlane = j31 * 8 + (g ^ ((j31 >> 1) & 7));
    bf16x8 fx[2][2];
    auto frag = [&](int kt, int s, int t) { return *(const bf16x8*)(rows + ((kt * kTileUnits + xlane) ^ (2 * s)) + t * 256); };
#pragma unroll
    for (int t = 0; t < 2; ++t) fx[0][t] = frag(0, 0, t);
#pragma unroll
    for (int kt = 0; kt < 4; ++kt)
#pragma unroll
        for (int s = 0; s < 4; ++s) {
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                if (kt < 3 || s < 3) fx[(s + 1) & 1][t] = frag(s < 3 ? kt : kt + 1, (s + 1) & 3, t);
#pragma unroll
                for (int i = 0; i < 2; ++i) a[i][t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(w[kt & 1][s][i], fx[s & 1][t], a[i][t], 0, 0, 0);
            }
            request(kt, s);
            __builtin_amdgcn_sched_barrier(0);
        }
}
__device__ __forceinline__ void set_bias(Acc& a, const float* b, int g)    // b: of the wave's 64 features
{
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int v4 = 0; v4 < 4; ++v4) {
            const f32x4 b4 = *(const f32x4*)(b + 32 * i + 8 * v4 + 4 * g);
#pragma unroll
            for (int t = 0; t < 2; ++t)
#pragma unroll
                for (int e = 0; e < 4; ++e) a[i][t][4 * v4 + e] = b4[e];
        }
}
// four features of a token in a wave's k-tile
__device__ __forceinline__ bf16x4* cell(uint4* tile, int i, int t, int v4, int j31, int g)
{
    const int r = 32 * t + j31;
    return (bf16x4*)((char*)tile + r * 128 + (((4 * i + v4) ^ ((r >> 1) & 7)) << 4) + 8 * g);
}
__device__ __forceinline__ void put(uint4* tile, const Acc& a, int j31, int g)
{
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int v4 = 0; v4 < 4; ++v4) {
                bf16x4 o;
#pragma unroll
                for (int e = 0; e < 4; ++e) o[e] = (bf16)a[i][t][4 * v4 + e];
                *cell(tile, i, t, v4, j31, g) = o;
            }
}
// a wave's k-tile to the rows at dst (row stride ld), 128 bytes of each
__device__ __forceinline__ void store_rows(const uint4* tile, bf16* dst, int ld, int lane)
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    const int rr = lane >> 3, cc = lane & 7;
#pragma unroll
    for (int q = 0; q < 8; ++q) {
        const int r = 8 * q + rr;
        store16_through<false>(dst + (size_t)r * ld + cc * 8, __builtin_bit_cast(u32x4, tile[r * 8 + (cc ^ ((r >> 1) & 7))]));
    }
}

// (out may be x: a workgroup has read its rows before it writes them.)
__global__ __launch_bounds__(256, 2) void layer_kernel(LayerArgs p)
{
    extern __shared__ uint4 smem[];
    uint4 *const X = smem, *const G = smem + 4 * kTileUnits;
    float* const prm = (float*)(smem + 8 * kTileUnits);      // bo, g1, be1, b2, g2, be2, b1
    float* const red = prm + 6 * kH + kMaxF;                // [2][wave][token]
    const int chunk = (p.total + 7) >> 3, lin = (int)(blockIdx.x & 7) * chunk + (int)(blockIdx.x >> 3);     // (contiguous runs per XCD)
    if ((int)(blockIdx.x >> 3) >= chunk || lin >= p.total) return;
    const int m = lin / p.mtiles, m0 = (lin - m * p.mtiles) * kTok, F = p.F;
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    int lane = tid & 63, j31 = lane & 31, g = lane >> 5;
    const char* sb = p.arena + (size_t)m * p.ss;
    const size_t row0 = (size_t)m * p.t_ss + (size_t)m0 * kH;

    // attention output and residual rows: wave-load (kt, i) is rows 8 (wave + 4 i) .. + 7 of k-tile kt, lane -> (row lane / 8, slot lane % 8)
    int aoff[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int r = 8 * (wave + 4 * i) + (lane >> 3);
        aoff[i] = 2 * (r * kH + ((lane & 7) ^ ((r >> 1) & 7)) * 8);
    }
    auto fetch = [&](const bf16* from, uint4* to) {
#pragma unroll
        for (int kt = 0; kt < 4; ++kt)
#pragma unroll
            for (int i = 0; i < 2; ++i) load_lds16(from + row0, (lds_void*)(to + kt * kTileUnits + (wave + 4 * i) * 64), aoff[i], kt * 128);
    };
    fetch(p.att, G);
    fetch(p.x, X);
    float pv[6], bv[kMaxF / 256];
    {
        const size_t at[6] = {p.bo, p.g1, p.be1, p.b2, p.g2, p.be2};
#pragma unroll
        for (int i = 0; i < 6; ++i) pv[i] = ((const float*)(sb + at[i]))[tid];
#pragma unroll
        for (int i = 0; i < kMaxF / 256; ++i) bv[i] = ((const float*)(sb + p.b1))[256 * i + tid < F ? 256 * i + tid : tid];
    }
    __builtin_amdgcn_sched_barrier(0);

    Weights w;
    const int lane_h = weights_lane(j31, g, kH), lane_f = weights_lane(j31, g, F);
    const char *wo = sb + p.wo + (size_t)wave * 128 * kH, *w1 = sb + p.w1 + (size_t)wave * 128 * kH, *w2 = sb + p.w2 + (size_t)wave * 128 * F;
    auto load_wo = [&](int slot, int s, int kt) { load_weights(w, slot, s, wo, lane_h, kH, kt * 2048); };
    auto load_w1 = [&](int slot, int s, int c, int kt) { load_weights(w, slot, s, w1, lane_h, kH, c * 512 * kH + kt * 2048); };
    auto load_w2 = [&](int slot, int s, int c, int kt) { load_weights(w, slot, s, w2, lane_f, F, (4 * c + kt) * 2048); };
#pragma unroll
    for (int kt = 0; kt < 2; ++kt)
#pragma unroll
        for (int s = 0; s < 4; ++s) load_wo(kt, s, kt);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < 6; ++i) prm[i * kH + tid] = pv[i];
#pragma unroll
    for (int i = 0; i < kMaxF / 256; ++i) prm[6 * kH + 256 * i + tid] = bv[i];
    wait_vmcnt<16>();                                       // the rows (behind them: two k-tiles of weights)
    barrier_lds();

    uint4* const own = X + wave * kTileUnits;               // the wave's features of the rows
    auto add_rows = [&](Acc& a) {
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int t = 0; t < 2; ++t)
#pragma unroll
                for (int v4 = 0; v4 < 4; ++v4) {
                    const bf16x4 x4 = *cell(own, i, t, v4, j31, g);
#pragma unroll
                    for (int e = 0; e < 4; ++e) a[i][t][4 * v4 + e] += (float)x4[e];
                }
    };
    // sums over all features of this lane's two tokens: over its own values, the other half's and the other waves'
    auto row_sums = [&](float s0, float s1, float* r, float (&out)[2]) {
        float a0 = s0, a1 = s1;
        swap_halves(s0, a0);
        swap_halves(s1, a1);
        s0 += a0;
        s1 += a1;
        r[wave * kTok + lane] = g ? s1 : s0;                // (token 32 g + l % 32 = lane)
        barrier_lds();
#pragma unroll
        for (int t = 0; t < 2; ++t) out[t] = (r[32 * t + j31] + r[kTok + 32 * t + j31]) + (r[2 * kTok + 32 * t + j31] + r[3 * kTok + 32 * t + j31]);
    };
    auto normalise = [&](Acc& a, const float* gam, const float* bet) {
        float s[2], mean[2], inv[2];
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            s[t] = 0.f;
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int v = 0; v < 16; ++v) s[t] += a[i][t][v];
        }
        row_sums(s[0], s[1], red, mean);
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            mean[t] *= 1.0f / kH;
            s[t] = 0.f;
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    a[i][t][v] -= mean[t];
                    s[t] = __builtin_fmaf(a[i][t][v], a[i][t][v], s[t]);
                }
        }
        row_sums(s[0], s[1], red + 4 * kTok, inv);
#pragma unroll
        for (int t = 0; t < 2; ++t) inv[t] = __builtin_amdgcn_rsqf(__builtin_fmaf(inv[t], 1.0f / kH, p.eps));
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int v4 = 0; v4 < 4; ++v4) {
                const int f = 64 * wave + 32 * i + 8 * v4 + 4 * g;
                const f32x4 ga = *(const f32x4*)(gam + f), be = *(const f32x4*)(bet + f);
#pragma unroll
                for (int t = 0; t < 2; ++t)
#pragma unroll
                    for (int e = 0; e < 4; ++e) a[i][t][4 * v4 + e] = ga[e] * (a[i][t][4 * v4 + e] * inv[t]) + be[e];
            }
    };

    Acc acc, up;
    set_bias(acc, prm + 64 * wave, g);
    multiply(acc, w, G, j31, g, [&](int kt, int s) { kt < 2 ? load_wo(kt & 1, s, kt + 2) : load_w1(kt & 1, s, 0, kt - 2); });
    add_rows(acc);
    normalise(acc, prm + kH, prm + 2 * kH);                 // (its barriers: every wave is done with the attention output)
    put(own, acc, j31, g);
    set_bias(acc, prm + 3 * kH + 64 * wave, g);
    barrier_lds();
    const int nc = F / 256;
    for (int c = 0; c < nc; ++c) {
        set_bias(up, prm + 6 * kH + 256 * c + 64 * wave, g);
        multiply(up, w, X, j31, g, [&](int kt, int s) { kt < 2 ? load_w1(kt & 1, s, c, kt + 2) : load_w2(kt & 1, s, c, kt - 2); });
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int t = 0; t < 2; ++t)
#pragma unroll
                for (int v = 0; v < 16; ++v) up[i][t][v] = gelu_erf_fast(up[i][t][v]);
        barrier_lds();                                      // everybody has read the activations before
        put(G + wave * kTileUnits, up, j31, g);
        barrier_lds();
        const int cn = c + 1 < nc ? c + 1 : c;              // (behind the last one: requested and not used)
        multiply(acc, w, G, j31, g, [&](int kt, int s) { kt < 2 ? load_w2(kt & 1, s, c, kt + 2) : load_w1(kt & 1, s, cn, kt - 2); });
    }
    // (counted anew, so that no address is kept through the loop)
    lane = (int)__builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
    j31 = lane & 31;
    g = lane >> 5;
    add_rows(acc);
    normalise(acc, prm + 4 * kH, prm + 5 * kH);
    put(own, acc, j31, g);
    store_rows(own, p.out + row0 + 64 * wave, kH, lane);
}

// -------------------------------------------------------------------------------------
// Embedding, LayerNorm and q|k|v of 64 tokens.  Sixteen lanes share a row (two pieces of eight features each), a wave sixteen rows, all of
// them requested together; the statistics take four data-parallel-primitive adds for four rows at once.  Behind the one barrier each
// wave multiplies and writes by itself.
// -------------------------------------------------------------------------------------
struct EmbedQkvArgs {
    const char* arena;
    size_t ss, tok, pos, ge, be, w, b;                      // byte offsets into a student slab
    const int32_t *ids, *cu;
    bf16 *x, *att, *qkv, *vt;
    size_t t_ss;                      // student stride of x, att and vt, elements
    int B, T, V, P, rows, mtiles, total;
    float eps;
};
constexpr size_t kEmbedLds = (size_t)8 * kTileUnits * 16;

__global__ __launch_bounds__(256, 2) void embed_qkv_kernel(EmbedQkvArgs p)
{
    extern __shared__ uint4 smem[];
    uint4* const X = smem;
    const int chunk = (p.total + 7) >> 3, lin = (int)(blockIdx.x & 7) * chunk + (int)(blockIdx.x >> 3);
    if ((int)(blockIdx.x >> 3) >= chunk || lin >= p.total) return;
    const int m = lin / p.mtiles, m0 = (lin - m * p.mtiles) * kTok;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int j31 = lane & 31, g = lane >> 5, l16 = lane & 15, rq = lane >> 4;
    const char* sb = p.arena + (size_t)m * p.ss;
    uint4* const own = smem + (4 + wave) * kTileUnits;      // where the wave's outputs are put together

    // token id and position of the wave's rows, a lane each: the sequence of the first row, then what begins in the rows behind it
    const int r0 = m0 + 16 * wave, first = r0 < p.T ? r0 : p.T - 1;
    int id = lane < 16 && r0 + lane < p.T ? p.ids[r0 + lane] : 0, c0, c1, at = 0;
    id = id < 0 ? 0 : (id >= p.V ? p.V - 1 : id);
    const int b = last_sequence(p.cu, p.B, lane, [&](int, int c) { return c <= first; }, c0, c1);
    const int begin = lane == 0 ? c0 : lane == 1 ? c1 : lane < 32 && b + lane < p.B ? p.cu[b + lane] : 0x7fffffff;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        const int nb = __popcll(__ballot(begin <= r0 + r)), pos = r0 + r - __builtin_amdgcn_readlane(begin, nb > 0 ? nb - 1 : 0);
        at = lane == r ? pos : at;
    }
    at = at < 0 ? 0 : (at >= p.P ? p.P - 1 : at);
    bf16x8 te[4][2], pe[4][2];                              // row 4 it + lane / 16 of the wave's
#pragma unroll
    for (int it = 0; it < 4; ++it) {
        const bf16* t = (const bf16*)(sb + p.tok) + (size_t)__shfl(id, 4 * it + rq) * kH + 8 * l16;
        const bf16* q = (const bf16*)(sb + p.pos) + (size_t)__shfl(at, 4 * it + rq) * kH + 8 * l16;
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            te[it][c] = *(const bf16x8*)(t + 128 * c);
            pe[it][c] = *(const bf16x8*)(q + 128 * c);
        }
    }
    f32x4 ga[4], be[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        ga[c] = *(const f32x4*)((const float*)(sb + p.ge) + 128 * (c >> 1) + 8 * l16 + 4 * (c & 1));
        be[c] = *(const f32x4*)((const float*)(sb + p.be) + 128 * (c >> 1) + 8 * l16 + 4 * (c & 1));
    }
    __builtin_amdgcn_sched_barrier(0);
    Weights w;
    const int lane_h = weights_lane(j31, g, kH);
    const char* wq = sb + p.w + (size_t)wave * 128 * kH;
    auto load = [&](int slot, int s, int c, int kt) { load_weights(w, slot, s, wq, lane_h, kH, c * 512 * kH + kt * 2048); };
#pragma unroll
    for (int kt = 0; kt < 2; ++kt)
#pragma unroll
        for (int s = 0; s < 4; ++s) load(kt, s, 0, kt);
    __builtin_amdgcn_sched_barrier(0);

#pragma unroll
    for (int it = 0; it < 4; ++it) {
        const int r = 16 * wave + 4 * it + rq;
        float v[16], s = 0.f, q = 0.f;
#pragma unroll
        for (int e = 0; e < 16; ++e) {
            v[e] = (float)te[it][e >> 3][e & 7] + (float)pe[it][e >> 3][e & 7];
            s += v[e];
        }
        auto over_row = [](float a) {
            a += dpp_moved<kDppPair>(a);
            a += dpp_moved<kDppQuad>(a);
            a += dpp_moved<kDppHalfRowMirror>(a);
            return a + dpp_moved<kDppRowMirror>(a);
        };
        const float mean = over_row(s) * (1.0f / kH);
#pragma unroll
        for (int e = 0; e < 16; ++e) {
            v[e] -= mean;
            q = __builtin_fmaf(v[e], v[e], q);
        }
        const float inv = __builtin_amdgcn_rsqf(__builtin_fmaf(over_row(q), 1.0f / kH, p.eps));
        const bool live = m0 + r < p.T;
        bf16* const xr = p.x + (size_t)m * p.t_ss + (size_t)(m0 + r) * kH + 8 * l16;
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            bf16x8 o;
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const int n = 8 * c + e;
                o[e] = (bf16)(live ? ga[n >> 2][n & 3] * (v[n] * inv) + be[n >> 2][n & 3] : 0.f);
            }
            *(bf16x8*)(X + (2 * c + (l16 >> 3)) * kTileUnits + r * 8 + ((l16 & 7) ^ ((r >> 1) & 7))) = o;
            *(bf16x8*)(xr + 128 * c) = o;
            // padding rows: zeros here and, once per call, in the attention output, which no kernel writes there (both are computed with)
            if (!live) *(bf16x8*)(p.att + (xr - p.x) + 128 * c) = o;
        }
    }
    barrier_lds();

    Acc acc;
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        set_bias(acc, (const float*)(sb + p.b) + c * kH + 64 * wave, g);
        multiply(acc, w, X, j31, g, [&](int kt, int s) {
            if (kt < 2) load(kt & 1, s, c, kt + 2);
            else if (c < 2) load(kt & 1, s, c + 1, kt - 2);
        });
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();                    // (the outputs before have been read)
        if (c < 2) {
            put(own, acc, j31, g);
            store_rows(own, p.qkv + 3 * ((size_t)m * p.t_ss + (size_t)m0 * kH) + c * kH + 64 * wave, 3 * kH, lane);
            continue;
        }
        // values: feature-major, rows of 64 tokens; chunk of eight tokens c of feature f in slot c ^ ((f / 4) % 8)
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int t = 0; t < 2; ++t)
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const int f = 32 * i + 8 * (v >> 2) + 4 * g, tk = 32 * t + j31;
                    *(bf16*)((char*)own + (f + (v & 3)) * 128 + (((tk >> 3) ^ (f >> 2 & 7)) << 4) + (tk & 7) * 2) = (bf16)acc[i][t][v];
                }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        bf16* dst = p.vt + (size_t)m * p.t_ss + (size_t)(64 * wave + (lane >> 3)) * p.rows + m0 + (lane & 7) * 8;
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const int f = 8 * q + (lane >> 3);
            store16_through<false>(dst + (size_t)8 * q * p.rows, __builtin_bit_cast(u32x4, own[f * 8 + ((lane & 7) ^ (f >> 2 & 7))]));
        }
    }
}

template <class Kernel, class Args>
hipError_t launch(Kernel kern, size_t lds, std::atomic<bool>& raised, const Args& a, hipStream_t s)
{
    if (!raised.load(std::memory_order_acquire)) {          // (the attribute is sticky for the process)
        const hipError_t e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
        raised.store(true, std::memory_order_release);
    }
    hipLaunchKernelGGL(kern, dim3((unsigned)((a.total + 7) / 8 * 8)), dim3(256), lds, s, a);
    return hipGetLastError();
}

}  // namespace

// (An FFN as narrow as the rows keeps the separate launches, although these would be quicker, us a call, three students on 14653 tokens 172 / 130, one
// on 1344 62 / 54: the folded attention on rows before their LayerNorm, which such calls of 256 take from 8192 tokens on, is checked bit for bit
// through the rows that it leaves in x.)
bool layer_supported(const sp_config& c)
{
    return bf16_path(c) && c.hidden == kH && c.ffn % 256 == 0 && c.ffn > kH && c.ffn <= kMaxF;
}

// A workgroup's chain is 1 + 2 F / 256 products behind one another, while separate launches spread their features over the chip: a call of few
// rows takes them unless the FFN is narrow.  us a call, separate / this, by tokens x students, two and six layers: FFN 512: 260 54 / 51 162 / 149, 1000 65 / 62
// 179 / 160, 3000 79 / 71 235 / 183; 768: 260 55 / 60 170 / 167, 600 60 / 62 176 / 177, 1020 60 / 63 186 / 180, 1250 63 / 64 and 63 / 58 196 / 181, 1400 67 / 65 209 / 186, 2000
// 71 / 67 228 / 190; 1024: 260 55 / 63 168 / 185, 600 59 / 66 179 / 194, 1020 61 / 66 187 / 197, 1250 65 / 68 200 / 199, 1600 67 / 69 209 / 203 and, two students, 69 / 69 217 /
// 203, 2000 70 / 69 224 / 207.  Twelve layers, 1024: 260 323 / 373, 1020 379 / 397, 1600 437 / 411.
bool layer_pays(const sp_config& c, int64_t rows_of_all_students)
{
    return layer_supported(c) && rows_of_all_students >= (c.ffn <= 512 ? 0 : c.ffn <= 768 ? 1280 : 1664);
}

hipError_t launch_layer(const sp_model* M, size_t lo, const void* att, const void* x, void* out, int rows, int mrows, int k, hipStream_t s)
{
    const sp_config& c = M->cfg;
    const ArenaLayout& L = M->L;
    if (!layer_supported(c) || mrows % kTok || mrows > rows) return hipErrorInvalidValue;
    static std::atomic<bool> raised{false};
    const LayerArgs a{M->arena, L.student_stride, lo + L.wo, lo + L.bo, lo + L.ln1g, lo + L.ln1b, lo + L.w1, lo + L.b1, lo + L.w2, lo + L.b2,
                      lo + L.ln2g, lo + L.ln2b, (const bf16*)att, (const bf16*)x, (bf16*)out, (size_t)rows * kH, c.ffn, mrows / kTok,
                      mrows / kTok * k, c.ln_eps};
    return launch(layer_kernel, kLayerLds, raised, a, s);
}

hipError_t launch_embed_qkv(const sp_model* M, size_t lo, const int32_t* ids, const int32_t* cu, int B, int T, void* x, void* att, void* qkv,
                            void* vt, int rows, int mrows, int k, hipStream_t s)
{
    const sp_config& c = M->cfg;
    const ArenaLayout& L = M->L;
    if (!layer_supported(c) || mrows % kTok || mrows > rows || T > mrows || T < 1) return hipErrorInvalidValue;
    static std::atomic<bool> raised{false};
    const EmbedQkvArgs a{M->arena, L.student_stride, L.tok, L.pos, L.emb_g, L.emb_b, lo + L.wqkv, lo + L.bqkv, ids, cu, (bf16*)x, (bf16*)att,
                         (bf16*)qkv, (bf16*)vt, (size_t)rows * kH, B, T, c.vocab, c.max_pos, rows, mrows / kTok, mrows / kTok * k, c.ln_eps};
    return launch(embed_qkv_kernel, kEmbedLds, raised, a, s);
}

}  // namespace sp
