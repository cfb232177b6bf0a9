// fp32 path, calls of few rows: everything of an encoder layer that follows the attention, and the q|k|v projection of the
// next layer, in one launch.
//
// Such a call is a chain of dependent launches of 4-6 us that leave the chip idle: five per layer after the attention and one
// for q|k|v.  All of it is row-wise, so a workgroup takes two rows through the whole chain with the rows in LDS and reads
// the layer's weights (768 KB at 128 x 512) from the L2, which is what bounds it: about 64 bytes per cycle and compute unit.
//   * sixteen lanes share an output feature and read 256 bytes in a row of its weights ([out][in]); eight waves x four
//     features per step, four steps (eight wave-loads) at a time, the next eight in flight, also across the barriers between
//     the projections;
//   * a lane's partial sums are added over the sixteen lanes by four data-parallel-primitive adds; then one lane per output
//     applies bias, GELU or residual.  Biases and LayerNorm parameters come through LDS, so nothing waits behind the weights.
// Measured, two students of 2 layers x 128 wide on 86 tokens: 19 launches, 83.6 us a call -> 8 launches, 57.7 us; relative difference
// from the separate launches' logits 1.9e-7.
#include "sp_internal.h"

namespace sp {

namespace {

constexpr int kWaves = 8, kRows = 2;

struct F32LayerArgs {
    const char* arena;
    size_t ss, wo, bo, g1, be1, w1, b1, w2, b2, g2, be2, wqkv, bqkv;   // byte offsets into a student slab
    const float* att;
    float *x, *qkv;                   // student strides: rows x H, rows x H, rows x 3 H
    int T, rows, H, F;
    float eps;
};

// Eight wave-loads: features f0 + 32 i (i < 4) of this lane group, reduction elements kc and kc + 64 on
__device__ inline void load_weights(f32x4 (&w)[8], const float* W, int K, int step, int kc, int lane, int wave)
{
    const float* p = W + (size_t)(step * 32 + wave * 4 + (lane >> 4)) * K + kc + (lane & 15) * 4;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        w[2 * i] = *(const f32x4*)(p + (size_t)i * 32 * K);
        w[2 * i + 1] = *(const f32x4*)(p + (size_t)i * 32 * K + 64);
    }
}

// emit(feature, row, sum) of xs[row][K] . W[feature][K] for N features (N and K multiples of 128).  w holds the first eight
// wave-loads of W on entry and those of Wn (reduction depth Kn), the next product's weights, on return.
template <class Emit>
__device__ inline void product(f32x4 (&w)[8], const float* W, int N, int K, const float* Wn, int Kn, const float* xs, int lane,
                               int wave, Emit emit)
{
    const int l16 = lane & 15, steps = N / 32;
    float acc[kRows][4];
#pragma unroll
    for (int r = 0; r < kRows; ++r)
#pragma unroll
        for (int i = 0; i < 4; ++i) acc[r][i] = 0.f;
    int s = 0, kc = 0;
    const int its = steps / 4 * (K / 128);
    for (int it = 0; it < its; ++it) {
        const bool wrap = kc + 128 == K, last = it + 1 == its;
        const int s1 = last ? 0 : wrap ? s + 4 : s, kc1 = wrap ? 0 : kc + 128;
        f32x4 wn[8];
        load_weights(wn, last ? Wn : W, last ? Kn : K, s1, kc1, lane, wave);
#pragma unroll
        for (int r = 0; r < kRows; ++r) {
            const f32x4 xa = *(const f32x4*)(xs + r * K + kc + l16 * 4), xb = *(const f32x4*)(xs + r * K + kc + 64 + l16 * 4);
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    acc[r][i] = fmaf(w[2 * i][e], xa[e], acc[r][i]);
                    acc[r][i] = fmaf(w[2 * i + 1][e], xb[e], acc[r][i]);
                }
        }
        if (wrap) {
            float out = 0.f;                                // lane l16 = 4 r + i of the group takes row r, step s + i
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
            if (l16 < 4 * kRows) emit((s + (l16 & 3)) * 32 + wave * 4 + (lane >> 4), l16 >> 2, out);
        }
        s = s1;
        kc = kc1;
#pragma unroll
        for (int i = 0; i < 8; ++i) w[i] = wn[i];
    }
}

// LayerNorm of a row of H <= 256 values in LDS, in place, by one wave; dst (may be null): the row once more
__device__ inline void layernorm_row(float* v, const float* g, const float* b, int H, float eps, int lane, float* dst)
{
    float x[4], s = 0.f, q = 0.f;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        x[i] = lane + 64 * i < H ? v[lane + 64 * i] : 0.f;
        s += x[i];
    }
    const float inv_h = __builtin_amdgcn_rcpf((float)H), mean = wave_sum(s) * inv_h;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const float d = x[i] - mean;
        if (lane + 64 * i < H) q += d * d;
    }
    const float inv = __builtin_amdgcn_rsqf(wave_sum(q) * inv_h + eps);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int c = lane + 64 * i;
        if (c < H) {
            const float o = g[c] * ((x[i] - mean) * inv) + b[c];
            v[c] = o;
            if (dst) dst[c] = o;
        }
    }
}

__global__ __launch_bounds__(64 * kWaves) void f32_layer_kernel(F32LayerArgs p)
{
    extern __shared__ float lds[];
    const int H = p.H, F = p.F, m = blockIdx.y, r0 = blockIdx.x * kRows;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    float *xa = lds, *xr = xa + kRows * H, *xg = xr + kRows * H, *bo = xg + kRows * F, *g1 = bo + H, *be1 = g1 + H, *b1 = be1 + H;
    float *b2 = b1 + F, *g2 = b2 + H, *be2 = g2 + H, *bq = be2 + H;
    const char* sb = p.arena + (size_t)m * p.ss;
    const bool tail = p.qkv != nullptr;
    const float *Wo = (const float*)(sb + p.wo), *W1 = (const float*)(sb + p.w1), *W2 = (const float*)(sb + p.w2);
    const float* Wq = tail ? (const float*)(sb + p.wqkv) : W2;          // (nothing follows: a load that nobody uses)

    auto fill = [&](float* dst, size_t off, int n) {
        for (int i = tid; i < n; i += 64 * kWaves) dst[i] = ((const float*)(sb + off))[i];
    };
    for (int i = tid; i < kRows * H; i += 64 * kWaves) {
        const int r = i / H, row = r0 + r < p.T ? r0 + r : p.T - 1;
        const size_t at = ((size_t)m * p.rows + row) * H + (i - r * H);
        xa[i] = p.att[at];
        xr[i] = p.x[at];
    }
    fill(bo, p.bo, H);
    fill(g1, p.g1, H);
    fill(be1, p.be1, H);
    fill(b1, p.b1, F);
    fill(b2, p.b2, H);
    fill(g2, p.g2, H);
    fill(be2, p.be2, H);
    if (tail) fill(bq, p.bqkv, 3 * H);
    f32x4 w[8];
    load_weights(w, Wo, H, 0, 0, lane, wave);
    barrier_lds();
    product(w, Wo, H, H, W1, H, xa, lane, wave, [&](int f, int r, float v) { xr[r * H + f] = v + bo[f] + xr[r * H + f]; });
    barrier_lds();
    if (wave < kRows) layernorm_row(xr + wave * H, g1, be1, H, p.eps, lane, nullptr);
    barrier_lds();
    product(w, W1, F, H, W2, F, xr, lane, wave, [&](int f, int r, float v) {
        const float u = v + b1[f];
        xg[r * F + f] = 0.5f * u * (1.0f + erff(u * 0.70710678118654752f));
    });
    barrier_lds();
    product(w, W2, H, F, Wq, tail ? H : F, xg, lane, wave, [&](int f, int r, float v) { xa[r * H + f] = v + b2[f] + xr[r * H + f]; });
    barrier_lds();
    if (wave < kRows)
        layernorm_row(xa + wave * H, g2, be2, H, p.eps, lane,
                      r0 + wave < p.T ? p.x + ((size_t)m * p.rows + r0 + wave) * H : nullptr);
    if (!tail) return;
    barrier_lds();
    product(w, Wq, 3 * H, H, Wq, H, xa, lane, wave, [&](int f, int r, float v) {
        if (r0 + r < p.T) p.qkv[((size_t)m * p.rows + r0 + r) * 3 * H + f] = v + bq[f];
    });
}

}  // namespace

// Every workgroup reads the layer's weights, so the kernel is for narrow students (1 MB of weights, i.e. hidden 128 with an FFN of up
// to 768: 7 us at the L2's rate; the separate launches spread them over the chip) and for calls of at most one workgroup per
// compute unit.
bool f32_layer_supported(const sp_config& c, long rows_of_all_students)
{
    const size_t H = c.hidden, F = c.ffn;
    return !bf16_path(c) && H == 128 && F % 128 == 0 && (4 * H * H + 2 * H * F) * sizeof(float) <= (1u << 20) &&
           rows_of_all_students <= 256 * kRows;
}

hipError_t launch_f32_layer(const sp_model* M, size_t lo, const void* att, void* x, void* qkv_next, int T, int rows, int k,
                            hipStream_t s)
{
    const sp_config& c = M->cfg;
    const ArenaLayout& L = M->L;
    const size_t nx = lo + L.layer_stride;
    const F32LayerArgs a{M->arena, L.student_stride, lo + L.wo, lo + L.bo, lo + L.ln1g, lo + L.ln1b, lo + L.w1, lo + L.b1,
                         lo + L.w2, lo + L.b2, lo + L.ln2g, lo + L.ln2b, nx + L.wqkv, nx + L.bqkv, (const float*)att, (float*)x,
                         (float*)qkv_next, T, rows, c.hidden, c.ffn, c.ln_eps};
    const size_t smem = sizeof(float) * ((size_t)kRows * (2 * c.hidden + c.ffn) + 9 * (size_t)c.hidden + c.ffn);
    if (smem > 48 * 1024) return hipErrorInvalidValue;
    hipLaunchKernelGGL(f32_layer_kernel, dim3((T + kRows - 1) / kRows, k), dim3(64 * kWaves), smem, s, a);
    return hipGetLastError();
}

}  // namespace sp
