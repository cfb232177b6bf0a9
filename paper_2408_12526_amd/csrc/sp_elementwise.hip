// Bandwidth-bound kernels of the student forward: embedding gather + LayerNorm,
// stand-alone LayerNorm, and the pooled head with the cross-student sum.
#include <type_traits>

#include "sp_internal.h"

namespace sp {

namespace {

constexpr int kMaxChunks = 4;  // 8-element chunks per lane: hidden <= 64 * 8 * kMaxChunks

__device__ inline void load8(const float* p, float (&v)[8])
{
    const f32x4 a = *(const f32x4*)p, b = *(const f32x4*)(p + 4);
    v[0] = a[0]; v[1] = a[1]; v[2] = a[2]; v[3] = a[3]; v[4] = b[0]; v[5] = b[1]; v[6] = b[2]; v[7] = b[3];
}
__device__ inline void load8(const bf16* p, float (&v)[8])
{
    const bf16x8 a = *(const bf16x8*)p;
#pragma unroll
    for (int i = 0; i < 8; ++i) v[i] = (float)a[i];
}
// eight values as they lie in memory
template <typename T> struct Raw8;
template <> struct Raw8<bf16> { bf16x8 v; };
template <> struct Raw8<float> { f32x4 v[2]; };
__device__ inline void widen(const Raw8<bf16>& r, float (&v)[8])
{
#pragma unroll
    for (int i = 0; i < 8; ++i) v[i] = (float)r.v[i];
}
__device__ inline void widen(const Raw8<float>& r, float (&v)[8])
{
#pragma unroll
    for (int i = 0; i < 8; ++i) v[i] = r.v[i >> 2][i & 3];
}
__device__ inline void store8(float* p, const float (&v)[8])
{
    *(f32x4*)p = f32x4{v[0], v[1], v[2], v[3]};
    *(f32x4*)(p + 4) = f32x4{v[4], v[5], v[6], v[7]};
}
__device__ inline void store8(bf16* p, const float (&v)[8])
{
    bf16x8 a;
#pragma unroll
    for (int i = 0; i < 8; ++i) a[i] = (bf16)v[i];
    *(bf16x8*)p = a;
}

// LayerNorm of one row held across a wave as v[chunk][8]; chunk c of lane l covers
// elements 8*(l + 64c) .. +7.  Two passes over registers: mean, then centred variance.
// gamma and beta are held the same way (a wave keeps them for all the rows it normalises).
// eight values -> eight fp8 (e4m3) codes of v * qscale, saturating, packed in 8 bytes
__device__ inline void store8_fp8(unsigned char* p, const float (&v)[8], float qscale)
{
    int lo = 0, hi = 0;
    lo = __builtin_amdgcn_cvt_pk_fp8_f32(v[0] * qscale, v[1] * qscale, lo, false);
    lo = __builtin_amdgcn_cvt_pk_fp8_f32(v[2] * qscale, v[3] * qscale, lo, true);
    hi = __builtin_amdgcn_cvt_pk_fp8_f32(v[4] * qscale, v[5] * qscale, hi, false);
    hi = __builtin_amdgcn_cvt_pk_fp8_f32(v[6] * qscale, v[7] * qscale, hi, true);
    *(int2*)p = int2{lo, hi};
}

// qout (may be null): the same row once more as fp8 codes of value * qscale, for the fp8 projections
// (Q8 is a template parameter: the plain bf16 / fp32 instantiations carry no trace of the second output)
template <typename T, int MAXC, bool Q8 = false>
__device__ inline void ln_row_store(float (&v)[MAXC][8], int nch, int lane, int H, const float (&gg)[MAXC][8],
                                    const float (&bb)[MAXC][8], float eps, T* out, unsigned char* qout = nullptr,
                                    float qscale = 1.f)
{
    float s = 0.f;
#pragma unroll
    for (int i = 0; i < MAXC; ++i)
        if (lane + 64 * i < nch)
#pragma unroll
            for (int e = 0; e < 8; ++e) s += v[i][e];
    // (1 / H once and the hardware reciprocal square root: a correctly rounded division is ten dependent instructions)
    const float inv_h = __builtin_amdgcn_rcpf((float)H);
    const float mean = wave_sum(s) * inv_h;
    float q = 0.f;
#pragma unroll
    for (int i = 0; i < MAXC; ++i)
        if (lane + 64 * i < nch)
#pragma unroll
            for (int e = 0; e < 8; ++e) { const float d = v[i][e] - mean; q += d * d; }
    const float inv = __builtin_amdgcn_rsqf(wave_sum(q) * inv_h + eps);
#pragma unroll
    for (int i = 0; i < MAXC; ++i) {
        const int c = lane + 64 * i;
        if (c < nch) {
            float o[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) o[e] = gg[i][e] * ((v[i][e] - mean) * inv) + bb[i][e];
            store8(out + c * 8, o);
            if (Q8) store8_fp8(qout + c * 8, o, qscale);
        }
    }
}

template <int MAXC>
__device__ inline void load_gamma_beta(const float* g, const float* b, int nch, int lane, float (&gg)[MAXC][8],
                                       float (&bb)[MAXC][8])
{
#pragma unroll
    for (int i = 0; i < MAXC; ++i) {
        const int c = lane + 64 * i;
        if (c < nch) { load8(g + c * 8, gg[i]); load8(b + c * 8, bb[i]); }
    }
}

// Consecutive rows normalised by one wave (gamma and beta are fetched once for them, and a row's loads run while the one before is
// normalised): few rows one each, where the row-parallelism is worth more.  us by rows a wave: 18432 rows of 1024: LayerNorm 1 14.1, 2 13.7, 4
// 15.0, embedding 22.6 / 20.6 / 20.8; 9216 of 768: 7.6 / 7.1 / 7.8, 12.7 / 12.0 / 11.4; 117 k rows of 768: LayerNorm 4 56.4, 8 57.9, embedding
// 83.4 / 76.8 (whose waves look for their sequence first); 110 k of 1024: LayerNorm 66.9 / 71.9, embedding 87.6 / 90.1.
inline int rows_per_wave(int mrows, int k, int many) { return (long)mrows * k >= 32768 ? many : (long)mrows * k >= 8192 ? 2 : 1; }

// One wave per rpw consecutive packed token rows, grid.y = student.
template <typename T, int MAXC, bool Q8>
__global__ __launch_bounds__(256) void embed_ln_kernel(const char* arena, size_t student_stride, size_t tok_off,
                                                       size_t pos_off, size_t g_off, size_t b_off,
                                                       const int32_t* __restrict__ ids,
                                                       const int32_t* __restrict__ cu, int B, int Tn, int rows,
                                                       int mrows, int H, int V, int P, float eps, T* __restrict__ x,
                                                       T* __restrict__ att, int rpw, unsigned char* __restrict__ xq,
                                                       float qscale, unsigned char* __restrict__ attq)
{
    const int m = blockIdx.y, lane = threadIdx.x & 63;
    const int row0 = (blockIdx.x * 4 + (threadIdx.x >> 6)) * rpw;
    if (row0 >= mrows) return;
    const int nch = H >> 3;
    const char* sb = arena + (size_t)m * student_stride;
    float gg[MAXC][8], bb[MAXC][8];
    load_gamma_beta<MAXC>((const float*)(sb + g_off), (const float*)(sb + b_off), nch, lane, gg, bb);
    // Token ids and sequence starts of the wave's rows, a lane each (rpw < 64), before any row is fetched, so that the row loop has
    // no dependent index loads: the sequence of the first row, then what begins in the rows behind it.
    const int first = row0 < Tn ? row0 : Tn - 1;
    int my_id = row0 + lane < Tn ? ids[row0 + lane] : 0, c0, c1;
    my_id = my_id < 0 ? 0 : (my_id >= V ? V - 1 : my_id);
    const int b = last_sequence(cu, B, lane, [&](int, int c) { return c <= first; }, c0, c1);
    const int begin = lane == 0 ? c0 : lane == 1 ? c1 : rpw > 1 && b + lane < B ? cu[b + lane] : 0x7fffffff;
    // Rows of tokens, the next one's fetched while one is normalised; then padding rows.
    const int end = row0 + rpw < mrows ? row0 + rpw : mrows, live = end < Tn ? end : Tn;
    Raw8<T> te[2][MAXC], pe[2][MAXC];
    auto fetch = [&](int row, int set) {
        const int id = __builtin_amdgcn_readlane(my_id, row - row0), nb = __popcll(__ballot(begin <= row));
        int pos = row - __builtin_amdgcn_readlane(begin, nb > 0 ? nb - 1 : 0);
        pos = pos < 0 ? 0 : (pos >= P ? P - 1 : pos);
        const T* t = (const T*)(sb + tok_off) + (size_t)id * H;
        const T* q = (const T*)(sb + pos_off) + (size_t)pos * H;
#pragma unroll
        for (int i = 0; i < MAXC; ++i) {
            const int c = lane + 64 * i;
            if (c < nch) {
                te[set][i] = *(const Raw8<T>*)(t + c * 8);
                pe[set][i] = *(const Raw8<T>*)(q + c * 8);
            }
        }
    };
    auto normalise = [&](int row, int set) {
        float v[MAXC][8];
#pragma unroll
        for (int i = 0; i < MAXC; ++i) {
            float p8[8];
            widen(te[set][i], v[i]);
            widen(pe[set][i], p8);
#pragma unroll
            for (int e = 0; e < 8; ++e) v[i][e] += p8[e];
        }
        const size_t at = ((size_t)m * rows + row) * H;
        ln_row_store<T, MAXC, Q8>(v, nch, lane, H, gg, bb, eps, x + at, Q8 ? xq + at : nullptr, qscale);
    };
    if (row0 < live) fetch(row0, 0);
    for (int row = row0; row < live; row += 2) {
        if (row + 1 < live) fetch(row + 1, 1);
        __builtin_amdgcn_sched_barrier(0);
        normalise(row, 0);
        if (row + 1 >= live) break;
        if (row + 2 < live) fetch(row + 2, 0);
        __builtin_amdgcn_sched_barrier(0);
        normalise(row + 1, 1);
    }
    // Padding rows of the token tile.  They never reach a result, but the projections compute them and the attention kernels fetch values in
    // chunks of eight tokens, so they must hold finite numbers: zero the hidden state here and, once per call, the attention output rows
    // that no kernel writes.
    for (int row = row0 > Tn ? row0 : Tn; row < end; ++row) {
        const float zero8[8] = {0, 0, 0, 0, 0, 0, 0, 0};
        const size_t at = ((size_t)m * rows + row) * H;
        for (int c = lane; c < nch; c += 64) { store8(x + at + c * 8, zero8); store8(att + at + c * 8, zero8); }
        if (Q8)
            for (int c = lane; c < nch; c += 64) {
                *(int2*)(xq + at + c * 8) = int2{0, 0};
                if (attq) *(int2*)(attq + at + c * 8) = int2{0, 0};
            }
    }
}

template <typename T, int MAXC, bool Q8>
__global__ __launch_bounds__(256) void layernorm_kernel(const char* arena, size_t student_stride, size_t g_off,
                                                        size_t b_off, const T* __restrict__ u, T* __restrict__ out,
                                                        int rows, int mrows, int H, float eps, int rpw,
                                                        unsigned char* __restrict__ outq, float qscale)
{
    const int m = blockIdx.y, lane = threadIdx.x & 63;
    const int row0 = (blockIdx.x * 4 + (threadIdx.x >> 6)) * rpw;
    if (row0 >= mrows) return;
    const int nch = H >> 3;
    const char* sb = arena + (size_t)m * student_stride;
    float gg[MAXC][8], bb[MAXC][8];
    load_gamma_beta<MAXC>((const float*)(sb + g_off), (const float*)(sb + b_off), nch, lane, gg, bb);
    // (the next row is fetched while one is normalised)
    const int end = row0 + rpw < mrows ? row0 + rpw : mrows;
    Raw8<T> in[2][MAXC];
    auto fetch = [&](int row, int set) {
        const T* r = u + ((size_t)m * rows + row) * H;
#pragma unroll
        for (int i = 0; i < MAXC; ++i)
            if (lane + 64 * i < nch) in[set][i] = *(const Raw8<T>*)(r + (lane + 64 * i) * 8);
    };
    auto normalise = [&](int row, int set) {
        float v[MAXC][8];
#pragma unroll
        for (int i = 0; i < MAXC; ++i) widen(in[set][i], v[i]);
        const size_t at = ((size_t)m * rows + row) * H;
        ln_row_store<T, MAXC, Q8>(v, nch, lane, H, gg, bb, eps, out + at, Q8 ? outq + at : nullptr, qscale);
    };
    fetch(row0, 0);
    for (int row = row0; row < end; row += 2) {
        if (row + 1 < end) fetch(row + 1, 1);
        __builtin_amdgcn_sched_barrier(0);
        normalise(row, 0);
        if (row + 1 >= end) break;
        if (row + 2 < end) fetch(row + 2, 0);
        __builtin_amdgcn_sched_barrier(0);
        normalise(row + 1, 1);
    }
}

// The first tokens' rows alone, one wave per row.
template <int MAXC>
__global__ __launch_bounds__(256) void layernorm_first_kernel(const char* arena, size_t student_stride, size_t g_off, size_t b_off,
                                                              const bf16* __restrict__ u, bf16* __restrict__ out, int rows,
                                                              const int32_t* __restrict__ cu, int B, int Tn, int H, float eps)
{
    const int m = blockIdx.y, lane = threadIdx.x & 63, b = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (b >= B) return;
    const int nch = H >> 3;
    const char* sb = arena + (size_t)m * student_stride;
    float gg[MAXC][8], bb[MAXC][8], v[MAXC][8];
    int row = cu[b];
    row = row < 0 ? 0 : (row >= Tn ? Tn - 1 : row);
    load_gamma_beta<MAXC>((const float*)(sb + g_off), (const float*)(sb + b_off), nch, lane, gg, bb);
    const bf16* in = u + ((size_t)m * rows + row) * H;
#pragma unroll
    for (int i = 0; i < MAXC; ++i)
        if (lane + 64 * i < nch) load8(in + (lane + 64 * i) * 8, v[i]);
    ln_row_store<bf16, MAXC>(v, nch, lane, H, gg, bb, eps, out + ((size_t)m * rows + b) * H);
}

// Sum of the slices of a split reduction + bias + residual, then LayerNorm: one wave per row.  Rows T..mrows become zero:
// attention multiplies the values of up to seven of them by zero probabilities, so what the next layer forms there
// must be finite, and the operands of this projection need not be (the slices lie over the attention output's padding rows).
// All loads of a row are requested at once, without a branch between them (one per chunk made a second round trip to memory of it).
template <int MAXC, int SLICES>
__global__ __launch_bounds__(256) void ln_slices_kernel(const char* arena, size_t student_stride, size_t g_off, size_t b_off,
                                                        size_t bias_off, const float* __restrict__ part, size_t slice,
                                                        size_t p_ss, const bf16* __restrict__ res,
                                                        bf16* __restrict__ out, int rows, int T, int mrows, int H, float eps)
{
    const int m = blockIdx.y, lane = threadIdx.x & 63;
    const int row = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (row >= mrows) return;
    const int nch = H >> 3;
    bf16* orow = out + ((size_t)m * rows + row) * H;
    if (row >= T) {
        const float zero8[8] = {0, 0, 0, 0, 0, 0, 0, 0};
        for (int c = lane; c < nch; c += 64) store8(orow + c * 8, zero8);
        return;
    }
    const char* sb = arena + (size_t)m * student_stride;
    const float* bias = (const float*)(sb + bias_off);
    const bf16* rrow = res + ((size_t)m * rows + row) * H;
    const float* prow = part + (size_t)m * p_ss + (size_t)row * H;
    float v[MAXC][8], gg[MAXC][8], bb[MAXC][8];
    Raw8<bf16> r8[MAXC];
    Raw8<float> b8[MAXC], p8[SLICES][MAXC];
#pragma unroll
    for (int i = 0; i < MAXC; ++i) {                        // (lanes behind the row's end: its last chunk, and nothing comes of it)
        const int c = (lane + 64 * i < nch ? lane + 64 * i : nch - 1) * 8;
#pragma unroll
        for (int sl = 0; sl < SLICES; ++sl) p8[sl][i] = *(const Raw8<float>*)(prow + (size_t)sl * slice + c);
        r8[i] = *(const Raw8<bf16>*)(rrow + c);
        b8[i] = *(const Raw8<float>*)(bias + c);
    }
    load_gamma_beta<MAXC>((const float*)(sb + g_off), (const float*)(sb + b_off), nch, lane, gg, bb);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < MAXC; ++i) {
        float t[8];
        widen(r8[i], v[i]);
        widen(b8[i], t);
#pragma unroll
        for (int e = 0; e < 8; ++e) v[i][e] += t[e];
#pragma unroll
        for (int sl = 0; sl < SLICES; ++sl) {               // ascending
            widen(p8[sl][i], t);
#pragma unroll
            for (int e = 0; e < 8; ++e) v[i][e] += t[e];
        }
    }
    ln_row_store<bf16, MAXC>(v, nch, lane, H, gg, bb, eps, orow);
}

// ---- head -------------------------------------------------------------------------
// Stage 1: one workgroup = (group of kSeqPerWg sequences, student, slice of 64 pooler outputs).
// pooled[n] = tanh(bp[n] + sum_i cls[i] Wp[i][n]); the slice's share of the classifier,
// sum_{n in slice} pooled[n] Wc[n][c], goes to zpart[m][slice][b][c].
constexpr int kSeqPerWg = 8;

// Pooler pre-activations of one slice of 64 outputs for up to kSeqPerWg rows held in LDS (xs[s][H], fp32):
// red[(wave * kSeqPerWg + s) * 64 + n] = sum over the wave's quarter of the inputs i of xs[s][i] * Wp[i][slice * 64 + n].
// A lane fetches 16 bytes (8 outputs) of a weight row, so a wave instruction covers 8 rows of the slice and the wave's
// H / 4 rows are H / 32 instructions per lane, requested sixteen at a time (2-byte loads, one row per instruction,
// took four times as many round trips: the pooler was the longest kernel of a single-sequence call; requesting all
// rows before the token rows are gathered was measured slower than two batches afterwards).  The 8 lanes that share
// an output chunk are then added with shuffles.
template <typename T>
struct RawRow;
template <>
struct RawRow<bf16> {
    bf16x8 v;
    __device__ void load(const bf16* p) { v = *(const bf16x8*)p; }
    __device__ float get(int e) const { return (float)v[e]; }
};
template <>
struct RawRow<float> {
    f32x4 a, b;
    __device__ void load(const float* p) { a = *(const f32x4*)p; b = *(const f32x4*)(p + 4); }
    __device__ float get(int e) const { return e < 4 ? a[e] : b[e - 4]; }
};

template <typename T>
struct PoolerWeights {
    static constexpr int NB = sizeof(T) == 2 ? 16 : 8;       // weight rows in flight per lane
    RawRow<T> w[NB];
    const T* base;
    int nj, stride;
    __device__ void request(const T* Wp, int H, int slice, int lane, int wv)   // addresses only
    {
        nj = H / 32;                                          // rows per lane: the wave's H / 4 rows, 8 per instruction
        stride = 8 * H;
        base = Wp + (size_t)(wv * (H / 4) + (lane >> 3)) * H + slice * 64 + (lane & 7) * 8;
    }
    __device__ void multiply(const float* xs, float* red, int H, int nseq, int lane, int wv)
    {
        const int c8 = (lane & 7) * 8, rl = lane >> 3, row0 = wv * (H / 4) + rl;
        float acc[kSeqPerWg][8];
#pragma unroll
        for (int s = 0; s < kSeqPerWg; ++s)
#pragma unroll
            for (int e = 0; e < 8; ++e) acc[s][e] = 0.f;
        for (int j0 = 0; j0 < nj; j0 += NB) {
#pragma unroll
            for (int jj = 0; jj < NB; ++jj)
                if (j0 + jj < nj) w[jj].load(base + (size_t)(j0 + jj) * stride);
#pragma unroll
            for (int jj = 0; jj < NB; ++jj)
                if (j0 + jj < nj) {
                    const int i = row0 + (j0 + jj) * 8;
#pragma unroll
                    for (int s = 0; s < kSeqPerWg; ++s)
                        if (s < nseq) {
                            const float xv = xs[s * H + i];
#pragma unroll
                            for (int e = 0; e < 8; ++e) acc[s][e] += xv * w[jj].get(e);
                        }
                }
        }
#pragma unroll
        for (int s = 0; s < kSeqPerWg; ++s)
            if (s < nseq) {
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    // sum over the eight lanes that share lane % 8: other half of the row, other row of the pair,
                    // other half of the wave
                    float a = acc[s][e];
                    a += dpp_moved<0x128>(a);               // row_ror:8
                    float lo = a, hi = a;
                    swap_rows(lo, hi);
                    a = lo + hi;
                    lo = a;
                    hi = a;
                    swap_halves(lo, hi);
                    a = lo + hi;
                    if (rl == 0) red[(wv * kSeqPerWg + s) * 64 + c8 + e] = a;
                }
            }
    }
};

template <typename T>
__global__ __launch_bounds__(256) void head_pool_kernel(const char* arena, size_t student_stride, size_t wp_off,
                                                        size_t bp_off, size_t wc_off, const T* __restrict__ x,
                                                        const int32_t* __restrict__ cu, int B, int Tn, int rows, int H,
                                                        int C, float* __restrict__ zpart)
{
    extern __shared__ float smem[];
    float* xs = smem;                      // [kSeqPerWg][H]
    float* red = smem + kSeqPerWg * H;     // [4][kSeqPerWg][64]
    const int b0 = blockIdx.x * kSeqPerWg, m = blockIdx.y, slice = blockIdx.z, nslice = gridDim.z;
    const int tid = threadIdx.x, lane = tid & 63, part = tid >> 6;
    const int nseq = (B - b0) < kSeqPerWg ? (B - b0) : kSeqPerWg;
    const char* sb = arena + (size_t)m * student_stride;
    for (int s = 0; s < nseq; ++s) {
        int r = cu[b0 + s];                  // first token of the sequence
        r = r < 0 ? 0 : (r >= Tn ? Tn - 1 : r);
        const T* src = x + ((size_t)m * rows + r) * H;
        for (int i = tid; i < H; i += 256) xs[s * H + i] = (float)src[i];
    }
    __syncthreads();
    const int n = slice * 64 + lane;
    if (nseq <= 2) {
        // one or two sequences: latency of the weight fetch is all there is, wide loads (see PoolerWeights)
        PoolerWeights<T> pw;
        pw.request((const T*)(sb + wp_off), H, slice, lane, part);
        pw.multiply(xs, red, H, nseq, lane, part);
    } else {
        // a full group of sequences: a lane owns one output for all of them (measured faster than the wide loads,
        // whose eight-outputs-per-lane sums need 64 accumulators and a shuffle reduction per sequence)
        const T* Wp = (const T*)(sb + wp_off);
        float acc[kSeqPerWg];
#pragma unroll
        for (int s = 0; s < kSeqPerWg; ++s) acc[s] = 0.f;
        const int per = H / 4, i0 = part * per;   // this wave's share of the reduction index (a multiple of 16)
#pragma unroll 8
        for (int i = i0; i < i0 + per; i += 4) {     // unrolled: 32 weight loads in flight per lane
            float w[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) w[e] = (float)Wp[(size_t)(i + e) * H + n];
#pragma unroll
            for (int s = 0; s < kSeqPerWg; ++s) {    // rows beyond nseq hold stale data: their sums are never used
                const f32x4 xv = *(const f32x4*)&xs[s * H + i];
                acc[s] += xv[0] * w[0] + xv[1] * w[1] + xv[2] * w[2] + xv[3] * w[3];
            }
        }
#pragma unroll
        for (int s = 0; s < kSeqPerWg; ++s) red[(part * kSeqPerWg + s) * 64 + lane] = acc[s];
    }
    __syncthreads();
    // wave `part` finishes sequences part, part+4: fixed order over the four shares
    const float bpn = ((const float*)(sb + bp_off))[n];
    const T* Wc = (const T*)(sb + wc_off);
    for (int s = part; s < nseq; s += 4) {
        float p = bpn;
#pragma unroll
        for (int q = 0; q < 4; ++q) p += red[(q * kSeqPerWg + s) * 64 + lane];
        p = tanhf(p);
        for (int c = 0; c < C; ++c) {
            const float t = wave_sum(p * (float)Wc[(size_t)n * C + c]);
            if (lane == 0) zpart[(((size_t)m * nslice + slice) * B + (b0 + s)) * C + c] = t;
        }
    }
}

// Stage 2: z[m][b][c] = bc[m][c] + sum over slices (ascending); logits[b][c] = sum_m z (m ascending).
// 256 threads = 8 student lanes x 32 outputs: the students' slice sums run in parallel, the sum over students is taken
// in order by the first lane of each output.
constexpr int kSumStudents = 64;   // most students (sp_config.K is capped at this)
constexpr int kMaxSlices64 = 16;   // most slices of 64 pooled features

__global__ __launch_bounds__(256) void head_sum_kernel(const char* arena, size_t student_stride, size_t bc_off,
                                                       const float* __restrict__ zpart, int B, int C, int k, int nslice,
                                                       float* __restrict__ z, float* __restrict__ logits)
{
    __shared__ float zs[kSumStudents][32];
    const int ox = threadIdx.x & 31, my = threadIdx.x >> 5;
    const int idx = blockIdx.x * 32 + ox;
    const bool live = idx < B * C;
    const int c = live ? idx % C : 0;
    for (int m = my; m < k; m += 8) {
        float zm = 0.f;
        if (live) {
            float part[kMaxSlices64];                       // all slices requested at once, added in ascending order
#pragma unroll
            for (int sl = 0; sl < kMaxSlices64; ++sl) part[sl] = zpart[((size_t)m * nslice + (sl < nslice ? sl : nslice - 1)) * B * C + idx];
#pragma unroll
            for (int sl = 0; sl < kMaxSlices64; ++sl) zm += sl < nslice ? part[sl] : 0.f;
            zm += ((const float*)(arena + (size_t)m * student_stride + bc_off))[c];
            z[(size_t)m * B * C + idx] = zm;
        }
        zs[m][ox] = zm;
    }
    __syncthreads();
    if (logits && my == 0 && live) {
        float total = 0.f;
        for (int m = 0; m < k; ++m) total += zs[m][ox];
        logits[idx] = total;
    }
}

// logits[i] = sum over students of z[m][i], m ascending.
__global__ void sum_students_kernel(const float* __restrict__ z, int n, int k, float* __restrict__ logits)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    float total = 0.f;
#pragma unroll 4
    for (int m = 0; m < k; ++m) total += z[(size_t)m * n + i];
    logits[i] = total;
}

// Classifier and the cross-student sum where the first tokens are many: one workgroup per sequence, a wave per student (up to kClassifyWaves).
// One pass over the row for CB classes at a time and all its loads requested together: a student is one memory round trip
// (a pass per class, a chain of dependent iterations each, took 11.6 us for one sequence and eight students).
// The rows are the pooler's sums: bias and tanh are applied here.
constexpr int kClassifyWaves = 8;
template <int CB>
__global__ __launch_bounds__(64 * kClassifyWaves) void head_classify_kernel(const char* arena, size_t student_stride, size_t wc_off,
                                                            size_t bc_off, size_t bp_off, const float* __restrict__ pooled, size_t p_ss,
                                                            int B, int H, int C, int k, float* __restrict__ z,
                                                            float* __restrict__ logits)
{
    __shared__ float zs[64][16];                 // [student][class]
    const int b = blockIdx.x, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    for (int m = wave; m < k; m += (int)(blockDim.x >> 6)) {
        const char* sb = arena + (size_t)m * student_stride;
        const bf16* Wc = (const bf16*)(sb + wc_off);
        const float* p = pooled + (size_t)m * p_ss + (size_t)b * H;
        for (int c0 = 0; c0 < C; c0 += CB) {
            float pv[16];
            bf16 wv[16][CB];
#pragma unroll
            for (int i = 0; i < 16; ++i) {       // hidden <= 1024, a multiple of 64; pieces beyond it count as zero
                const int n = lane + (64 * i < H ? 64 * i : 0);
                pv[i] = tanhf(p[n] + ((const float*)(sb + bp_off))[n]);
#pragma unroll
                for (int c = 0; c < CB; ++c) wv[i][c] = Wc[(size_t)n * C + (c0 + c < C ? c0 + c : C - 1)];
            }
            float acc[CB];
#pragma unroll
            for (int c = 0; c < CB; ++c) {
                acc[c] = 0.f;
#pragma unroll
                for (int i = 0; i < 16; ++i) acc[c] += 64 * i < H ? pv[i] * (float)wv[i][c] : 0.f;
                acc[c] = wave_sum(acc[c]);
                if (lane == 0 && c0 + c < C) {
                    const float v = acc[c] + ((const float*)(sb + bc_off))[c0 + c];
                    zs[m][c0 + c] = v;
                    z[((size_t)m * B + b) * C + c0 + c] = v;
                }
            }
        }
    }
    __syncthreads();
    if (logits && threadIdx.x < C) {
        float total = 0.f;
        for (int m = 0; m < k; ++m) total += zs[m][threadIdx.x];   // students in training order
        logits[(size_t)b * C + threadIdx.x] = total;
    }
}

}  // namespace

hipError_t launch_head_classify(const sp_model* M, const float* sums, size_t p_ss, int B, int k, float* z, float* logits,
                                hipStream_t s)
{
    const sp_config& c = M->cfg;
    if (!bf16_path(c) || k > 64 || c.hidden > 1024 || c.hidden % 64) return hipErrorInvalidValue;
#define SP_CLASSIFY(CB)                                                                                             \
    hipLaunchKernelGGL(head_classify_kernel<CB>, dim3((unsigned)B), dim3(64 * (k < kClassifyWaves ? k : kClassifyWaves)), 0, s, \
                       M->arena, M->L.student_stride, M->L.wc, M->L.bc, M->L.bp, sums, p_ss, B, c.hidden, c.classes, k, z, logits)
    if (c.classes <= 2) SP_CLASSIFY(2); else SP_CLASSIFY(4);
#undef SP_CLASSIFY
    return hipGetLastError();
}

hipError_t launch_head_sum(const sp_model* M, const float* zpart, int B, int k, float* z, float* logits, hipStream_t s)
{
    const sp_config& c = M->cfg;
    const int n = B * c.classes, nslice = c.hidden / 64;
    if (k > kSumStudents || nslice > kMaxSlices64) return hipErrorInvalidValue;
    hipLaunchKernelGGL(head_sum_kernel, dim3((n + 31) / 32), dim3(256), 0, s, M->arena, M->L.student_stride, M->L.bc, zpart, B,
                       c.classes, k, nslice, z, logits);
    return hipGetLastError();
}

hipError_t launch_embed_ln(const sp_model* M, const int32_t* ids, const int32_t* cu, int B, int T, int rows, int mrows,
                           int k, void* x, void* att, hipStream_t s, void* xq, float qscale, void* attq)
{
    const sp_config& c = M->cfg;
    const ArenaLayout& L = M->L;
    const int rpw = rows_per_wave(mrows, k, 8);
    dim3 grid((mrows + 4 * rpw - 1) / (4 * rpw), k);
    const int maxc = (c.hidden / 8 + 63) / 64;              // 8-element chunks per lane
#define SP_EMBED(T, MAXC) do {                                                                                     \
    if (xq && std::is_same<T, bf16>::value)                                                                        \
        hipLaunchKernelGGL((embed_ln_kernel<bf16, MAXC, true>), grid, dim3(256), 0, s, M->arena, L.student_stride, L.tok, \
                           L.pos, L.emb_g, L.emb_b, ids, cu, B, T_, rows, mrows, c.hidden, c.vocab, c.max_pos, c.ln_eps,  \
                           (bf16*)x, (bf16*)att, rpw, (unsigned char*)xq, qscale, (unsigned char*)attq);               \
    else                                                                                                           \
    hipLaunchKernelGGL((embed_ln_kernel<T, MAXC, false>), grid, dim3(256), 0, s, M->arena, L.student_stride, L.tok, L.pos, \
                       L.emb_g, L.emb_b, ids, cu, B, T_, rows, mrows, c.hidden, c.vocab, c.max_pos, c.ln_eps, (T*)x, \
                       (T*)att, rpw, (unsigned char*)xq, qscale, (unsigned char*)attq); } while (0)
    const int T_ = T;
    if (maxc > kMaxChunks) return hipErrorInvalidValue;
    if (bf16_path(c)) {
        if (maxc <= 1) SP_EMBED(bf16, 1); else if (maxc == 2) SP_EMBED(bf16, 2); else SP_EMBED(bf16, 4);
    } else {
        if (maxc <= 1) SP_EMBED(float, 1); else if (maxc == 2) SP_EMBED(float, 2); else SP_EMBED(float, 4);
    }
#undef SP_EMBED
    return hipGetLastError();
}

hipError_t launch_layernorm(const sp_model* M, const void* u, void* out, int rows, int mrows, int k, size_t g_off,
                            size_t b_off, hipStream_t s, void* outq, float qscale)
{
    const sp_config& c = M->cfg;
    const int rpw = rows_per_wave(mrows, k, 4);
    dim3 grid((mrows + 4 * rpw - 1) / (4 * rpw), k);
    const int maxc = (c.hidden / 8 + 63) / 64;              // 8-element chunks per lane
    if (maxc > kMaxChunks) return hipErrorInvalidValue;
#define SP_LN(T, MAXC) do {                                                                                         \
    if (outq && std::is_same<T, bf16>::value)                                                                       \
        hipLaunchKernelGGL((layernorm_kernel<bf16, MAXC, true>), grid, dim3(256), 0, s, M->arena, M->L.student_stride, \
                           g_off, b_off, (const bf16*)u, (bf16*)out, rows, mrows, c.hidden, c.ln_eps, rpw,         \
                           (unsigned char*)outq, qscale);                                                          \
    else                                                                                                            \
    hipLaunchKernelGGL((layernorm_kernel<T, MAXC, false>), grid, dim3(256), 0, s, M->arena, M->L.student_stride, g_off,    \
                       b_off, (const T*)u, (T*)out, rows, mrows, c.hidden, c.ln_eps, rpw, (unsigned char*)outq, qscale); } while (0)
    if (bf16_path(c)) {
        if (maxc <= 1) SP_LN(bf16, 1); else if (maxc == 2) SP_LN(bf16, 2); else SP_LN(bf16, 4);
    } else {
        if (maxc <= 1) SP_LN(float, 1); else if (maxc == 2) SP_LN(float, 2); else SP_LN(float, 4);
    }
#undef SP_LN
    return hipGetLastError();
}

hipError_t launch_layernorm_first(const sp_model* M, const void* u, void* out, int rows, const int32_t* cu, int B, int T, int k,
                                  size_t g_off, size_t b_off, hipStream_t s)
{
    const sp_config& c = M->cfg;
    if (!bf16_path(c) || B < 1 || B > rows || c.hidden > 1024) return hipErrorInvalidValue;
    const dim3 grid((unsigned)((B + 3) / 4), (unsigned)k);
#define SP_GO(MAXC) hipLaunchKernelGGL(layernorm_first_kernel<MAXC>, grid, dim3(256), 0, s, M->arena, M->L.student_stride, g_off, \
                                       b_off, (const bf16*)u, (bf16*)out, rows, cu, B, T, c.hidden, c.ln_eps)
    if (c.hidden <= 512) SP_GO(1); else SP_GO(2);
#undef SP_GO
    return hipGetLastError();
}

// Contents check of a forward's inputs (sp_check_inputs): every thread looks at a strided share of the ids and of the
// offsets and ORs what it finds into one word.
__global__ void clear_word_kernel(unsigned* w) { *w = 0u; }

__global__ __launch_bounds__(256) void check_inputs_kernel(const int32_t* __restrict__ ids,
                                                           const int32_t* __restrict__ cu, int B, int Tn, int max_seqlen,
                                                           int V, unsigned* flags)
{
    unsigned bad = 0;
    const int stride = gridDim.x * blockDim.x, first = blockIdx.x * blockDim.x + threadIdx.x;
    for (int i = first; i < Tn; i += stride) {
        const int id = ids[i];
        if (id < 0 || id >= V) bad |= SP_BAD_ID;
    }
    for (int b = first; b < B; b += stride) {
        const int a = cu[b], e = cu[b + 1];
        if (e <= a) bad |= SP_BAD_ORDER;
        else if (e - a > max_seqlen) bad |= SP_BAD_LENGTH;
    }
    if (first == 0) {
        if (cu[0] != 0) bad |= SP_BAD_CU0;
        if (cu[B] != Tn) bad |= SP_BAD_TOTAL;
    }
    if (bad) atomicOr(flags, bad);
}

hipError_t launch_check_inputs(const int32_t* ids, const int32_t* cu, int B, int T, int max_seqlen, int vocab,
                               unsigned* flags, hipStream_t s)
{
    hipLaunchKernelGGL(clear_word_kernel, dim3(1), dim3(1), 0, s, flags);
    const int blocks = (T + 255) / 256 < 1024 ? (T + 255) / 256 : 1024;
    hipLaunchKernelGGL(check_inputs_kernel, dim3(blocks < 1 ? 1 : blocks), dim3(256), 0, s, ids, cu, B, T, max_seqlen,
                       vocab, flags);
    return hipGetLastError();
}

hipError_t launch_ln_slices(const sp_model* M, const float* part, size_t slice, size_t p_ss, int splits, size_t bias_off,
                            const void* residual, void* out, int rows, int T, int mrows, int k, size_t g_off, size_t b_off,
                            hipStream_t s)
{
    const sp_config& c = M->cfg;
    if (!bf16_path(c) || c.hidden > 1024) return hipErrorInvalidValue;
    dim3 grid((mrows + 3) / 4, k);
#define SP_LNS(MAXC, SLICES)                                                                                       \
    hipLaunchKernelGGL((ln_slices_kernel<MAXC, SLICES>), grid, dim3(256), 0, s, M->arena, M->L.student_stride, g_off, b_off, bias_off, \
                       part, slice, p_ss, (const bf16*)residual, (bf16*)out, rows, T, mrows, c.hidden, c.ln_eps)
#define SP_GO(SLICES) case SLICES: if (c.hidden <= 512) SP_LNS(1, SLICES); else SP_LNS(2, SLICES); break
    switch (splits) {                                       // (what callers choose from)
        SP_GO(2); SP_GO(3); SP_GO(4); SP_GO(6); SP_GO(8);
        default: return hipErrorInvalidValue;
    }
#undef SP_GO
#undef SP_LNS
    return hipGetLastError();
}

hipError_t launch_sum_students(const float* z, int n, int k, float* logits, hipStream_t s)
{
    hipLaunchKernelGGL(sum_students_kernel, dim3((n + 255) / 256), dim3(256), 0, s, z, n, k, logits);
    return hipGetLastError();
}

hipError_t launch_head(const sp_model* M, const void* x, const int32_t* cu, int B, int T, int rows, int k, float* z,
                       float* zpart, float* logits, hipStream_t s)
{
    const sp_config& c = M->cfg;
    const ArenaLayout& L = M->L;
    const int nslice = c.hidden / 64;
    dim3 grid((B + kSeqPerWg - 1) / kSeqPerWg, k, nslice);
    const size_t smem = (size_t)(kSeqPerWg * c.hidden + 4 * kSeqPerWg * 64) * sizeof(float);
    if (bf16_path(c))
        hipLaunchKernelGGL(head_pool_kernel<bf16>, grid, dim3(256), smem, s, M->arena, L.student_stride, L.wp, L.bp,
                           L.wc, (const bf16*)x, cu, B, T, rows, c.hidden, c.classes, zpart);
    else
        hipLaunchKernelGGL(head_pool_kernel<float>, grid, dim3(256), smem, s, M->arena, L.student_stride, L.wp, L.bp,
                           L.wc, (const float*)x, cu, B, T, rows, c.hidden, c.classes, zpart);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    return launch_head_sum(M, zpart, B, k, z, logits, s);
}

}  // namespace sp
