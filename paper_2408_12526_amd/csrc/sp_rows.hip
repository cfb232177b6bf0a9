// Projections of few rows (bf16 path): the all-token layers of calls of up to kRowsMaxTokens tokens, and the last layer
// on the first-token rows (one row per sequence) of calls of any size.
//
// At these sizes a 64 x 64 tile that walks the reduction range through LDS is a serial chain of k-tiles, and a call is
// a chain of dependent launches of 4-8 us each in which neither the matrix cores nor the memory are busy.  Two changes
// of shape shorten both chains:
//   * a wave owns sixteen output features (the "A" rows of v_mfma_f32_16x16x32_bf16) and requests its whole share of
//     the weight matrix (16 rows x up to 1024 elements, up to 128 registers per lane) straight into registers before it
//     looks at anything else: one memory round trip, which runs while the activations are being prepared.  The weights
//     lie in memory in operand blocks (see ArenaLayout), so a wave-load is 1 KB in a row: with the rows of a plain
//     [out][in] matrix instead, four neighbouring lanes touch four cache lines, the load path delivers 16 bytes per
//     cycle instead of 64, and these kernels took 1.5 to 3 times as long;
//   * what produces the activations rides in the same launch while the rows are few: the kernels of the projections that
//     follow a LayerNorm (q|k|v, FFN up, pooler) normalise the fp32 rows the previous projection left (or gather and
//     normalise the embedding rows) into LDS themselves.
// One sequence of 64 tokens, hidden 768, one student: twelve launches, 57 us a call, where fifteen launches took 84.
// Rounding points: operands bf16, accumulation fp32, the rows before a LayerNorm stay fp32, x, x1, g, the attention
// output and the final hidden state are rounded to bf16.
#include <atomic>
#include <type_traits>

#include "sp_internal.h"

namespace sp {

namespace {

__device__ inline f32x4 mfma16(bf16x8 a, bf16x8 b, f32x4 c) { return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0); }

__device__ inline int first_row(const int32_t* cu, int b, int Tn)
{
    const int r = cu[b];
    return r < 0 ? 0 : (r >= Tn ? Tn - 1 : r);
}

// -------------------------------------------------------------------------------------
// LayerNorm (or embedding + LayerNorm) of sixteen rows, then the projection of those rows.
// Workgroup = 4 waves x 16 features, whole reduction range (H <= 32 NS) in one pass; a wave normalises four of the rows.
//   grid: ((student * nrb + row block) * nfb8 + feature block); nfb8 is a multiple of 8, so the row blocks that read one
//   slice of the weights run on one XCD and share its L2.
// Bound by latency: launch, the rows (just written, from beyond the L2), the statistics, 24 LDS reads and matrix
// instructions; 5.4-5.8 us for one student's FFN up-projection of up to 64 rows, where the LayerNorm launch and the tile
// kernel took 4.6 + 7.7 us.  The statistics are repeated by every workgroup of a row block (36 to 48 of them), which is
// what bounds it once the rows of all students exceed a few hundred: the callers then normalise in a launch of its own and
// take the tile kernel.  (Tried against that: 32 and 64 rows per workgroup, eight waves with 32 features each, sixteen
// lanes per row: 8 to 25 us where this takes 6 to 12.)
// -------------------------------------------------------------------------------------
struct RowsLnArgs {
    const char* arena;
    size_t ss;                        // student stride of the arena (bytes)
    size_t w, b, g, beta;             // weights, bias, LayerNorm scale and shift (byte offsets into a student slab)
    float eps;
    const float* u;                   // rows before the LayerNorm: [student][u_ss], row stride H
    size_t u_ss;
    const int32_t *ids, *cu;          // embedding prologue
    size_t tok, pos;
    int B, V, P;
    bf16* xout;                       // normalised rows once more, row stride H (null: not needed)
    size_t x_ss;
    void* out;                        // [student][o_ss] (elements of the output type)
    size_t o_ss;
    RowsLayout ol;
    bf16* out2;                       // value third, transposed: [student][o2_ss], row stride ld2
    size_t o2_ss;
    int ld2, n_split;
    size_t wc;                        // pooler: classifier, [in][out]; out: [student][feature block][row][class]
    int C;
    int M, H, N, nfb, nfb8, nrb;
};

constexpr int kMaxClasses = 16;
enum RowsPrologue { PRO_LN = 0, PRO_EMBED = 1 };

// (No branches between the loads: behind one, the compiler waits for everything in flight at the first use.)
template <int PRO, int EPI, int NS>
__global__ __launch_bounds__(256) void rows_ln_gemm_kernel(RowsLnArgs p)
{
    constexpr int H = 32 * NS, NC = (NS + 7) / 8;           // NC: chunks of four elements per lane and row
    constexpr int PITCH = NS * 64 + 16;                     // bytes per LDS row: sixteen rows, one chunk: 16 bank groups
    constexpr int RW = 4;                                   // rows a wave normalises
    __shared__ __attribute__((aligned(16))) char rowbuf[16 * PITCH];
    const int fb = (int)blockIdx.x % p.nfb8, rm = (int)blockIdx.x / p.nfb8;
    if (fb >= p.nfb) return;
    const int m = rm / p.nrb, r0 = (rm % p.nrb) * 16;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int l16 = lane & 15, kg = lane >> 4;
    const char* sb = p.arena + (size_t)m * p.ss;
    const int n0 = fb * 64 + wave * 16;
    // element of chunk c of a row for this lane; chunks beyond H (its last half chunk of 128) repeat the last one and do not count
    auto in_row = [&](int c) { return 256 * (c + 1) <= H || 4 * (lane + 64 * c) < H; };
    auto el = [&](int c) { return in_row(c) ? 4 * (lane + 64 * c) : H - 4; };
    // rows beyond M repeat the last one; what comes of them is written where no result looks
    auto row_of = [&](int r) { return r < p.M ? r : p.M - 1; };

    // the rows first (they are on the critical path), then the weights, both in flight together
    const int rw = r0 + wave * RW;                          // this wave's first row
    f32x4 v[RW][NC];
    if constexpr (PRO == PRO_LN) {
        const float* ub = p.u + (size_t)m * p.u_ss;
#pragma unroll
        for (int i = 0; i < RW; ++i)
#pragma unroll
            for (int c = 0; c < NC; ++c) v[i][c] = *(const f32x4*)(ub + (size_t)row_of(rw + i) * H + el(c));
    }
    bf16x4 te[PRO == PRO_EMBED ? RW : 1][NC], pe[PRO == PRO_EMBED ? RW : 1][NC];
    if constexpr (PRO == PRO_EMBED) {
        // Start of each row's sequence: the number of boundaries cu[1 .. B - 1] that are <= row, counted by the whole wave
        // 64 at a time, so that there is no chain of dependent loads.
        int ids[RW], start[RW];
#pragma unroll
        for (int i = 0; i < RW; ++i) { ids[i] = p.ids[row_of(rw + i)]; start[i] = 0; }
        for (int b0 = 0; b0 < p.B; b0 += 64) {
            const int bi = b0 + lane;
            const int cv = bi < p.B ? p.cu[bi] : 0x7fffffff;
#pragma unroll
            for (int i = 0; i < RW; ++i) {
                const int cnt = __popcll(__ballot(cv <= row_of(rw + i)));
                // (boundaries ascend: the last one counted so far is the start of the row's sequence)
                if (cnt > 0) start[i] = __builtin_amdgcn_readlane(cv, cnt - 1);
            }
        }
#pragma unroll
        for (int i = 0; i < RW; ++i) {
            int pos = row_of(rw + i) - start[i], id = ids[i];
            pos = pos < 0 ? 0 : (pos >= p.P ? p.P - 1 : pos);
            id = id < 0 ? 0 : (id >= p.V ? p.V - 1 : id);
            const bf16* t = (const bf16*)(sb + p.tok) + (size_t)id * H;
            const bf16* q = (const bf16*)(sb + p.pos) + (size_t)pos * H;
#pragma unroll
            for (int c = 0; c < NC; ++c) { te[i][c] = *(const bf16x4*)(t + el(c)); pe[i][c] = *(const bf16x4*)(q + el(c)); }
        }
    }
    f32x4 gg[NC], bb[NC];
    {
        const float* gam = (const float*)(sb + p.g);
        const float* bet = (const float*)(sb + p.beta);
#pragma unroll
        for (int c = 0; c < NC; ++c) { gg[c] = *(const f32x4*)(gam + el(c)); bb[c] = *(const f32x4*)(bet + el(c)); }
    }
    __builtin_amdgcn_sched_barrier(0);
    bf16x8 fw[NS];
    {
        const bf16* wp = (const bf16*)(sb + p.w) + (size_t)n0 * H + kg * 128 + l16 * 8;
#pragma unroll
        for (int s = 0; s < NS; ++s) fw[s] = *(const bf16x8*)(wp + 512 * s);
    }
    const bool transposed = EPI == EPI_QKV && fb * 64 >= p.n_split;    // (uniform: n_split is a multiple of 64)
    f32x4 acc;
    {
        const float* bias = (const float*)(sb + p.b) + n0;
        if (transposed) { const float bs = bias[l16]; acc = f32x4{bs, bs, bs, bs}; }
        else acc = *(const f32x4*)(bias + 4 * kg);
    }
    // pooler: this lane's four features of the classifier's matrix, all of them if there are two classes
    const bf16* wc = (const bf16*)(sb + p.wc) + (size_t)(n0 + 4 * kg) * p.C;
    bf16x4 wc2[2];
    if constexpr (EPI == EPI_BIAS_TANH) {
        const bf16* at = (n0 + 4 * kg) * p.C + 8 <= H * p.C ? wc : wc - 4;      // (one class: the last lanes' eight would pass the end)
        wc2[0] = *(const bf16x4*)at;
        wc2[1] = *(const bf16x4*)(at + 4);
    }
    __builtin_amdgcn_sched_barrier(0);

    if constexpr (PRO == PRO_EMBED) {
#pragma unroll
        for (int i = 0; i < RW; ++i)
#pragma unroll
            for (int c = 0; c < NC; ++c)
#pragma unroll
                for (int e = 0; e < 4; ++e) v[i][c][e] = (float)te[i][c][e] + (float)pe[i][c][e];
    }
    const float inv_h = __builtin_amdgcn_rcpf((float)H);
    float mean[RW], inv[RW];
#pragma unroll
    for (int i = 0; i < RW; ++i) {
        float s = 0.f;
#pragma unroll
        for (int c = 0; c < NC; ++c)
#pragma unroll
            for (int e = 0; e < 4; ++e) s += in_row(c) ? v[i][c][e] : 0.f;
        mean[i] = s;
    }
#pragma unroll
    for (int i = 0; i < RW; ++i) mean[i] = wave_sum(mean[i]) * inv_h;
#pragma unroll
    for (int i = 0; i < RW; ++i) {
        float q = 0.f;
#pragma unroll
        for (int c = 0; c < NC; ++c)
#pragma unroll
            for (int e = 0; e < 4; ++e) { const float d = in_row(c) ? v[i][c][e] - mean[i] : 0.f; q += d * d; }
        inv[i] = q;
    }
#pragma unroll
    for (int i = 0; i < RW; ++i) inv[i] = __builtin_amdgcn_rsqf(wave_sum(inv[i]) * inv_h + p.eps);
#pragma unroll
    for (int i = 0; i < RW; ++i)
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            bf16x4 o;
#pragma unroll
            for (int e = 0; e < 4; ++e) o[e] = (bf16)(gg[c][e] * ((v[i][c][e] - mean[i]) * inv[i]) + bb[c][e]);
            if (in_row(c)) *(bf16x4*)(rowbuf + (wave * RW + i) * PITCH + 8 * (lane + 64 * c)) = o;
        }
    barrier_lds();

    auto rows_frag = [&](int s) { return *(const bf16x8*)(rowbuf + l16 * PITCH + (4 * s + kg) * 16); };
    if (EPI == EPI_QKV && transposed) {                     // rows: tokens, columns: features
#pragma unroll
        for (int s = 0; s < NS; ++s) acc = mfma16(rows_frag(s), fw[s], acc);
    } else {                                                // rows: features, columns: tokens
#pragma unroll
        for (int s = 0; s < NS; ++s) acc = mfma16(fw[s], rows_frag(s), acc);
    }
    // the rows once more for whoever adds them as a residual
    if (fb == 0 && p.xout)
        for (int i = 0; i < RW && rw + i < p.M; ++i)
            for (int e = 8 * lane; e < H; e += 512)
                *(bf16x8*)(p.xout + (size_t)m * p.x_ss + (size_t)(rw + i) * H + e) = *(const bf16x8*)(rowbuf + (wave * RW + i) * PITCH + 2 * e);
    if (EPI == EPI_QKV && transposed) {
        bf16x4 o;
#pragma unroll
        for (int e = 0; e < 4; ++e) o[e] = (bf16)acc[e];
        *(bf16x4*)(p.out2 + (size_t)m * p.o2_ss + (size_t)(n0 - p.n_split + l16) * p.ld2 + r0 + 4 * kg) = o;
        return;
    }
    if constexpr (EPI == EPI_BIAS_TANH) {
        // This workgroup's share of the classifier: 64 of the pooled features, so that the launch behind it adds a dozen numbers
        // per output where it read every pooled row (and, with the classifier's matrix cold, took 6 us for eight students).
        __shared__ float zs[4][16][kMaxClasses];
        float t[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) t[e] = tanhf(acc[e]);
        for (int c = 0; c < p.C; ++c) {
            float z = 0.f;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float w2 = (float)(c ? wc2[e >> 1][2 * (e & 1) + 1] : wc2[e >> 1][2 * (e & 1)]);
                z = __builtin_fmaf(t[e], p.C == 2 ? w2 : (float)wc[(size_t)e * p.C + c], z);
            }
            float a = z, b = z;                             // over the four lanes of a row: 16 features
            swap_rows(a, b);
            z = a + b;
            a = z;
            b = z;
            swap_halves(a, b);
            if (kg == 0) zs[wave][l16][c] = a + b;
        }
        __syncthreads();
        for (int i = threadIdx.x; i < 16 * p.C; i += 256) {
            const int r = i / p.C, c = i - r * p.C;
            if (r0 + r < p.M)
                ((float*)p.out)[(((size_t)m * p.nfb + fb) * p.M + r0 + r) * p.C + c] = (zs[0][r][c] + zs[1][r][c]) + (zs[2][r][c] + zs[3][r][c]);
        }
        return;
    }
    const int f = n0 + 4 * kg;
    const size_t at = (size_t)m * p.o_ss + (size_t)(r0 / 16) * p.ol.rb + (size_t)l16 * p.ol.rs + (size_t)(f >> 3) * p.ol.cs + (f & 7);
    bf16x4 o;
#pragma unroll
    for (int e = 0; e < 4; ++e) o[e] = (bf16)(EPI == EPI_BIAS_GELU ? gelu_erf_fast(acc[e]) : acc[e]);
    *(bf16x4*)((bf16*)p.out + at) = o;
}

// -------------------------------------------------------------------------------------
// Projection of bf16 rows with the reduction range split over the four waves of a workgroup: 16 TF features x 16 TM rows
// per workgroup (see launch_rows_k for the choice; 768 features from a depth of 3072: 4.4 us for one student and 64 rows, 12.4 us
// for eight), wave w reduces over the w-th quarter (at most 32 NS elements at a time), weights and rows straight from
// global memory in operand layout; the four partial tiles meet in LDS and are added in wave order.
//   F32OUT: out (fp32) = sum + bias + residual row;  else out (bf16) = sum + bias.
//   Row r of the operand: row r, or the token row cu[r] (a_first); the same for the residual (r_first).
//   a_hs != 0: the operand row depends on the head of the feature (64 features per head): + head * a_hs elements.
// -------------------------------------------------------------------------------------
struct RowsKArgs {
    const char* arena;
    size_t ss, w, b;
    const bf16* A;
    size_t a_ss;
    RowsLayout al;
    int a_hs, a_first;
    const bf16* res;
    size_t r_ss;
    int ldr, r_first;
    void* out;
    size_t o_ss;
    int ldo;
    const int32_t* cu;
    int Tn, M, N, Kd, nfb, nfb8, nrb;
};

// Outputs are four neighbouring features of a row per thread and round: threads per row, rows per round, rounds.
template <int TM, int TF>
struct KsplitOut {
    static constexpr int TPR = 4 * TF, RPR = 256 / TPR, ROUNDS = 16 * TM / RPR < 1 ? 1 : 16 * TM / RPR;
};

// what the last step needs (requested first)
template <bool F32OUT, int TM, int TF>
__device__ __forceinline__ void ksplit_inputs(const RowsKArgs& p, bf16x4 (&rv)[KsplitOut<TM, TF>::ROUNDS], f32x4& bias,
                                              const char* sb, int m, int r0, int n0)
{
    using O = KsplitOut<TM, TF>;
    const int f = 4 * ((int)threadIdx.x % O::TPR), rr = (int)threadIdx.x / O::TPR;
    bias = *(const f32x4*)((const float*)(sb + p.b) + n0 + f);
    if (!F32OUT) return;
#pragma unroll
    for (int i = 0; i < O::ROUNDS; ++i) {
        int r = r0 + (rr + O::RPR * i) % (16 * TM);
        r = r < p.M ? r : p.M - 1;
        rv[i] = *(const bf16x4*)(p.res + (size_t)m * p.r_ss + (size_t)(p.r_first ? first_row(p.cu, r, p.Tn) : r) * p.ldr + n0 + f);
    }
}

// the four waves' partial tiles through LDS, added in wave order, then bias and residual
template <bool F32OUT, int TM, int TF>
__device__ __forceinline__ void ksplit_finish(const RowsKArgs& p, float (*part)[16 * TM][16 * TF + 4], const f32x4 (&acc)[TF][TM],
                                              const bf16x4 (&rv)[KsplitOut<TM, TF>::ROUNDS], f32x4 bias, int m, int r0, int n0)
{
    using O = KsplitOut<TM, TF>;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, l16 = lane & 15, kg = lane >> 4;
    const int f = 4 * ((int)threadIdx.x % O::TPR), rr = (int)threadIdx.x / O::TPR;
#pragma unroll
    for (int fi = 0; fi < TF; ++fi)
#pragma unroll
        for (int t = 0; t < TM; ++t) *(f32x4*)&part[wave][16 * t + l16][16 * fi + 4 * kg] = acc[fi][t];
    __syncthreads();
#pragma unroll
    for (int i = 0; i < O::ROUNDS; ++i) {
        const int rl = rr + O::RPR * i, r = r0 + rl;
        if (rl >= 16 * TM || r >= p.M) continue;
        f32x4 s = *(const f32x4*)&part[0][rl][f];
#pragma unroll
        for (int w = 1; w < 4; ++w) s += *(const f32x4*)&part[w][rl][f];
        s += bias;
        const size_t at = (size_t)m * p.o_ss + (size_t)r * p.ldo + n0 + f;
        if (F32OUT) {
#pragma unroll
            for (int e = 0; e < 4; ++e) s[e] += (float)rv[i][e];
            *(f32x4*)((float*)p.out + at) = s;
        } else {
            bf16x4 o;
#pragma unroll
            for (int e = 0; e < 4; ++e) o[e] = (bf16)s[e];
            *(bf16x4*)((bf16*)p.out + at) = o;
        }
    }
}

template <bool F32OUT, int TM, int TF, int NS, bool EXACT>
__global__ __launch_bounds__(256) void rows_ksplit_kernel(RowsKArgs p)
{
    __shared__ __attribute__((aligned(16))) float part[4][16 * TM][16 * TF + 4];  // [wave][row][feature], padded
    const int fb = (int)blockIdx.x % p.nfb8, rm = (int)blockIdx.x / p.nfb8;
    if (fb >= p.nfb) return;
    const int m = rm / p.nrb, r0 = (rm % p.nrb) * 16 * TM;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int l16 = lane & 15, kg = lane >> 4;
    const char* sb = p.arena + (size_t)m * p.ss;
    const int Kd = EXACT ? 128 * NS : p.Kd, n0 = fb * 16 * TF, kw = Kd >> 2, k0 = wave * kw;
    const bf16* wp = (const bf16*)(sb + p.w) + (size_t)n0 * Kd + (size_t)(k0 / 8 + kg) * 128 + l16 * 8;
    const bf16* ab = p.A + (size_t)m * p.a_ss + (size_t)(n0 >> 6) * p.a_hs + (size_t)(k0 / 8 + kg) * p.al.cs;
    const int step = 4 * p.al.cs;                           // 32 elements further along the reduction
    const bf16* ar[TM];
#pragma unroll
    for (int t = 0; t < TM; ++t) {
        int r = r0 + 16 * t + l16;
        r = r < p.M ? r : p.M - 1;
        if (p.a_first) r = first_row(p.cu, r, p.Tn);
        ar[t] = ab + (size_t)(r >> 4) * p.al.rb + (size_t)(r & 15) * p.al.rs;
    }
    bf16x4 rv[KsplitOut<TM, TF>::ROUNDS];
    f32x4 bias;
    ksplit_inputs<F32OUT, TM, TF>(p, rv, bias, sb, m, r0, n0);
    f32x4 acc[TF][TM];
#pragma unroll
    for (int fi = 0; fi < TF; ++fi)
#pragma unroll
        for (int t = 0; t < TM; ++t) acc[fi][t] = f32x4{0.f, 0.f, 0.f, 0.f};
    // (!EXACT: several passes, the last one's steps beyond the range repeat its last step with zero weights)
    for (int c0 = 0; c0 < (EXACT ? 1 : kw); c0 += 32 * NS) {
        bf16x8 fw[TF][NS], fa[2][NS];
        auto at = [&](int s) { const int e = c0 / 32 + s; return EXACT || 32 * e < kw ? e : kw / 32 - 1; };
#pragma unroll
        for (int fi = 0; fi < TF; ++fi)
#pragma unroll
            for (int s = 0; s < NS; ++s) {
                fw[fi][s] = *(const bf16x8*)(wp + (size_t)fi * 16 * Kd + (size_t)at(s) * 512);
                if (!EXACT && c0 + 32 * s >= kw) fw[fi][s] = bf16x8{};
            }
#pragma unroll
        for (int s = 0; s < NS; ++s) fa[0][s] = *(const bf16x8*)(ar[0] + (size_t)at(s) * step);
#pragma unroll
        for (int t = 0; t < TM; ++t) {
            if (t + 1 < TM) {
#pragma unroll
                for (int s = 0; s < NS; ++s) fa[(t + 1) & 1][s] = *(const bf16x8*)(ar[t + 1] + (size_t)at(s) * step);
                __builtin_amdgcn_sched_barrier(0);
            }
#pragma unroll
            for (int s = 0; s < NS; ++s)
#pragma unroll
                for (int fi = 0; fi < TF; ++fi) acc[fi][t] = mfma16(fw[fi][s], fa[t & 1][s], acc[fi][t]);   // rows: features
        }
    }
    ksplit_finish<F32OUT, TM, TF>(p, part, acc, rv, bias, m, r0, n0);
}

// -------------------------------------------------------------------------------------
// Queries of the first tokens, folded through the key projection (see the first-token attention): one workgroup =
// (student, head, 16 sequences).  q_h = x[first token] Wq_h^T + bq_h (sixteen of the head's 64 features per wave),
// exchanged through LDS as bf16, then q~_h = Wk_h q_h (a quarter of the H features per wave, reduction over 64).  Both
// weight slices (64 x H each) are requested at once, so the two products cost one memory round trip: 9-13 us for four
// students and up to 32 sequences where gathering the rows and two launches took 22 us.  The weights fill the register file
// of a compute unit, so a launch of more workgroups than that repeats the round trip: there a workgroup takes several blocks
// of 16 sequences, the weights staying in its registers.  Its token rows, a quarter per wave, go through registers into one of
// two LDS buffers, two blocks ahead, and its results through LDS out in whole row pieces.  What bounds it then is the way of
// rows and results through memory.  us at hidden 768, each wave fetching all rows when it needs them / this: eight students, 256
// sequences 41 / 29; four, 1024 sequences 118 / 71; two, 4096 sequences 259 / 148.
// A-operand row i of block j of a pair of blocks stands for feature 8 (i / 4) + 4 (j % 2) + i % 4 of the pair's 32, so
// that a lane ends with eight neighbouring features and writes 16 bytes.
// SCALED: the results times a LayerNorm's scale, feature by feature from LDS, before they are rounded (the attention behind it then
// rounds nothing again): 26.3 -> 28.6 us for eight students of 768 on 256 sequences.
// -------------------------------------------------------------------------------------
struct FoldQArgs {
    const char* arena;
    size_t ss, wq, bq, wk;            // wk: the key projection with rows = inputs
    const bf16* x;
    size_t x_ss;
    const int32_t* cu;
    bf16* q;                          // [student][q_ss], row stride H
    size_t q_ss;
    bf16* qt;                         // [student][qt_ss], row stride heads * H
    size_t qt_ss;
    size_t g;                         // SCALED: what feature f of a folded query is multiplied with (fp32, byte offset into a student slab)
    int Tn, M, H, heads, heads8, nrb, rpw;                  // nrb: groups of rpw blocks of 16 sequences
};

constexpr int kFoldQPitch = 64 * 2 + 16;                    // bytes per staged query row
constexpr int fold_x_pitch(int ns) { return ns * 64 + 16; } // bytes per staged token row
constexpr int fold_o_pitch(int ns) { return ns * 16 + 16; } // bytes per row of a wave's staged output
constexpr size_t fold_query_smem(int ns, bool scaled)
{
    return 2 * 16 * (size_t)(fold_x_pitch(ns) + kFoldQPitch) + 4 * 16 * (size_t)fold_o_pitch(ns) + (scaled ? 32 * (size_t)ns * 4 : 0);
}

template <int NS, bool SCALED>
__global__ __launch_bounds__(256) void fold_query_kernel(FoldQArgs p)
{
    constexpr int H = 32 * NS, XP = fold_x_pitch(NS), QP = kFoldQPitch;
    constexpr int CPR = H / 8, NL = 4 * CPR / 64;           // 16-byte chunks of a row; chunks a lane moves (a wave: four rows)
    constexpr int OP = fold_o_pitch(NS), CO = NS, NO = CO / 4;   // 16-byte chunks of a staged output row; chunks a lane stores
    extern __shared__ __attribute__((aligned(16))) char fold_lds[];
    char *const xbuf = fold_lds, *const qbuf = fold_lds + 2 * 16 * XP;
    char* const obuf = qbuf + 2 * 16 * QP + (threadIdx.x >> 6) * 16 * OP;   // wave-private
    float* const gbuf = (float*)(qbuf + 2 * 16 * QP + 4 * 16 * OP);         // the H scales
    const int h = (int)blockIdx.x % p.heads8, rm = (int)blockIdx.x / p.heads8;
    if (h >= p.heads) return;
    const int m = rm / p.nrb, rb = (rm % p.nrb) * p.rpw * 16;
    const int re = rb + p.rpw * 16 < p.M ? rb + p.rpw * 16 : p.M;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int l16 = lane & 15, kg = lane >> 4;
    const char* sb = p.arena + (size_t)m * p.ss;
    const int n0 = h * 64 + wave * 16;
    const bf16* xs = p.x + (size_t)m * p.x_ss;
    // this wave's four of a block's sixteen rows: chunk lane + 64 i of the four together (rows beyond the last sequence repeat it)
    bf16x8 xr[2][NL];                                       // two blocks in flight: a block's set by its number's last bit
    // (The rows' token indices come through the scalar path: vector loads would be waited for together with the stores before
    // them, which put several microseconds between two blocks.)
    auto load_x = [&](int r0, auto set) {
        const auto* cu = (const __attribute__((address_space(4))) int32_t*)p.cu;
        int t[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int r = r0 + 4 * wave + q < p.M ? r0 + 4 * wave + q : p.M - 1, v = cu ? cu[r] : r;
            t[q] = v < 0 ? 0 : (v >= p.Tn ? p.Tn - 1 : v);
        }
#pragma unroll
        for (int i = 0; i < NL; ++i) {
            const int c = lane + 64 * i, q = c / CPR;
            xr[set()][i] = *(const bf16x8*)(xs + (size_t)(q == 0 ? t[0] : q == 1 ? t[1] : q == 2 ? t[2] : t[3]) * H + (c % CPR) * 8);
        }
    };
    auto write_x = [&](auto set) {
#pragma unroll
        for (int i = 0; i < NL; ++i) {
            const int c = lane + 64 * i;
            *(bf16x8*)(xbuf + (set() * 16 + 4 * wave + c / CPR) * XP + (c % CPR) * 16) = xr[set()][i];
        }
    };
    constexpr std::integral_constant<int, 0> S0{};
    constexpr std::integral_constant<int, 1> S1{};
    load_x(rb, S0);
    bf16x8 fw[NS];
    const bf16* wp = (const bf16*)(sb + p.wq) + (size_t)n0 * H + kg * 128 + l16 * 8;
#pragma unroll
    for (int s = 0; s < NS; ++s) fw[s] = *(const bf16x8*)(wp + 512 * s);
    const f32x4 bias = *(const f32x4*)((const float*)(sb + p.bq) + n0 + 4 * kg);
    // key slice: this wave's H / 4 features in pairs of 16-row blocks, two reduction steps each
    const int f0 = wave * (H / 4);                          // (a multiple of 32)
    const int prow = 8 * (l16 >> 2) + (l16 & 3);
    // (rows prow and prow + 4 of a pair lie in the same block of sixteen)
    const bf16* kp = (const bf16*)(sb + p.wk) + (size_t)(f0 + (prow & 16)) * H + (size_t)(h * 8 + kg) * 128 + (prow & 15) * 8;
    bf16x8 fk[NS / 2][2];                                   // [block of 16 features][reduction step]
#pragma unroll
    for (int j = 0; j < NS / 2; ++j)
#pragma unroll
        for (int s = 0; s < 2; ++s) fk[j][s] = *(const bf16x8*)(kp + (size_t)(j >> 1) * 32 * H + 32 * (j & 1) + 512 * s);
    f32x4 gv = {};
    if (SCALED && 4 * threadIdx.x < H) gv = *(const f32x4*)((const float*)(sb + p.g) + 4 * threadIdx.x);
    __builtin_amdgcn_sched_barrier(0);
    write_x(S0);
    if (SCALED && 4 * threadIdx.x < H) *(f32x4*)(gbuf + 4 * threadIdx.x) = gv;
    if (rb + 16 < re) load_x(rb + 16, S1);
    if (rb + 32 < re) load_x(rb + 32, S0);
    barrier_lds();
    // A block's rows are in LDS when its turn begins.  During it the next one's, two turns in flight, are put down and their
    // registers requested again for the block two after that.  Either buffer's readers are behind a barrier by then.
    auto block = [&](int r0, auto set, auto other) {
        constexpr int buf = decltype(set)::value;
        const int r = r0 + l16;                             // this lane's sequence
        f32x4 acc = bias, acc1 = {0.f, 0.f, 0.f, 0.f};
        const char* xrow = xbuf + (buf * 16 + l16) * XP + 16 * kg;
#pragma unroll
        for (int s = 0; s < NS; s += 2) {
            acc = mfma16(fw[s], *(const bf16x8*)(xrow + 64 * s), acc);
            acc1 = mfma16(fw[s + 1], *(const bf16x8*)(xrow + 64 * (s + 1)), acc1);
        }
        acc += acc1;
        bf16x4 o4;
#pragma unroll
        for (int e = 0; e < 4; ++e) o4[e] = (bf16)acc[e];
        *(bf16x4*)(qbuf + (buf * 16 + l16) * QP + (wave * 16 + 4 * kg) * 2) = o4;
        if (r0 + 16 < re) {
            write_x(other);
            if (r0 + 48 < re) load_x(r0 + 48, other);
        }
        if (r < p.M) *(bf16x4*)(p.q + (size_t)m * p.q_ss + (size_t)r * H + n0 + 4 * kg) = o4;
        barrier_lds();
        bf16x8 fq[2];
#pragma unroll
        for (int s = 0; s < 2; ++s) fq[s] = *(const bf16x8*)(qbuf + (buf * 16 + l16) * QP + (4 * s + kg) * 16);
#pragma unroll
        for (int j = 0; j < NS / 2; j += 2) {
            f32x4 a = {0.f, 0.f, 0.f, 0.f}, b = a;
#pragma unroll
            for (int s = 0; s < 2; ++s) { a = mfma16(fk[j][s], fq[s], a); b = mfma16(fk[j + 1][s], fq[s], b); }
            if (SCALED) {
                a *= *(const f32x4*)(gbuf + f0 + 16 * j + 8 * kg);
                b *= *(const f32x4*)(gbuf + f0 + 16 * j + 8 * kg + 4);
            }
            bf16x8 o;
#pragma unroll
            for (int e = 0; e < 4; ++e) { o[e] = (bf16)a[e]; o[4 + e] = (bf16)b[e]; }
            *(bf16x8*)(obuf + l16 * OP + 32 * j + 16 * kg) = o;
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int i = 0; i < NO; ++i) {
            const int c = lane + 64 * i, ro = r0 + c / CO;
            if (ro < p.M)
                *(bf16x8*)(p.qt + (size_t)m * p.qt_ss + ((size_t)ro * p.heads + h) * H + f0 + (c % CO) * 8) =
                    *(const bf16x8*)(obuf + (c / CO) * OP + (c % CO) * 16);
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
    };
    for (int r0 = rb; r0 < re; r0 += 32) {
        block(r0, S0, S1);
        if (r0 + 16 < re) block(r0 + 16, S1, S0);
    }
}

// -------------------------------------------------------------------------------------
// Attention of the first token of each sequence on formed queries, keys and values (calls whose q|k|v projection covers
// every token): WPH waves share one (student, sequence, head), 64 keys per step and wave, a lane per key for the scores
// and a lane per dimension for the values (feature-major rows, eight tokens per 16 bytes).  Probabilities are rounded to
// bf16 for the product and summed in fp32 as in the all-token kernel, and each tile of 32 keys against the maximum of
// the keys up to its end, as there in sequences of up to 128 tokens (64 keys in longer ones): up to that length the two round alike.
// -------------------------------------------------------------------------------------
template <int WPH>
__global__ __launch_bounds__(256) void attention_first_kernel(const bf16* __restrict__ qkv, const bf16* __restrict__ vt,
                                                              bf16* __restrict__ att, const int32_t* __restrict__ cu,
                                                              int B, int Tn, int rows, int H, int heads, int max_seqlen)
{
    __shared__ __attribute__((aligned(16))) float ps[4][72];            // a wave's probabilities, slots of its step
    __shared__ float po[4][64], pl[4], tm[2][8];                        // partial outputs and sums; maxima of a step's tiles
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int m = blockIdx.y, item = (int)blockIdx.x * (4 / WPH) + wave / WPH, part = wave % WPH;
    const bool on = item < B * heads;                       // (whole waves; WPH == 4: every item exists)
    const int b = on ? item / heads : 0, h = on ? item % heads : 0;
    int t0 = cu[b], t1 = cu[b + 1];
    t0 = t0 < 0 ? 0 : (t0 > Tn - 1 ? Tn - 1 : t0);
    int L = t1 - t0;
    L = L < 1 ? 1 : L;
    L = L > max_seqlen ? max_seqlen : L;
    L = L > Tn - t0 ? Tn - t0 : L;
    if (!on) return;
    const size_t ld = (size_t)3 * H;
    const bf16* base = qkv + ((size_t)m * rows + t0) * ld + h * 64;
    const int lead = t0 & 7;                                // value rows are fetched in chunks of eight tokens
    const bf16* vrow = vt + ((size_t)m * H + h * 64 + lane) * rows + (t0 - lead);
    const float sl2 = 0.125f * 1.44269504088896341f;
    bf16x8 q[8];
#pragma unroll
    for (int c = 0; c < 8; ++c) q[c] = *(const bf16x8*)(base + 8 * c);
    float mrun = -INFINITY, lrun = 0.f, o = 0.f;
    // steps of 64 WPH slots; slot i is token i - lead of the sequence
    for (int st = 0, sb0 = 0; sb0 < L + lead; sb0 += 64 * WPH, st ^= 1) {
        const int s0 = sb0 + 64 * part, key = s0 + lane - lead;
        const bool ok = key >= 0 && key < L;
        const bf16* kr = base + H + (size_t)(ok ? key : 0) * ld;
        bf16x8 kv[8], vv[8];
#pragma unroll
        for (int c = 0; c < 8; ++c) kv[c] = *(const bf16x8*)(kr + 8 * c);
#pragma unroll
        for (int c = 0; c < 8; ++c) {
            vv[c] = bf16x8{};
            if (s0 + 8 * c < L + lead) vv[c] = *(const bf16x8*)(vrow + s0 + 8 * c);
        }
        float sc = 0.f;
#pragma unroll
        for (int c = 0; c < 8; ++c)
#pragma unroll
            for (int e = 0; e < 8; ++e) sc = __builtin_fmaf((float)q[c][e], (float)kv[c][e], sc);
        sc = ok ? sc : -INFINITY;
        // maxima of the step's tiles, 32 slots (half a wave) each, then of everything up to a tile's end
        float mh = fmaxf(sc, dpp_moved<kDppPair>(sc));
        mh = fmaxf(mh, dpp_moved<kDppQuad>(mh));
        mh = fmaxf(mh, dpp_moved<kDppHalfRowMirror>(mh));
        mh = fmaxf(mh, dpp_moved<kDppRowMirror>(mh));
        float x0 = mh, x1 = mh;
        swap_rows(x0, x1);
        mh = fmaxf(x0, x1);
        x0 = mh;
        x1 = mh;
        swap_halves(x0, x1);                                // x0: the lower half's maximum, x1: the upper half's
        float mlow, mhigh, mend;                            // reference of the two tiles; of the whole step
        if (WPH == 1) {
            mlow = fmaxf(mrun, x0);
            mhigh = mend = fmaxf(mlow, x1);
        } else {
            if (lane == 0) { tm[st][2 * part] = x0; tm[st][2 * part + 1] = x1; }
            __syncthreads();
            float run = mrun;
            mlow = mhigh = mrun;
#pragma unroll
            for (int t = 0; t < 8; ++t) {
                run = fmaxf(run, tm[st][t]);
                if (t == 2 * part) mlow = run;
                if (t == 2 * part + 1) mhigh = run;
            }
            mend = run;
        }
        const float ref = lane < 32 ? mlow : mhigh;         // (finite: the first tile has a key of the sequence)
        const float pr = __builtin_amdgcn_exp2f((sc - ref) * sl2);
        const float down = __builtin_amdgcn_exp2f((ref - mend) * sl2), alpha = __builtin_amdgcn_exp2f((mrun - mend) * sl2);
        mrun = mend;
        lrun = lrun * alpha + pr * down;                    // this lane's share
        o *= alpha;
        ps[wave][lane] = (float)(bf16)pr * down;
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int c = 0; c < 8; ++c) {
            const f32x4 p0 = *(const f32x4*)&ps[wave][8 * c], p1 = *(const f32x4*)&ps[wave][8 * c + 4];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                o = __builtin_fmaf(p0[e], (float)vv[c][e], o);
                o = __builtin_fmaf(p1[e], (float)vv[c][4 + e], o);
            }
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
    }
    float l = wave_sum(lrun);
    if (WPH > 1) {                                          // (all waves ended on the same maximum)
        po[wave][lane] = o;
        if (lane == 0) pl[wave] = l;
        __syncthreads();
        if (part != 0) return;
#pragma unroll
        for (int w = 1; w < WPH; ++w) { o += po[w][lane]; l += pl[w]; }
    }
    att[((size_t)m * rows + t0) * H + h * 64 + lane] = (bf16)(o / l);
}

// fp32 rows -> LayerNorm -> bf16 rows, one wave per row.  ADD: the rows are bare sums of a projection, bias and residual are
// added first (residual row r, or the token row cu[r]).
struct RowsAdd {
    size_t bias;                      // byte offset into a student slab
    const bf16* res;
    size_t r_ss;
    const int32_t* cu;                // null: residual row r
    int Tn;
};
// NC: chunks of 256 features, the last one perhaps half.  Everything that a row takes is requested at once, without a branch between the
// loads: one per chunk, in front of the chunk's sums and again of its scale and shift, made six memory round trips of one.
template <int NC, bool ADD>
__global__ __launch_bounds__(256) void rows_ln_kernel(const char* arena, size_t ss, size_t g_off, size_t b_off,
                                                      const float* __restrict__ u, size_t u_ss, RowsAdd add,
                                                      bf16* __restrict__ out, size_t o_ss, int M, int H, float eps)
{
    const int m = blockIdx.y, lane = threadIdx.x & 63, row = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (row >= M) return;
    const char* sb = arena + (size_t)m * ss;
    const float* ur = u + (size_t)m * u_ss + (size_t)row * H;
    const bf16* rr = ADD ? add.res + (size_t)m * add.r_ss + (size_t)(add.cu ? first_row(add.cu, row, add.Tn) : row) * H : nullptr;
    // (lanes behind the row's end: its last four features, which do not count)
    auto in_row = [&](int c) { return c + 1 < NC || 4 * (lane + 64 * c) < H; };
    auto el = [&](int c) { return in_row(c) ? 4 * (lane + 64 * c) : H - 4; };
    f32x4 v[NC], bias[NC], g[NC], b[NC];
    bf16x4 r[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c) {
        v[c] = *(const f32x4*)(ur + el(c));
        if (ADD) {
            bias[c] = *(const f32x4*)((const float*)(sb + add.bias) + el(c));
            r[c] = *(const bf16x4*)(rr + el(c));
        }
        g[c] = *(const f32x4*)((const float*)(sb + g_off) + el(c));
        b[c] = *(const f32x4*)((const float*)(sb + b_off) + el(c));
    }
    __builtin_amdgcn_sched_barrier(0);
    float s = 0.f;
#pragma unroll
    for (int c = 0; c < NC; ++c) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            if (ADD) v[c][e] = v[c][e] + bias[c][e] + (float)r[c][e];
            s += in_row(c) ? v[c][e] : 0.f;
        }
    }
    const float inv_h = __builtin_amdgcn_rcpf((float)H), mean = wave_sum(s) * inv_h;
    float q = 0.f;
#pragma unroll
    for (int c = 0; c < NC; ++c)
#pragma unroll
        for (int e = 0; e < 4; ++e) { const float d = in_row(c) ? v[c][e] - mean : 0.f; q += d * d; }
    const float inv = __builtin_amdgcn_rsqf(wave_sum(q) * inv_h + eps);
#pragma unroll
    for (int c = 0; c < NC; ++c) {
        bf16x4 o;
#pragma unroll
        for (int e = 0; e < 4; ++e) o[e] = (bf16)(g[c][e] * ((v[c][e] - mean) * inv) + b[c][e]);
        if (in_row(c)) *(bf16x4*)(out + (size_t)m * o_ss + (size_t)row * H + el(c)) = o;
    }
}

inline int up8(int v) { return (v + 7) & ~7; }

// Workgroups of a launch with a tile of 16 tm rows and n features.
inline long tile_count(int M, int N, int k, int tm, int n) { return (long)((M + 16 * tm - 1) / (16 * tm)) * (N / n) * k; }

template <int PRO, int EPI>
hipError_t launch_rows_ln(RowsLnArgs a, int k, hipStream_t s)
{
    a.nfb = a.N / 64;
    a.nfb8 = up8(a.nfb);
    a.nrb = (a.M + 15) / 16;
    const dim3 grid((unsigned)(a.nfb8 * a.nrb * k));
    // (an instance for every hidden width there is: multiples of 128 up to 1024)
#define SP_GO(NS) case 32 * NS: hipLaunchKernelGGL((rows_ln_gemm_kernel<PRO, EPI, NS>), grid, dim3(256), 0, s, a); break
    switch (a.H) {
        SP_GO(4); SP_GO(8); SP_GO(12); SP_GO(16); SP_GO(20); SP_GO(24); SP_GO(28); SP_GO(32);
        default: return hipErrorInvalidValue;
    }
#undef SP_GO
    return hipGetLastError();
}

// A wave's quarter of the reduction range has Kd / 128 steps of 32.  Up to eight (every hidden width): one pass of an instance of
// that length.  FFN depths: one pass of 24 steps, or of 32 where the rows are few enough for the registers; any other depth takes
// passes of 10, 12, 14 or 16 steps, whichever makes them cheapest: a pass costs a memory round trip, about six steps, and the
// steps that it has, the unused ones of the last pass among them.  Instances for listed depths only, and 16-step passes for all
// others, cost depth 640 three times its loads (four students, 200 rows, one launch: 19.9 us against 7.2 now).
template <bool F32OUT, int TM, int TF>
hipError_t launch_rows_k_tile(const RowsKArgs& a, dim3 grid, hipStream_t s)
{
#define SP_GO(NS, X) hipLaunchKernelGGL((rows_ksplit_kernel<F32OUT, TM, TF, NS, X>), grid, dim3(256), 0, s, a)
    const int steps = a.Kd / 128;
    switch (steps) {
        case 2: SP_GO(2, true); return hipGetLastError();
        case 4: SP_GO(4, true); return hipGetLastError();
        case 6: SP_GO(6, true); return hipGetLastError();
        case 8: SP_GO(8, true); return hipGetLastError();
        default: break;
    }
    if constexpr (F32OUT) {
        switch (steps) {
            case 1: SP_GO(1, true); return hipGetLastError();
            case 3: SP_GO(3, true); return hipGetLastError();
            case 5: SP_GO(5, true); return hipGetLastError();
            case 7: SP_GO(7, true); return hipGetLastError();
            default: break;
        }
        if (steps == 24) { SP_GO(24, true); return hipGetLastError(); }
        if constexpr (TM == 1)
            if (steps == 32) { SP_GO(32, true); return hipGetLastError(); }
        int best = 0, least = 0;
        for (int ns : {16, 14, 12, 10}) {
            const int cost = (steps + ns - 1) / ns * (ns + 6);
            if (!best || cost < least) { best = ns; least = cost; }
        }
        switch (best) {
            case 10: SP_GO(10, false); break;
            case 12: SP_GO(12, false); break;
            case 14: SP_GO(14, false); break;
            default: SP_GO(16, false); break;
        }
        return hipGetLastError();
    }
#undef SP_GO
    return hipErrorInvalidValue;                            // (bf16 outputs: the value projection, as deep as the folded attention's widths)
}

template <bool F32OUT>
hipError_t launch_rows_k(RowsKArgs a, int k, hipStream_t s)
{
    // the smallest tile whose grid the chip takes at once: about a workgroup per compute unit with a deep reduction (eight
    // students, 64 rows, depth 3072: tile 1 x 1 16.7 us, 1 x 2 14.1, 4 x 2 12.4), else three (depth 768: 9.3, 6.6, 8.0)
    const long most = a.Kd > 1024 ? 256 : 768;
    int tm = 1, tf = 1;
    if (tile_count(a.M, a.N, k, tm, 16 * tf) > most) tf = 2;
    if (tile_count(a.M, a.N, k, tm, 16 * tf) > most && a.M > 16) tm = 2;
    if (tile_count(a.M, a.N, k, tm, 16 * tf) > most && a.M > 32) tm = 4;
    a.nfb = a.N / (16 * tf);
    a.nfb8 = up8(a.nfb);
    a.nrb = (a.M + 16 * tm - 1) / (16 * tm);
    const dim3 grid((unsigned)(a.nfb8 * a.nrb * k));
    if (tm == 1 && tf == 1) return launch_rows_k_tile<F32OUT, 1, 1>(a, grid, s);
    if (tm == 1) return launch_rows_k_tile<F32OUT, 1, 2>(a, grid, s);
    if (tm == 2) return launch_rows_k_tile<F32OUT, 2, 2>(a, grid, s);
    return launch_rows_k_tile<F32OUT, 4, 2>(a, grid, s);
}

template <int NS, bool SCALED>
hipError_t launch_fold(const FoldQArgs& a, int k, hipStream_t s)
{
    constexpr size_t smem = fold_query_smem(NS, SCALED);
    auto kern = fold_query_kernel<NS, SCALED>;
    if (smem > 48 * 1024) {
        static std::atomic<bool> raised{false};             // per instantiation; the attribute is sticky for the process
        if (!raised.load(std::memory_order_acquire)) {
            const hipError_t e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
            if (e != hipSuccess) return e;
            raised.store(true, std::memory_order_release);
        }
    }
    hipLaunchKernelGGL(kern, dim3((unsigned)(a.heads8 * a.nrb * k)), dim3(256), smem, s, a);
    return hipGetLastError();
}

RowsLnArgs ln_args(const sp_model* M, size_t w, size_t b, size_t g, size_t beta)
{
    RowsLnArgs a{};
    a.arena = M->arena; a.ss = M->L.student_stride; a.w = w; a.b = b; a.g = g; a.beta = beta; a.eps = M->cfg.ln_eps;
    a.H = M->cfg.hidden;
    return a;
}

}  // namespace

hipError_t launch_rows_qkv(const sp_model* M, size_t lo, const float* u, size_t u_ss, size_t g_off, size_t b_off,
                           const int32_t* ids, const int32_t* cu, int B, int T, void* x, void* qkv, void* vt, int rows,
                           int k, hipStream_t s)
{
    const sp_config& c = M->cfg;
    if (!bf16_path(c) || T > rows || rows % 64) return hipErrorInvalidValue;
    const int H = c.hidden;
    RowsLnArgs a = ln_args(M, lo + M->L.wqkv, lo + M->L.bqkv, g_off, b_off);
    a.u = u; a.u_ss = u_ss; a.ids = ids; a.cu = cu; a.tok = M->L.tok; a.pos = M->L.pos; a.B = B; a.V = c.vocab; a.P = c.max_pos;
    a.xout = (bf16*)x; a.x_ss = (size_t)rows * H;
    a.out = qkv; a.o_ss = (size_t)rows * 3 * H; a.ol = rows_layout(3 * H);
    a.out2 = (bf16*)vt; a.o2_ss = (size_t)rows * H; a.ld2 = rows; a.n_split = 2 * H;
    a.M = T; a.N = 3 * H;
    return u ? launch_rows_ln<PRO_LN, EPI_QKV>(a, k, s) : launch_rows_ln<PRO_EMBED, EPI_QKV>(a, k, s);
}

hipError_t launch_rows_ffn_up(const sp_model* M, size_t lo, const float* u, size_t u_ss, int nrows, void* x1, size_t x1_ss,
                              void* g, size_t g_ss, RowsLayout gl, int k, hipStream_t s)
{
    const sp_config& c = M->cfg;
    if (!bf16_path(c) || nrows < 1) return hipErrorInvalidValue;
    RowsLnArgs a = ln_args(M, lo + M->L.w1, lo + M->L.b1, lo + M->L.ln1g, lo + M->L.ln1b);
    a.u = u; a.u_ss = u_ss;
    a.xout = (bf16*)x1; a.x_ss = x1_ss;
    a.out = g; a.o_ss = g_ss; a.ol = gl;
    a.M = nrows; a.N = c.ffn;
    return launch_rows_ln<PRO_LN, EPI_BIAS_GELU>(a, k, s);
}

hipError_t launch_rows_pooler(const sp_model* M, size_t lo, const float* u, size_t u_ss, int nrows, float* zpart, int k,
                              hipStream_t s)
{
    const sp_config& c = M->cfg;
    if (!bf16_path(c) || nrows < 1 || c.classes > kMaxClasses) return hipErrorInvalidValue;
    RowsLnArgs a = ln_args(M, M->L.wp_t, M->L.bp, lo + M->L.ln2g, lo + M->L.ln2b);
    a.u = u; a.u_ss = u_ss;
    a.out = zpart; a.wc = M->L.wc; a.C = c.classes;
    a.M = nrows; a.N = c.hidden;
    return launch_rows_ln<PRO_LN, EPI_BIAS_TANH>(a, k, s);
}

hipError_t launch_rows_residual(const sp_model* M, size_t w_off, size_t b_off, const bf16* A, size_t a_ss, RowsLayout al,
                                int Kd, bool a_first, const bf16* res, size_t r_ss, bool r_first, float* out, size_t o_ss,
                                const int32_t* cu, int T, int nrows, int k, hipStream_t s)
{
    const sp_config& c = M->cfg;
    if (!bf16_path(c) || nrows < 1 || Kd % 128) return hipErrorInvalidValue;
    RowsKArgs a{};
    a.arena = M->arena; a.ss = M->L.student_stride; a.w = w_off; a.b = b_off;
    a.A = A; a.a_ss = a_ss; a.al = al; a.a_first = a_first;
    a.res = res; a.r_ss = r_ss; a.ldr = c.hidden; a.r_first = r_first;
    a.out = out; a.o_ss = o_ss; a.ldo = c.hidden;
    a.cu = cu; a.Tn = T; a.M = nrows; a.N = c.hidden; a.Kd = Kd;
    return launch_rows_k<true>(a, k, s);
}

hipError_t launch_rows_head_values(const sp_model* M, size_t lo, const void* xbar, size_t xb_ss, void* att, size_t att_ss,
                                   int nrows, int k, hipStream_t s)
{
    const sp_config& c = M->cfg;
    if (!bf16_path(c) || nrows < 1) return hipErrorInvalidValue;
    const int H = c.hidden;
    RowsKArgs a{};
    a.arena = M->arena; a.ss = M->L.student_stride;
    a.w = lo + M->L.wqkv + (size_t)2 * H * H * 2; a.b = lo + M->L.bqkv + (size_t)2 * H * 4;
    a.A = (const bf16*)xbar; a.a_ss = xb_ss; a.al = rows_layout(c.heads * H); a.a_hs = H;
    a.out = att; a.o_ss = att_ss; a.ldo = H;
    a.M = nrows; a.N = H; a.Kd = H;
    return launch_rows_k<false>(a, k, s);
}

hipError_t launch_fold_query(const sp_model* M, size_t lo, const void* x, int rows, const int32_t* cu, int T, int B,
                             void* q, size_t q_ss, void* qt, size_t qt_ss, int k, hipStream_t s, bool scaled, size_t g_off)
{
    const sp_config& c = M->cfg;
    if (!bf16_path(c) || c.heads * 64 != c.hidden || B < 1) return hipErrorInvalidValue;
    FoldQArgs a{};
    a.g = g_off;
    a.arena = M->arena; a.ss = M->L.student_stride; a.wq = lo + M->L.wqkv; a.bq = lo + M->L.bqkv; a.wk = lo + M->L.wk_io;
    a.x = (const bf16*)x; a.x_ss = (size_t)rows * c.hidden; a.cu = cu;
    a.q = (bf16*)q; a.q_ss = q_ss; a.qt = (bf16*)qt; a.qt_ss = qt_ss;
    a.Tn = T; a.M = B; a.H = c.hidden; a.heads = c.heads; a.heads8 = up8(c.heads);
    // (one workgroup per compute unit: the fewest blocks per workgroup that need no second round)
    const int blocks = (B + 15) / 16, groups = 256 / (c.heads * k) < 1 ? 1 : 256 / (c.heads * k);
    a.rpw = (blocks + groups - 1) / groups;
    a.nrb = (blocks + a.rpw - 1) / a.rpw;
    switch (a.H) {                                          // (the folded attention's widths)
        case 256: return scaled ? launch_fold<8, true>(a, k, s) : launch_fold<8, false>(a, k, s);
        case 512: return scaled ? launch_fold<16, true>(a, k, s) : launch_fold<16, false>(a, k, s);
        case 768: return scaled ? launch_fold<24, true>(a, k, s) : launch_fold<24, false>(a, k, s);
        case 1024: return scaled ? launch_fold<32, true>(a, k, s) : launch_fold<32, false>(a, k, s);
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_attention_first(const sp_model* M, const void* qkv, const void* vt, void* att, const int32_t* cu, int B,
                                  int T, int max_seqlen, int rows, int k, hipStream_t s)
{
    const sp_config& c = M->cfg;
    if (!bf16_path(c) || c.heads * 64 != c.hidden) return hipErrorInvalidValue;
    const int items = B * c.heads;
    // (57: a sequence of up to 57 tokens fits one step of 64 slots wherever it starts)
    if (max_seqlen <= 57)
        hipLaunchKernelGGL(attention_first_kernel<1>, dim3((unsigned)((items + 3) / 4), k), dim3(256), 0, s, (const bf16*)qkv,
                           (const bf16*)vt, (bf16*)att, cu, B, T, rows, c.hidden, c.heads, max_seqlen);
    else
        hipLaunchKernelGGL(attention_first_kernel<4>, dim3((unsigned)items, k), dim3(256), 0, s, (const bf16*)qkv,
                           (const bf16*)vt, (bf16*)att, cu, B, T, rows, c.hidden, c.heads, max_seqlen);
    return hipGetLastError();
}

namespace {
template <bool ADD>
hipError_t launch_rows_ln_any(const sp_model* M, size_t g_off, size_t b_off, const float* u, size_t u_ss, const RowsAdd& add,
                              void* out, size_t o_ss, int nrows, int k, hipStream_t s)
{
    const sp_config& c = M->cfg;
    if (!bf16_path(c) || nrows < 1) return hipErrorInvalidValue;
    const dim3 grid((unsigned)((nrows + 3) / 4), (unsigned)k);
#define SP_GO(NC) case NC: hipLaunchKernelGGL((rows_ln_kernel<NC, ADD>), grid, dim3(256), 0, s, M->arena, M->L.student_stride, g_off, \
                                       b_off, u, u_ss, add, (bf16*)out, o_ss, nrows, c.hidden, c.ln_eps); break
    switch ((c.hidden + 255) / 256) {
        SP_GO(1); SP_GO(2); SP_GO(3); SP_GO(4);
        default: return hipErrorInvalidValue;
    }
#undef SP_GO
    return hipGetLastError();
}
}  // namespace

hipError_t launch_rows_ln_out(const sp_model* M, size_t g_off, size_t b_off, const float* u, size_t u_ss, void* out,
                              size_t o_ss, int nrows, int k, hipStream_t s)
{
    return launch_rows_ln_any<false>(M, g_off, b_off, u, u_ss, RowsAdd{}, out, o_ss, nrows, k, s);
}

hipError_t launch_rows_ln_add(const sp_model* M, size_t g_off, size_t b_off, const float* u, size_t u_ss, size_t bias_off,
                              const void* res, size_t r_ss, const int32_t* cu, int T, void* out, size_t o_ss, int nrows, int k,
                              hipStream_t s)
{
    return launch_rows_ln_any<true>(M, g_off, b_off, u, u_ss, RowsAdd{bias_off, (const bf16*)res, r_ss, cu, T}, out, o_ss, nrows,
                                    k, s);
}

}  // namespace sp
