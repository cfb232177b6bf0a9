// Student-grouped projections on fp8 (e4m3) operands for large calls of quantised students:
//   out[m] = epilogue((A8[m] . W8[m]^T) * (sw[m][n] / qa) + bias[m][n])
// A8 are activations quantised by their producer as e4m3(value * qa) (one power-of-two scale per tensor), W8 the
// weights quantised at load per output feature n as e4m3(W[n][:] / sw[n]); the products are accumulated in fp32
// by v_mfma_f32_32x32x64_f8f6f4 (both block scales 1).
//
// The bf16 kernel's plan on eight-bit operands: tile 32 TM tokens x 256 features, four waves, each with all the tile's
// tokens and 64 features of its own, two workgroups per compute unit (one's first loads, epilogue arithmetic and stores
// run while the other multiplies).  A matrix instruction consumes 64 reduction elements, 32 bytes per lane: the 16-byte
// chunks 2 g and 2 g + 1 of the step for lane half g; both operands use the same map, so the order inside the reduction is
// immaterial.
//   * weights: from memory straight to the registers of the one wave that uses them, in operand blocks (see ArenaLayout: a
//     load is 1 KB in a row); a step's registers are requested again, for the next k-tile of 128 reduction elements, as soon as
//     its matrix instructions are issued;
//   * activations: by direct-to-LDS loads into one of three stages (rows of eight 16-byte slots; slot s of row r holds chunk
//     s ^ ((r >> 1) & 7): no bank conflicts), requested two k-tiles ahead.  Fragments have one register set: a block of 32
//     tokens is read for the next step as soon as its two matrix instructions are issued (2 (TM - 1) instructions of 64 cycles
//     to arrive), so the barrier of a k-tile sits behind the first block of its second step.
// Bytes per matrix-core cycle are those of the bf16 kernel: 48 from the L2, 80 from and to the LDS at 128 tokens.
#include <atomic>
#include <type_traits>

#include "sp_internal.h"

namespace sp {

namespace {

typedef int v8i __attribute__((ext_vector_type(8)));
typedef int v4i __attribute__((ext_vector_type(4)));

struct Fp8Args {
    const unsigned char* A;
    size_t a_ss;                      // student strides: elements of their tensors
    const char* arena;
    size_t ss, w_off, s_off, b_off;
    float inv_qa, q_out;
    void* out;
    size_t o_ss;
    const bf16* res;
    size_t r_ss;
    bf16* out2;
    size_t o2_ss;
    int lda, ldo, ldr, ld2, n_split, Kd, mrows, mtiles, ntiles, total, mb;
};

constexpr int F8_NW = 4, F8_BN = 64 * F8_NW;                // waves; features of a tile
// three activation stages or the staged output tile, then scales and biases of the tile's features
constexpr size_t fp8_tile_bytes(int tm) { return (size_t)32 * tm * 128 * F8_NW; }
constexpr size_t fp8_smem_bytes(int tm) { return fp8_tile_bytes(tm) + 2 * F8_BN * sizeof(float); }

template <int TM, int EPI>
__global__ __launch_bounds__(256, 2) void gemm_fp8_kernel(Fp8Args p)
{
    constexpr int BM = 32 * TM, NA = TM;                    // NA: wave-loads (eight rows) of an activation k-tile per wave
    constexpr int STAGE = BM * 8;                           // 16-byte units
    constexpr int TKEY = TM == 3 ? 3 : TM * 4 - 1;          // swizzle of the transposed staging: bits of the chunk
    extern __shared__ uint4 smem[];
    float* coef = (float*)((char*)smem + fp8_tile_bytes(TM));   // [scales | biases] of the tile's features
    const int chunk = (p.total + 7) >> 3;
    const int lin = (int)(blockIdx.x & 7) * chunk + (int)(blockIdx.x >> 3);
    if ((int)(blockIdx.x >> 3) >= chunk || lin >= p.total) return;
    const int tiles = p.ntiles * p.mtiles, tl = lin % tiles, m = lin / tiles;
    const int gi = tl / (p.mb * p.ntiles), rb = tl - gi * p.mb * p.ntiles;
    const int mbe = p.mtiles - gi * p.mb < p.mb ? p.mtiles - gi * p.mb : p.mb;
    const int nt = rb / mbe, mt = gi * p.mb + rb % mbe;
    const int m0 = mt * BM, n0 = nt * F8_BN;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int j31 = lane & 31, g = lane >> 5, nf = n0 + 64 * wave;
    const char* sb = p.arena + (size_t)m * p.ss;
    const int Kd = p.Kd, nk = Kd >> 7;

    // activations: wave-load i of a k-tile is rows 8 (wave + 4 i) .. + 7, lane -> (row lane / 8, slot lane % 8), which holds chunk
    // slot ^ ((row >> 1) & 7); rows beyond mrows repeat the last one (64-bit base of the tile, 32-bit offsets inside it: a buffer may hold
    // more than 2^32 elements)
    const unsigned char* Ag = p.A + (size_t)m * p.a_ss + (size_t)m0 * p.lda;
    int aoff[NA];
#pragma unroll
    for (int i = 0; i < NA; ++i) {
        const int r = 8 * (wave + F8_NW * i) + (lane >> 3);
        const int rr = m0 + r < p.mrows ? r : p.mrows - 1 - m0;
        aoff[i] = rr * p.lda + ((lane & 7) ^ ((r >> 1) & 7)) * 16;
    }
    // weights: operand blocks of 32 features x 64 reduction elements, 2 KB, lane after lane in both halves
    const char* Wg = sb + p.w_off + (size_t)nf * Kd;
    const int wlane = lane * 16;

    v8i w[2][2], fx[TM];
    auto dma_a = [&](int kt, int stage) {
#pragma unroll
        for (int i = 0; i < NA; ++i) load_lds16(Ag, (lds_void*)(smem + stage * STAGE + (wave + F8_NW * i) * 64), aoff[i], kt * 128);
    };
    auto load_w = [&](int kt, int s) {
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int at = i * 32 * Kd + (2 * kt + s) * 2048;
            w[s][i] = __builtin_shufflevector(__builtin_bit_cast(v4i, load16(Wg, wlane, at)), __builtin_bit_cast(v4i, load16(Wg, wlane + 1024, at)), 0, 1, 2, 3, 4, 5, 6, 7);
        }
    };
    const int xrow = j31 * 8, xkey = (j31 >> 1) & 7;
    auto frag = [&](int stage, int s, int t) {
        const v4i* base = (const v4i*)(smem + stage * STAGE + t * 256 + xrow);
        return __builtin_shufflevector(base[(4 * s + 2 * g) ^ xkey], base[(4 * s + 2 * g + 1) ^ xkey], 0, 1, 2, 3, 4, 5, 6, 7);
    };

    f32x16 acc[2][TM];
    dma_a(0, 0);
    const float scale = ((const float*)(sb + p.s_off))[n0 + tid], bias = ((const float*)(sb + p.b_off))[n0 + tid];
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int s = 0; s < 2; ++s) load_w(0, s);
    __builtin_amdgcn_sched_barrier(0);
    dma_a(1, 1);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int t = 0; t < TM; ++t)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[i][t][e] = 0.f;
    {
        // (GELU: the output scale rides in the factors)
        const float q = EPI == EPI_BIAS_GELU ? p.q_out : 1.f;
        coef[tid] = scale * (p.inv_qa * q);
        coef[F8_BN + tid] = bias * q;
    }
    __builtin_amdgcn_sched_barrier(0);
    wait_vmcnt<8 + NA>();                                   // activations of k-tile 0
    barrier_lds();
#pragma unroll
    for (int t = 0; t < TM; ++t) fx[t] = frag(0, 0, t);

    // One k-tile, j.  Requested during it: the weights of k-tile j + 1 (NEXT), a step's when its registers are free, and the activations of
    // k-tile j + 2 (AL) in the stage that k-tile j - 1 has left: its last fragments were in registers at the barrier of that k-tile.  V: loads
    // that may be in flight when the activations of k-tile j + 1 have to be there, those requested behind them.
    int prev = 2, cur = 0, next = 1;                        // stages of k-tiles j - 1, j and j + 1
    auto ktile = [&](int j, auto next_c, auto a_c, auto v_c) {
        constexpr bool NEXT = decltype(next_c)::value, AL = decltype(a_c)::value;
#pragma unroll
        for (int s = 0; s < 2; ++s) {
#pragma unroll
            for (int t = 0; t < TM; ++t) {
#pragma unroll
                for (int i = 0; i < 2; ++i)
                    acc[i][t] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(w[s][i], fx[t], acc[i][t], 0, 0, 0, 0x7f7f7f7f, 0, 0x7f7f7f7f);
                __builtin_amdgcn_sched_barrier(0);
                if (s == 1 && t == 0 && NEXT) {
                    wait_vmcnt<decltype(v_c)::value>();
                    barrier_lds();
                }
                if (s == 0) fx[t] = frag(cur, 1, t);
                else if (NEXT) fx[t] = frag(next, 0, t);
                if (s == 0 && t == 0 && AL) dma_a(j + 2, prev);
                __builtin_amdgcn_sched_barrier(0);
            }
            if (NEXT) load_w(j + 1, s);
            __builtin_amdgcn_sched_barrier(0);
        }
        prev = cur;
        cur = next;
        next = next == 2 ? 0 : next + 1;
    };
    constexpr std::true_type Y{};
    constexpr std::false_type N{};
    constexpr std::integral_constant<int, 8 + NA + 4> V{};  // both steps' weights, activations and weights of a step since
    int j = 0;
    if (nk > 2) {                                           // (nk is even)
        ktile(0, Y, Y, std::integral_constant<int, NA + 4>{});
        ktile(1, Y, Y, V);
        for (j = 2; j + 2 < nk; j += 2) {
            ktile(j, Y, Y, V);
            ktile(j + 1, Y, Y, V);
        }
    }
    ktile(j, Y, N, std::integral_constant<int, 4>{});
    ktile(j + 1, N, N, V);

    // ---- epilogue: accumulator element v of lane l in block (i, t): token 32 t + l % 32, feature 32 i + 8 (v / 4) +
    // 4 (l / 32) + v % 4.
    barrier_lds();                                          // everybody has read the last activations
    f32x4 sc, bs;                                           // of the four features at hand
    auto coefficients = [&](int i, int v4) {
        __builtin_amdgcn_sched_barrier(0);                  // (all features' at once would not fit the registers)
        const int f = 64 * wave + 32 * i + 8 * v4 + 4 * g;
        sc = *(const f32x4*)(coef + f);
        bs = *(const f32x4*)(coef + F8_BN + f);
    };
    auto values = [&](int i, int t, int v4, float (&r)[4]) {
#pragma unroll
        for (int e = 0; e < 4; ++e) r[e] = __builtin_fmaf(acc[i][t][4 * v4 + e], sc[e], bs[e]);
    };
    if (EPI == EPI_BIAS_GELU) {
        // fp8 output, e4m3(gelu(.) * q_out), staged by all waves together as [tokens][256 bytes], chunk (feature / 16) ^
        // (token & 15), so that rows leave in whole 256-byte pieces.  The fit's coefficients are scaled as the values are.
        const float iq = 1.0f / p.q_out;
        const float k0 = kGeluQ8C0 * iq, k1 = kGeluQ8C1 * iq * iq, k2 = kGeluQ8C2 * iq * iq * iq;
        char* stg = (char*)smem;
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int v4 = 0; v4 < 4; ++v4) {
                coefficients(i, v4);
#pragma unroll
                for (int t = 0; t < TM; ++t) {
                    const int f = 64 * wave + 32 * i + 8 * v4 + 4 * g, tok = t * 32 + j31;
                    float r[4];
                    values(i, t, v4, r);
#pragma unroll
                    for (int e = 0; e < 4; ++e) r[e] = gelu_erf_q8_scaled(r[e], k0, k1, k2);
                    int c = 0;
                    c = __builtin_amdgcn_cvt_pk_fp8_f32(r[0], r[1], c, false);
                    c = __builtin_amdgcn_cvt_pk_fp8_f32(r[2], r[3], c, true);
                    *(int*)(stg + tok * 256 + (((f >> 4) ^ (tok & 15)) << 4) + (f & 15)) = c;
                }
            }
        barrier_lds();
        unsigned char* dst = (unsigned char*)p.out + (size_t)m * p.o_ss + n0;
        const int rr = tid >> 4, cc = tid & 15;
#pragma unroll
        for (int q = 0; q < BM / 16; ++q) {
            const int r = q * 16 + rr, row = m0 + r;
            if (row < p.mrows) *(uint4*)(dst + (size_t)row * p.ldo + cc * 16) = *(const uint4*)(stg + r * 256 + ((cc ^ (r & 15)) << 4));
        }
        return;
    }

    // bf16 output: each wave stages its tile in its own slice and stores whole row segments
    char* stg = (char*)smem + (size_t)wave * BM * 128;
    if (EPI == EPI_QKV && n0 >= p.n_split) {                // values: rows are features, 2 BM bytes each
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int v4 = 0; v4 < 4; ++v4) {
                coefficients(i, v4);
                const int f = i * 32 + 8 * v4 + 4 * g;
#pragma unroll
                for (int t = 0; t < TM; ++t) {
                    const int tok = t * 32 + j31;
                    float r[4];
                    values(i, t, v4, r);
                    char* c = stg + f * (BM * 2) + (((tok >> 3) ^ (f >> 2 & TKEY)) << 4) + (tok & 7) * 2;
#pragma unroll
                    for (int e = 0; e < 4; ++e) *(bf16*)(c + e * (BM * 2)) = (bf16)r[e];
                }
            }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        constexpr int CPR = TM * 4, RPI = 64 / CPR;         // chunks per feature row, rows per instruction
        const int fr = lane / CPR, fc = lane % CPR;
        bf16* dst = p.out2 + (size_t)m * p.o2_ss + (size_t)(nf - p.n_split) * p.ld2 + m0 + fc * 8;
        if (fr < RPI && m0 + fc * 8 < p.mrows)
#pragma unroll 4
            for (int f = fr; f < 64; f += RPI)
                *(uint4*)(dst + (size_t)f * p.ld2) = *(const uint4*)(stg + f * (BM * 2) + ((fc ^ (f >> 2 & TKEY)) << 4));
        return;
    }
    const int rr = lane >> 3, cc = lane & 7;
    if (EPI == EPI_BIAS_RESIDUAL) {
        const bf16* rg = p.res + (size_t)m * p.r_ss + nf;
#pragma unroll
        for (int q = 0; q < BM / 8; ++q) {
            const int r = q * 8 + rr, row = m0 + r < p.mrows ? m0 + r : p.mrows - 1;
            __builtin_amdgcn_global_load_lds((gbl_void*)(rg + (size_t)row * p.ldr + (cc ^ ((r >> 1) & 7)) * 8),
                                             (lds_void*)(stg + q * 1024), 16, 0, 0);
        }
        wait_vmcnt<0>();
    }
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int v4 = 0; v4 < 4; ++v4) {
            coefficients(i, v4);
#pragma unroll
            for (int t = 0; t < TM; ++t) {
                const int f = i * 32 + 8 * v4 + 4 * g, tok = t * 32 + j31;
                float r[4];
                values(i, t, v4, r);
                char* c = stg + tok * 128 + (((f >> 3) ^ ((tok >> 1) & 7)) << 4) + (f & 7) * 2;
                if (EPI == EPI_BIAS_RESIDUAL) {
                    const bf16x4 x4 = *(const bf16x4*)c;
#pragma unroll
                    for (int e = 0; e < 4; ++e) r[e] += (float)x4[e];
                }
                bf16x4 o4;
#pragma unroll
                for (int e = 0; e < 4; ++e) o4[e] = (bf16)r[e];
                *(bf16x4*)c = o4;
            }
        }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    bf16* dst = (bf16*)p.out + (size_t)m * p.o_ss + nf + cc * 8;
#pragma unroll 4
    for (int q = 0; q < BM / 8; ++q) {
        const int r = q * 8 + rr, row = m0 + r;
        if (row < p.mrows) *(uint4*)(dst + (size_t)row * p.ldo) = *(const uint4*)(stg + r * 128 + ((cc ^ ((r >> 1) & 7)) << 4));
    }
}

template <int TM, int EPI>
hipError_t launch_fp8_tile(Fp8Args a, int N, int k, hipStream_t s)
{
    constexpr size_t smem = fp8_smem_bytes(TM);
    auto kern = gemm_fp8_kernel<TM, EPI>;
    if (smem > 48 * 1024) {
        static std::atomic<bool> raised{false};             // per instantiation; the attribute is sticky for the process
        if (!raised.load(std::memory_order_acquire)) {
            hipError_t e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
            if (e != hipSuccess) return e;
            raised.store(true, std::memory_order_release);
        }
    }
    a.mtiles = (a.mrows + 32 * TM - 1) / (32 * TM);
    a.ntiles = N / F8_BN;
    a.total = k * a.mtiles * a.ntiles;
    a.mb = 32 / TM;                                         // (about a thousand tokens, as in the bf16 kernel)
    hipLaunchKernelGGL(kern, dim3((unsigned)((a.total + 7) / 8 * 8)), dim3(64 * F8_NW), smem, s, a);
    return hipGetLastError();
}

// Tile height.  A depth of 256 is two k-tiles: low tiles hide the first loads and the epilogue better, as in the bf16 kernel, whose costs
// are good here as well; deeper reductions have costs of their own.  us a call on 14653 tokens, the costs of a bf16 projection half as
// deep / these: 512 wide, eight students 896 / 850, four 467 / 452, two 271 / 264, one 162 / 163; 768 wide, four 774 / 766; 1024 wide, two 605 / 590,
// the others within 1 %.  At a depth of 256, bf16's / these: eight 402 / 409, two 151 / 155.  us per launch at 128 / 96 / 64 tokens, eight
// students: q|k|v from 256 56 / 58 / 59, from 512 133 / 143 / 147, from 768 238 / 247 / 262; FFN up from 256 68 / 67 / 61, from 512 172 / 163 / 167, from
// 768 299 / 305 / 310; FFN down from 1024 58 / 61 / 62, from 2048 162 / 163 / 192, from 3072 270 / 298 / 346.
constexpr double kFp8TokenCost[5] = {0, 1.7, 1.2, 1.1, 1.0};

template <int EPI>
hipError_t launch_fp8(const Fp8Args& a, int N, int k, hipStream_t s)
{
    switch (gemm_tile_height(a.mrows, N, k, a.Kd <= 256 ? gemm_token_cost(a.Kd) : kFp8TokenCost)) {
        case 1: return launch_fp8_tile<1, EPI>(a, N, k, s);
        case 2: return launch_fp8_tile<2, EPI>(a, N, k, s);
        case 3: return launch_fp8_tile<3, EPI>(a, N, k, s);
        default: return launch_fp8_tile<4, EPI>(a, N, k, s);
    }
}

// y[i] = the GELU of the fp8 epilogue evaluated on x[i], before the scaling and the rounding to e4m3 (test aid)
__global__ void gelu_q8_probe_kernel(const float* __restrict__ x, float* __restrict__ y, long n)
{
    const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) y[i] = gelu_erf_q8(x[i]);
}

}  // namespace

hipError_t launch_gelu_q8_probe(const float* x, float* y, long n, hipStream_t s)
{
    if (n < 1) return hipErrorInvalidValue;
    hipLaunchKernelGGL(gelu_q8_probe_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, x, y, n);
    return hipGetLastError();
}

hipError_t launch_gemm_fp8(const sp_model* M, const void* A8, int lda, size_t w_off, size_t s_off, size_t b_off,
                           float a_qscale, void* out, int ldo, const void* residual, int ldr, int mrows, int N, int Kd,
                           int k, Epilogue epi, size_t a_student_stride, size_t o_student_stride,
                           size_t r_student_stride, hipStream_t s, void* out2, int n_split, int ld2,
                           size_t o2_student_stride, float out_qscale)
{
    if (M->cfg.dtype != SP_DTYPE_FP8 || mrows < 64 || mrows % 64 || N % 256 || Kd < 256 || Kd % 256 || lda % 16 || !(a_qscale > 0.f))
        return hipErrorInvalidValue;
    if (epi == EPI_BIAS_RESIDUAL && !residual) return hipErrorInvalidValue;
    if (epi == EPI_QKV && (!out2 || n_split % 256 || ld2 % 8)) return hipErrorInvalidValue;
    const size_t osz = epi == EPI_BIAS_GELU ? 1 : 2;        // bytes per output element
    const Fp8Args a{(const unsigned char*)A8, a_student_stride, M->arena, M->L.student_stride, w_off, s_off, b_off, 1.0f / a_qscale,
                    out_qscale, out, o_student_stride / osz, (const bf16*)residual, r_student_stride / 2, (bf16*)out2,
                    o2_student_stride / 2, lda, ldo, ldr, ld2, n_split, Kd, mrows, 0, 0, 0, 0};
    switch (epi) {
        case EPI_QKV: return launch_fp8<EPI_QKV>(a, N, k, s);
        case EPI_BIAS_GELU: return launch_fp8<EPI_BIAS_GELU>(a, N, k, s);
        case EPI_BIAS_RESIDUAL: return launch_fp8<EPI_BIAS_RESIDUAL>(a, N, k, s);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace sp
