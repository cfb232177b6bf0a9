// Student-grouped projections: out[m] = epilogue(A[m] . W[m]^T + bias[m]) for every active
// student m.  The bf16 kernel runs on the matrix cores (v_mfma_f32_32x32x16_bf16, fp32
// accumulate); the fp32 kernel is a plain FMA tile kernel used by the fp32 path.
#include <atomic>
#include <type_traits>

#include "sp_internal.h"

namespace sp {

namespace {

__device__ inline float gelu_erf(float u) { return 0.5f * u * (1.0f + erff(u * 0.70710678118654752f)); }

// -------------------------------------------------------------------------------------
// bf16 MFMA kernel with the weights in registers (v_mfma_f32_32x32x16_bf16): tile 32 TM tokens x 64 NW features, NW waves,
// each with all the tile's tokens and 64 features of its own; two workgroups per compute unit.  D: k-tiles of weights in flight.
//
// Operand roles are swapped with respect to the textbook picture: the weights are the MFMA "A" operand (rows = output
// features) and the activations the "B" operand (columns = tokens), so a lane of the 32x32 accumulator owns one token and
// runs of four consecutive features.
//   * weights: a feature's weights are used by one wave only, so they go from memory straight to its registers, in operand
//     blocks (see ArenaLayout: a load is 256-byte runs).  A step's registers are requested again, for the next k-tile of 64
//     reduction elements (D = 2: the one after), as soon as its matrix instructions are issued: four steps (1024 matrix-core
//     cycles at 128 tokens) to arrive, twice that while the other workgroup has the matrix cores.  Buffer loads as well: one register of
//     address.
//   * activations: by direct-to-LDS loads into one of D + 2 stages (rows of eight 16-byte slots; slot s of row r holds chunk
//     s ^ ((r >> 1) & 7): no bank conflicts), requested D + 1 k-tiles ahead, one barrier per k-tile, in front of which a wave waits for
//     its own share of the next one.  In their buffer form (load_lds16) they can be mixed with loads to registers.  A k-tile's are
//     requested together: spread over its steps, the workgroups that share a row fetch it from beyond the L2 more often (FFN down of
//     eight students of 768, 14653 tokens: 1070 MB and 510 us, together 482).  Through registers they held sixteen more and cost
//     the LDS writes: us at hidden 1024, 18387 tokens, six students, before / this: q|k|v 634 / 611, attention output 240 / 236, FFN up 835 / 810,
//     FFN down 770 / 744; eight of 768 on 14653 tokens 391 / 380, 161 / 158, 546 / 532, 481 / 482.  (Two k-tiles of weights in flight at 128
//     tokens, requested step by step or together: no gain; another 32 registers.  256 x 256 tiles of eight waves whose halves share the weights through
//     the L1: 652 / 266 / 958 / 780 on the first; 128 x 512: 624 / 249 / 903 / 736, and worse for fewer tokens.)
//   * per matrix-core cycle at the full rate and 128 tokens a compute unit needs 48 bytes from the L2 (52-60 is what the load
//     path delivers) and 80 from and to the LDS (of 128).  With both operands through LDS a 128 x 128 tile needs 192: that kernel
//     stopped at half of this one's rate.
//   * two workgroups per compute unit (three of 96 tokens): one's first loads, epilogue arithmetic and stores run while the other multiplies.  (One
//     workgroup with a 256 x 256 tile and a five-slot LDS ring moves a third less through the load path but leaves the
//     matrix cores idle for 44 % of a tile at depth 768.)
//   * epilogue through LDS: each wave stages its tile in its own slice and stores whole 16-byte-per-lane row segments; the
//     residual rows arrive there by direct-to-LDS loads.
// What bounds large launches (eight students of 768, 14.7 k tokens): the wait for operands first (matrix cores 52-57 % busy, waves waiting 47-59 %
// of their time, address units 69-83 % busy), then the package power limit (1.85-2.1 GHz of 2.4; on operands that are all zero a launch takes
// 8-20 % less, and the same loop without its loads runs at 1.8 PFLOP/s).
// -------------------------------------------------------------------------------------
struct GemmArgs {
    const bf16* A;
    size_t a_ss;
    const char* arena;
    size_t ss, w_off, b_off;
    bf16* out;
    size_t o_ss;
    const bf16* res;
    size_t r_ss;
    bf16* out2;
    size_t o2_ss;
    RowsLayout ol;
    int lda, ldr, ld2, n_split, Kd, Kper, splits, mrows, mtiles, ntiles, total, mb;     // Kper: reduction elements per split
    size_t slice;                     // EPI_PARTIAL: elements between the slices of a split reduction
    bool stream;                      // output not kept in the memory-side cache
};

template <int TM, int NW, int D, int EPI>
__global__ __launch_bounds__(64 * NW, 2) void gemm_wreg_kernel(GemmArgs p)
{
    constexpr int BM = 32 * TM, BN = 64 * NW, NA = TM * 4 / NW;   // NA: wave-loads (eight rows) of an activation k-tile per wave
    constexpr int STAGE = BM * 8;                           // 16-byte units
    constexpr int TKEY = TM == 3 ? 3 : TM * 4 - 1;          // swizzle of the transposed staging: bits of the chunk
    static_assert(NA >= 1, "every wave moves activations");
    extern __shared__ uint4 smem[];
    const int chunk = (p.total + 7) >> 3;
    const int lin = (int)(blockIdx.x & 7) * chunk + (int)(blockIdx.x >> 3);
    if ((int)(blockIdx.x >> 3) >= chunk || lin >= p.total) return;
    const int tiles = p.ntiles * p.mtiles, tl = lin % tiles, sp = EPI == EPI_PARTIAL ? (lin / tiles) % p.splits : 0;
    const int m = EPI == EPI_PARTIAL ? lin / (tiles * p.splits) : lin / tiles;
    const int gi = tl / (p.mb * p.ntiles), rb = tl - gi * p.mb * p.ntiles;
    const int mbe = p.mtiles - gi * p.mb < p.mb ? p.mtiles - gi * p.mb : p.mb;
    const int nt = rb / mbe, mt = gi * p.mb + rb % mbe;
    const int m0 = mt * BM, n0 = nt * BN;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int j31 = lane & 31, g = lane >> 5, nf = n0 + 64 * wave;
    const char* sb = p.arena + (size_t)m * p.ss;
    const int Kd = p.Kd, nk = (EPI == EPI_PARTIAL ? p.Kper : Kd) >> 6;

    // activations: wave-load i of a k-tile is rows 8 (wave + NW i) .. + 7, lane -> (row lane / 8, slot lane % 8), which holds chunk
    // slot ^ ((row >> 1) & 7); rows beyond mrows repeat the last one (64-bit base of the tile, 32-bit offsets inside it: a buffer may hold
    // more than 2^32 elements)
    const bf16* Ag = p.A + (size_t)m * p.a_ss + (size_t)m0 * p.lda + (EPI == EPI_PARTIAL ? sp * p.Kper : 0);
    int aoff[NA];
#pragma unroll
    for (int i = 0; i < NA; ++i) {
        const int r = 8 * (wave + NW * i) + (lane >> 3);
        const int rr = m0 + r < p.mrows ? r : p.mrows - 1 - m0;
        aoff[i] = 2 * (rr * p.lda + ((lane & 7) ^ ((r >> 1) & 7)) * 8);
    }
    // weights: lane -> row j31 of a 32-feature block, chunk g of a 16-element step
    const bf16* Wg = (const bf16*)(sb + p.w_off) + (size_t)(nf >> 4) * 16 * Kd + (EPI == EPI_PARTIAL ? (size_t)sp * p.Kper * 16 : 0);
    const int wlane = 2 * ((j31 >> 4) * 16 * Kd + g * 128 + (j31 & 15) * 8);

    bf16x8 w[D][4][2];
    auto dma_a = [&](int kt, int stage) {
#pragma unroll
        for (int i = 0; i < NA; ++i) load_lds16(Ag, (lds_void*)(smem + stage * STAGE + (wave + NW * i) * 64), aoff[i], kt * 128);
    };
    auto load_w = [&](int kt, int slot, int s) {
#pragma unroll
        for (int i = 0; i < 2; ++i) w[slot][s][i] = __builtin_bit_cast(bf16x8, load16(Wg, wlane + s * 512, kt * 2048 + i * 64 * Kd));
    };
    const int xlane = j31 * 8 + (g ^ ((j31 >> 1) & 7));     // slot of step 0; that of step s is at xlane ^ 2 s
    bf16x8 fx[2][TM];
    auto frag = [&](int stage, int s, int t) { return *(const bf16x8*)(smem + ((stage * STAGE + xlane) ^ (2 * s)) + t * 256); };

    f32x16 acc[2][TM];
    dma_a(0, 0);
    f32x4 b4[2][4];
    {
        const float* bias = (const float*)(sb + p.b_off) + nf + 4 * g;
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int v4 = 0; v4 < 4; ++v4) b4[i][v4] = EPI == EPI_PARTIAL ? f32x4{0.f, 0.f, 0.f, 0.f} : *(const f32x4*)(bias + 32 * i + 8 * v4);
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int s = 0; s < 4; ++s) load_w(0, 0, s);
    __builtin_amdgcn_sched_barrier(0);
    dma_a(1, 1);
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (D > 1) {
#pragma unroll
        for (int s = 0; s < 4; ++s) load_w(1, 1, s);
        __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int t = 0; t < TM; ++t)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[i][t][e] = b4[i][e >> 2][e & 3];
    __builtin_amdgcn_sched_barrier(0);
    wait_vmcnt<8 * D + NA>();                               // activations of k-tile 0
    barrier_lds();
    if (D > 1 && nk > 2) dma_a(2, 2);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int t = 0; t < TM; ++t) fx[0][t] = frag(0, 0, t);

    // One k-tile, j, weights in slot j % D.  Requested during it: W: the weights of k-tile j + D, a step's when its registers are free; AL:
    // the activations of k-tile j + 1 + D, all together.  NEXT: k-tile j + 1 exists; V: loads that may be in flight when its activations have
    // to be there, those requested behind them.
    int prev = D + 1, cur = 0, next = 1;                    // stages of k-tiles j - 1 (free: the one requested goes there), j and j + 1
    auto ktile = [&](int j, auto slot_c, auto w_c, auto a_c, auto next_c, auto v_c) {
        constexpr int slot = decltype(slot_c)::value % D;
        constexpr bool W = decltype(w_c)::value, AL = decltype(a_c)::value, NEXT = decltype(next_c)::value;
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            if (s == 3 && NEXT) {
                wait_vmcnt<decltype(v_c)::value>();
                barrier_lds();
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int t = 0; t < TM; ++t) {
                if (s < 3) fx[(s + 1) & 1][t] = frag(cur, s + 1, t);
                else if (NEXT) fx[0][t] = frag(next, 0, t);
#pragma unroll
                for (int i = 0; i < 2; ++i) acc[i][t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(w[slot][s][i], fx[s & 1][t], acc[i][t], 0, 0, 0);
                __builtin_amdgcn_sched_barrier(0);
            }
            if (AL && s == 1) dma_a(j + 1 + D, prev);
            if (W) load_w(j + D, slot, s);
            __builtin_amdgcn_sched_barrier(0);
        }
        prev = cur;
        cur = next;
        next = next == D + 1 ? 0 : next + 1;
    };
    constexpr std::true_type Y{};
    constexpr std::false_type N{};
    constexpr std::integral_constant<int, 0> S0{};
    constexpr std::integral_constant<int, 1> S1{};
    int j = 0;                                              // (nk is even)
    if constexpr (D == 1) {
        constexpr std::integral_constant<int, 12 + NA> V{};     // W of the last three steps before, A and W of three steps since
        if (nk > 2) {
            ktile(0, S0, Y, Y, Y, std::integral_constant<int, 6 + NA>{});
            ktile(1, S0, Y, Y, Y, V);
            for (j = 2; j + 2 < nk; j += 2) {
                ktile(j, S0, Y, Y, Y, V);
                ktile(j + 1, S0, Y, Y, Y, V);
            }
        }
        ktile(j, S0, Y, N, Y, std::integral_constant<int, 6>{});
        ktile(j + 1, S0, N, N, N, S0);
    } else {
        constexpr std::integral_constant<int, 14 + 2 * NA> V{};
        for (; j + 4 < nk; j += 2) {
            ktile(j, S0, Y, Y, Y, V);
            ktile(j + 1, S1, Y, Y, Y, V);
        }
        if (nk > 2) {
            ktile(j, S0, Y, Y, Y, V);
            ktile(j + 1, S1, Y, N, Y, std::integral_constant<int, 14 + NA>{});
            j += 2;
        }
        ktile(j, S0, N, N, Y, std::integral_constant<int, 8>{});
        ktile(j + 1, S1, N, N, N, S0);
    }

    // ---- epilogue: accumulator element v of lane l in block (i, t): token 32 t + l % 32, feature 32 i + 8 (v / 4) +
    // 4 (l / 32) + v % 4.  Each wave stages its tile in its own slice of LDS and stores whole row segments.
    if (EPI == EPI_PARTIAL) {                               // fp32 sums of this split of the reduction, no bias
        float* po = (float*)p.out + (size_t)sp * p.slice + (size_t)m * p.o_ss + nf + 4 * g;
#pragma unroll
        for (int t = 0; t < TM; ++t) {
            const int row = m0 + 32 * t + j31;
            if (row < p.mrows)
#pragma unroll
                for (int i = 0; i < 2; ++i)
#pragma unroll
                    for (int v4 = 0; v4 < 4; ++v4)
                        *(f32x4*)(po + (size_t)row * p.ol.rs + 32 * i + 8 * v4) =
                            f32x4{acc[i][t][4 * v4], acc[i][t][4 * v4 + 1], acc[i][t][4 * v4 + 2], acc[i][t][4 * v4 + 3]};
        }
        return;
    }
    char* stg = (char*)smem + (size_t)wave * BM * 128;
    const bool transposed = EPI == EPI_QKV && n0 >= p.n_split;
    const int rr = lane >> 3, cc = lane & 7;
    auto cell = [&](int r, int f) { return stg + r * 128 + (((f >> 3) ^ ((r >> 1) & 7)) << 4) + (f & 7) * 2; };
    barrier_lds();                                          // everybody has read the last activations
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
    for (int t = 0; t < TM; ++t)
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int v4 = 0; v4 < 4; ++v4) {
                const int f = i * 32 + 8 * v4 + 4 * g;
                float r[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) r[e] = acc[i][t][4 * v4 + e];
                if (EPI == EPI_BIAS_GELU) {
#pragma unroll
                    for (int e = 0; e < 4; ++e) r[e] = gelu_erf_fast(r[e]);
                }
                if (EPI == EPI_QKV && transposed) {
                    const int tok = t * 32 + j31;
#pragma unroll
                    for (int e = 0; e < 4; ++e)             // rows: features, 2 BM bytes each
                        *(bf16*)(stg + (f + e) * (BM * 2) + (((tok >> 3) ^ (f >> 2 & TKEY)) << 4) + (tok & 7) * 2) = (bf16)r[e];
                } else {
                    char* c = cell(t * 32 + j31, f);
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
    if (EPI == EPI_QKV && transposed) {
        constexpr int CPR = TM * 4, RPI = 64 / CPR;         // chunks per feature row, rows per instruction
        const int fr = lane / CPR, fc = lane % CPR;
        bf16* dst = p.out2 + (size_t)m * p.o2_ss + (size_t)(nf - p.n_split) * p.ld2 + m0 + fc * 8;
        auto store = [&](auto stream) {
            if (fr < RPI && m0 + fc * 8 < p.mrows)
#pragma unroll 4
                for (int f = fr; f < 64; f += RPI)
                    store16_through<decltype(stream)::value>(dst + (size_t)f * p.ld2, *(const u32x4*)(stg + f * (BM * 2) + ((fc ^ (f >> 2 & TKEY)) << 4)));
        };
        if (p.stream) store(Y); else store(N);
        return;
    }
    bf16* dst = p.out + (size_t)m * p.o_ss + (size_t)(nf / 8 + cc) * p.ol.cs;
    auto store = [&](auto stream) {
#pragma unroll
        for (int q0 = 0; q0 < BM / 8; q0 += 4) {
            u32x4 v[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int r = (q0 + q) * 8 + rr;
                v[q] = *(const u32x4*)(stg + r * 128 + ((cc ^ ((r >> 1) & 7)) << 4));
            }
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int row = m0 + (q0 + q) * 8 + rr;
                if (row < p.mrows)
                    store16_through<decltype(stream)::value>(dst + (size_t)(row >> 4) * p.ol.rb + (size_t)(row & 15) * p.ol.rs, v[q]);
            }
        }
    };
    if (p.stream) store(Y); else store(N);
}

template <int TM, int NW, int D, int EPI>
hipError_t launch_wreg_tile(const sp_model* M, GemmArgs a, int N, int k, hipStream_t s)
{
    constexpr size_t smem = (size_t)32 * TM * 128 * (D + 2 > NW ? D + 2 : NW);
    auto kern = gemm_wreg_kernel<TM, NW, D, EPI>;
    if (smem > 48 * 1024) {
        static std::atomic<bool> raised{false};
        if (!raised.load(std::memory_order_acquire)) {
            hipError_t e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
            if (e != hipSuccess) return e;
            raised.store(true, std::memory_order_release);
        }
    }
    a.mtiles = (a.mrows + 32 * TM - 1) / (32 * TM);
    a.ntiles = N / (64 * NW);
    a.total = k * a.splits * a.mtiles * a.ntiles;
    a.mb = 32 / TM;                                         // (about a thousand tokens: see the tile order)
    hipLaunchKernelGGL(kern, dim3((unsigned)((a.total + 7) / 8 * 8)), dim3(64 * NW), smem, s, a);
    return hipGetLastError();
}

// Tile height.  The chip has 256 compute units and two workgroups of one run side by side, sharing its matrix cores, so a
// launch takes about as long as the compute unit with the most work: workgroups per unit (rounded up) x tokens per tile x
// what a token costs at that height.  A lower tile reads the weights more often, which counts the more the deeper the reduction; at 256
// the first loads and the epilogue take longer than the four k-tiles, and lower tiles, of which three fit a unit, hide them better.
// Measured against it, us at 128 / 96 / 64 tokens: 14653 tokens x 2 students, 768 from 256: 27.5 / 26.8 / 23.1, 1024 from 256 36.6 / 31.6 / 32.5;
// 2304 features from 768 98.7 / 96.4 / 109; 768 from 3072 131 / 141 / 171; 4608 tokens x 2, 3072 from 768: 55.1 / 50.3 / 52.5; x 8, 768 from 3072: 177 / 188 /
// 219; 18432 tokens, 1024 from 4096: 147 / 132 / 163; 640 tokens, 768 from 768, at 64 and 32: 11.2 / 8.8.  (A split reduction goes by the depth of a share,
// 256 at least: one student of 768 or 1024, 1600-5300 tokens, the height that costs of 1.2 and 1.1 choose as well, and the quickest of the three.)
}  // namespace

constexpr double kHalfTokenCost[5] = {0, 1.7, 1.2, 1.1, 1.0};       // tiles of half the features
constexpr double kTokenCost[3][5] = {{0, 1.7, 0.88, 0.95, 1.0}, {0, 1.7, 1.2, 1.05, 1.0}, {0, 1.7, 1.25, 1.15, 1.0}};

// wide: tiles side by side; round: how many the chip takes at once; tallest: the largest height there is; cost: of a token by height
static int tile_height(int mrows, long wide, long round, int tallest, const double* cost)
{
    int best = tallest;
    double least = 0;
    for (int tm = tallest; tm >= 1; --tm) {
        const double t = (double)(((mrows + 32 * tm - 1) / (32 * tm) * wide + round - 1) / round) * tm * cost[tm];
        if (tm == tallest || t < least) { best = tm; least = t; }
    }
    return best;
}

int gemm_tile_height(int mrows, int N, int k, const double* cost) { return tile_height(mrows, (long)(N / 256) * k, 256, 4, cost); }
const double* gemm_token_cost(int Kd) { return kTokenCost[Kd <= 256 ? 0 : Kd < 2048 ? 1 : 2]; }

namespace {

template <int EPI>
hipError_t launch_bf16(const sp_model* M, const GemmArgs& a, int N, int k, hipStream_t s)
{
    // Widths that are not multiples of 256: half the features, two waves, so a round is twice as many workgroups; 96 tokens (128
    // do not fit the registers: 665 us where these take 471) only from two rounds on.  Measured, us, 64 tokens always / this: 14521
    // tokens x 4 students, hidden 896: q|k|v 322 / 289, attention output 144 / 127, FFN down 507 / 471; calls of few tiles are
    // chains of k-tiles that a lower tile shortens: 1851 tokens, hidden 384: attention output 7.5 / 5.9, FFN down from 640 10 / 8.
    if (N % 256 || a.n_split % 256) {
        // (Two k-tiles in flight while there is a workgroup per compute unit at most, as below, were measured here as well: no rule for all
        // widths.  us a call, one in flight / two: one student, twelve sequences: hidden 128 70 / 73, 384 100 / 95, 640 124 / 117, 896 153 / 145;
        // four students 79 / 81, 128 / 130, 177 / 177, 259 / 259; 64 tokens at hidden 128 47 / 50.)
        const long wide = (long)(N / 128) * k * a.splits;
        switch (tile_height(a.mrows, wide, 512, (a.mrows + 95) / 96 * wide >= 1024 ? 3 : 2, kHalfTokenCost)) {
            case 1: return launch_wreg_tile<1, 2, 1, EPI>(M, a, N, k, s);
            case 2: return launch_wreg_tile<2, 2, 1, EPI>(M, a, N, k, s);
            default: return launch_wreg_tile<3, 2, 1, EPI>(M, a, N, k, s);
        }
    }
    // Few tiles: a workgroup is alone on its compute unit, and what a launch takes is its chain of k-tiles, each of which waits for
    // its weights.  Half the features per tile bring twice the workgroups, and two k-tiles of weights are in flight: 32 tokens
    // while those are at most a workgroup per compute unit, 64 (the weights read half as often) while that holds there.  us, 32 x
    // 256 with one k-tile in flight / 32 x 128 / 64 x 128: 2304 features from 768, 192 rows x 2 students 8.3 / 5.9 / 8.2, 64 x 4 8.3 /
    // 5.9 / 8.0, 64 x 8 12.1 / 12.1 / 10.2; 3072 features, 256 rows x 1 8.4 / 6.5 / 9.0, 64 x 8 14.0 / 14.0 / 12.6; with one k-tile in
    // flight 32 x 128 takes 7.7 for the first.  (Four in flight: no change.  Taller tiles of 256 features, alone or two to a unit:
    // none from two in flight, -4 to +25 %.)
    const long half = (long)(N / 128) * k * a.splits;
    if ((a.mrows + 31) / 32 * half <= 256) return launch_wreg_tile<1, 2, 2, EPI>(M, a, N, k, s);
    if ((a.mrows + 63) / 64 * half <= 256) return launch_wreg_tile<2, 2, 2, EPI>(M, a, N, k, s);
    switch (gemm_tile_height(a.mrows, N, k * a.splits, gemm_token_cost(a.Kper))) {
        case 1: return launch_wreg_tile<1, 4, 1, EPI>(M, a, N, k, s);
        case 2: return launch_wreg_tile<2, 4, 1, EPI>(M, a, N, k, s);
        case 3: return launch_wreg_tile<3, 4, 1, EPI>(M, a, N, k, s);
        default: return launch_wreg_tile<4, 4, 1, EPI>(M, a, N, k, s);
    }
}

// -------------------------------------------------------------------------------------
// fp32 kernel: square tile of 16 TS rows x 16 TS features (TS = 4: 64 x 64, TS = 2: 32 x 32 for calls whose larger
// tiles would leave most compute units idle), 16 x 16 threads with TS x TS outputs each, FMA only, the reduction index
// ascending for every output.  Slabs of 64 along the reduction: the next slab's rows are requested (into registers)
// before the current one is multiplied, so a slab costs one memory round trip or its arithmetic, whichever is longer.
// -------------------------------------------------------------------------------------
template <int EPI, int TS>
__global__ __launch_bounds__(256) void gemm_f32_kernel(const float* __restrict__ A, int lda, size_t a_ss,
                                                       const char* __restrict__ arena, size_t student_stride,
                                                       size_t w_off, size_t b_off, float* __restrict__ out, int ldo,
                                                       size_t o_ss, const float* __restrict__ res, int ldr,
                                                       size_t r_ss, int Kd)
{
    constexpr int BT = 16 * TS, BK = 64, PITCH = BT + 4;
    constexpr int LPT = BT * BK / 4 / 256;                  // 16-byte loads per thread and operand: 16 rows apart
    typedef float fts __attribute__((ext_vector_type(TS)));
    __shared__ float As[BK][PITCH], Ws[BK][PITCH];
    const int m = blockIdx.z, m0 = blockIdx.y * BT, n0 = blockIdx.x * BT;
    const int tid = threadIdx.x, tx = tid & 15, ty = tid >> 4;
    const float* Ag = A + (size_t)m * a_ss + (size_t)m0 * lda;
    const float* Wg = (const float*)(arena + (size_t)m * student_stride + w_off) + (size_t)n0 * Kd;
    const int lr = tid >> 4, lk = (tid & 15) * 4;           // loader: row lr + 16 i of the tile, reduction elements lk .. lk + 3
    f32x4 pa[LPT], pw[LPT];
    auto request = [&](int k0) {
#pragma unroll
        for (int i = 0; i < LPT; ++i) {
            pa[i] = *(const f32x4*)(Ag + (size_t)(lr + 16 * i) * lda + k0 + lk);
            pw[i] = *(const f32x4*)(Wg + (size_t)(lr + 16 * i) * Kd + k0 + lk);
        }
    };
    float acc[TS][TS] = {};
    request(0);
    for (int k0 = 0; k0 < Kd; k0 += BK) {
#pragma unroll
        for (int i = 0; i < LPT; ++i)
#pragma unroll
            for (int e = 0; e < 4; ++e) { As[lk + e][lr + 16 * i] = pa[i][e]; Ws[lk + e][lr + 16 * i] = pw[i][e]; }
        __syncthreads();
        if (k0 + BK < Kd) request(k0 + BK);
#pragma unroll 16
        for (int kk = 0; kk < BK; ++kk) {
            const fts a = *(const fts*)&As[kk][ty * TS];
            const fts w = *(const fts*)&Ws[kk][tx * TS];
#pragma unroll
            for (int i = 0; i < TS; ++i)
#pragma unroll
                for (int j = 0; j < TS; ++j) acc[i][j] = fmaf(a[i], w[j], acc[i][j]);
        }
        __syncthreads();
    }
    const float* bias = (const float*)(arena + (size_t)m * student_stride + b_off);
    const fts bv = *(const fts*)(bias + n0 + tx * TS);
#pragma unroll
    for (int i = 0; i < TS; ++i) {
        const size_t row = (size_t)(m0 + ty * TS + i);
        fts r;
#pragma unroll
        for (int j = 0; j < TS; ++j) r[j] = acc[i][j] + bv[j];
        if (EPI == EPI_BIAS_GELU) {
#pragma unroll
            for (int j = 0; j < TS; ++j) r[j] = gelu_erf(r[j]);
        }
        if (EPI == EPI_BIAS_RESIDUAL) r += *(const fts*)(res + (size_t)m * r_ss + row * ldr + n0 + tx * TS);
        *(fts*)(out + (size_t)m * o_ss + row * ldo + n0 + tx * TS) = r;
    }
}

// The same product for deep reductions on small grids (the FFN down-projection of a call of a few dozen tokens): one
// 32 x 32 tile per workgroup, the reduction range split over its four waves (a quarter each, ascending inside it, 4 x 4
// outputs per lane, wave-private slabs of 32 along the reduction), the four partial tiles added in wave order through
// LDS.  A single chain over the whole depth costs one memory round trip per slab; here a wave has four slabs in flight
// at once and a quarter of the depth to walk.  Kd must be a multiple of 512 (a wave's quarter: whole groups of four slabs).
template <int EPI, int TS>
__global__ __launch_bounds__(256) void gemm_f32_ksplit_kernel(const float* __restrict__ A, int lda, size_t a_ss,
                                                              const char* __restrict__ arena, size_t student_stride,
                                                              size_t w_off, size_t b_off, float* __restrict__ out,
                                                              int ldo, size_t o_ss, const float* __restrict__ res,
                                                              int ldr, size_t r_ss, int Kd)
{
    // tile of 8 TS x 8 TS outputs (TS = 4: 32 x 32; TS = 2: 16 x 16, four times the workgroups, when even the 32 x 32
    // tiles would leave most of the chip idle); a lane owns TS x TS of them
    constexpr int BT = 8 * TS, BK = 32, PITCH = BT + 4, SLAB = BK * PITCH;
    typedef float fts __attribute__((ext_vector_type(TS)));
    __shared__ __attribute__((aligned(16))) float lds[4 * 2 * SLAB];   // per wave: activation slab, weight slab
    const int m = blockIdx.z, m0 = blockIdx.y * BT, n0 = blockIdx.x * BT;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int tx = lane & 7, ty = lane >> 3;                // this lane's outputs: rows TS ty .., features TS tx ..
    const int kw = Kd / 4, kb = wave * kw;
    const float* Ag = A + (size_t)m * a_ss + (size_t)m0 * lda + kb;
    const float* Wg = (const float*)(arena + (size_t)m * student_stride + w_off) + (size_t)n0 * Kd + kb;
    float* As = lds + wave * 2 * SLAB;
    float* Ws = As + SLAB;
    // A wave requests four slabs (128 of its reduction range: all of it at a depth of 512) before it uses the first, so
    // their memory round trips overlap; then slab after slab goes through the wave's LDS and is multiplied.
    constexpr int NSL = 4, LPT = BT * BK / 4 / 64;          // 16-byte loads per lane, slab and operand
    f32x4 pa[NSL][LPT], pw[NSL][LPT];
    float acc[TS][TS] = {};
    for (int kc0 = 0; kc0 < kw; kc0 += NSL * BK) {
#pragma unroll
        for (int sl = 0; sl < NSL; ++sl)
#pragma unroll
            for (int i = 0; i < LPT; ++i) {
                const int idx = lane + 64 * i, row = idx >> 3, kc = (idx & 7) * 4;
                pa[sl][i] = *(const f32x4*)(Ag + (size_t)row * lda + kc0 + sl * BK + kc);
                pw[sl][i] = *(const f32x4*)(Wg + (size_t)row * Kd + kc0 + sl * BK + kc);
            }
#pragma unroll
        for (int sl = 0; sl < NSL; ++sl) {
#pragma unroll
            for (int i = 0; i < LPT; ++i) {
                const int idx = lane + 64 * i, row = idx >> 3, kc = (idx & 7) * 4;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    As[(kc + e) * PITCH + row] = pa[sl][i][e];
                    Ws[(kc + e) * PITCH + row] = pw[sl][i][e];
                }
            }
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
#pragma unroll 8
            for (int kk = 0; kk < BK; ++kk) {
                const fts a = *(const fts*)&As[kk * PITCH + ty * TS];
                const fts w = *(const fts*)&Ws[kk * PITCH + tx * TS];
#pragma unroll
                for (int i = 0; i < TS; ++i)
#pragma unroll
                    for (int j = 0; j < TS; ++j) acc[i][j] = fmaf(a[i], w[j], acc[i][j]);
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();                // the slab is rewritten only after every lane has read it
        }
    }
    // partial tiles -> LDS (over the slabs, which nobody reads any more), then summed in wave order
    __syncthreads();
    float* red = lds;                                       // [wave][row][PITCH]
#pragma unroll
    for (int i = 0; i < TS; ++i)
#pragma unroll
        for (int jj = 0; jj < TS; ++jj) red[(wave * BT + ty * TS + i) * PITCH + tx * TS + jj] = acc[i][jj];
    __syncthreads();
    constexpr int OUTS = BT * BT / 256, TPR = BT / OUTS;    // outputs per thread (neighbours in a row); threads per row
    const int r = tid / TPR, c0 = (tid % TPR) * OUTS;
    const float* bias = (const float*)(arena + (size_t)m * student_stride + b_off);
    const size_t row = (size_t)(m0 + r);
#pragma unroll
    for (int o = 0; o < OUTS; ++o) {
        const int c = c0 + o;
        float v = red[r * PITCH + c];
#pragma unroll
        for (int wv = 1; wv < 4; ++wv) v += red[(wv * BT + r) * PITCH + c];
        v += bias[n0 + c];
        if (EPI == EPI_BIAS_GELU) v = gelu_erf(v);
        if (EPI == EPI_BIAS_RESIDUAL) v += res[(size_t)m * r_ss + row * ldr + n0 + c];
        out[(size_t)m * o_ss + row * ldo + n0 + c] = v;
    }
}

template <int EPI>
hipError_t launch_f32(const sp_model* M, const void* A, int lda, size_t w_off, size_t b_off, void* out, int ldo,
                      const void* residual, int ldr, int mrows, int N, int Kd, int k, size_t a_ss, size_t o_ss,
                      size_t r_ss, hipStream_t s)
{
    // (rows and widths are multiples of 64 and the reduction depth of 128: the launcher's callers see to that)
    if (mrows % 64 || N % 64 || Kd % 64) return hipErrorInvalidValue;
    // 64 x 64 tiles when they give every compute unit a few workgroups; else 32 x 32 tiles, four times as many
    if ((long)(N / 64) * (mrows / 64) * k >= 1024) {
        hipLaunchKernelGGL((gemm_f32_kernel<EPI, 4>), dim3(N / 64, mrows / 64, k), dim3(256), 0, s, (const float*)A, lda,
                           a_ss / 4, M->arena, M->L.student_stride, w_off, b_off, (float*)out, ldo, o_ss / 4,
                           (const float*)residual, ldr, r_ss / 4, Kd);
    } else if (Kd >= 512 && Kd % 512 == 0 && (long)(N / 32) * (mrows / 32) * k <= 256) {
        // few tiles and a deep reduction: the reduction range over the four waves of a workgroup
        if ((long)(N / 32) * (mrows / 32) * k < 128)
            hipLaunchKernelGGL((gemm_f32_ksplit_kernel<EPI, 2>), dim3(N / 16, mrows / 16, k), dim3(256), 0, s,
                               (const float*)A, lda, a_ss / 4, M->arena, M->L.student_stride, w_off, b_off, (float*)out,
                               ldo, o_ss / 4, (const float*)residual, ldr, r_ss / 4, Kd);
        else
            hipLaunchKernelGGL((gemm_f32_ksplit_kernel<EPI, 4>), dim3(N / 32, mrows / 32, k), dim3(256), 0, s,
                               (const float*)A, lda, a_ss / 4, M->arena, M->L.student_stride, w_off, b_off, (float*)out,
                               ldo, o_ss / 4, (const float*)residual, ldr, r_ss / 4, Kd);
    } else {
        hipLaunchKernelGGL((gemm_f32_kernel<EPI, 2>), dim3(N / 32, mrows / 32, k), dim3(256), 0, s, (const float*)A, lda,
                           a_ss / 4, M->arena, M->L.student_stride, w_off, b_off, (float*)out, ldo, o_ss / 4,
                           (const float*)residual, ldr, r_ss / 4, Kd);
    }
    return hipGetLastError();
}

// y[i] = the GELU of the bf16 epilogue evaluated on x[i], before any rounding to bf16 (test aid)
__global__ void gelu_probe_kernel(const float* __restrict__ x, float* __restrict__ y, long n)
{
    const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) y[i] = gelu_erf_fast(x[i]);
}

}  // namespace

hipError_t launch_gelu_probe(const float* x, float* y, long n, hipStream_t s)
{
    if (n < 1) return hipErrorInvalidValue;
    hipLaunchKernelGGL(gelu_probe_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, x, y, n);
    return hipGetLastError();
}

hipError_t launch_gemm_split(const sp_model* M, const void* A, int lda, size_t w_off, float* part, size_t slice, int mrows,
                             int N, int Kd, int k, int splits, size_t a_student_stride, size_t p_student_stride, hipStream_t s)
{
    if (!bf16_path(M->cfg) || mrows % 64 || N % 128 || splits < 1 || Kd % (128 * splits)) return hipErrorInvalidValue;
    const GemmArgs a{(const bf16*)A, a_student_stride / 2, M->arena, M->L.student_stride, w_off, 0, (bf16*)part, p_student_stride,
                     nullptr, 0, nullptr, 0, rows_layout(N), lda, 0, 0, 0, Kd, Kd / splits, splits, mrows, 0, 0, 0, 0, slice, false};
    return launch_bf16<EPI_PARTIAL>(M, a, N, k, s);
}

hipError_t launch_gemm(const sp_model* M, const void* A, int lda, size_t w_off, size_t b_off, void* out, int ldo,
                       const void* residual, int ldr, int mrows, int N, int Kd, int k, Epilogue epi,
                       size_t a_student_stride, size_t o_student_stride, size_t r_student_stride, hipStream_t s,
                       void* out2, int n_split, int ld2, size_t o2_student_stride, bool packed_out)
{
    // shapes the kernels assume; config_supported() guarantees them for every model that loads
    if (mrows % 64 || N % 128 || Kd % 128 || (epi == EPI_BIAS_RESIDUAL && !residual)) return hipErrorInvalidValue;
    if (epi == EPI_QKV && (!bf16_path(M->cfg) || !out2 || n_split % 128 || ld2 % 8)) return hipErrorInvalidValue;
#define SP_ARGS M, A, lda, w_off, b_off, out, ldo, residual, ldr, mrows, N, Kd, k, a_student_stride, \
                o_student_stride, r_student_stride, s
    if (packed_out && (!bf16_path(M->cfg) || epi == EPI_QKV)) return hipErrorInvalidValue;
    if (bf16_path(M->cfg)) {
        const GemmArgs a{(const bf16*)A, a_student_stride / 2, M->arena, M->L.student_stride, w_off, b_off, (bf16*)out,
                         o_student_stride / 2, (const bf16*)residual, r_student_stride / 2, (bf16*)out2, o2_student_stride / 2,
                         packed_out ? packed_layout(ldo) : rows_layout(ldo), lda, ldr, ld2, n_split, Kd, Kd, 1, mrows, 0, 0, 0, 0, 0,
                         (size_t)k * mrows * N * 2 >= kStreamBytes};
        switch (epi) {
            case EPI_BIAS_GELU: return launch_bf16<EPI_BIAS_GELU>(M, a, N, k, s);
            case EPI_QKV: return launch_bf16<EPI_QKV>(M, a, N, k, s);
            case EPI_BIAS_RESIDUAL: return launch_bf16<EPI_BIAS_RESIDUAL>(M, a, N, k, s);
            default: return hipErrorInvalidValue;
        }
    }
    if (epi == EPI_QKV || epi == EPI_BIAS_TANH) return hipErrorInvalidValue;   // bf16 path only
    switch (epi) {
        case EPI_BIAS: return launch_f32<EPI_BIAS>(SP_ARGS);
        case EPI_BIAS_GELU: return launch_f32<EPI_BIAS_GELU>(SP_ARGS);
        default: return launch_f32<EPI_BIAS_RESIDUAL>(SP_ARGS);
    }
#undef SP_ARGS
}

}  // namespace sp
