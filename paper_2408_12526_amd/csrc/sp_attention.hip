// Multi-head self-attention over a packed batch: every sequence attends to itself only,
// over exactly its own tokens (cu_seqlens gives the boundaries); head width is 64.
#include <atomic>
#include <type_traits>

#include "sp_attn_offsets.h"
#include "sp_internal.h"

namespace sp {

namespace {

constexpr int kD = 64;          // head width
// 2^x by the hardware instruction alone.  (exp2f() wraps it in a range test, a scaling and an ldexp so that results
// below 2^-126 come out as denormals: four more instructions per value, which a softmax numerator does not need;
// arguments here are <= 0, and what underflows is flushed to zero.)
__device__ inline float exp2_raw(float x) { return __builtin_amdgcn_exp2f(x); }

// A query's keys sit in lanes l and l ^ 32: maximum and sum over the two (every lane active).
__device__ inline float max_across_halves(float x) { float lo = x, hi = x; swap_halves(lo, hi); return fmaxf(lo, hi); }
__device__ inline float sum_across_halves(float x) { float lo = x, hi = x; swap_halves(lo, hi); return lo + hi; }

// eight bf16 values (one 16-byte chunk of an output row) -> eight e4m3 codes of value * qscale
__device__ inline uint2 chunk_to_fp8(uint4 c, float qscale)
{
    const bf16x8 v = __builtin_bit_cast(bf16x8, c);
    int lo = 0, hi = 0;
    lo = __builtin_amdgcn_cvt_pk_fp8_f32((float)v[0] * qscale, (float)v[1] * qscale, lo, false);
    lo = __builtin_amdgcn_cvt_pk_fp8_f32((float)v[2] * qscale, (float)v[3] * qscale, lo, true);
    hi = __builtin_amdgcn_cvt_pk_fp8_f32((float)v[4] * qscale, (float)v[5] * qscale, hi, false);
    hi = __builtin_amdgcn_cvt_pk_fp8_f32((float)v[6] * qscale, (float)v[7] * qscale, hi, true);
    return uint2{(unsigned)lo, (unsigned)hi};
}

// -------------------------------------------------------------------------------------
// bf16 kernel on the matrix cores (v_mfma_f32_32x32x16_bf16, fp32 accumulate).  A workgroup takes 128 queries of one sequence
// and head, a wave 32 of them.  Keys and values go through LDS in tiles of 64 keys that the four waves share; per block of 32 keys:
//   S^T = K Q^T      (A operand: key rows from LDS, B operand: the queries, in registers throughout)
//   online softmax   a query is a lane column, its keys sit in the registers of lanes l and l + 32; the
//                    1/sqrt(d) log2(e) factor rides in the multiply-add in front of the exponential
//   O^T += V^T P^T   (A operand: transposed value tile from LDS; B operand: the probabilities as they are)
// The tiles are double-buffered and travel through registers, keys and values in turn: the next tile's keys are put down once
// the scores are formed and its values requested, the values put down at the end and the keys of the tile after it requested; one
// barrier per tile, which waits for LDS traffic only.  Rows of eight 16-byte slots, slot = chunk ^ ((row / 2) % 8).
//
// The running maximum moves per tile of 64 keys, in sequences of up to 128 tokens per block of 32.
//
// Work item i belongs to the last sequence b with cu[b] / 128 + b <= i: a sequence of L tokens gets at least ceil(L / 128)
// consecutive numbers, T / 128 + B numbers are enough for any lengths, and which sequence it is takes one look at 64 boundaries
// by the whole wave (two beyond 64 sequences, three beyond 4096).
//
// What bounds it: vector instructions (about seven issue slots per score, four of them the exponential) and the read of
// queries, keys and values, neither saturated: a wave's chain of products, maximum, exponentials and products is issued in
// order, so waves in flight are what counts.  Hence 32 queries a wave and 128 registers, four waves per SIMD (with 64 queries a
// wave a key fragment served two products, but two waves per SIMD was all the registers held).  Sequences of up to 32 tokens would leave
// three of the four waves idle: batches of them have a part of their own (attention_short).  us per launch, a wave per
// sequence and head up to 128 tokens and 64 queries per wave above / this: 64 sequences of 64-512 tokens, 16 heads, one student
// 84 / 66, six 466 / 335; 256 sequences of 8-256, 12 heads, eight students 238 / 214, two 65 / 54; 32 of 16-128, four students
// 31 / 21; one of 64, one student 9.9 / 6.9.  With the next tile's keys in flight across the loop's end (they were waited for there, for
// the sake of a copy) and a loop of their own for waves without queries 60.0 / 58.9, 345 / 339, two students of the third 32.3 / 31.6.  Tried: keys and values in flight together (141 registers, three waves) 65, 357, 237,
// 60, 22 and 6.6; two heads per workgroup side by side where a sequence fits one tile: 382 for the second where one head took 340.
// A reference that moves only when it is outgrown by 2^8 saves most rescaling (317 for the second), but then the largest
// probability is no longer 1 and is rounded: up to 1.2 times the error against 64 bits on sharp distributions.
// -------------------------------------------------------------------------------------
constexpr int kQItem = 128;     // queries of a work item: four waves x 32
constexpr int kKeyTile = 64;    // keys staged in LDS per step
constexpr int kNarrowLen = 128; // longest sequence whose softmax goes by blocks of 32 keys
constexpr int kTileBytes = kKeyTile * kD * 2;       // keys: rows of 64 dimensions; values: rows of 64 keys; eight 16-byte slots each
constexpr int kOutPitch = kD * 2 + 16;              // bytes per staged output row
constexpr int kAttnLdsBytes = 4 * kTileBytes;       // two buffers of a key and a value tile
static_assert(4 * 32 * kOutPitch <= kAttnLdsBytes && (2 * kTileBytes & (2 * kTileBytes - 1)) == 0, "the output tiles reuse the key/value buffers; offsets change buffers by an exclusive or");

constexpr int kShortLen = 32;   // longest sequence that one wave takes with all its queries
constexpr int kShortBytes = kAttnLdsBytes / 4;      // LDS of such a wave: a key and a value tile of 32 keys
constexpr int kShortKeys = kShortLen * kD * 2;      // bytes of the key tile
static_assert(2 * kShortKeys == kShortBytes && kShortLen * kOutPitch <= kShortBytes, "the output tile reuses the wave's key/value tiles");

struct AttnArgs {
    const bf16 *qkv, *vt;
    bf16* att;                        // null: the fp8 copy alone
    unsigned char* attq;              // null: none
    const int32_t* cu;
    float qscale;
    int B, Tn, rows, H, heads, max_seqlen;
    int items, run;                   // work items per head; neighbouring items that stay on one XCD
    int pairs, whole;                 // (student, head) pairs; how many of them an XCD has to itself (0: one row of the grid per student)
    int general;                      // workgroups of the general part; those behind it take sequences of up to kShortLen tokens
};

// Scores of a block of 32 keys (a query is a lane column): accumulator register v of a lane of half g is key 8 (v / 4) + 4 g + v % 4.  Only
// the first and the last block of a sequence of L keys have keys to mask (k0: the block's first key, at least -7).
__device__ __forceinline__ void mask_block(f32x16& sc, int k0, int L, int g)
{
    if (k0 >= 0 && k0 + 32 <= L) return;
    const int g4 = 4 * g;
#pragma unroll
    for (int v = 0; v < 16; ++v) {
        const int c = 8 * (v >> 2) + (v & 3);
        bool ok = g4 < L - k0 - c;
        if (v < 4) ok = ok && g4 >= -k0 - c;
        if (!ok) sc[v] = -INFINITY;
    }
}
__device__ __forceinline__ float block_maximum(const f32x16& sc)
{
    float mx = sc[0];
#pragma unroll
    for (int v = 1; v < 16; ++v) mx = fmaxf(mx, sc[v]);
    return mx;
}
// New maximum of the queries; what the sums so far have to be multiplied by (no rescaling where no maximum moves).
__device__ __forceinline__ float rescale_sums(float mx, float& mrun, f32x16 (&o)[2], float sl2)
{
    mx = max_across_halves(mx);
    float alpha = 1.f;
    if (__any(mx > mrun)) {
        mx = fmaxf(mx, mrun);
        alpha = exp2_raw((mrun - mx) * sl2);    // first block: exp2(-inf) = 0
        mrun = mx;
#pragma unroll
        for (int db = 0; db < 2; ++db)
#pragma unroll
            for (int e = 0; e < 16; ++e) o[db][e] *= alpha;
    }
    return alpha;
}
// probabilities of a block as the second operand of the values' product: reduction slot e of step s2 is the key of register 8 s2 + e
__device__ __forceinline__ void probabilities(const f32x16& sc, float mrun, float sl2, float& psum, bf16x8 (&pf)[2])
{
    const float nm = -mrun * sl2;
#pragma unroll
    for (int v = 0; v < 16; ++v) {
        const float e = exp2_raw(fmaf(sc[v], sl2, nm));
        psum += e;
        pf[v >> 3][v & 7] = (bf16)e;
    }
}
// A wave's 32 x 64 output block leaves through its own LDS tile (the key/value buffers are idle) as whole 128-byte rows, the first n of
// them; at: element of the first row's first dimension.
__device__ __forceinline__ void store_outputs(char* stg, const f32x16 (&o)[2], float lrun, int ln, int n, bf16* att, unsigned char* attq, size_t at,
                                              int H, float qscale)
{
    const int oq = ln & 31, og = ln >> 5 & 1, orow = ln >> 3 & 7, oc = ln & 7;
    const float inv = 1.0f / sum_across_halves(lrun);
#pragma unroll
    for (int db = 0; db < 2; ++db)
#pragma unroll
        for (int v4 = 0; v4 < 4; ++v4) {
            bf16x4 w;
#pragma unroll
            for (int e = 0; e < 4; ++e) w[e] = (bf16)(o[db][4 * v4 + e] * inv);
            *(bf16x4*)(stg + oq * kOutPitch + (db * 32 + 8 * v4 + 4 * og) * 2) = w;
        }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    at += oc * 8;
#pragma unroll
    for (int r0 = 0; r0 < 32; r0 += 8)
        if (r0 + orow < n) {
            const uint4 c = *(const uint4*)(stg + (r0 + orow) * kOutPitch + oc * 16);
            if (att) *(uint4*)(att + at + (size_t)(r0 + orow) * H) = c;   // (null: the fp8 copy alone)
            if (attq) *(uint2*)(attq + at + (size_t)(r0 + orow) * H) = chunk_to_fp8(c, qscale);
        }
}

// A sequence of up to kShortLen tokens: a wave takes it for one head, the four waves of a workgroup four heads, with nothing to wait for one
// another for.  The keys' blocks and their order are the general part's, so the bits are too: the block in front may begin up to seven
// tokens before the sequence, so there are one or two.  Bound by a chain of one memory round trip, products and exponentials per wave, of
// which sixteen to a compute unit are in flight (128 registers).  us per launch, general part / this: eight students of 768, 256
// sequences of 16 tokens 103 / 44, of 32 131 / 73, 1024 of 4 348 / 90; two students, 256 of 16 28.6 / 13.9.
__device__ __forceinline__ void attention_short(const AttnArgs& p, char* lds, int bid)
{
    // Contiguous runs of (sequence, head group) per XCD (workgroup id mod 8): the lines of the token-contiguous value rows that
    // neighbouring sequences share come into one L2.
    const int groups = (p.heads + 3) >> 2, total = p.B * groups, chunk = (total + 7) >> 3, lin = (bid & 7) * chunk + (bid >> 3);
    if ((bid >> 3) >= chunk || lin >= total) return;
    const int b = lin / groups, m = blockIdx.y;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), h = (lin % groups) * 4 + wave;
    int t0 = p.cu[b], t1 = p.cu[b + 1];
    t0 = t0 < 0 ? 0 : (t0 > p.Tn - 1 ? p.Tn - 1 : t0);
    int L = t1 - t0;
    L = L < 1 ? 1 : L;
    L = L > p.max_seqlen ? p.max_seqlen : L;
    L = L > p.Tn - t0 ? p.Tn - t0 : L;
    if (L > kShortLen || h >= p.heads) return;              // (whole waves, and no barrier below)
    lds += wave * kShortBytes;
    const int j = lane & 31, g = lane >> 5, H = p.H, rows = p.rows;
    const int lead = t0 & 7, vlast = (L + lead - 1) & ~7;
    const bf16* base = p.qkv + ((size_t)m * rows + t0) * (3 * H) + h * kD;
    const bf16* vrows = p.vt + ((size_t)m * H + h * kD) * rows + (t0 - lead);
    const float sl2 = 0.125f * 1.44269504088896341f;        // 1/sqrt(64) * log2(e)
    // 16-byte pieces per lane: keys lane / 8 + 8 i, chunk lane % 8; dimensions lane / 4 + 16 i, chunk lane % 4.  Slots as in the general part
    // (values: four of them per row, slot ^ ((row / 2) % 4)); what lies outside the sequence repeats its first or last row (chunk).
    const bf16* keys = base + H + (lane & 7) * 8;
    const int vc = (lane & 3) * 8;
    bf16x8 kr[4], vr[4], qf[4], k2, v2;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        kr[i] = *(const bf16x8*)(keys + key_tile_offset(-lead, 3 * H) + key_row_offset(-lead, (lane >> 3) + 8 * i, L, 3 * H));
        vr[i] = *(const bf16x8*)(vrows + value_row_offset((lane >> 2) + 16 * i, rows) + (vc < vlast ? vc : vlast));
    }
#pragma unroll
    for (int s4 = 0; s4 < 4; ++s4) qf[s4] = *(const bf16x8*)(base + (size_t)(j < L ? j : L - 1) * (3 * H) + 16 * s4 + 8 * g);
    const bool two = 32 - lead < L;                         // (at most seven keys in the second block: eight rows, a chunk per dimension)
    if (two) {
        k2 = *(const bf16x8*)(keys + key_tile_offset(32 - lead, 3 * H) + key_row_offset(32 - lead, lane >> 3, L, 3 * H));
        v2 = *(const bf16x8*)(vrows + value_row_offset(lane, rows) + 32);
    }
    f32x16 o[2];
    float mrun = -INFINITY, lrun = 0.f;
#pragma unroll
    for (int db = 0; db < 2; ++db)
#pragma unroll
        for (int e = 0; e < 16; ++e) o[db][e] = 0.f;
    const int kdst = (lane >> 3) * 128 + (((lane & 7) ^ (lane >> 4)) << 4);
    auto stage_values = [&](int to, const bf16x8& r) {
        *(bf16x4*)(lds + to) = bf16x4{r[0], r[1], r[2], r[3]};
        *(bf16x4*)(lds + (to ^ 16)) = bf16x4{r[4], r[5], r[6], r[7]};
    };
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        *(bf16x8*)(lds + (kdst ^ (i & 1) * 64) + i * 8 * 128) = kr[i];
        stage_values(kShortKeys + ((lane >> 2) + 16 * i) * 64 + (((lane & 2) ^ (lane >> 3 & 3)) << 4) + 8 * (lane & 1), vr[i]);
    }
    const int krow = j * 128 + ((g ^ ((j >> 1) & 7)) << 4), vrow = kShortKeys + j * 64 + ((g ^ ((j >> 1) & 3)) << 4);
    for (int kt0 = -lead; kt0 < L; kt0 += 32) {
        if (kt0 + lead) {                                   // second block: over the first keys of the first (the others are masked, and finite)
            *(bf16x8*)(lds + kdst) = k2;
            stage_values(kShortKeys + lane * 64 + ((lane >> 1 & 3) << 4), v2);
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        f32x16 sc;
#pragma unroll
        for (int e = 0; e < 16; ++e) sc[e] = 0.f;
#pragma unroll
        for (int s4 = 0; s4 < 4; ++s4) sc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(*(const bf16x8*)(lds + (krow ^ (32 * s4))), qf[s4], sc, 0, 0, 0);
        mask_block(sc, kt0, L, g);
        const float alpha = rescale_sums(block_maximum(sc), mrun, o, sl2);
        float psum = 0.f;
        bf16x8 pf[2];
        probabilities(sc, mrun, sl2, psum, pf);
#pragma unroll
        for (int s2 = 0; s2 < 2; ++s2)
#pragma unroll
            for (int db = 0; db < 2; ++db)
                o[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(*(const bf16x8*)(lds + (vrow ^ (32 * s2)) + db * 32 * 64), pf[s2], o[db], 0, 0, 0);
        lrun = lrun * alpha + psum;
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();                    // (the tiles are written again)
    }
    store_outputs(lds, o, lrun, lane, L, p.att, p.attq, ((size_t)m * rows + t0) * H + h * kD, H, p.qscale);
}

// SHORT: sequences of up to kShortLen tokens are taken by the workgroups behind the general part.
template <bool SHORT>
__global__ __launch_bounds__(256, 4) void attention_bf16_kernel(AttnArgs p)
{
    __shared__ __attribute__((aligned(16))) char lds[kAttnLdsBytes];
    if (SHORT && (int)blockIdx.x >= p.general) return attention_short(p, lds, (int)blockIdx.x - p.general);
    // Workgroup id mod 8 selects the XCD.  Runs of neighbouring items (they share lines of the token-contiguous value rows) stay on one XCD
    // and go round the XCDs, another way for every student.  Long sequences: an XCD takes every eighth (student, head) with all its
    // items, so that the XCDs have the same work whatever the lengths; only the items of the pairs left over go round.
    const int xcd = (int)blockIdx.x & 7, y = (int)blockIdx.x >> 3, rest = y - p.whole * p.items;
    int m = blockIdx.y, h, item;
    if (rest < 0) {
        const int pair = y / p.items * 8 + xcd;
        m = pair / p.heads;
        h = pair - m * p.heads;
        item = y % p.items;
    } else {
        const int pairs = p.whole ? p.pairs - 8 * p.whole : p.heads, s = rest / pairs;
        h = rest - s * pairs;
        item = ((s / p.run) * 8 + ((xcd + m) & 7)) * p.run + s % p.run;
        if (p.whole) {
            h += 8 * p.whole;
            m = h / p.heads;
            h -= m * p.heads;
        }
        if (item >= p.items) return;
    }
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    int t0, t1;
    const int b = last_sequence(p.cu, p.B, lane, [&](int i, int c) { return (c >> 7) + i <= item; }, t0, t1);
    const int q0 = (item - ((t0 >> 7) + b)) * kQItem;
    t0 = t0 < 0 ? 0 : (t0 > p.Tn - 1 ? p.Tn - 1 : t0);
    int L = t1 - t0;
    L = L < 1 ? 1 : L;
    L = L > p.max_seqlen ? p.max_seqlen : L;
    L = L > p.Tn - t0 ? p.Tn - t0 : L;
    if (q0 < 0 || q0 >= L || (SHORT && L <= kShortLen)) return;   // (the whole workgroup)

    const int j = lane & 31, g = lane >> 5;
    const int H = p.H, rows = p.rows;
    const size_t ld = (size_t)3 * H;
    const bf16* base = p.qkv + ((size_t)m * rows + t0) * ld + h * kD;
    // Key tiles start at a token index that is a multiple of 8, so that the values can be fetched 16 bytes at a time; tokens in
    // front of the sequence are masked.
    const int lead = t0 & 7;
    const bf16* vbase = p.vt + ((size_t)m * H + h * kD) * rows + (t0 - lead);
    const bf16* vrows = vbase + value_row_offset(threadIdx.x >> 3, rows);
    const int vlast = (L + lead - 1) & ~7;          // last chunk of eight tokens that holds one of the sequence
    const float sl2 = 0.125f * 1.44269504088896341f;   // 1/sqrt(64) * log2(e)

    // 16-byte pieces of a tile per thread: rows tid / 8 and tid / 8 + 32, chunk tid % 8 in slot (tid % 8) ^ ((row / 2) % 8).  What lies
    // outside the sequence repeats its first or last row (chunk): finite values that get probability zero.
    const int lrow = tid >> 3, lc = tid & 7;
    int dst = lrow * 128 + ((lc ^ ((lrow >> 1) & 7)) << 4);
    auto fetch_keys = [&](int kt0, bf16x8 (&r)[2]) {
#pragma unroll
        for (int i = 0; i < 2; ++i)
            r[i] = *(const bf16x8*)(base + key_tile_offset(kt0, 3 * H) + (key_row_offset(kt0, lrow + 32 * i, L, 3 * H) + (unsigned)(H + lc * 8)));
    };
    auto fetch_values = [&](int kt0, bf16x8 (&r)[2]) {
        const int c = kt0 + lead + lc * 8;
#pragma unroll
        for (int i = 0; i < 2; ++i) r[i] = *(const bf16x8*)(vrows + value_row_offset(32 * i, rows) + (c < vlast ? c : vlast));
    };
    // (values: the two halves of a lane's share of a reduction step, four keys each, side by side: half p of chunk c goes to half
    // c % 2 of slot (c - c % 2 + p) ^ ...)
    int vdst = kTileBytes + lrow * 128 + (((lc & 6) ^ ((lrow >> 1) & 7)) << 4) + 8 * (lc & 1);
    auto stage_keys = [&](int to, const bf16x8 (&r)[2]) {
#pragma unroll
        for (int i = 0; i < 2; ++i) *(bf16x8*)(lds + to + i * 32 * 128) = r[i];
    };
    auto stage_values = [&](int to, const bf16x8 (&r)[2]) {
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            *(bf16x4*)(lds + to + i * 32 * 128) = bf16x4{r[i][0], r[i][1], r[i][2], r[i][3]};
            *(bf16x4*)(lds + (to ^ 16) + i * 32 * 128) = bf16x4{r[i][4], r[i][5], r[i][6], r[i][7]};
        }
    };
    const int q = q0 + 32 * wave;                   // the wave's first query
    bf16x8 qf[4], kr[2], vr[2];
    f32x16 o[2];
    float mrun = -INFINITY, lrun = 0.f;             // running maximum (raw scores); sum over this lane's keys
    // LDS offsets of this lane's row in the current buffer, slot g; slot g + 2 n is at offset ^ 32 n
    int krow = j * 128 + ((g ^ ((j >> 1) & 7)) << 4), vrow = kTileBytes + krow;
    auto scores = [&](int kb) {
        f32x16 sc;
#pragma unroll
        for (int e = 0; e < 16; ++e) sc[e] = 0.f;
#pragma unroll
        for (int s4 = 0; s4 < 4; ++s4) {
            const bf16x8 kf = *(const bf16x8*)(lds + (krow ^ (32 * s4)) + kb * 32 * 128);
            sc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf, qf[s4], sc, 0, 0, 0);
        }
        return sc;
    };
    // a block's values weighted with its probabilities
    auto weigh = [&](const f32x16& sc, int kb, float& psum) {
        bf16x8 pf[2];
        probabilities(sc, mrun, sl2, psum, pf);
#pragma unroll
        for (int s2 = 0; s2 < 2; ++s2)
#pragma unroll
            for (int db = 0; db < 2; ++db) {
                const bf16x8 vf = *(const bf16x8*)(lds + (vrow ^ (64 * kb + 32 * s2)) + db * 32 * 128);
                o[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf, pf[s2], o[db], 0, 0, 0);
            }
    };
    const bool wide = L > kNarrowLen;
    auto tile = [&](int kt0, auto busy) {            // busy: the wave has queries
        const bool more = kt0 + kKeyTile < L, two = kt0 + 32 < L;
        // (the other buffer is idle since the barrier of the previous tile)
        auto next_keys = [&] {                      // keys of the next tile down, its values requested
            if (!more) return;
            stage_keys(dst ^ 2 * kTileBytes, kr);
            __builtin_amdgcn_sched_barrier(0);
            fetch_values(kt0 + kKeyTile, vr);
        };
        // (Without a condition, in front of the last tile those of the last once more: behind a branch the compiler copies what is
        // requested to the registers that the next tile expects it in, and waits for it before it can.)
        auto keys_after = [&] { fetch_keys(kt0 + 2 * kKeyTile < L ? kt0 + 2 * kKeyTile : kt0 + kKeyTile, kr); };
        if constexpr (decltype(busy)::value) {
            f32x16 s0 = scores(0), s1;
            if (two) s1 = scores(1);
            next_keys();
            mask_block(s0, kt0, L, g);
            float mx = block_maximum(s0), mx1 = -INFINITY;
            if (two) {
                mask_block(s1, kt0 + 32, L, g);
                mx1 = block_maximum(s1);
            }
            if (wide) mx = fmaxf(mx, mx1);
            float alpha = rescale_sums(mx, mrun, o, sl2), psum = 0.f;
            weigh(s0, 0, psum);
            if (two) {
                if (!wide) {
                    lrun = lrun * alpha + psum;
                    psum = 0.f;
                    alpha = rescale_sums(mx1, mrun, o, sl2);
                }
                weigh(s1, 1, psum);
            }
            lrun = lrun * alpha + psum;
            if (more) {
                stage_values(vdst ^ 2 * kTileBytes, vr);
                __builtin_amdgcn_sched_barrier(0);
                keys_after();
            }
        } else if (more) {
            next_keys();
            keys_after();
            __builtin_amdgcn_sched_barrier(0);
            stage_values(vdst ^ 2 * kTileBytes, vr);
        }
        barrier_lds();
        dst ^= 2 * kTileBytes;
        vdst ^= 2 * kTileBytes;
        krow ^= 2 * kTileBytes;
        vrow ^= 2 * kTileBytes;
    };
    {
        bf16x8 k0[2], v0[2];
        fetch_keys(-lead, k0);
        fetch_values(-lead, v0);
        const int r = q + j < L ? q + j : L - 1;
#pragma unroll
        for (int s4 = 0; s4 < 4; ++s4) qf[s4] = *(const bf16x8*)(base + (size_t)r * ld + 16 * s4 + 8 * g);
        if (kKeyTile - lead < L) fetch_keys(kKeyTile - lead, kr);
#pragma unroll
        for (int db = 0; db < 2; ++db)
#pragma unroll
            for (int e = 0; e < 16; ++e) o[db][e] = 0.f;
        stage_keys(dst, k0);
        stage_values(vdst, v0);
    }
    barrier_lds();
    // (Two loops, a barrier per tile in either: where the two meet inside one, the compiler waits for the keys on their way.)
    if (q >= L) {
        for (int kt0 = -lead; kt0 < L; kt0 += kKeyTile) tile(kt0, std::false_type{});
        return;
    }
    for (int kt0 = -lead; kt0 < L; kt0 += kKeyTile) tile(kt0, std::true_type{});

    int ln = tid;
    asm volatile("" : "+v"(ln));                    // (what follows from it is not kept through the loop)
    store_outputs(lds + wave * (32 * kOutPitch), o, lrun, ln, L - q, p.att, p.attq, ((size_t)m * rows + t0 + q) * H + h * kD, H, p.qscale);
}

// -------------------------------------------------------------------------------------
// Attention of one query per sequence (its first token), used when only the first-token rows of the last layer are
// needed.  With a single query q per (sequence, head) the key and value projections of the other tokens never
// have to be formed:
//     score_t = q . (Wk^T x_t + bk) = (Wk q) . x_t + q . bk        (q . bk is the same for every t: softmax drops it)
//     out     = sum_t p_t (Wv^T x_t + bv) = Wv^T (sum_t p_t x_t) + bv          (the p_t sum to one)
// so the layer needs q~ = Wk q (one small product per head), one pass over the token rows x that yields the
// p-weighted mean row x^ per head, and Wv^T x^ + bv (another small product per head).  That replaces a projection
// of every token onto 2 H features, and reading those back, by one read of x.
// -------------------------------------------------------------------------------------

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));

// Maximum / sum over the four lanes l % 16 + {0, 16, 32, 48} (every lane active).
__device__ inline float max_across_rows(float v)
{
    float a = v, b = v;
    swap_rows(a, b);
    v = fmaxf(a, b);
    a = v;
    b = v;
    swap_halves(a, b);
    return fmaxf(a, b);
}
__device__ inline float sum_across_rows(float v)
{
    float a = v, b = v;
    swap_rows(a, b);
    v = a + b;
    a = v;
    b = v;
    swap_halves(a, b);
    return a + b;
}

// One workgroup (eight waves, four at hidden 256) per (student, sequence); the sequence's token rows x are read from global
// memory once, in tiles of 32 tokens, and every wave touches only its own share of the features (FW = H / 8 of them):
//   scores: heads x tokens on the matrix cores (16 x 16 x 32 shape: two blocks of 16 tokens, FW / 32 steps of 32
//           features); the token rows arrive in registers in operand layout (lane: token l % 16, eight features); the
//           waves' partial tiles are added in a fixed order through LDS;
//   weighted rows: features x heads, reduction over the tile's 32 tokens in one instruction.  That operand wants eight
//           tokens of one feature per lane, so the wave writes its registers to its own LDS slab (16-byte chunks
//           XOR-swizzled by the token) and reads them back as 4-byte pieces (two neighbouring features) of eight
//           tokens, unzipped into two operands: row r of operand c is feature 2 r + c of a block of 32.  The softmax
//           is the running one (maximum and sum per head, accumulators rescaled when the maximum moves); every wave
//           keeps the statistics of all heads: lane l holds head l % 16 and tokens 8 (l / 16) ... + 8 of the tile.
// The next tile's rows are requested as soon as the current ones are in LDS.  Two workgroup barriers per tile; about
// 66 KB of LDS at hidden width 768 and at most 128 registers, so two workgroups share a compute unit and one's
// start-up and barrier waits are covered by the other.
//   qt   [m][b][head][H]   folded queries (row stride HEADS * H)
//   xbar [m][b][head][H]   output
//
// RAW: the token rows are u, before their LayerNorm x = g (u - mu) r + b (mu and r = 1 / deviation, per token), which nobody else
// needs of all tokens, so that the LayerNorm launch (a read and a write of every row) falls away:
//     q~ . x_t = r_t ((g q~) . u_t - mu_t sum(g q~)) + const,    sum_t p_t x_t = g (a - mean(a)) + b sum_t p_t,  a = sum_t p_t r_t u_t.
// What is rounded to bf16, compared with the fold of x: g q~ in the place of q~ (fold_query_kernel applies g in fp32), w_t = p_t r_t
// in the place of p_t, and x no more.  The weights are normalised by sum_t w_t / r_t over the rounded w_t, so that what their rounding
// has in common cancels: the weight of a token that has all of it is 1 again, to fp32.  sum(g q~) and mean(a) are likewise formed
// from the rounded g q~ and w, so that a mean common to the row's features cancels to fp32.  The variance is a two-pass one: a
// wave's sum of its features (a product with ones), squares about that mean, and the waves' parts joined about the row's mean;
// both numbers cross the waves with the partial scores.  Error of the first tokens' attention output against 64 bits, relative to the
// fold of x, over four widths, flat to very sharp scores, rows of outliers or of a mean of up to 100 deviations: 0.77-0.95, one
// token 1.00.  (E[u^2] - mu^2 from the matrix cores, g applied to the rounded q~ and weights normalised by the sum of the p_t were
// 0.90-1.12, one token 1.0-1.8, and 1-2 us a call faster: eight students of hidden 768 on 14.3 k tokens 2166 / 2174 us, three of 256
// 228.6 / 230.9.)
template <int HEADS, bool RAW>
struct FoldLds {
    // (Four heads: a wave's 32 features would be mostly the exchange between the waves.  Eight heads, 64 features: four waves and eight measured
    // the same, 1061 / 1056 us for eight students on 256 sequences, 574 / 571 for four, 2155 / 2169 on 1024.)
    static constexpr int NW = HEADS == 4 ? 4 : 8;               // waves
    static constexpr int H = HEADS * kD, FW = H / NW;           // features per wave
    static constexpr int SCP = 36;                          // pitch of a head's 32 scores (floats)
    static constexpr size_t slab_bytes = (size_t)32 * FW * 2;   // per wave: 32 tokens x FW features
    static constexpr size_t stats = NW * (slab_bytes + 16 * 32 * 4) + (size_t)16 * SCP * 4;
    static constexpr size_t bytes = stats + (RAW ? 32 * NW * 8 + 2 * 32 * 4 + NW * 16 * 4 : 0);
    static_assert(FW % 32 == 0 && HEADS <= 2 * NW && bytes <= 160 * 1024, "whole reduction steps per wave, a thread per score of a tile");
};

struct FoldArgs {
    const bf16 *x, *qt;
    bf16* xbar;
    size_t qt_ss, xb_ss;
    const int32_t* cu;
    int Tn, rows, max_seqlen;
    const char* arena;                // RAW: scale and shift (byte offsets into a student slab)
    size_t ss, g, b;
    float eps;
    float* parts;                     // SPLIT: [student][p_ss], per item the unscaled rows of its heads (HEADS * H), then maximum and sum of each
    size_t p_ss;
    int B;
};

// SPLIT: sequences in parts of up to kFoldPart tokens, a workgroup each.  Item i belongs to the last sequence b with cu[b] / kFoldPart + b
// <= i, as in the all-token kernel; a sequence's tiles of 32 tokens are dealt evenly over its parts, none of which is empty.  A sequence of
// one part leaves its result, one of several its parts' unscaled sums for fold_join_kernel.
constexpr int kFoldPartLog = 7, kFoldPart = 1 << kFoldPartLog;
__device__ __forceinline__ int fold_parts(int L) { return (L + kFoldPart - 1) >> kFoldPartLog; }
template <int HEADS>
constexpr size_t fold_item_floats() { return (size_t)HEADS * HEADS * kD + 2 * HEADS; }

template <int HEADS, bool RAW, bool SPLIT>
__global__ __launch_bounds__((64 * FoldLds<HEADS, RAW>::NW), (HEADS == 16 ? 2 : 4)) void attention_first_fold_kernel(FoldArgs p)
{
    using F = FoldLds<HEADS, RAW>;
    constexpr int H = F::H, FW = F::FW, SCP = F::SCP, NW = F::NW;
    constexpr int KS = FW / 32;                             // 32-feature steps (scores) = 32-feature blocks (output)
    constexpr int PITCH = FW * 2;                           // slab row, bytes
    extern __shared__ uint4 fold_smem[];
    float* part = (float*)((char*)fold_smem + NW * F::slab_bytes);   // [waves][16][32] partial score tiles
    float* sc = part + NW * 16 * 32;                        // [16][SCP] scores of the current tile, log2 units
    float* stat = (float*)((char*)fold_smem + F::stats);    // [32][waves][2] a wave's features of the tile's rows: sum, squares about their mean
    float* norm = stat + 32 * NW * 2;                       // [2][32] 1 / deviation, deviation
    float* qsum = norm + 2 * 32;                            // [waves][16] sums of the scaled folded queries, later of the weighted rows
    const bf16 *x = p.x, *qt = p.qt;
    const int32_t* cu = p.cu;
    const int Tn = p.Tn, rows = p.rows, max_seqlen = p.max_seqlen;
    const size_t qt_ss = p.qt_ss;
    const int m = blockIdx.y, item = blockIdx.x;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    int t0, t1, b = item;
    if (SPLIT) b = last_sequence(cu, p.B, lane, [&](int i, int c) { return (c >> kFoldPartLog) + i <= item; }, t0, t1);
    else { t0 = cu[b]; t1 = cu[b + 1]; }
    const int part_of = SPLIT ? item - ((t0 >> kFoldPartLog) + b) : 0;
    char* slab = (char*)fold_smem + wave * F::slab_bytes;   // this wave's features of the tile: [token][FW / 8 chunks]
    bf16* xb = p.xbar + (size_t)m * p.xb_ss + (size_t)b * HEADS * H;
    t0 = t0 < 0 ? 0 : (t0 > Tn - 1 ? Tn - 1 : t0);
    int L = t1 - t0;
    L = L < 1 ? 1 : L;
    L = L > max_seqlen ? max_seqlen : L;
    L = L > Tn - t0 ? Tn - t0 : L;
    bool whole = true;
    if (SPLIT) {
        const int n = fold_parts(L), each = ((L + 31) / 32 + n - 1) / n * 32;
        if (part_of < 0 || part_of >= n) return;            // (the whole workgroup: an item without tokens)
        t0 += part_of * each;
        L = L - part_of * each < each ? L - part_of * each : each;
        whole = n == 1;
    }
    const int l16 = lane & 15, kg = lane >> 4;
    const bf16* xw = x + ((size_t)m * rows + t0) * H + wave * FW + 8 * kg;   // this lane's features of the first token
    const int nt = (L + 31) >> 5;

    // folded-query operands: row = head, the wave's features in steps of 32 (lane: eight of them)
    bf16x8 fq[KS];
    {
        const bf16* qr = qt + (size_t)m * qt_ss + ((size_t)b * HEADS + (l16 < HEADS ? l16 : 0)) * H + wave * FW + 8 * kg;
#pragma unroll
        for (int st = 0; st < KS; ++st) {
            fq[st] = *(const bf16x8*)(qr + 32 * st);
            if (l16 >= HEADS) {
#pragma unroll
                for (int e = 0; e < 8; ++e) fq[st][e] = (bf16)0.f;
            }
        }
    }
    bf16x8 ones;
#pragma unroll
    for (int e = 0; e < 8; ++e) ones[e] = (bf16)1.f;
    // token rows of a tile in operand layout: block nb holds tokens 16 nb + l16.  Rows beyond the sequence repeat its
    // last row (they get probability zero).
    bf16x8 xr[2][KS];
    auto load_tile = [&](int tile) {
#pragma unroll
        for (int nb = 0; nb < 2; ++nb) {
            int tok = tile * 32 + 16 * nb + l16;
            tok = tok < L ? tok : L - 1;
#pragma unroll
            for (int st = 0; st < KS; ++st) xr[nb][st] = *(const bf16x8*)(xw + (size_t)tok * H + 32 * st);
        }
    };
    load_tile(0);

    const float scale = 0.125f * 1.44269504088896341f;
    f32x4 acc[2 * KS];                                      // [block of 32 features][c]: feature 2 row + c, column = head
#pragma unroll
    for (int a = 0; a < 2 * KS; ++a) acc[a] = f32x4{0.f, 0.f, 0.f, 0.f};
    float mrun = -INFINITY, lrun = 0.f, qs = 0.f;            // qs: sum of this thread's head's scaled query
    if (RAW) {
        f32x4 a = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int st = 0; st < KS; ++st) a = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fq[st], ones, a, 0, 0, 0);   // rows: heads, columns alike
        if (l16 == 0) *(f32x4*)(qsum + wave * 16 + 4 * kg) = a;
    }
    for (int tile = 0; tile < nt; ++tile) {
        // partial scores[head][token] over this wave's features
        f32x4 sa[2] = {f32x4{0.f, 0.f, 0.f, 0.f}, f32x4{0.f, 0.f, 0.f, 0.f}};
#pragma unroll
        for (int st = 0; st < KS; ++st)
#pragma unroll
            for (int nb = 0; nb < 2; ++nb)
                sa[nb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fq[st], xr[nb][st], sa[nb], 0, 0, 0);   // rows: heads, columns: tokens
#pragma unroll
        for (int nb = 0; nb < 2; ++nb)
#pragma unroll
            for (int v = 0; v < 4; ++v) part[(wave * 16 + 4 * kg + v) * 32 + 16 * nb + l16] = sa[nb][v];
        if (RAW) {
#pragma unroll
            for (int nb = 0; nb < 2; ++nb) {
                f32x4 us = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int st = 0; st < KS; ++st)
                    us = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ones, xr[nb][st], us, 0, 0, 0);       // columns: tokens, rows alike
                const float mean = us[0] * (1.0f / FW);
                float sq = 0.f;
#pragma unroll
                for (int st = 0; st < KS; ++st)
#pragma unroll
                    for (int e = 0; e < 8; ++e) {
                        const float d = (float)xr[nb][st][e] - mean;
                        sq = __builtin_fmaf(d, d, sq);
                    }
                sq = sum_across_rows(sq);
                if (kg == nb) *(f32x2*)(stat + ((16 * nb + l16) * NW + wave) * 2) = f32x2{us[0], sq};
            }
        }
        // the rows into the wave's slab: chunk ch of token r sits in slot ch ^ ((r / 2) % 4).  (The wave's previous
        // reads of the slab are behind it: LDS accesses of one wave execute in order.)
#pragma unroll
        for (int nb = 0; nb < 2; ++nb)
#pragma unroll
            for (int st = 0; st < KS; ++st)
                *(bf16x8*)(slab + (16 * nb + l16) * PITCH + (((4 * st + kg) ^ ((l16 >> 1) & 3)) << 4)) = xr[nb][st];
        __builtin_amdgcn_sched_barrier(0);                  // (the next rows take over the registers of these)
        if (tile + 1 < nt) load_tile(tile + 1);
        barrier_lds();
        {
            int id = tid;
            // (What follows from it is not kept through the loop: with 12 heads three addresses did not fit the registers.  us for the last layer,
            // kept / not, 768 wide, four students on 32 sequences of 340: 100 / 95.)
            if (RAW && SPLIT) asm volatile("" : "+v"(id));
            const int hh = id >> 5, t = id & 31;            // 2 NW heads x 32 sums, one per thread, waves in a fixed order
            float sum = 0.f;
#pragma unroll
            for (int w = 0; w < NW; ++w) sum += part[(w * 16 + hh) * 32 + t];
            if (RAW) {
                if (tile == 0)
#pragma unroll
                    for (int w = 0; w < NW; ++w) qs += qsum[w * 16 + hh];
                f32x4 v[NW / 2];
                float s1 = 0.f, s2 = 0.f;
#pragma unroll
                for (int w = 0; w < NW / 2; ++w) {
                    v[w] = *(const f32x4*)(stat + (t * NW + 2 * w) * 2);
                    s1 += v[w][0];
                    s1 += v[w][2];
                }
                const float mu = s1 * (1.0f / H);
#pragma unroll
                for (int w = 0; w < NW / 2; ++w) {
                    const float d0 = v[w][0] * (1.0f / FW) - mu, d1 = v[w][2] * (1.0f / FW) - mu;
                    s2 += __builtin_fmaf((float)FW * d0, d0, v[w][1]);
                    s2 += __builtin_fmaf((float)FW * d1, d1, v[w][3]);
                }
                const float var = __builtin_fmaf(s2, 1.0f / H, p.eps), r = __builtin_amdgcn_rsqf(var);
                sum = (sum - mu * qs) * r;
                if (hh == 0) {
                    norm[t] = r;
                    norm[32 + t] = var * r;
                }
            }
            sc[hh * SCP + t] = tile * 32 + t < L ? sum * scale : -INFINITY;
        }
        barrier_lds();

        // xbar^T[feature][head] += sum_t x[t][feature] p[head][t]
        const float* sr = sc + (l16 < HEADS ? l16 : 0) * SCP + 8 * kg;
        const f32x4 s0 = *(const f32x4*)sr, s1 = *(const f32x4*)(sr + 4);
        float pr[8];
        float mx = -INFINITY;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            pr[e] = s0[e];
            pr[4 + e] = s1[e];
            mx = fmaxf(mx, fmaxf(s0[e], s1[e]));
        }
        mx = fmaxf(mrun, max_across_rows(mx));              // finite: the tile has at least one token of the sequence
        const float alpha = exp2_raw(mrun - mx);            // first tile: exp2(-inf) = 0
        mrun = mx;
        float ls = 0.f;
#pragma unroll
        for (int e = 0; e < 8; ++e) pr[e] = exp2_raw(pr[e] - mx);
#pragma unroll
        for (int a = 0; a < 2 * KS; ++a) acc[a] *= alpha;
        bf16x8 fp;
        if (RAW) {
            const f32x4 n0 = *(const f32x4*)(norm + 8 * kg), n1 = *(const f32x4*)(norm + 8 * kg + 4);
            const f32x4 d0 = *(const f32x4*)(norm + 32 + 8 * kg), d1 = *(const f32x4*)(norm + 32 + 8 * kg + 4);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                fp[e] = (bf16)(l16 < HEADS ? pr[e] * n0[e] : 0.f);
                fp[4 + e] = (bf16)(l16 < HEADS ? pr[4 + e] * n1[e] : 0.f);
                ls = __builtin_fmaf((float)fp[e], d0[e], ls);
                ls = __builtin_fmaf((float)fp[4 + e], d1[e], ls);
            }
        } else {
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                fp[e] = (bf16)(l16 < HEADS ? pr[e] : 0.f);
                ls += pr[e];
            }
        }
        lrun = fmaf(lrun, alpha, ls);
#pragma unroll
        for (int gq = 0; gq < KS; ++gq) {
            bf16x2 xv[8];
#pragma unroll
            for (int e = 0; e < 8; ++e)                     // token 8 kg + e of the tile: (token / 2) % 4 = e / 2
                xv[e] = *(const bf16x2*)(slab + (8 * kg + e) * PITCH + (((4 * gq + (l16 >> 2)) ^ (e >> 1)) << 4) + (l16 & 3) * 4);
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                bf16x8 fx;
#pragma unroll
                for (int e = 0; e < 8; ++e) fx[e] = xv[e][c];
                acc[2 * gq + c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fx, fp, acc[2 * gq + c], 0, 0, 0);   // rows: features, columns: heads
            }
        }
    }
    // (the lane is counted anew, so that nothing that follows from it is kept through the loop)
    const int ln = (int)__builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
    const int fh = ln & 15, fk = ln >> 4;                   // head; group of four rows
    const float sum = sum_across_rows(lrun), inv = 1.0f / sum;
    if (SPLIT && !whole) {
        float* const out = p.parts + (size_t)m * p.p_ss + (size_t)item * fold_item_floats<HEADS>();
        if (fh < HEADS) {
#pragma unroll
            for (int gq = 0; gq < KS; ++gq)
#pragma unroll
                for (int i = 0; i < 8; i += 4)
                    *(f32x4*)(out + (size_t)fh * H + wave * FW + 32 * gq + 8 * fk + i) =
                        f32x4{acc[2 * gq][i >> 1], acc[2 * gq + 1][i >> 1], acc[2 * gq][(i >> 1) + 1], acc[2 * gq + 1][(i >> 1) + 1]};
            if (wave == 0 && fk == 0) *(f32x2*)(out + HEADS * H + 2 * fh) = f32x2{mrun, sum};
        }
        return;
    }
    const float *gam = (const float*)(p.arena + (size_t)m * p.ss + p.g) + wave * FW, *bet = (const float*)(p.arena + (size_t)m * p.ss + p.b) + wave * FW;
    float common = 0.f;                                     // mean of the head's weighted row over the features
    if (RAW) {
        float t = 0.f;
#pragma unroll
        for (int a = 0; a < 2 * KS; ++a) t += acc[a][0] + acc[a][1] + (acc[a][2] + acc[a][3]);
        t = sum_across_rows(t);
        if (fk == 0) qsum[wave * 16 + fh] = t;              // (the queries' sums were read before the last tile's barriers)
        barrier_lds();
#pragma unroll
        for (int w = 0; w < NW; ++w) common += qsum[w * 16 + fh];
        common *= 1.0f / H;
    }
    // lane: head fh; element v of acc[2 gq + c] is feature 32 gq + 2 (4 fk + v) + c of the wave's FW
    if (fh < HEADS) {
#pragma unroll
        for (int gq = 0; gq < KS; ++gq) {
            bf16x8 r;
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                float v = acc[2 * gq + (i & 1)][i >> 1];
                if (RAW) v = gam[32 * gq + 8 * fk + i] * ((v - common) * inv) + bet[32 * gq + 8 * fk + i];
                else v *= inv;
                r[i] = (bf16)v;
            }
            *(bf16x8*)(xb + (size_t)fh * H + wave * FW + 32 * gq + 8 * fk) = r;
        }
    }
}

// Sequences of several parts: their sums at a common maximum, scaled (RAW: with the LayerNorm's scale and shift as above); a wave per head.
template <int HEADS, bool RAW>
__global__ __launch_bounds__(256) void fold_join_kernel(FoldArgs p)
{
    constexpr int H = HEADS * kD, NC = (H / 4 + 63) / 64;   // chunks of four features per lane
    const int m = blockIdx.y, b = blockIdx.x / (HEADS / 4), lane = threadIdx.x & 63;
    const int h = (int)(blockIdx.x % (HEADS / 4)) * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    int t0 = p.cu[b], t1 = p.cu[b + 1];
    int first = (t0 >> kFoldPartLog) + b;
    t0 = t0 < 0 ? 0 : (t0 > p.Tn - 1 ? p.Tn - 1 : t0);
    int L = t1 - t0;
    L = L < 1 ? 1 : L;
    L = L > p.max_seqlen ? p.max_seqlen : L;
    L = L > p.Tn - t0 ? p.Tn - t0 : L;
    const int n = fold_parts(L);
    if (n == 1) return;
    const int last = (p.Tn >> kFoldPartLog) + p.B - n;      // (boundaries out of order: some items, but no others than there are)
    first = first < 0 ? 0 : (first > last ? last : first);
    const float* from = p.parts + (size_t)m * p.p_ss + (size_t)first * fold_item_floats<HEADS>();
    f32x4 acc[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c) acc[c] = f32x4{0.f, 0.f, 0.f, 0.f};
    float mrun = -INFINITY, lrun = 0.f;
    for (int i = 0; i < n; ++i, from += fold_item_floats<HEADS>()) {
        const f32x2 ml = *(const f32x2*)(from + HEADS * H + 2 * h);
        f32x4 v[NC];
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            const int e = 4 * (lane + 64 * c);
            v[c] = e < H ? *(const f32x4*)(from + (size_t)h * H + e) : f32x4{0.f, 0.f, 0.f, 0.f};
        }
        const float mx = fmaxf(mrun, ml[0]), down = exp2_raw(mrun - mx), w = exp2_raw(ml[0] - mx);      // (first part: exp2(-inf) = 0)
        mrun = mx;
        lrun = fmaf(lrun, down, ml[1] * w);
#pragma unroll
        for (int c = 0; c < NC; ++c) acc[c] = acc[c] * down + v[c] * w;
    }
    const float inv = 1.0f / lrun;
    float common = 0.f;
    if (RAW) {
#pragma unroll
        for (int c = 0; c < NC; ++c) common += acc[c][0] + acc[c][1] + (acc[c][2] + acc[c][3]);
        common = wave_sum(common) * (1.0f / H);
    }
    const char* sb = p.arena + (size_t)m * p.ss;
    bf16* out = p.xbar + (size_t)m * p.xb_ss + ((size_t)b * HEADS + h) * H;
#pragma unroll
    for (int c = 0; c < NC; ++c) {
        const int e0 = 4 * (lane + 64 * c);
        if (e0 >= H) continue;
        bf16x4 o;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            float v = (acc[c][e] - common) * inv;
            if (RAW) v = ((const float*)(sb + p.g))[e0 + e] * v + ((const float*)(sb + p.b))[e0 + e];
            o[e] = (bf16)v;
        }
        *(bf16x4*)(out + e0) = o;
    }
}

// -------------------------------------------------------------------------------------
// fp32 kernel: one workgroup per (student, sequence, head, block of 256 / LQ queries); LQ neighbouring lanes share a query,
// 64 / LQ of the head's dimensions each (a score is summed over them, every lane rescales and accumulates its own output
// dimensions).  Keys and values come through LDS in chunks of 64 tokens; the queries of a wave read the same key row (a
// broadcast).  Online softmax in registers by blocks of eight keys, whose scores do not wait for one another; exact
// exponentials and division.
// Bound by latency in small calls (two launches of them are a third of the smallest fp32 call): a chain of keys per query, so
// sixteen lanes share one while the workgroups are few; four (fewer instructions in all) where they fill the chip.  us, key by key
// with four lanes / this: two students, four sequences of 8-32 tokens 10.8 / 6.0.
// -------------------------------------------------------------------------------------
template <int LQ>
__global__ __launch_bounds__(256) void attention_f32_kernel(const float* __restrict__ qkv, float* __restrict__ att,
                                                            const int32_t* __restrict__ cu, int B, int Tn, int rows,
                                                            int H, int heads, int max_seqlen, int nqc)
{
    constexpr int KC = 64, DP = kD / LQ, QW = 256 / LQ, KB = 8;   // keys per chunk; dimensions per lane; queries per workgroup; keys per block
    __shared__ __attribute__((aligned(16))) float Ks[KC][kD], Vs[KC][kD];
    const int m = blockIdx.y;
    int idx = blockIdx.x;
    const int qc = idx % nqc; idx /= nqc;
    const int h = idx % heads;
    const int b = idx / heads;
    int t0 = cu[b], t1 = cu[b + 1];
    t0 = t0 < 0 ? 0 : (t0 > Tn - 1 ? Tn - 1 : t0);
    int L = t1 - t0;
    L = L < 1 ? 1 : L;
    L = L > max_seqlen ? max_seqlen : L;
    L = L > Tn - t0 ? Tn - t0 : L;
    if (qc * QW >= L) return;                               // (uniform over the workgroup)
    const int tid = threadIdx.x, part = tid % LQ, q = qc * QW + tid / LQ;
    const bool live = q < L;
    const size_t ld = (size_t)3 * H;
    const float* base = qkv + ((size_t)m * rows + t0) * ld + h * kD;
    float qv[DP], o[DP];
#pragma unroll
    for (int e4 = 0; e4 < DP; e4 += 4) {
        const f32x4 t = live ? *(const f32x4*)(base + (size_t)q * ld + DP * part + e4) : f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int e = 0; e < 4; ++e) { qv[e4 + e] = t[e]; o[e4 + e] = 0.f; }
    }
    float mrun = -INFINITY, lrun = 0.f;
    for (int kt0 = 0; kt0 < L; kt0 += KC) {
        const int nk = L - kt0 < KC ? L - kt0 : KC;
        __syncthreads();                                    // the previous chunk has been read by everybody
#pragma unroll
        for (int i = 0; i < KC * kD / 4 / 256; ++i) {
            const int c = tid + 256 * i, key = c >> 4, d = (c & 15) * 4;
            if (key < nk) {
                const float* kr = base + (size_t)(kt0 + key) * ld + H + d;
                *(f32x4*)&Ks[key][d] = *(const f32x4*)kr;
                *(f32x4*)&Vs[key][d] = *(const f32x4*)(kr + H);
            }
        }
        __syncthreads();
        for (int k0 = 0; k0 < nk; k0 += KB) {
            float s[KB], mx = mrun;                         // (keys behind the last one repeat it, with probability zero)
#pragma unroll
            for (int i = 0; i < KB; ++i) {
                const int key = k0 + i < nk ? k0 + i : nk - 1;
                s[i] = 0.f;
#pragma unroll
                for (int e4 = 0; e4 < DP; e4 += 4) {
                    const f32x4 kv = *(const f32x4*)&Ks[key][DP * part + e4];
#pragma unroll
                    for (int e = 0; e < 4; ++e) s[i] = fmaf(qv[e4 + e], kv[e], s[i]);
                }
            }
#pragma unroll
            for (int i = 0; i < KB; ++i) {                  // over the lanes of a query: every one ends with the whole sum
                s[i] += dpp_moved<kDppPair>(s[i]);
                s[i] += dpp_moved<kDppQuad>(s[i]);
                if (LQ == 16) {
                    s[i] += dpp_moved<kDppHalfRowMirror>(s[i]);
                    s[i] += dpp_moved<kDppRowMirror>(s[i]);
                }
                s[i] *= 0.125f;
                mx = fmaxf(mx, s[i]);
            }
            const float alpha = expf(mrun - mx);
            lrun *= alpha;
#pragma unroll
            for (int e = 0; e < DP; ++e) o[e] *= alpha;
#pragma unroll
            for (int i = 0; i < KB; ++i) {
                const int key = k0 + i < nk ? k0 + i : nk - 1;
                const float p = k0 + i < nk ? expf(s[i] - mx) : 0.f;
                lrun += p;
#pragma unroll
                for (int e4 = 0; e4 < DP; e4 += 4) {
                    const f32x4 vv = *(const f32x4*)&Vs[key][DP * part + e4];
#pragma unroll
                    for (int e = 0; e < 4; ++e) o[e4 + e] = fmaf(p, vv[e], o[e4 + e]);
                }
            }
            mrun = mx;
        }
    }
    if (live) {
        float* dst = att + ((size_t)m * rows + t0 + q) * H + h * kD + DP * part;
#pragma unroll
        for (int e4 = 0; e4 < DP; e4 += 4)
            *(f32x4*)(dst + e4) = f32x4{o[e4] / lrun, o[e4 + 1] / lrun, o[e4 + 2] / lrun, o[e4 + 3] / lrun};
    }
}

}  // namespace

hipError_t launch_attention(const sp_model* M, const void* qkv, const void* vt, void* att, const int32_t* cu, int B,
                            int T, int max_seqlen, int rows, int k, hipStream_t s, void* attq, float qscale)
{
    const sp_config& c = M->cfg;
    if (c.hidden / c.heads != kD) return hipErrorInvalidValue;
    if (!att && !(attq && bf16_path(c))) return hipErrorInvalidValue;   // (no bf16 output: the fp8 copy alone)
    if (bf16_path(c)) {
        // Runs of neighbouring items that stay on one XCD: 1, 2, 4, 8 and 16 measured 208 / 208 / 207 / 210 / 211 us on 371 items of
        // short sequences (eight students), 325 / 322 / 326 / 328 / 347 on 208 of long ones (six); few items go round one by one.
        AttnArgs a{(const bf16*)qkv, (const bf16*)vt, (bf16*)att, (unsigned char*)attq, cu, qscale, B, T, rows, c.hidden, c.heads,
                   max_seqlen, T / kQItem + B, 1, c.heads * k, max_seqlen > kShortLen && T >= (int64_t)kQItem * B ? c.heads * k / 8 : 0, 0};
        // A pair's items all on one XCD from a mean of 128 tokens on (all the host knows): going round the XCDs, what an XCD gets of long and
        // short sequences evens out over the students only.  us per launch, round / this: 64 sequences of 64-512 tokens, 16 heads, one student
        // 65.0 / 60.0, six 348 / 345; 256 of 8-256 (mean 57), 12 heads, eight students, whose heads then are read by different XCDs: 214 / 221.
        a.run = a.items < 128 ? 1 : (a.items < 256 ? 2 : 4);
        const int nitems = (a.items + 8 * a.run - 1) / (8 * a.run) * (8 * a.run), nshort = (B * ((c.heads + 3) / 4) + 7) / 8 * 8;
        // Sequences of up to 32 tokens by single waves: alone where there are no others; beside the general part, whose workgroups then leave for
        // those, where most are short (by the mean, all the host knows) and half a workgroup per compute unit comes together.  us a call,
        // general part alone / this.  768 wide, eight students: 300 sequences of 4 tokens 496 / 426, 256 of 16 793 / 736, of 32 1290 / 1244; 256
        // lognormal ones of mean 15 782 / 755, 24 1095 / 1075, 39 1588 / 1577, 58 2213 / 2207; two students, 24 of mean 25 102 / 102, 42 124 / 125.
        // 256 wide, three students: 256 of 16 122 / 114, mean 24 144 / 142; 24 of mean 25 67.6 / 68.2, 36 71.3 / 71.9.
        const bool few = (long)B * ((c.heads + 3) / 4) * k < 128, only = max_seqlen <= kShortLen, mixed = !only && !few && T <= (int64_t)32 * B;
        a.general = only ? 0 : 8 * a.whole * a.items + nitems * (a.whole ? a.pairs - 8 * a.whole : c.heads);
        const dim3 grid((unsigned)(a.general + (only || mixed ? nshort : 0)), a.whole ? 1 : k);
        if (only || mixed) hipLaunchKernelGGL(attention_bf16_kernel<true>, grid, dim3(256), 0, s, a);
        else hipLaunchKernelGGL(attention_bf16_kernel<false>, grid, dim3(256), 0, s, a);
    } else {
        // Sixteen lanes per query: four times the workgroups; up to about two of them per compute unit.  us a call, four lanes / sixteen, two
        // students, by workgroups of the latter: hidden 128: 16 44.5 / 38.5, 128 113 / 107, 256 (sequences of 128-256) 211 / 173, 512 182 / 179 and,
        // of long sequences, 276 / 255, 960 344 / 356; hidden 768: 96 310 / 304, 384 776 / 773, 768 1252 / 1251, 1536 1661 / 1664 and 1799 / 1847.
        const int nq16 = (max_seqlen + 15) / 16, nq4 = (max_seqlen + 63) / 64;
        if ((long)B * c.heads * nq16 * k <= 512)
            hipLaunchKernelGGL(attention_f32_kernel<16>, dim3((unsigned)(B * c.heads * nq16), k), dim3(256), 0, s, (const float*)qkv,
                               (float*)att, cu, B, T, rows, c.hidden, c.heads, max_seqlen, nq16);
        else
            hipLaunchKernelGGL(attention_f32_kernel<4>, dim3((unsigned)(B * c.heads * nq4), k), dim3(256), 0, s, (const float*)qkv,
                               (float*)att, cu, B, T, rows, c.hidden, c.heads, max_seqlen, nq4);
    }
    return hipGetLastError();
}

bool attention_first_fold_supported(const sp_config& c, int max_seqlen)
{
    (void)max_seqlen;                                       // any length: the softmax is a running one
    return bf16_path(c) && c.hidden / c.heads == kD && c.heads % 4 == 0 && c.heads <= 16;
}

// Whether sequences are split, in calls that have the buffers for it.  work: sequences x students.  Few long sequences alone, by the mean
// length, all the host knows: a part costs the way to its first rows (3-4 us; a tile of 32 tokens takes 1.4-3 us) and its sums a write, a
// read and one more launch.  us a call, whole / split, by sequences x students, mean: 768 wide: 4 400 130 / 117, 16 512 228 / 215, 32 140 161 / 163,
// 64 190 316 / 316, 256 140 697 / 710, 256 319 804 / 790; six layers: 32 382 1231 / 1220; 1024 wide: 4 377 148 / 136, 96 191 594 / 594, 252 287
// 2093 / 2117; 256 wide: 48 317 98.6 / 95.7, 255 192 161.5 / 163.8.
bool fold_splits(const sp_config& c, int B, int T, long work, size_t bytes)
{
    const size_t items = (size_t)(T >> kFoldPartLog) + B, floats = (size_t)c.heads * c.hidden + 2 * c.heads;
    return T >= (int64_t)2 * kFoldPart * B && work <= 128 && items * floats * 4 <= bytes;
}

hipError_t launch_attention_first_fold(const sp_model* M, const void* x, const void* qt, size_t qt_ss, void* xbar,
                                       size_t xb_ss, const int32_t* cu, int B, int T, int max_seqlen, int rows, int k,
                                       hipStream_t s, bool raw, size_t g_off, size_t b_off, float* parts, size_t p_ss)
{
    const sp_config& c = M->cfg;
    if (!attention_first_fold_supported(c, max_seqlen)) return hipErrorInvalidValue;
    const FoldArgs a{(const bf16*)x, (const bf16*)qt, (bf16*)xbar, qt_ss, xb_ss, cu, T, rows, max_seqlen, M->arena, M->L.student_stride,
                     g_off, b_off, c.ln_eps, parts, p_ss, B};
    const dim3 grid((unsigned)(parts ? (T >> kFoldPartLog) + B : B), (unsigned)k);
#define SP_FOLD(HEADS, RAW, SPLIT)                                                                                  \
    do {                                                                                                            \
        auto kern = attention_first_fold_kernel<HEADS, RAW, SPLIT>;                                                 \
        constexpr size_t smem = FoldLds<HEADS, RAW>::bytes;                                                         \
        static std::atomic<bool> raised{false}; /* the attribute is sticky for the process */                      \
        if (smem > 48 * 1024 && !raised) {                                                                          \
            hipError_t e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize,      \
                                               (int)smem);                                                          \
            if (e != hipSuccess) return e;                                                                          \
            raised = true;                                                                                          \
        }                                                                                                           \
        hipLaunchKernelGGL(kern, grid, dim3((64 * FoldLds<HEADS, RAW>::NW)), smem, s, a);                           \
        if (SPLIT) {                                                                                                \
            const hipError_t e = hipGetLastError();                                                                 \
            if (e != hipSuccess) return e;                                                                          \
            hipLaunchKernelGGL((fold_join_kernel<HEADS, RAW>), dim3((unsigned)(B * (HEADS / 4)), (unsigned)k), dim3(256), 0, s, a); \
        }                                                                                                           \
    } while (0)
#define SP_FOLD_RAW(HEADS, RAW) do { if (parts) SP_FOLD(HEADS, RAW, true); else SP_FOLD(HEADS, RAW, false); } while (0)
#define SP_FOLD_ANY(HEADS) do { if (raw) SP_FOLD_RAW(HEADS, true); else SP_FOLD_RAW(HEADS, false); } while (0)
    switch (c.heads) {
        case 4: SP_FOLD_ANY(4); break;
        case 8: SP_FOLD_ANY(8); break;
        case 12: SP_FOLD_ANY(12); break;
        default: SP_FOLD_ANY(16); break;
    }
#undef SP_FOLD_ANY
#undef SP_FOLD_RAW
#undef SP_FOLD
    return hipGetLastError();
}

}  // namespace sp
