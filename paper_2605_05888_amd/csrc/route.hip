// Routing (Section II-A, step 1): gating logits in the fixed fp32 order that makes
// the top-K selection reproducible bit for bit, then selection and normalisation.
//
// Order of the logit sum ("R64"): 64 partial sums, partial l takes
// h = l, l+64, ... ascending with one fused multiply-add per term; the partials
// are folded in six pairwise rounds s = 32,...,1 (p[l] + p[l^s]); bias last.
//
// The products run on the matrix cores without giving up that order.  v_mfma_f32_16x16x1_4B_f32 multiplies
// four independent 16x1 by 1x16 pairs: with a reduction length of ONE every output is exactly one fused
// multiply-add, d = fma(a, b, c) (checked bit for bit against fmaf, signed zeros and subnormal products
// included), so nothing about the summation order is left to the hardware.  The four blocks of an
// instruction are four different partials; sixteen instructions cover all 64 for 16 tokens x 16 experts:
//   a operand, lane (blk = lane / 16, c = lane % 16):  x[token c, h]       h = 64 step + l
//   b operand:                                         W_r[h, expert c]
//   result register 4 b + t of lane (q, c):            partial of block b, token 4 q + t, expert c
// A wavefront takes a share of the partials (64 / kSplit of them, kG = 16 / kSplit instructions per step of
// 64 columns): wavefront `ps` of a group of kSplit has l = 4 kG ps + kG blk + g.  The rounds of the fold that
// pair partials of different wavefronts (the high bits of l) come first and go through LDS; all the others
// pair registers of one lane.
//
// Tokens past N and experts past E repeat the last one (their results are not stored).  Rows of W_r past H
// count as zeros, and so do columns of x past H: adding a zero product never changes a partial
// sum (partials start at +0 and can never become -0), so a ragged last step gives the R64 sum bit for bit.
#include <math.h>

#include <type_traits>

#include "common.h"

namespace moe {

constexpr int kRouteWaves = 4; // wavefronts per workgroup of the selection kernel
constexpr int kRtExp = 16, kRtTok = 16;

__device__ const u32x4 kZeroColumns = {0u, 0u, 0u, 0u}; // 16 bytes of x past H

// Four columns of x (bf16: two per register) or fewer, as fetched; see x_value.
template <bool kBf16, int kG>
struct XChunk {
    static constexpr int kRegs = kBf16 ? kG / 2 : kG;
    uint32_t r[kRegs];
};
template <bool kBf16, int kG>
__device__ __forceinline__ float x_value(const XChunk<kBf16, kG> &c, int g)
{
    if (kBf16)
        return __uint_as_float(g & 1 ? c.r[g / 2] & 0xFFFF0000u : c.r[g / 2] << 16);
    return __uint_as_float(c.r[g]);
}
template <bool kBf16, int kG>
__device__ __forceinline__ XChunk<kBf16, kG> load_chunk(const unsigned char *p)
{
    XChunk<kBf16, kG> c;
    constexpr int n = XChunk<kBf16, kG>::kRegs;
    if constexpr (n % 4 == 0) {
#pragma unroll
        for (int i = 0; i < n / 4; ++i) {
            const u32x4 v = *reinterpret_cast<const u32x4 *>(p + 16 * i);
#pragma unroll
            for (int j = 0; j < 4; ++j)
                c.r[4 * i + j] = v[j];
        }
    } else if constexpr (n == 2) {
        const u32x2 v = *reinterpret_cast<const u32x2 *>(p);
        c.r[0] = v[0], c.r[1] = v[1];
    } else {
        static_assert(n == 1, "chunk of one, two or a multiple of four registers");
        c.r[0] = *reinterpret_cast<const uint32_t *>(p);
    }
    return c;
}

// Rounds of the fold inside a lane: v[b * kG + g] over blocks b (two bits, high first), then g.
template <int kG>
__device__ __forceinline__ float fold_in_lane(float *v)
{
#pragma unroll
    for (int s = 2 * kG; s >= 1; s >>= 1)
#pragma unroll
        for (int i = 0; i < s; ++i)
            v[i] = v[i] + v[i + s];
    return v[0];
}

// Value of the lane `kRor` places away inside a row of sixteen lanes.
template <int kRor, class T>
__device__ __forceinline__ T row_ror(T v)
{
    return __builtin_bit_cast(T, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x120 + kRor, 0xf, 0xf, true));
}
__device__ __forceinline__ float row_max16(float v)
{
    v = fmaxf(v, row_ror<8>(v));
    v = fmaxf(v, row_ror<4>(v));
    v = fmaxf(v, row_ror<2>(v));
    return fmaxf(v, row_ror<1>(v));
}
__device__ __forceinline__ float row_sum16(float v)
{
    v += row_ror<8>(v);
    v += row_ror<4>(v);
    v += row_ror<2>(v);
    return v + row_ror<1>(v);
}

// (value, index) order of the selection: larger logit first, equal logits to the lower index.
__device__ __forceinline__ bool better(float va, int ia, float vb, int ib)
{
    return (va > vb) || (va == vb && ia < ib);
}

__device__ __forceinline__ float score(float logit, float top, int score_mode)
{
    return score_mode == MOE_SCORE_SOFTMAX_TOPK ? expf(logit - top) : 1.0f / (1.0f + expf(-logit));
}

template <int kStep>
__device__ __forceinline__ int count_better(float v, int e, int rank)
{
    if constexpr (kStep == 16) {
        return rank;
    } else {
        if (better(row_ror<kStep>(v), row_ror<kStep>(e), v, e))
            ++rank;
        return count_better<kStep + 1>(v, e, rank);
    }
}

// ------------------------------------------------------------------------
// Small launches (and any E): a workgroup of eight wavefronts computes 16 tokens x 16 experts, every
// wavefront an eighth of the partials (two instructions per step).  What bounds it is latency, so operands are
// fetched three batches of kBatch steps ahead.  A wavefront's rows of W_r are its own and go straight to
// registers; x goes through LDS (loaded there directly): in the operand layout neighbouring lanes hold different
// tokens, and fetching it like that costs the vector cache one access per lane instead of one per 64 bytes.
// With at most 16 experts a row of sixteen lanes holds all logits of a token and selects its top K at once
// (kSelect): no second launch.
// Routing with selection, 4x4x1 instructions on 32 tokens per workgroup before -> now: 1 token, H = 7168, 256
// experts 45 -> 21 us; 37 tokens, H = 2880, 128 experts 24 -> 13; 128 / 4096 tokens, H = 4096, 8 experts 26 / 28 ->
// 12 / 13; 4096 tokens, H = 1024, 30 experts 28 -> 13.
// ------------------------------------------------------------------------
template <bool kBf16, bool kSelect>
__global__ __launch_bounds__(512, 2) void router_logits_small(
    const void *__restrict__ x, int64_t N, int64_t H, const float *__restrict__ W_r, const float *__restrict__ bias,
    int E, float *__restrict__ logits, int K, int score_mode, int32_t *__restrict__ topk_idx,
    float *__restrict__ topk_w, int row_tiles)
{
#if defined(__HIP_DEVICE_COMPILE__)
    constexpr int kSplit = 8, kG = 2, kXb = kBf16 ? 2 : 4, kBatch = 8, kSets = 4;
    constexpr int kCols = kBatch * kWave;            // columns of a batch
    constexpr int kXRow = kCols * kXb;               // bytes of a token's columns: 1 or 2 KiB
    constexpr int kXStage = kRtTok * kXRow;
    constexpr int kXLoads = kXStage / 1024 / kSplit; // per wavefront and batch
    constexpr int kFold = kSplit * kG * 16 * kWave * 4;
    __shared__ __attribute__((aligned(1024))) unsigned char lds[kSets * kXStage > kFold ? kSets * kXStage : kFold];
    const int lane = threadIdx.x % kWave;
    const int ps = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int blk = lane / 16, c = lane % 16;
    const int e_tiles = (E + kRtExp - 1) / kRtExp;
    const int e0 = (int)(blockIdx.x % e_tiles) * kRtExp;
    const int64_t n0 = ((int64_t)blockIdx.y * row_tiles + blockIdx.x / e_tiles) * kRtTok;
    if (n0 >= N) // (the last row of the grid)
        return;
    const int l0 = 4 * kG * ps + kG * blk; // first of the lane's kG partials
    const float *pw = W_r + (int64_t)l0 * E + (e0 + c < E ? e0 + c : E - 1);

    // x: a load instruction of a wavefront fills 1 KiB; the 16-byte chunk at position p of token row r is chunk
    // p ^ r, so that the operand reads (sixteen rows at one column) spread over the banks
    const unsigned char *px[kXLoads];
    int x_col[kXLoads]; // first column of the lane's chunk inside a batch
#pragma unroll
    for (int i = 0; i < kXLoads; ++i) {
        const int at = (ps * kXLoads + i) * 1024 + lane * 16, r = at / kXRow;
        x_col[i] = (((at % kXRow) / 16) ^ r) * (16 / kXb);
        const int64_t tok = n0 + r < N ? n0 + r : N - 1;
        px[i] = static_cast<const unsigned char *>(x) + (tok * H + x_col[i]) * kXb;
    }
    struct Weights {
        float w[kBatch][kG];
    };
    // batch i: x into LDS stage `set`, W_r into registers.  Chunks of x past H: zeros (the row's own values would do as
    // long as they are finite; an infinity among them would make every logit of the token NaN).
    auto fetch = [&](Weights &b, int64_t i, int set) {
        const int64_t h0 = i * kCols;
        const bool whole = h0 + kCols <= H;
#pragma unroll
        for (int j = 0; j < kXLoads; ++j) {
            const unsigned char *const from = whole || h0 + x_col[j] < H
                                                  ? px[j] + h0 * kXb
                                                  : reinterpret_cast<const unsigned char *>(&kZeroColumns);
            __builtin_amdgcn_global_load_lds(
                (const __attribute__((address_space(1))) void *)from,
                (__attribute__((address_space(3))) void *)(lds + set * kXStage + (ps * kXLoads + j) * 1024), 16, 0, 0);
        }
        if (whole) {
#pragma unroll
            for (int s = 0; s < kBatch; ++s)
#pragma unroll
                for (int g = 0; g < kG; ++g)
                    b.w[s][g] = pw[(h0 + s * kWave + g) * E];
        } else {
#pragma unroll
            for (int s = 0; s < kBatch; ++s)
#pragma unroll
                for (int g = 0; g < kG; ++g) { // (H is even: both of the lane's columns or none)
                    const bool in = h0 + s * kWave + l0 < H;
                    const float v = pw[(in ? h0 + s * kWave + g : -(int64_t)l0) * E];
                    b.w[s][g] = in ? v : 0.0f;
                }
        }
    };

    f32x16 acc[kG];
#pragma unroll
    for (int g = 0; g < kG; ++g)
#pragma unroll
        for (int r = 0; r < 16; ++r)
            acc[g][r] = 0.0f;
    auto multiply = [&](const Weights &b, int set) {
        const unsigned char *row = lds + set * kXStage + c * kXRow;
        XChunk<kBf16, kG> xv[kBatch];
#pragma unroll
        for (int s = 0; s < kBatch; ++s) {
            const int byte = (s * kWave + l0) * kXb;
            xv[s] = load_chunk<kBf16, kG>(row + (((byte / 16) ^ c) * 16 + byte % 16));
        }
#pragma unroll
        for (int s = 0; s < kBatch; ++s)
#pragma unroll
            for (int g = 0; g < kG; ++g)
                acc[g] = __builtin_amdgcn_mfma_f32_16x16x1f32(x_value(xv[s], g), b.w[s][g], acc[g], 0, 0, 0);
    };
    const int64_t batches = (H + kCols - 1) / kCols;
    // batch i has landed (own loads: all but the ones of the two batches after it; everyone's: the barrier)
    auto turn = [&](int64_t i, int set, const Weights &now, Weights &later) {
        constexpr int kInFlight = 2 * (kXLoads + kBatch * kG);
        __builtin_amdgcn_s_waitcnt(0x0070 | (kInFlight & 15) | (kInFlight >> 4 << 14)); // (and my reads of i - 1)
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        fetch(later, i + 3 < batches ? i + 3 : batches - 1, (set + 3) % kSets); // (past the last: once more, unused)
        __builtin_amdgcn_sched_barrier(0);
        multiply(now, set);
    };
    Weights w0, w1, w2, w3;
    fetch(w0, 0, 0);
    fetch(w1, 1 < batches ? 1 : batches - 1, 1);
    fetch(w2, 2 < batches ? 2 : batches - 1, 2);
    int64_t i = 0;
    for (; i + 3 < batches; i += 4) {
        turn(i, 0, w0, w3);
        turn(i + 1, 1, w1, w0);
        turn(i + 2, 2, w2, w1);
        turn(i + 3, 3, w3, w2);
    }
    if (i < batches)
        turn(i, 0, w0, w3);
    if (i + 1 < batches)
        turn(i + 1, 1, w1, w0);
    if (i + 2 < batches)
        turn(i + 2, 2, w2, w1);
    __builtin_amdgcn_s_waitcnt(0x0F70); // the loads past the last batch (they write LDS too)
    __syncthreads();

    // fold: rounds 32, 16, 8 pair wavefronts ps and ps ^ 4, ^ 2, ^ 1
    float *const part = reinterpret_cast<float *>(lds); // [wavefront][kG * 16][lane]
#pragma unroll
    for (int g = 0; g < kG; ++g)
#pragma unroll
        for (int r = 0; r < 16; ++r)
            part[(ps * kG * 16 + g * 16 + r) * kWave + lane] = acc[g][r];
    __syncthreads();
    if (ps >= 4)
        return;
    const int t = ps; // this wavefront finishes tokens 4 q + t
    float v[4 * kG];
#pragma unroll
    for (int b = 0; b < 4; ++b)
#pragma unroll
        for (int g = 0; g < kG; ++g) {
            float p[kSplit];
#pragma unroll
            for (int w = 0; w < kSplit; ++w)
                p[w] = part[(w * kG * 16 + g * 16 + 4 * b + t) * kWave + lane];
#pragma unroll
            for (int s = 4; s >= 1; s >>= 1)
#pragma unroll
                for (int w = 0; w < s; ++w)
                    p[w] = p[w] + p[w + s];
            v[b * kG + g] = p[0];
        }
    float val = fold_in_lane<kG>(v);
    const int64_t n = n0 + 4 * blk + t;
    const int e = e0 + c;
    const bool there = n < N && e < E;
    if (bias && there)
        val = val + bias[e];
    if (there && logits)
        logits[n * E + e] = val;
    if constexpr (kSelect) {
        const float key = e < E && val > -INFINITY ? val : -INFINITY; // (NaN counts as -infinity)
        const int rank = count_better<1>(key, e, 0);
        const float top = row_max16(key);
        const bool chosen = e < E && rank < K;
        const float s = chosen ? score(val, top, score_mode) : 0.0f;
        // summed by rank like router_topk's scores, for the same bits: lane `rank` of the row receives the score
        const float by_rank = __uint_as_float((uint32_t)__builtin_amdgcn_ds_permute(((lane & ~15) + rank) * 4, (int)__float_as_uint(s)));
        const float sum = row_sum16(by_rank);
        if (chosen && n < N) {
            topk_idx[n * K + rank] = e;
            topk_w[n * K + rank] = s / sum;
        }
    }
#endif
}

// ------------------------------------------------------------------------
// Large launches (E % 4 == 0): tiles of 32 tokens x 32 experts, a persistent workgroup of eight wavefronts per
// compute unit.  A wavefront has 16 tokens x 16 experts and half of the partials (128 accumulators per lane, eight
// instructions per step of 64 columns, two wavefronts per SIMD).  Operands go through LDS in K tiles of 128
// columns, five stages (fp32: four), by loads that write LDS directly; the K tiles of a workgroup's successive
// tiles are one stream, so that a tile starts with its operands in LDS and the fold runs under the next tile's
// loads.  x chunks are XOR-placed by token, rows of W_r so that the operand reads of an instruction are linear in
// the lane number: no bank conflicts.  The operands of step s + 1 are read under the multiplications of step s; the
// barrier of a K tile stands before its last step's multiplications, and the loads that refill its stage go out
// under them, with running addresses: both wavefronts of a SIMD are at the barrier together, and what they do
// between it and the next multiplication leaves the matrix pipe idle.
// 16384 tokens, H = 7168, 256 experts (60 GFLOP), selection included: 785 us with 4x4x1 instructions on tiles of
// 32 x 16, two workgroups per compute unit -> 607 us, 99 of 157 TFLOP/s.  Those smaller tiles with the instruction
// used here: 735 us, bound by their loads from L2 (14 TB/s, 550 us by themselves in a timing build; this tile asks
// for half as much).  This form with the addresses worked out per K tile and a register shared by all values of x:
// 822 us.
// ------------------------------------------------------------------------
constexpr int kRbTok = 32, kRbExp = 32, kRbWaves = 8;

template <bool kBf16>
__global__ __launch_bounds__(kWave *kRbWaves, 2) void router_logits_large(
    const void *__restrict__ x, int64_t N, int H, const float *__restrict__ W_r, const float *__restrict__ bias,
    int E, float *__restrict__ logits, bool by_expert)
{
#if defined(__HIP_DEVICE_COMPILE__)
    constexpr int kG = 8, kXb = kBf16 ? 2 : 4;
    constexpr int kTile = 128, kXRow = kTile * kXb;     // columns of a K tile
    constexpr int kXPart = kRbTok * kXRow, kWPart = kTile * kRbExp * 4, kStage = kXPart + kWPart;
    constexpr int kStages = kBf16 ? 5 : 4;              // 120 or 128 KiB
    constexpr int kXLoads = kXPart / 1024 / kRbWaves, kWLoads = kWPart / 1024 / kRbWaves; // per wavefront and K tile
    constexpr int kBox = kRbWaves * 2 * kG * kWave * 4; // the fold's exchange, 32 KiB
    __shared__ __attribute__((aligned(1024))) unsigned char lds[kStages * kStage + kBox];
    const int lane = threadIdx.x % kWave;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int ps = wave % 2, tg = wave / 2 % 2, eg = wave / 4;
    const int blk = lane / 16, c = lane % 16;

    // ---- tiles.  Workgroup ids are dealt round-robin to the XCDs; each XCD takes an eighth of the tiles, one run of the
    //      list.  The list goes token tile by token tile, so the tokens' rows are fetched into one L2 and W_r into all of
    //      them, or, with `by_expert` (W_r is the larger one), the other way round.  (All expert tiles of a token tile to
    //      the XCD of its number: 582 tokens, 384 experts are 19 x 12 tiles, three XCDs had 36 of them on 32 workgroups.)
    const unsigned e_tiles = (E + kRbExp - 1) / kRbExp, tok_tiles = (unsigned)((N + kRbTok - 1) / kRbTok);
    const unsigned tiles = tok_tiles * e_tiles; // (below 2^31: N < 2^31 and at most 32 expert tiles)
    const unsigned inner = by_expert ? tok_tiles : e_tiles; // tiles that follow each other over one row of the list
    const unsigned xcd = blockIdx.x % 8, per_xcd = gridDim.x / 8, share = tiles / 8, rest = tiles % 8;
    struct Place {
        unsigned outer, inner; // position in the list
        int left;              // tiles of this XCD from here on; <= 0: none
    };
    const unsigned from = xcd * share + (xcd < rest ? xcd : rest) + blockIdx.x / 8;
    const Place step = {per_xcd / inner, per_xcd % inner, (int)per_xcd};
    const Place first = {from / inner, from % inner, (int)(share + (xcd < rest)) - (int)(blockIdx.x / 8)};
    auto advance = [&](Place &p) { // by per_xcd tiles
        p.outer += step.outer;
        p.inner += step.inner;
        if (p.inner >= inner)
            p.inner -= inner, ++p.outer;
        p.left -= step.left;
    };
    auto token_of = [&](const Place &p) { return (int64_t)(by_expert ? p.inner : p.outer) * kRbTok; };
    auto expert_of = [&](const Place &p) { return (int)(by_expert ? p.outer : p.inner) * kRbExp; };

    // ---- loads of a K tile
    const int KT = (H + kTile - 1) / kTile;
    int x_off[kXLoads], x_off_last[kXLoads], w_off[kWLoads]; // (of the last K tile: past the end where columns are past H)
#pragma unroll
    for (int i = 0; i < kXLoads; ++i) {
        constexpr int kChunks = kXRow / 16;
        const int r = (wave * kXLoads + i) * (kWave / kChunks) + lane / kChunks;
        const int in_row = ((lane % kChunks) ^ (r & 15)) << 4;
        x_off[i] = r * H * kXb + in_row;
        x_off_last[i] = in_row < (H - (KT - 1) * kTile) * kXb ? x_off[i] : 0x7FFFFFF0;
    }
#pragma unroll
    for (int i = 0; i < kWLoads; ++i) {
        // block of 1 KiB = [expert half][eight slots][16 experts]; slot 4 u + b of block 8 s + 4 p + v holds row
        // 64 s + 32 p + 8 b + 2 v + u
        const int block = wave * kWLoads + i, slot = lane % 32 / 4;
        const int row = (block / 8) * 64 + (block / 4 % 2) * 32 + (slot % 4) * 8 + (block % 4) * 2 + slot / 4;
        w_off[i] = (row * E + (lane / 32) * kRtExp + (lane % 4) * 4) * 4;
    }
    // The position of a K tile goes into the base addresses and the byte counts of the resources: the range check
    // covers the per-lane offset, and rows of W_r past H and tokens past N have to come back as zeros.  Columns past H
    // would be the start of the next token's row; they come back as zeros too, so that an infinity there stays there.
    // Kept as running values: little scalar work per K tile.
    Place load = first; // of the stream's next K tile: its tile ...
    int load_kt = 0;    // ... and its position there
    const unsigned char *x_at, *w_at;
    int x_bytes, w_bytes;
    auto load_from = [&]() { // (past the last tile: no bytes, so that the number of loads in flight stays)
        const bool there = load.left > 0;
        const int64_t n = there ? token_of(load) : 0;
        const int e = there ? expert_of(load) : 0;
        x_at = static_cast<const unsigned char *>(x) + n * H * kXb;
        w_at = reinterpret_cast<const unsigned char *>(W_r + e);
        x_bytes = there ? (int)(N - n < kRbTok ? N - n : kRbTok) * H * kXb : 0;
        w_bytes = there ? (H * E - e) * 4 : 0;
    };
    load_from();
    int x_now[kXLoads];
#pragma unroll
    for (int i = 0; i < kXLoads; ++i)
        x_now[i] = KT == 1 ? x_off_last[i] : x_off[i];
    auto issue = [&](int stage) {
        const __amdgpu_buffer_rsrc_t rs_x =
            __builtin_amdgcn_make_buffer_rsrc(const_cast<unsigned char *>(x_at), 0, x_bytes, 0x00020000);
        const __amdgpu_buffer_rsrc_t rs_w =
            __builtin_amdgcn_make_buffer_rsrc(const_cast<unsigned char *>(w_at), 0, w_bytes, 0x00020000);
        __attribute__((address_space(3))) unsigned char *const st =
            (__attribute__((address_space(3))) unsigned char *)lds + stage * kStage;
#pragma unroll
        for (int i = 0; i < kXLoads; ++i)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(
                rs_x, (__attribute__((address_space(3))) void *)(st + (wave * kXLoads + i) * 1024), 16, x_now[i], 0, 0, 0);
#pragma unroll
        for (int i = 0; i < kWLoads; ++i)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(
                rs_w, (__attribute__((address_space(3))) void *)(st + kXPart + (wave * kWLoads + i) * 1024), 16, w_off[i], 0,
                0, 0);
        x_at += kTile * kXb;
        x_bytes = x_bytes > kTile * kXb ? x_bytes - kTile * kXb : 0;
        w_at += kTile * E * 4;
        w_bytes = w_bytes > kTile * E * 4 ? w_bytes - kTile * E * 4 : 0;
        if (++load_kt >= KT - 1) {
            if (load_kt == KT) {
                load_kt = 0;
                advance(load);
                load_from();
            }
#pragma unroll
            for (int i = 0; i < kXLoads; ++i)
                x_now[i] = load_kt == KT - 1 ? x_off_last[i] : x_off[i];
        }
    };

    // ---- operands of a step
    struct Operands {
        XChunk<kBf16, kG> x;
        float w[kG];
    };
    auto read = [&](Operands &o, int stage, int s) {
        const unsigned char *st = lds + stage * kStage;
        const unsigned char *row = st + (tg * kRtTok + c) * kXRow;
        const int chunk = (64 * s + 32 * ps + 8 * blk) * kXb / 16; // one (bf16) or two (fp32) neighbouring chunks
        if constexpr (kBf16) {
            o.x = load_chunk<kBf16, kG>(row + ((chunk ^ c) << 4));
        } else {
            const u32x4 lo = *reinterpret_cast<const u32x4 *>(row + ((chunk ^ c) << 4));
            const u32x4 hi = *reinterpret_cast<const u32x4 *>(row + (((chunk + 1) ^ c) << 4));
#pragma unroll
            for (int t = 0; t < 4; ++t)
                o.x.r[t] = lo[t], o.x.r[kG / 2 + t] = hi[t];
        }
        const unsigned char *pw = st + kXPart + ps * 4096 + eg * 512 + lane * 4;
#pragma unroll
        for (int g = 0; g < kG; ++g)
            o.w[g] = *reinterpret_cast<const float *>(pw + s * 8192 + (g / 2) * 1024 + (g % 2) * 256);
    };
    f32x16 acc[kG];
    float xv[kG];
    auto unpack = [&](const Operands &o) {
        // all eight values before the first multiplication: one register for all of them would make every
        // instruction wait for the one before it
#pragma unroll
        for (int g = 0; g < kG; ++g)
            xv[g] = x_value(o.x, g);
        asm volatile("" : "+v"(xv[0]), "+v"(xv[1]), "+v"(xv[2]), "+v"(xv[3]), "+v"(xv[4]), "+v"(xv[5]), "+v"(xv[6]), "+v"(xv[7]));
    };
    auto multiply = [&](const Operands &o, auto lo, auto hi) {
#pragma unroll
        for (int g = decltype(lo)::value; g < decltype(hi)::value; ++g)
            acc[g] = __builtin_amdgcn_mfma_f32_16x16x1f32(xv[g], o.w[g], acc[g], 0, 0, 0);
    };
    using from0 = std::integral_constant<int, 0>;
    using from4 = std::integral_constant<int, kG / 2>;
    using to8 = std::integral_constant<int, kG>;
    auto barrier = [&]() { // (not __syncthreads, whose fence would wait for the loads in flight)
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
    };
    // my loads of the next K tile have landed (those of the tiles after it may be in flight), my reads are done
    auto tile_barrier = [&]() {
        constexpr int kInFlight = (kStages - 2) * (kXLoads + kWLoads);
        __builtin_amdgcn_s_waitcnt(0x0070 | (kInFlight & 15) | (kInFlight >> 4 << 14));
        barrier();
    };
    Operands o0, o1;
#pragma unroll
    for (int t = 0; t + 1 < kStages; ++t)
        issue(t);
    tile_barrier();
    issue(kStages - 1);
    read(o0, 0, 0);
    int stage = 0;
    float *const box = reinterpret_cast<float *>(lds + kStages * kStage); // [wavefront][2 * kG][lane]
    for (Place at = first; at.left > 0; advance(at)) {
#pragma unroll
        for (int g = 0; g < kG; ++g)
#pragma unroll
            for (int r = 0; r < 16; ++r)
                acc[g][r] = 0.0f;
        for (int kt = 0; kt < KT; ++kt) {
            read(o1, stage, 1); // (under the multiplications of the step before)
            unpack(o0);
            __builtin_amdgcn_sched_barrier(0);
            multiply(o0, from0{}, to8{});
            __builtin_amdgcn_sched_barrier(0);
            unpack(o1);
            tile_barrier();
            multiply(o1, from0{}, from4{});
            __builtin_amdgcn_sched_barrier(0);
            issue(stage); // all of this K tile is read: its stage takes another
            stage = stage == kStages - 1 ? 0 : stage + 1;
            read(o0, stage, 0);
            __builtin_amdgcn_sched_barrier(0);
            multiply(o1, from4{}, to8{});
            __builtin_amdgcn_sched_barrier(0);
        }

        // Round 32 pairs the two wavefronts ps: each keeps tokens 4 q + 2 ps, + 1 of a block of 16 and sends the other
        // two rows' partials, a block of partials at a time.
        float v[2][4 * kG];
#pragma unroll
        for (int b = 0; b < 4; ++b) {
#pragma unroll
            for (int g = 0; g < kG; ++g)
#pragma unroll
                for (int u = 0; u < 2; ++u)
                    box[((wave ^ 1) * 2 * kG + 2 * g + u) * kWave + lane] = ps ? acc[g][4 * b + u] : acc[g][4 * b + 2 + u];
            __builtin_amdgcn_s_waitcnt(0xC07F); // lgkmcnt(0)
            barrier();
#pragma unroll
            for (int g = 0; g < kG; ++g)
#pragma unroll
                for (int u = 0; u < 2; ++u)
                    v[u][b * kG + g] = (ps ? acc[g][4 * b + 2 + u] : acc[g][4 * b + u]) +
                                       box[(wave * 2 * kG + 2 * g + u) * kWave + lane];
            __builtin_amdgcn_s_waitcnt(0xC07F);
            barrier();
        }
        const int64_t n_tile = token_of(at);
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            float val = fold_in_lane<kG>(v[u]);
            const int64_t n = n_tile + tg * kRtTok + 4 * blk + 2 * ps + u;
            const int e = expert_of(at) + eg * kRtExp + c;
            if (n < N && e < E) {
                if (bias)
                    val = val + bias[e];
                logits[n * E + e] = val;
            }
        }
    }
    __builtin_amdgcn_s_waitcnt(0x0070); // the loads past the last K tile (they write LDS too)
#endif
}

// ------------------------------------------------------------------------
// Selection.  One wavefront per token, lane l holds experts l, l+64, ... (kPer of them).  A round takes the
// largest value over the wavefront by data-parallel-primitive moves (no LDS), then the lowest index that has it
// (experts in ascending order are ballots of ascending i, lanes from the lowest).
// The K picks are distinct experts of [0, E) whatever the logits are: an overflowed token has infinities or NaN, a
// masked expert a bias of -infinity.  NaN counts as -infinity, so NaN can stand for "taken" and "not there": it never is
// the maximum as long as an expert is left (K <= E), and never equals it.  (With these in a bit mask beside the values:
// 1 token, 1024 experts, top-32 43 us instead of 33.)
// kTakeRows: every routed row also takes its local row id from its expert's row pointer as it is
// produced (Section IV-A3: the allocation unit hands out the next free row of a region on arrival);
// rank[n*K + k] receives it, and the pointers end up as the experts' counts.
// ------------------------------------------------------------------------
// lane 63's copy after folding all rows into it, for every lane
__device__ __forceinline__ float wave_max(float v)
{
    v = row_max16(v);
    auto move = [](float f, auto ctrl, auto rows) { // rows that do not take part keep their own value
        const int i = __builtin_bit_cast(int, f);
        return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(i, i, decltype(ctrl)::value, decltype(rows)::value, 0xf, false));
    };
    v = fmaxf(v, move(v, std::integral_constant<int, 0x142>{}, std::integral_constant<int, 0xa>{})); // row_bcast:15
    v = fmaxf(v, move(v, std::integral_constant<int, 0x143>{}, std::integral_constant<int, 0xc>{})); // row_bcast:31
    return __uint_as_float((uint32_t)__builtin_amdgcn_readlane((int)__float_as_uint(v), 63));
}

template <int kPer, bool kTakeRows>
__global__ __launch_bounds__(kWave *kRouteWaves) void router_topk(
    const float *__restrict__ logits, int64_t N, int E, int K, int score_mode,
    int32_t *__restrict__ topk_idx, float *__restrict__ topk_w, int32_t *__restrict__ row_pointer,
    int32_t *__restrict__ rank)
{
    const int lane = threadIdx.x % kWave;
    const int64_t n = (int64_t)blockIdx.x * kRouteWaves + threadIdx.x / kWave;
    if (n >= N)
        return;
    const float *row = logits + n * E;
    float val[kPer]; // NaN: taken, or not there
    bool odd = false;
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
        const int e = i * kWave + lane;
        const float f = e < E ? row[e] : 0.0f;
        odd |= f != f;
        val[i] = e < E ? (f == f ? f : -INFINITY) : NAN;
    }
    float my_logit = 0.0f, top = 0.0f; // lane k keeps the k-th pick
    int my_pick = 0;
    for (int k = 0; k < K; ++k) {
        float best = val[0];
#pragma unroll
        for (int i = 1; i < kPer; ++i)
            best = fmaxf(best, val[i]);
        best = wave_max(best);
        int pick = -1;
#pragma unroll
        for (int i = 0; i < kPer; ++i) {
            const uint64_t m = __ballot(val[i] == best);
            if (pick < 0 && m != 0) {
                const int at = __builtin_ctzll(m);
                pick = i * kWave + at;
                if (lane == at)
                    val[i] = NAN;
            }
        }
        if (k == 0)
            top = best;
        if (lane == k) {
            my_logit = best;
            my_pick = pick;
        }
    }
    if (__ballot(odd) != 0) { // the weights are those of the logits themselves
        my_logit = lane < K ? row[my_pick] : 0.0f;
        top = __uint_as_float((uint32_t)__builtin_amdgcn_readlane((int)__float_as_uint(my_logit), 0));
    }
    const float s = lane < K ? score(my_logit, top, score_mode) : 0.0f;
    // Sum in pairs of ranks that are 16, 8, 4, 2, 1 apart (K <= 32: the first two rows of sixteen lanes)
    const float pairs = K > 16 ? s + __shfl_xor(s, 16) : s;
    float sum = row_sum16(pairs);
    sum = __uint_as_float((uint32_t)__builtin_amdgcn_readlane((int)__float_as_uint(sum), 0));
    if (lane < K) {
        topk_idx[n * K + lane] = my_pick;
        topk_w[n * K + lane] = s / sum;
        if constexpr (kTakeRows)
            rank[n * K + lane] = atomicAdd(&row_pointer[my_pick], 1);
    }
}

template <bool kTakeRows>
static void launch_topk(const float *logits, int64_t N, int E, int K, int score_mode, int32_t *topk_idx,
                        float *topk_w, int32_t *row_pointer, int32_t *rank, hipStream_t st)
{
    auto kern = E <= kWave       ? router_topk<1, kTakeRows>
                : E <= 2 * kWave ? router_topk<2, kTakeRows>
                : E <= 4 * kWave ? router_topk<4, kTakeRows>
                                 : router_topk<MOE_MAX_EXPERTS / kWave, kTakeRows>;
    hipLaunchKernelGGL(kern, dim3((unsigned)ceil_div(N, kRouteWaves)), dim3(kWave * kRouteWaves), 0, st, logits, N, E, K,
                       score_mode, topk_idx, topk_w, row_pointer, rank);
}

template <bool kBf16>
static void launch_logits(const void *x, int64_t N, int64_t H, const float *W_r, const float *bias, int E, int K,
                          int score_mode, int32_t *topk_idx, float *topk_w, float *logits, bool select, hipStream_t st)
{
    const int64_t e_tiles = ceil_div(E, kRtExp);
    // The large form (its 16-byte loads of W_r aligned) once the small one has more workgroups than there are compute
    // units; a workgroup of the small form then waits for, or shares a unit with, another.  Small / large, us: 256
    // workgroups: 250 tokens, H 3584, 256 experts, fp32 21 / 30; 260: 1033 tokens, H 2944, 64 experts 25 / 24; 272: 532
    // tokens, H 1152, 128 experts, fp32 18 / 15; 426: 1136 tokens, H 5696, 96 experts, fp32 51 / 38; 490: 3920 tokens, H
    // 2304, 32 experts 28 / 22.  (Between 300 and 400 two of fourteen were better off small, 4 - 6 %.)
    const int64_t tok_tiles = ceil_div(N, kRtTok), tiles = ceil_div(N, kRbTok) * ceil_div(E, kRbExp);
    if (!select && E % 4 == 0 && tok_tiles * e_tiles > 256 && H * kRbTok * 4 < ((int64_t)1 << 31) && H * (int64_t)E * 4 < ((int64_t)1 << 31)) {
        const int64_t groups = ceil_div(tiles, 8) * 8;
        hipLaunchKernelGGL(router_logits_large<kBf16>, dim3((unsigned)(groups < 256 ? groups : 256)), dim3(kWave * kRbWaves), 0,
                           st, x, N, (int)H, W_r, bias, E, logits, N * (kBf16 ? 2 : 4) < (int64_t)E * 4);
        return;
    }
    // One dimension of a grid holds fewer than 2^32 threads (2^23 of these workgroups): the token tiles go in rows.
    const int64_t fit = ((int64_t)1 << 22) / e_tiles, per_row = tok_tiles < fit ? tok_tiles : fit;
    const dim3 grid((unsigned)(per_row * e_tiles), (unsigned)ceil_div(tok_tiles, per_row));
    if (select)
        hipLaunchKernelGGL((router_logits_small<kBf16, true>), grid, dim3(512), 0, st, x, N, H, W_r, bias, E, logits, K,
                           score_mode, topk_idx, topk_w, (int)per_row);
    else
        hipLaunchKernelGGL((router_logits_small<kBf16, false>), grid, dim3(512), 0, st, x, N, H, W_r, bias, E, logits, K,
                           score_mode, topk_idx, topk_w, (int)per_row);
}

int launch_route(const void *x, int dtype, int64_t N, int64_t H, const float *W_r,
                 const float *bias, int E, int K, int score_mode, int32_t *topk_idx,
                 float *topk_w, float *logits, hipStream_t st, int32_t *row_pointer, int32_t *rank)
{
    const bool select = E <= kRtExp && !row_pointer; // the logits kernel selects as well
    if (dtype == MOE_BF16)
        launch_logits<true>(x, N, H, W_r, bias, E, K, score_mode, topk_idx, topk_w, logits, select, st);
    else
        launch_logits<false>(x, N, H, W_r, bias, E, K, score_mode, topk_idx, topk_w, logits, select, st);
    if (row_pointer)
        launch_topk<true>(logits, N, E, K, score_mode, topk_idx, topk_w, row_pointer, rank, st);
    else if (!select)
        launch_topk<false>(logits, N, E, K, score_mode, topk_idx, topk_w, nullptr, nullptr, st);
    return check_launch("moe_route");
}

}  // namespace moe
