// Expert computation in fp32: the two GEMMs of the grouped SwiGLU FFN on the fp32 matrix cores.
//
// v_mfma_f32_16x16x4_f32 multiplies exactly and adds in fp32, so the precision is that of a chain of fused
// multiply-adds (checked against 64-bit arithmetic by the parity tests).
//
// One workgroup of four wavefronts computes 32 rows x 64 columns (the gate/up projection: 64 gate columns and the
// same 64 up columns, so that the activation is applied to the accumulators).  Large launches are bound by the matrix
// pipe (157 TFLOP/s): a K tile of 32 columns keeps it busy for 1024 cycles (gate/up), against 20 KiB of loads and
// 64 KiB of operand reads per workgroup, below what L2 and LDS deliver; small ones by the latency of a K tile.  So
// the tile is kept small: experts often have a few dozen rows only at the sizes this type is used for (64 x 64 tiles
// of 32x32x2 instructions: gate/up 97 instead of 92 us on 3003 rows over 12 experts, 10.8 instead of 7.8 us on 512
// rows over 8).  K tiles go global -> LDS by 16-byte loads that write LDS directly, XOR-swizzled by 16-byte chunk so
// that the operand reads (16 bytes per lane: four consecutive k) are free of bank conflicts.  Which expert a
// workgroup's rows belong to is worked out from the segment offsets by every wavefront itself (a scan over the
// experts), so this type needs no tile table and no workspace beyond the activation.
//
// Measured, before (one thread per output element, every lane reading another weight row) and now:
//   1001 tokens, H = 516, F = 1028, 12 experts, top-3 (9.6 GFLOP): 17.4 ms -> 92 + 53 us (66 TFLOP/s; half of it
//   the last rounds of workgroups, on 12288 rows it is 106 TFLOP/s);
//   256 tokens, H = 128, F = 256, 8 experts, top-2: 130 + 36 us -> 7.8 + 7.4 us.
#include <type_traits>

#include "common.h"

namespace moe {

constexpr int kF32Rows = 32;  // rows of an output tile
constexpr int kF32Cols = 64;  // columns (of the gate and of the up projection)
constexpr int kF32K = 32;     // K tile: 128-byte rows, 8 chunks of 16 bytes
constexpr int kF32Threads = 256;
constexpr int kF32PartA = kF32Rows * kF32K * 4, kF32PartB = kF32Cols * kF32K * 4; // bytes of an operand's K tile
constexpr int kXcdCount = 8;
constexpr int kBand = 8;      // row tiles that follow each other over one weight tile

__device__ const f32x4 kZeroChunk = {0.0f, 0.0f, 0.0f, 0.0f};

// 16-byte chunk c of row r sits at chunk position c ^ key: any 8 and any 16 consecutive rows spread over the banks
__device__ __forceinline__ int f32_row_key(int r) { return ((r ^ (r >> 3)) & 1) | (r & 6); }

struct RowTile {
    int expert; // -1: no such tile
    int m0, m_end;
};

// Row tile `t` of the launch: experts in order, ceil(rows / kF32Rows) tiles each.  Every lane owns a run of experts.
__device__ __forceinline__ RowTile find_row_tile(const int32_t *__restrict__ seg, int E_local, int64_t M, int64_t t)
{
    const int lane = threadIdx.x % kWave;
    const int per = (E_local + kWave - 1) / kWave;
    auto rows_of = [&](int e, int64_t &lo) {
        int64_t hi = seg[e + 1];
        lo = seg[e];
        lo = lo < 0 ? 0 : (lo > M ? M : lo);
        hi = hi < lo ? lo : (hi > M ? M : hi);
        return hi - lo;
    };
    int64_t lo;
    int mine = 0;
    for (int j = 0; j < per; ++j) {
        const int e = lane * per + j;
        if (e < E_local)
            mine += (int)((rows_of(e, lo) + kF32Rows - 1) / kF32Rows);
    }
    int inc = mine;
    for (int d = 1; d < kWave; d <<= 1) {
        const int up = __shfl_up(inc, d);
        if (lane >= d)
            inc += up;
    }
    int first = inc - mine;
    RowTile r = {-1, 0, 0};
    const uint64_t owner = __ballot(t >= first && t < inc);
    if (owner == 0)
        return r;
    if (t >= first && t < inc) {
        for (int j = 0; j < per; ++j) {
            const int e = lane * per + j;
            if (e >= E_local)
                break;
            const int64_t rows = rows_of(e, lo);
            const int tiles = (int)((rows + kF32Rows - 1) / kF32Rows);
            if (t < first + tiles) {
                r.expert = e;
                r.m0 = (int)lo + (int)(t - first) * kF32Rows;
                r.m_end = (int)(lo + rows);
                break;
            }
            first += tiles;
        }
    }
    const int src = __builtin_ctzll(owner);
    r.expert = __builtin_amdgcn_readlane(r.expert, src);
    r.m0 = __builtin_amdgcn_readlane(r.m0, src);
    r.m_end = __builtin_amdgcn_readlane(r.m_end, src);
    return r;
}

// gather_rows != nullptr: row m of A is row gather_rows[m] / gather_div of `A`.
// kStages: K tiles in LDS; see the launcher.
template <bool kSwiglu, int kStages>
__global__ __launch_bounds__(kF32Threads, (kStages > 3 ? 2 : 4)) void ffn_f32_tiles(
    const float *__restrict__ A, int64_t M, int Kdim, int Ndim, int E_local, const int32_t *__restrict__ seg,
    const float *__restrict__ B0, const float *__restrict__ B1, float *__restrict__ C,
    const int32_t *__restrict__ gather_rows, int gather_div, int col_tiles)
{
#if defined(__HIP_DEVICE_COMPILE__)
    constexpr int kParts = kSwiglu ? 2 : 1;              // column parts: gate and up columns, or one range
    constexpr int kStage = kF32PartA + kParts * kF32PartB;
    constexpr int kLoads = 1 + 2 * kParts;               // per lane and K tile
    __shared__ __attribute__((aligned(1024))) unsigned char lds[kStages * kStage];
    const int lane = threadIdx.x % kWave;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    // Tiles in bands of kBand row tiles, column by column; workgroup ids are dealt round-robin to the XCDs, and the
    // kBand tiles of a band that share a weight tile go to one XCD, one after the other.
    // (A row of the grid is a multiple of kXcdCount * kBand workgroups long.)
    const int64_t slot = (int64_t)blockIdx.y * gridDim.x + blockIdx.x / (kXcdCount * kBand) * (kXcdCount * kBand) +
                         blockIdx.x % kXcdCount * kBand + blockIdx.x / kXcdCount % kBand;
    const int64_t band = slot / ((int64_t)kBand * col_tiles);
    const int in_band = (int)(slot - band * kBand * col_tiles);
    const RowTile rt = find_row_tile(seg, E_local, M, band * kBand + in_band % kBand);
    if (rt.expert < 0)
        return;
    const int n0 = in_band / kBand * kF32Cols;

    // ---- loads: an instruction of a wavefront fills 8 rows of a part; a lane fetches the chunk that belongs at its
    //      place.  Rows past the segment and columns past Ndim are clamped (their results are not stored), chunks
    //      past Kdim come from a chunk of zeros.  Load 0: rows of A; 1, 2: the first column part; 3, 4: the second.
    const float *src[kLoads];
    int k_of[3]; // first column of the lane's chunk inside a K tile, loads 0, 1 and 3, 2 and 4
    {
        const int r = wave * 8 + lane / 8;
        k_of[0] = ((lane % 8) ^ f32_row_key(r)) * 4;
        int64_t m = rt.m0 + r < rt.m_end ? rt.m0 + r : rt.m_end - 1;
        if (gather_rows)
            m = gather_rows[m] / gather_div;
        src[0] = A + m * Kdim + k_of[0];
    }
#pragma unroll
    for (int g = 0; g < 2; ++g) {
        const int r = wave * 16 + g * 8 + lane / 8;
        k_of[1 + g] = ((lane % 8) ^ f32_row_key(r)) * 4;
#pragma unroll
        for (int p = 0; p < kParts; ++p) {
            const int n = n0 + r < Ndim ? n0 + r : Ndim - 1;
            src[1 + 2 * p + g] = (p ? B1 : B0) + ((int64_t)rt.expert * Ndim + n) * Kdim + k_of[1 + g];
        }
    }
    auto load_chunk = [&](int i, int k, int kt, int at) {
        const float *s = kt * kF32K + k < Kdim ? src[i] + kt * kF32K : reinterpret_cast<const float *>(&kZeroChunk);
        __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)s,
                                         (__attribute__((address_space(3))) void *)(lds + at), 16, 0, 0);
    };
    auto issue = [&](int kt, int stage) {
        const int base = stage * kStage;
        load_chunk(0, k_of[0], kt, base + wave * 1024);
#pragma unroll
        for (int p = 0; p < kParts; ++p)
#pragma unroll
            for (int g = 0; g < 2; ++g)
                load_chunk(1 + 2 * p + g, k_of[1 + g], kt, base + kF32PartA + p * kF32PartB + (wave * 2 + g) * 1024);
    };

    // ---- operands: lane (i = lane % 16, q = lane / 16) holds k = 16 g + 4 q + s of row i for the four instructions
    //      s of a group g of sixteen columns (both operands alike, so the order of k does not matter).  A wavefront
    //      owns columns 16 wave .. + 16 of every column part and all 32 rows.
    const int i = lane % 16, q = lane / 16;
    const int key = f32_row_key(i), key_hi = f32_row_key(i + 16);
    const int a_at = i * 128, b_at = kF32PartA + (wave * 16 + i) * 128, b_key = f32_row_key(wave * 16 + i);
    const bool two_rows = rt.m0 + 16 < rt.m_end; // (else the second block of 16 rows is empty)
    f32x4 acc[2][kParts]; // [16-row block][column part]
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
        for (int p = 0; p < kParts; ++p)
            acc[b][p] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};

    const int KT = (Kdim + kF32K - 1) / kF32K;
#pragma unroll
    for (int t = 0; t + 1 < kStages; ++t)
        issue(t, t);
    auto k_loop = [&](auto rows_tag) {
        constexpr int kBlocks = decltype(rows_tag)::value;
        constexpr int kInFlight = (kStages - 2) * kLoads; // the loads of the K tiles after kt
        int stage = 0;
        for (int kt = 0; kt < KT; ++kt) {
            // my part of K tile kt is there (vmcnt), my reads of K tile kt - 1 are done (lgkmcnt) ...
            __builtin_amdgcn_s_waitcnt(0x0070 | (kInFlight & 15) | (kInFlight >> 4 << 14));
            asm volatile("" ::: "memory");
            __builtin_amdgcn_s_barrier(); // ... and everyone's
            asm volatile("" ::: "memory");
            issue(kt + kStages - 1, stage == 0 ? kStages - 1 : stage - 1); // (past the last K tile: zeros, the count stays)
            const unsigned char *st = lds + stage * kStage;
            stage = stage == kStages - 1 ? 0 : stage + 1;
            f32x4 a[2][2], w[2][kParts]; // [k group][row block], [k group][column part]: all reads of the K tile first
#pragma unroll
            for (int g = 0; g < 2; ++g) {
                const int c = 4 * g + q;
                a[g][0] = *reinterpret_cast<const f32x4 *>(st + a_at + ((c ^ key) << 4));
                if (kBlocks > 1)
                    a[g][1] = *reinterpret_cast<const f32x4 *>(st + a_at + 16 * 128 + ((c ^ key_hi) << 4));
#pragma unroll
                for (int p = 0; p < kParts; ++p)
                    w[g][p] = *reinterpret_cast<const f32x4 *>(st + b_at + p * kF32PartB + ((c ^ b_key) << 4));
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int g = 0; g < 2; ++g)
#pragma unroll
                for (int s = 0; s < 4; ++s)
#pragma unroll
                    for (int b = 0; b < kBlocks; ++b)
#pragma unroll
                        for (int p = 0; p < kParts; ++p) // weights first: a lane ends up with consecutive columns of a row
                            acc[b][p] = __builtin_amdgcn_mfma_f32_16x16x4f32(w[g][p][s], a[g][b][s], acc[b][p], 0, 0, 0);
        }
    };
    if (two_rows)
        k_loop(std::integral_constant<int, 2>{});
    else
        k_loop(std::integral_constant<int, 1>{});
    __builtin_amdgcn_s_waitcnt(0x0F70); // the loads past the last K tile still write LDS

    // ---- register r of lane l: output row l % 16, column 4 (l / 16) + r of a 16 x 16 block
#pragma unroll
    for (int b = 0; b < 2; ++b) {
        const int64_t m = (int64_t)rt.m0 + b * 16 + i;
        if (m >= rt.m_end)
            return;
        float *row = C + m * Ndim;
        const int n = n0 + wave * 16 + q * 4; // (Ndim is a multiple of four)
        f32x4 v = acc[b][0];
        if constexpr (kSwiglu) {
#pragma unroll
            for (int t = 0; t < 4; ++t)
                v[t] = v[t] / (1.0f + expf(-v[t])) * acc[b][kParts - 1][t];
        }
        if (n < Ndim)
            *reinterpret_cast<f32x4 *>(row + n) = v;
    }
#endif
}

template <bool kSwiglu>
static int launch_tiles(const float *A, int64_t M, int64_t Kdim, int64_t Ndim, int E_local, const int32_t *seg,
                        const float *B0, const float *B1, float *C, const int32_t *gather_rows, int gather_div,
                        hipStream_t st, const char *what)
{
    const int col_tiles = (int)ceil_div(Ndim, kF32Cols);
    // an upper bound of the row tiles: workgroups that find none leave at once
    const int64_t row_tiles = M / kF32Rows + E_local < M ? M / kF32Rows + E_local : M;
    const int64_t blocks = ceil_div(ceil_div(row_tiles, kBand) * kBand * col_tiles, kXcdCount * kBand) * (kXcdCount * kBand);
    // one dimension of a grid holds fewer than 2^32 threads: rows of 2^23 workgroups beyond that
    constexpr int64_t kGridRow = (int64_t)1 << 23;
    const dim3 grid((unsigned)(blocks < kGridRow ? blocks : kGridRow), (unsigned)ceil_div(blocks, kGridRow));
    // A launch that is resident at once with two workgroups per compute unit waits for latency, not for the matrix
    // pipe: as many K tiles in flight as two workgroups have LDS for.  Larger ones: four workgroups per unit.
    constexpr int kDeep = kSwiglu ? 4 : 6, kShallow = kSwiglu ? 2 : 3;
    auto kern = blocks <= 512 ? ffn_f32_tiles<kSwiglu, kDeep> : ffn_f32_tiles<kSwiglu, kShallow>;
    hipLaunchKernelGGL(kern, grid, dim3(kF32Threads), 0, st, A, M, (int)Kdim,
                       (int)Ndim, E_local, seg, B0, B1, C, gather_rows, gather_div, col_tiles);
    return check_launch(what);
}

int launch_ffn_f32_gate_up(const float *xp, int64_t M, int64_t H, int64_t F, int E_local, const int32_t *seg_offsets,
                           const float *W_gate, const float *W_up, float *a, const int32_t *gather_rows, int K,
                           hipStream_t st)
{
    return launch_tiles<true>(xp, M, H, F, E_local, seg_offsets, W_gate, W_up, a, gather_rows, K, st,
                              "moe_ffn_gate_up(f32)");
}

int launch_ffn_f32_down(const float *a, int64_t M, int64_t H, int64_t F, int E_local, const int32_t *seg_offsets,
                        const float *W_down, float *y, hipStream_t st)
{
    return launch_tiles<false>(a, M, F, H, E_local, seg_offsets, W_down, nullptr, y, nullptr, 1, st,
                               "moe_ffn_down(f32)");
}

}  // namespace moe
