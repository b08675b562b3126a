// Expert computation (bf16) of launches with few rows: both GEMMs as streams of weights.
//
// With a handful of rows the FFN is bound by reading the weights of the experts that got one.  The tiled kernel
// (grouped_gemm.h) gives a workgroup 256 columns, so such a launch is a few dozen workgroups and every one of them pulls
// its panel at what one compute unit can pull (about 55 GB/s).  Here a workgroup takes 32 weight rows (the gate/up
// projection: 16 gate columns and the same 16 up columns; the down projection: 32 columns), or 64 where that leaves
// enough workgroups, and its four wavefronts share the reduction, 128 bytes of every row in turn, so the launch is
// thousands of wavefronts that each keep some 20 KiB in flight.  A weight is used by one wavefront only and goes straight to registers in the operand layout of
// v_mfma_f32_16x16x32_bf16: four neighbouring lanes read 64 consecutive bytes of a row.  The rows of A (up to 64, in
// blocks of 16) come the same way, from L2.  The partial sums of the four wavefronts meet in LDS in a fixed order.
// One token of a 4-expert layer (H 2048, F 1408): gate/up 40 -> 16 us, down 23 -> 12 us (69 MB in all); 16 rows for each
// of 8 experts (H 7168, F 2048): 135 -> 102, 63 -> 56 us (4.6 and 4.2 TB/s).  Where the line lies: use_thin in ffn.hip.
#include <type_traits>

#include "common.h"
#include "ffn_thin.h"
#include "grouped_gemm.h"

namespace moe {

constexpr int kThinWaves = 4;

struct ThinArgs {
    const uint16_t *A;
    int64_t M;
    int Kdim, Ndim;
    const uint16_t *B0, *B1;
    uint16_t *C; // kScatter: fp32 sums
    TileTableHeader *hdr;
    const TileEntry *table; // one entry per row tile
    int out_cols;
    const int32_t *gather_rows;
    int gather_div;
    uint32_t gather_bytes;
    const float *scatter_w;
};

#if defined(__HIP_DEVICE_COMPILE__)
// One workgroup's tile: kB blocks of 16 rows by kParts blocks of 16 weight rows.
template <int kParts, int kB, bool kSwiglu, bool kGather, bool kScatter>
__device__ __forceinline__ void thin_tile(const ThinArgs &g, const TileEntry &t, f32x4 *red)
{
    // 128-byte lines of a row per turn; two turns' operands are in registers
    constexpr int kLines = kParts == 2 && kB == 1 ? 2 : 1, kSteps = 2 * kLines;
    constexpr int kHalf = kSwiglu ? kParts / 2 : kParts; // blocks of output columns
    const int lane = threadIdx.x % kWave;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int i = lane % 16, q = lane / 16;
    const int Kdim = g.Kdim, n0 = (int)blockIdx.x * g.out_cols;
    const int64_t first = (int64_t)t.expert * g.Ndim + n0;
    // block p of the weight rows: gate columns first, then the same up columns; 16 rows at a time
    const uint16_t *const w_gate = g.B0 + first * Kdim;
    const uint16_t *const w_up = kSwiglu ? g.B1 + first * Kdim : nullptr;
    const uint32_t w_bytes = 16u * kHalf * (uint32_t)Kdim * 2u;
    const uint16_t *const a = kGather ? g.A : g.A + (int64_t)t.m0 * Kdim;
    const int rows = t.m_end - t.m0;
    const uint32_t a_bytes = kGather ? g.gather_bytes : (uint32_t)(rows < 16 * kB ? rows : 16 * kB) * (uint32_t)Kdim * 2u;
    const uint32_t w_off = (uint32_t)(i * Kdim + q * 8) * 2u;
    uint32_t a_off[kB]; // rows past the segment lie past the byte count: zeros
#pragma unroll
    for (int b = 0; b < kB; ++b) {
        const int r = 16 * b + i;
        uint32_t at = (uint32_t)r * (uint32_t)Kdim * 2u;
        if constexpr (kGather)
            at = r < rows ? (uint32_t)(g.gather_rows[t.m0 + r] / g.gather_div) * (uint32_t)(Kdim * 2) : g.gather_bytes;
        a_off[b] = at + (uint32_t)q * 16u;
    }
    const int lines = Kdim / 64;
    // Where in the rows this workgroup starts.  Rows are often a power of two apart; with everyone at the same column
    // the requests of a moment meet in a few memory channels (8 experts, K = 4096: 408 us all from 0, 323 us like this).
    const int start = (int)(blockIdx.x * 16u % (uint32_t)lines);
    struct Operands {
        u32x4 w[kParts][kSteps], a[kB][kSteps];
    };
    // turn j of this wavefront: lines wave + 4 (kLines j + u); those past the end have no bytes and read as zeros
    auto fetch = [&](Operands &o, int j) {
#pragma unroll
        for (int u = 0; u < kLines; ++u) {
            const int line = wave + kThinWaves * (kLines * j + u);
            const bool there = line < lines;
            const auto rg = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t *>(w_gate), 0, there ? w_bytes : 0u, 0x00020000);
            const auto ru = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t *>(w_up), 0, there && kSwiglu ? w_bytes : 0u, 0x00020000);
            const auto ra = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t *>(a), 0, there ? a_bytes : 0u, 0x00020000);
            const int turned = line + start;
            const uint32_t at = (uint32_t)(turned < lines ? turned : turned - lines) * 128u;
#pragma unroll
            for (int p = 0; p < kParts; ++p)
#pragma unroll
                for (int s = 0; s < 2; ++s) // (weights are read once: non-temporal)
                    o.w[p][2 * u + s] = __builtin_amdgcn_raw_buffer_load_b128(
                        p < kHalf ? rg : ru, (int)(w_off + (uint32_t)(p % kHalf) * 32u * (uint32_t)Kdim + at + 64 * s), 0, 2);
#pragma unroll
            for (int b = 0; b < kB; ++b)
#pragma unroll
                for (int s = 0; s < 2; ++s)
                    o.a[b][2 * u + s] = __builtin_amdgcn_raw_buffer_load_b128(ra, (int)(a_off[b] + at + 64 * s), 0, 0);
            // one order of the loads everywhere: else the wait at the top of the loop is for all of them
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    f32x4 acc[kB][kParts];
#pragma unroll
    for (int b = 0; b < kB; ++b)
#pragma unroll
        for (int p = 0; p < kParts; ++p)
            acc[b][p] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    auto multiply = [&](const Operands &o) {
#pragma unroll
        for (int s = 0; s < kSteps; ++s)
#pragma unroll
            for (int b = 0; b < kB; ++b)
#pragma unroll
                for (int p = 0; p < kParts; ++p) // weights first: a lane ends up with consecutive columns of a row
                    acc[b][p] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, o.w[p][s]),
                                                                        __builtin_bit_cast(bf16x8, o.a[b][s]), acc[b][p], 0, 0, 0);
    };
    const int turns = (lines + kThinWaves * kLines - 1) / (kThinWaves * kLines);
    Operands o0, o1;
    fetch(o0, 0);
    for (int j = 0; j < turns; j += 2) { // (turns past the end: no bytes)
        fetch(o1, j + 1);
        multiply(o0);
        __builtin_amdgcn_sched_barrier(0);
        fetch(o0, j + 2);
        multiply(o1);
        __builtin_amdgcn_sched_barrier(0);
    }

    // ---- red[wavefront][block][lane]; register r of lane (q, i): row i, column 4 q + r of a block
    constexpr int kBlocks = kB * kParts;
#pragma unroll
    for (int b = 0; b < kB; ++b)
#pragma unroll
        for (int p = 0; p < kParts; ++p)
            red[(wave * kBlocks + b * kParts + p) * kWave + lane] = acc[b][p];
    __syncthreads();
    auto total = [&](int block) {
        f32x4 s = red[block * kWave + lane];
#pragma unroll
        for (int w = 1; w < kThinWaves; ++w) {
            const f32x4 v = red[(w * kBlocks + block) * kWave + lane];
#pragma unroll
            for (int r = 0; r < 4; ++r)
                s[r] += v[r];
        }
        return s;
    };
    for (int o = wave; o < kB * kHalf; o += kThinWaves) {
        const int b = o / kHalf, p = o % kHalf;
        f32x4 v = total(b * kParts + p);
        if constexpr (kSwiglu) {
            const f32x4 up = total(b * kParts + kHalf + p);
#pragma unroll
            for (int r = 0; r < 4; ++r)
                v[r] = silu_mul(v[r], up[r]);
        }
        const int64_t m = (int64_t)t.m0 + 16 * b + i;
        const int n = n0 + 16 * p + 4 * q;
        if (m >= t.m_end || n >= g.Ndim)
            continue;
        if constexpr (kScatter) {
            const int32_t r = g.gather_rows[m];
            const float sw = g.scatter_w[r];
            float *const sums = reinterpret_cast<float *>(g.C) + (int64_t)(r / g.gather_div) * g.Ndim + n;
#pragma unroll
            for (int k = 0; k < 4; ++k)
                unsafeAtomicAdd(sums + k, sw * v[k]);
        } else {
            u32x2 out;
            out[0] = pack_bf16x2(v[0], v[1]);
            out[1] = pack_bf16x2(v[2], v[3]);
            *reinterpret_cast<u32x2 *>(g.C + m * g.Ndim + n) = out;
        }
    }
}
#endif

// Workgroup (x, y): columns x, row tile y of the table.
template <int kParts, int kMaxB, bool kSwiglu, bool kGather, bool kScatter>
__global__ __launch_bounds__(kWave *kThinWaves, kMaxB == 1 ? 4 : 2) void ffn_thin(ThinArgs g)
{
#if defined(__HIP_DEVICE_COMPILE__)
    __shared__ f32x4 red[kThinWaves * kMaxB * kParts * kWave];
    const TileTableHeader *const hdr = g.hdr;
    if (hdr->magic != kTableMagic || hdr->rows != (int32_t)g.M || hdr->out_cols != g.out_cols) {
        // no schedule for these rows in this workspace: leave the word that moe_ffn_status finds
        if (blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0)
            g.hdr->error = kNoScheduleError;
        return;
    }
    if ((int)blockIdx.y >= hdr->len[0] + hdr->len[1])
        return;
    const TileEntry t = g.table[blockIdx.y];
    const int rows = t.m_end - t.m0;
    if (kMaxB == 1 || rows <= 16)
        thin_tile<kParts, 1, kSwiglu, kGather, kScatter>(g, t, red);
    else if (kMaxB == 2 || rows <= 32)
        thin_tile<kParts, (kMaxB < 2 ? kMaxB : 2), kSwiglu, kGather, kScatter>(g, t, red);
    else
        thin_tile<kParts, kMaxB, kSwiglu, kGather, kScatter>(g, t, red);
#endif
}

template <int kParts, bool kSwiglu, bool kGather, bool kScatter>
static void launch_parts(const ThinArgs &g, int row_tiles, hipStream_t st)
{
    const dim3 grid((unsigned)ceil_div(g.Ndim, g.out_cols), (unsigned)row_tiles);
    if (g.M <= 16) // no expert can have more rows
        hipLaunchKernelGGL((ffn_thin<kParts, 1, kSwiglu, kGather, kScatter>), grid, dim3(kWave * kThinWaves), 0, st, g);
    else
        hipLaunchKernelGGL((ffn_thin<kParts, 4, kSwiglu, kGather, kScatter>), grid, dim3(kWave * kThinWaves), 0, st, g);
}

template <bool kSwiglu, bool kGather, bool kScatter>
static void launch(const ThinArgs &g, int row_tiles, hipStream_t st)
{
    if (g.out_cols * (kSwiglu ? 2 : 1) == 16 * 4)
        launch_parts<4, kSwiglu, kGather, kScatter>(g, row_tiles, st);
    else
        launch_parts<2, kSwiglu, kGather, kScatter>(g, row_tiles, st);
}

void launch_thin_gate_up(const uint16_t *A, int64_t M, int64_t H, int64_t F, const uint16_t *W_gate, const uint16_t *W_up,
                         uint16_t *a, TileTableHeader *hdr, const TileEntry *table, int row_tiles, int out_cols,
                         const int32_t *gather_rows, int gather_div, uint32_t gather_bytes, hipStream_t st)
{
    const ThinArgs g = {A, M, (int)H, (int)F, W_gate, W_up, a, hdr, table, out_cols, gather_rows, gather_div, gather_bytes, nullptr};
    if (gather_rows)
        launch<true, true, false>(g, row_tiles, st);
    else
        launch<true, false, false>(g, row_tiles, st);
}

void launch_thin_down(const uint16_t *a, int64_t M, int64_t H, int64_t F, const uint16_t *W_down, void *y,
                      TileTableHeader *hdr, const TileEntry *table, int row_tiles, int out_cols, const int32_t *row_of_slot, int K,
                      const float *scatter_w, hipStream_t st)
{
    const ThinArgs g = {a, M, (int)F, (int)H, W_down, nullptr, static_cast<uint16_t *>(y), hdr, table, out_cols, row_of_slot, K, 0u, scatter_w};
    if (scatter_w)
        launch<false, false, true>(g, row_tiles, st);
    else
        launch<false, false, false>(g, row_tiles, st);
}

}  // namespace moe
