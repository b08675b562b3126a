// Row moves of the dispatch and combine steps (Section II-A, steps 2, 4, 5).
// Both are pure HBM traffic: 16-byte vector accesses, one wavefront per token,
// whole rows contiguous so every access is fully coalesced.
//
//   permute : x[n,:] is read once and written to its K slots.
//             algorithmic bytes = N*H*b (read) + N*K*H*b (write) + 4*N*K (slots)
//   combine : K rows are gathered per token, scaled, summed in fp32 (k ascending)
//             and rounded once.  bytes = N*K*H*b (read) + N*H*b (write) + 8*N*K
#include <type_traits>

#include "common.h"

namespace moe {

constexpr int kTokensPerBlock = 4; // one wavefront each (combine of long rows: one token, all four)

// Value of lane k (k wave-uniform) whatever lanes are active: the chunk loops below run a different
// number of times per lane, and a cross-lane read that honours the execution mask (__shfl) returns 0
// for a lane that has already left the loop.
__device__ __forceinline__ int32_t lane_value(int32_t v, int k) { return __builtin_amdgcn_readlane(v, k); }
__device__ __forceinline__ float lane_value(float v, int k)
{
    return __uint_as_float((uint32_t)__builtin_amdgcn_readlane((int32_t)__float_as_uint(v), k));
}

// x has just been read by the router and may still lie in the 256 MB memory-side cache, and xp is read next.  kPassX, kPassXp:
// non-temporal loads of x, stores of xp, which leave that cache to the other (launch_permute says when).
template <bool kPassX, bool kPassXp>
__global__ __launch_bounds__(kWave *kTokensPerBlock) void permute_rows(
    const u32x4 *__restrict__ x, int chunks, int64_t N, int K,
    const int32_t *__restrict__ slot_of_row, u32x4 *__restrict__ xp)
{
    const int lane = threadIdx.x % kWave;
    const int64_t n = (int64_t)blockIdx.x * kTokensPerBlock + threadIdx.x / kWave;
    if (n >= N)
        return;
    // lane k keeps slot k of this token
    int32_t my_slot = (lane < K) ? slot_of_row[n * K + lane] : 0;
    const u32x4 *src = x + n * chunks;
    auto get = [](const u32x4 *from) {
        if constexpr (kPassX)
            return __builtin_nontemporal_load(from);
        else
            return *from;
    };
    auto put = [](u32x4 v, u32x4 *to) {
        if constexpr (kPassXp)
            __builtin_nontemporal_store(v, to);
        else
            *to = v;
    };
    int c = lane;
    for (; c + 3 * kWave < chunks; c += 4 * kWave) {
        const u32x4 v0 = get(src + c), v1 = get(src + c + kWave), v2 = get(src + c + 2 * kWave), v3 = get(src + c + 3 * kWave);
        for (int k = 0; k < K; ++k) {
            u32x4 *dst = xp + (int64_t)lane_value(my_slot, k) * chunks + c;
            put(v0, dst);
            put(v1, dst + kWave);
            put(v2, dst + 2 * kWave);
            put(v3, dst + 3 * kWave);
        }
    }
    for (; c < chunks; c += kWave) {
        const u32x4 v = get(src + c);
        for (int k = 0; k < K; ++k)
            put(v, xp + (int64_t)lane_value(my_slot, k) * chunks + c);
    }
}

// kWaves wavefronts per token: the chunks of a row are dealt to them in turn, so that a workgroup reads whole rows at a time
// (long rows; 16384 tokens, H 7168, K 8: one wavefront per token 406 us, four 380 us, 5.6 TB/s).  A lane keeps four gathers
// in flight, of four chunks of a row or, where a row has fewer per lane, of several rows.
template <bool kBf16, int kWaves>
__global__ __launch_bounds__(kWave *kTokensPerBlock) void combine_rows(
    const u32x4 *__restrict__ y, int chunks, int64_t N, int K,
    const int32_t *__restrict__ slot_of_row, const float *__restrict__ topk_w,
    u32x4 *__restrict__ out)
{
    constexpr int kStep = kWaves * kWave; // chunks from one of a lane's to its next
    const int lane = threadIdx.x % kWave;
    const int64_t n = (int64_t)blockIdx.x * (kTokensPerBlock / kWaves) + threadIdx.x / kStep;
    if (n >= N)
        return;
    int32_t my_slot = (lane < K) ? slot_of_row[n * K + lane] : 0;
    float my_w = (lane < K) ? topk_w[n * K + lane] : 0.0f;
    auto rows_of = [&](auto u_tag, int c) {
        constexpr int kU = decltype(u_tag)::value;
        float acc[kU][8];
#pragma unroll
        for (int u = 0; u < kU; ++u)
#pragma unroll
            for (int i = 0; i < 8; ++i)
                acc[u][i] = 0.0f;
        auto rows = [&](auto count_tag, int k0) { // ascending k: the order of the sum is part of the contract
            constexpr int kRows = decltype(count_tag)::value;
            u32x4 v[kRows][kU];
#pragma unroll
            for (int k = 0; k < kRows; ++k) {
                const u32x4 *src = y + (int64_t)lane_value(my_slot, k0 + k) * chunks + c;
#pragma unroll
                for (int u = 0; u < kU; ++u)
                    v[k][u] = __builtin_nontemporal_load(&src[u * kStep]); // read once: no need to keep it cached
            }
#pragma unroll
            for (int k = 0; k < kRows; ++k) {
                const float w = lane_value(my_w, k0 + k);
#pragma unroll
                for (int u = 0; u < kU; ++u) {
                    if (kBf16) {
#pragma unroll
                        for (int i = 0; i < 4; ++i) {
                            acc[u][2 * i] = fmaf(w, bf16_bits_to_f32(v[k][u][i] & 0xFFFFu), acc[u][2 * i]);
                            acc[u][2 * i + 1] = fmaf(w, __uint_as_float(v[k][u][i] & 0xFFFF0000u), acc[u][2 * i + 1]);
                        }
                    } else {
#pragma unroll
                        for (int i = 0; i < 4; ++i)
                            acc[u][i] = fmaf(w, __uint_as_float(v[k][u][i]), acc[u][i]);
                    }
                }
            }
        };
        constexpr int kRows = 4 / kU;
        int k = 0;
        for (; k + kRows <= K; k += kRows)
            rows(std::integral_constant<int, kRows>{}, k);
        if constexpr (kRows > 1) {
            for (; k < K; ++k)
                rows(std::integral_constant<int, 1>{}, k);
        }
#pragma unroll
        for (int u = 0; u < kU; ++u) {
            u32x4 o;
            if (kBf16) {
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    o[i] = pack_bf16x2(acc[u][2 * i], acc[u][2 * i + 1]);
            } else {
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    o[i] = __float_as_uint(acc[u][i]);
            }
            __builtin_nontemporal_store(o, &out[n * chunks + c + u * kStep]);
        }
    };
    int c = threadIdx.x % kStep;
    for (; c + 3 * kStep < chunks; c += 4 * kStep)
        rows_of(std::integral_constant<int, 4>{}, c);
    for (; c + kStep < chunks; c += 2 * kStep)
        rows_of(std::integral_constant<int, 2>{}, c);
    for (; c < chunks; c += kStep)
        rows_of(std::integral_constant<int, 1>{}, c);
}

int launch_permute(const void *x, int64_t row_bytes, int64_t N, int K, const int32_t *slot_of_row,
                   void *xp, hipStream_t st)
{
    const int chunks = (int)(row_bytes / 16);
    const unsigned blocks = (unsigned)ceil_div(N, kTokensPerBlock);
    // What is to stay in the memory-side cache has to fit: x and xp, or x only, or xp only (an eighth more than fits: the rest of it
    // still is there).  270 random launches, x read before and xp after; MiB, us of the move and the read of xp (of which the move),
    // nothing past the cache -> x -> xp -> both: x 44, xp 176: 118 (39) -> 126 (47) -> 159 (53) -> 159 (53); x 180, xp 180: 173 (62)
    // -> 140 (61) -> 167 (59) -> 167 (59); x 44, xp 266: 223 (57) -> 199 (56) -> 212 (59) -> 211 (59); x 151, xp 302: 266 (79) ->
    // 268 (81) -> 244 (73) -> 244 (73); x 85, xp 687: 552 (143) -> 554 (141) -> 516 (144) -> 517 (145); x 396, xp 396: 381 (145) ->
    // 375 (129) -> 386 (166) -> 357 (137).  Rows that share lines of 128 bytes write those in two parts past the cache: below 4 KiB
    // 1.01 of the time (the move 1.2 - 1.5), above 0.95 (1.1), whole lines 0.92 (1.0).
    constexpr int64_t kMemoryCache = (int64_t)256 << 20;
    const int64_t x_bytes = N * row_bytes, xp_bytes = x_bytes * K;
    const bool pass_xp = xp_bytes > kMemoryCache / 8 * 9 && (row_bytes % 128 == 0 || row_bytes > 4096);
    const bool pass_x = x_bytes + (pass_xp ? 0 : xp_bytes) > kMemoryCache;
    auto kern = pass_xp ? (pass_x ? permute_rows<true, true> : permute_rows<false, true>)
                        : (pass_x ? permute_rows<true, false> : permute_rows<false, false>);
    hipLaunchKernelGGL(kern, dim3(blocks), dim3(kWave * kTokensPerBlock), 0, st,
                       static_cast<const u32x4 *>(x), chunks, N, K, slot_of_row,
                       static_cast<u32x4 *>(xp));
    return check_launch("moe_permute");
}

// rows from this many 16-byte chunks on: a workgroup per token (one chunk per lane or more); at 256 - 512 chunks both forms
// are within 3 % of each other
constexpr int kLongRow = 256;

template <bool kBf16>
static void launch_combine_of(const void *y, int64_t N, int chunks, int K, const int32_t *slot_of_row, const float *topk_w,
                              void *out, hipStream_t st)
{
    const bool long_row = chunks >= kLongRow && N <= 0xFFFFFF; // (a grid holds fewer than 2^32 threads)
    auto kern = long_row ? combine_rows<kBf16, 4> : combine_rows<kBf16, 1>;
    const unsigned blocks = (unsigned)(long_row ? N : ceil_div(N, kTokensPerBlock));
    hipLaunchKernelGGL(kern, dim3(blocks), dim3(kWave * kTokensPerBlock), 0, st, static_cast<const u32x4 *>(y), chunks, N, K,
                       slot_of_row, topk_w, static_cast<u32x4 *>(out));
}

int launch_combine(const void *y, int dtype, int64_t N, int64_t H, int K,
                   const int32_t *slot_of_row, const float *topk_w, void *out, hipStream_t st)
{
    if (dtype == MOE_BF16)
        launch_combine_of<true>(y, N, (int)(H * 2 / 16), K, slot_of_row, topk_w, out, st);
    else
        launch_combine_of<false>(y, N, (int)(H * 4 / 16), K, slot_of_row, topk_w, out, st);
    return check_launch("moe_combine");
}

}  // namespace moe
