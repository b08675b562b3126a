// Geometries of the expert computation's GEMMs and their launches.  The kernels are instantiated in several translation units
// (ffn_gate_up.hip, ffn_down.hip, ...), which compile side by side.
#pragma once

#include <atomic>

#include "common.h"
#include "grouped_gemm.h"

namespace moe {

// Geometries, by the rows of an expert.
//   up to 64: Shallow, 64x256x64, four (A, B) unit pairs, so that three K tiles of weights are in flight while one is multiplied.
//   65 - 160: Mid, 160x256x64, three pairs, every wavefront all rows of 64 columns.  Such a tile waits for memory; in Big, whose
//     A rows are fetched less than a K tile ahead and return in order behind the weights, a K tile took 2 us of which 1 was
//     arithmetic.  160 rows is the most three pairs have room for.
//   more: Big, 256x256x64, ring of 5 units (all 160 KiB of LDS); per window the 8 B loads of a wavefront go out under the first
//     two k-steps after the barrier, the 8 A loads under the other two.  An expert's last full tile also takes a remainder of up
//     to 64 rows ("tall" tile).
// The weights of the first two, which one workgroup reads once, are fetched with the non-temporal hint: they do not push out what
// is shared.  Experts of several row tiles share them in L2 and lose with it (256 experts of 425 - 616 rows, layer 11.6 ->
// 12.2 ms).  Gate/up, down, us, 16 experts, H 4096, F 6400, Big and ordinary loads -> Big and non-temporal -> as it is:
// 72 rows 350, 167 -> 342, 159 -> 317, 155; 128 rows 373, 177 -> 354, 168 -> 332, 166; 160 rows 382, 183 -> 363, 173 -> 343, 171.
// Experts of 161 - 320 rows, one Big tile, read their weights once too.  As a class of their own with the hint they took 0.98 of
// the time in 26 random launches of nothing larger and more than 512 MB of weights (64 experts of 170 rows, K 5696, N 960 178 ->
// 153 us), but 1.02 below that, 1.03 beside larger experts (a workgroup starts cold where the class changes) and 1.07 where the
// weights stay in the memory-side cache, which the hint passes by (438 launches, up to 1.3): ordinary loads.
// MOE_WEIGHTS_AHEAD: the operand that uses the ring's spare unit to run one K tile further ahead is the
// weights (1) or the activations (0).
#ifndef MOE_WEIGHTS_AHEAD
#define MOE_WEIGHTS_AHEAD 1
#endif
template <bool kSwiglu>
using BigTile = GemmCfg<256, 256, 2, 2, kSwiglu, 64, 5, (MOE_WEIGHTS_AHEAD ? 0x4400 : 0x0044),
                        (MOE_WEIGHTS_AHEAD ? 0x0044 : 0x4400), 0, 64, (MOE_WEIGHTS_AHEAD != 0)>;
#ifndef MOE_SHALLOW_UNITS
#define MOE_SHALLOW_UNITS 8
#endif
template <bool kSwiglu> using ShallowTile = GemmCfg<64, 256, 1, 4, kSwiglu, 64, MOE_SHALLOW_UNITS, 0x1010, 0x2222, 1>;

// The down projection with 128-column tiles, for launches with fewer tiles than compute units (few
// tokens): every tile of such a launch streams its whole weight panel alone and the launch lasts as
// long as one tile, so half as wide a panel on twice as many compute units halves it.  Where reductions
// are not turned (turn_of in ffn.hip) every output element is the same sum in the same order as with the
// 256-column tiles, so y has the same bits; a turned one starts at a K tile that depends on the tile's width.
// NarrowMid: four K tiles deep.  131 random launches (2 - 32 experts of 66 - 160 rows, K 512 - 14336) take 0.97 of the time of
// NarrowBig in the mean (singly 0.71 - 1.18).
template <bool kSwiglu> using NarrowBig = GemmCfg<256, 128, 2, 2, kSwiglu, 64, 6, 0x2222, 0x1111, 0, 64>;
template <bool kSwiglu> using NarrowShallow = GemmCfg<64, 128, 1, 4, kSwiglu, 64, 8, 0x1010, 0x1111, 1>;
template <bool kSwiglu> using MidTile = GemmCfg<160, 256, 1, 4, kSwiglu, 64, 6, 0x1121, 0x2222, 2>;
template <bool kSwiglu> using NarrowMid = GemmCfg<160, 128, 1, 4, kSwiglu, 64, 8, 0x1121, 0x1111, 2>;
constexpr int kMidRows = MidTile<true>::BM;
static_assert(MidTile<false>::BM == kMidRows && NarrowMid<false>::BM == kMidRows, "the tables' row tiles serve either geometry");

// a geometry of each kind
template <bool kSwiglu> struct WideSet {
    using Main = BigTile<kSwiglu>;
    using Mid = MidTile<kSwiglu>;
    using Light = ShallowTile<kSwiglu>;
};
struct NarrowSet {
    using Main = NarrowBig<false>;
    using Mid = NarrowMid<false>;
    using Light = NarrowShallow<false>;
};

int workgroup_slots(); // of the device, whole rounds over the XCDs
// Raises a kernel's dynamic LDS limit once per device (idempotent, so a race only repeats it).
void allow_lds(const void *kern, size_t lds_bytes, std::atomic<uint64_t> &raised);

template <class Set>
constexpr size_t lds_bytes_of()
{
    const size_t b = Set::Mid::kLdsBytes > Set::Light::kLdsBytes ? Set::Mid::kLdsBytes : Set::Light::kLdsBytes;
    return Set::Main::kLdsBytes > b ? Set::Main::kLdsBytes : b;
}

template <class Set, bool kSwiglu, bool kGather, bool kScatter, bool kTurn>
static void launch_gemm_form(const GemmArgs &g, hipStream_t st)
{
    auto kern = grouped_gemm_bf16<Set, kSwiglu, kGather, kScatter, kTurn>;
    static std::atomic<uint64_t> raised{0};
    allow_lds(reinterpret_cast<const void *>(kern), lds_bytes_of<Set>(), raised);
    // persistent grid: the workgroups draw their tiles from the table's counters
    hipLaunchKernelGGL(kern, dim3(workgroup_slots()), dim3(Set::Main::kThreads), lds_bytes_of<Set>(), st, g);
}

template <class Set, bool kSwiglu, bool kGather, bool kScatter>
static void launch_gemm(const GemmArgs &g, hipStream_t st)
{
    if (g.k_turn)
        launch_gemm_form<Set, kSwiglu, kGather, kScatter, true>(g, st);
    else
        launch_gemm_form<Set, kSwiglu, kGather, kScatter, false>(g, st);
}

// Both GEMMs in one launch, the second consuming the first's rows tile by tile.
template <class Set2, bool kTurn1, bool kTurn2>
static void launch_both_form(const GemmArgs &g1, const GemmArgs &g2, hipStream_t st)
{
    using Set1 = WideSet<true>;
    auto kern = grouped_ffn_bf16<Set1, Set2, kTurn1, kTurn2>;
    constexpr size_t lds_bytes = lds_bytes_of<Set1>() > lds_bytes_of<Set2>() ? lds_bytes_of<Set1>() : lds_bytes_of<Set2>();
    static std::atomic<uint64_t> raised{0};
    allow_lds(reinterpret_cast<const void *>(kern), lds_bytes, raised);
    hipLaunchKernelGGL(kern, dim3(workgroup_slots()), dim3(Set1::Main::kThreads), lds_bytes, st, g1, g2);
}

template <class Set2>
static void launch_both(const GemmArgs &g1, const GemmArgs &g2, hipStream_t st)
{
    if (g1.k_turn && g2.k_turn)
        launch_both_form<Set2, true, true>(g1, g2, st);
    else if (g1.k_turn)
        launch_both_form<Set2, true, false>(g1, g2, st);
    else if (g2.k_turn)
        launch_both_form<Set2, false, true>(g1, g2, st);
    else
        launch_both_form<Set2, false, false>(g1, g2, st);
}

void launch_gate_up(const GemmArgs &g, hipStream_t st);
void launch_gate_up_gather(const GemmArgs &g, hipStream_t st);
void launch_down(const GemmArgs &g, hipStream_t st);
void launch_down_narrow(const GemmArgs &g, hipStream_t st);
void launch_down_scatter(const GemmArgs &g, hipStream_t st);
void launch_down_scatter_narrow(const GemmArgs &g, hipStream_t st);
void launch_gate_up_and_down(const GemmArgs &g1, const GemmArgs &g2, hipStream_t st);
void launch_gate_up_and_down_narrow(const GemmArgs &g1, const GemmArgs &g2, hipStream_t st);

}  // namespace moe
