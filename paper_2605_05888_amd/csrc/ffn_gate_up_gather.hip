// Expert computation: gate/up projection of rows fetched through the slot map (grouped_gemm.h; geometries and launches in ffn_gemm.h).
#include "ffn_gemm.h"

namespace moe {

void launch_gate_up_gather(const GemmArgs &g, hipStream_t st) { launch_gemm<WideSet<true>, true, true, false>(g, st); }

}  // namespace moe
