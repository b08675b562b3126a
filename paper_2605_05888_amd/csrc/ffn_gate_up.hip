// Expert computation: gate/up projection of rows that lie in expert order (grouped_gemm.h; geometries and launches in ffn_gemm.h).
#include "ffn_gemm.h"

namespace moe {

void launch_gate_up(const GemmArgs &g, hipStream_t st) { launch_gemm<WideSet<true>, true, false, false>(g, st); }

}  // namespace moe
