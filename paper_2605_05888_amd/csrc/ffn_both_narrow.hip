// Expert computation: both GEMMs in one launch, the second with 128-column tiles (grouped_gemm.h; geometries and launches in ffn_gemm.h).
#include "ffn_gemm.h"

namespace moe {

void launch_gate_up_and_down_narrow(const GemmArgs &g1, const GemmArgs &g2, hipStream_t st) { launch_both<NarrowSet>(g1, g2, st); }

}  // namespace moe
