// Expert computation: down projection with 256-column tiles (grouped_gemm.h; geometries and launches in ffn_gemm.h).
#include "ffn_gemm.h"

namespace moe {

void launch_down(const GemmArgs &g, hipStream_t st) { launch_gemm<WideSet<false>, false, false, false>(g, st); }

}  // namespace moe
