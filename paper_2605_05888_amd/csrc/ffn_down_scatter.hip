// Expert computation: down projection with the combine in its epilogue (grouped_gemm.h; geometries and launches in ffn_gemm.h).
#include "ffn_gemm.h"

namespace moe {

void launch_down_scatter(const GemmArgs &g, hipStream_t st) { launch_gemm<WideSet<false>, false, false, true>(g, st); }
void launch_down_scatter_narrow(const GemmArgs &g, hipStream_t st) { launch_gemm<NarrowSet, false, false, true>(g, st); }

}  // namespace moe
