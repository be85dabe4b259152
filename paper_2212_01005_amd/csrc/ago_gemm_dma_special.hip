// The products of ago_gemm_dma.hpp on row-major weights with a residual or a head-major store.
#include "ago_gemm_dma.hpp"

namespace ago {
hipError_t gemm_dma_special(int tiling, const GemmDmaParams& p, bool head_major, hipStream_t s) {
    if (head_major) return gemm_dma_tiling<kNone, kEpHeadMajor, false>(tiling, p, s);
    if (p.act == kNone) return gemm_dma_tiling<kNone, kEpResidual, false>(tiling, p, s);
    return gemm_dma_tiling<kActRuntime, kEpResidual, false>(tiling, p, s);
}
}  // namespace ago
