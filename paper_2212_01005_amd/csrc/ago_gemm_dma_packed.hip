// The products of ago_gemm_dma.hpp on packed weights.
#include "ago_gemm_dma.hpp"

namespace ago {
hipError_t gemm_dma_packed(int tiling, const GemmDmaParams& p, hipStream_t s) {
    if (p.act == kNone) return gemm_dma_tiling<kNone, kEpPlain, true>(tiling, p, s);
    if (p.act == kGeluTanh) return gemm_dma_tiling<kGeluTanh, kEpPlain, true>(tiling, p, s);
    return gemm_dma_tiling<kActRuntime, kEpPlain, true>(tiling, p, s);
}
}  // namespace ago
