// The products of ago_gemm_dma.hpp on row-major weights, plain epilogue.
#include "ago_gemm_dma.hpp"

namespace ago {
hipError_t gemm_dma_rows(int tiling, const GemmDmaParams& p, hipStream_t s) {
    if (p.act == kNone) return gemm_dma_tiling<kNone, kEpPlain, false>(tiling, p, s);
    if (p.act == kGeluTanh) return gemm_dma_tiling<kGeluTanh, kEpPlain, false>(tiling, p, s);
    return gemm_dma_tiling<kActRuntime, kEpPlain, false>(tiling, p, s);
}
}  // namespace ago
