// Instantiations of ago_invres_reg.hpp: fp32, stride 1, depthwise 3 x 3.
#include "ago_invres_reg.hpp"

namespace ago {
hipError_t invres_reg_f13(int ropt, int xr, int nco, const InvresRegParams& p, unsigned grid, unsigned threads, size_t smem, hipStream_t s) {
    return invres_reg_run<false, 1, 3>(ropt, xr, nco, p, grid, threads, smem, s);
}
}  // namespace ago
